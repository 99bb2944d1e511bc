// Integers held across a wavefront: limb 64 c + lane of a number is word c of
// that lane, so additions, small multiples and comparisons take a few
// instructions whatever the length.  Carries between the limbs are resolved
// for all lanes at once: with masks G (limbs that carry out by themselves) and
// P (limbs of all ones, which pass a carry on), the 64-bit sum (G << 1) + P
// on the scalar unit ripples every carry through the P runs.
#pragma once

#include "arith.hpp"

namespace rnsrsa {

// Carry into each lane from masks g and p (never both set for a lane) and the
// carry cin into lane 0; cin becomes the carry out of lane 63.
__device__ __forceinline__ uint64_t limb_carries(uint64_t g, uint64_t p, uint32_t &cin) {
    const uint64_t y = (g << 1) | cin, s = y + p;
    cin = (uint32_t)(g >> 63) | (s < p ? 1u : 0u);
    return s ^ p;
}

__device__ __forceinline__ uint32_t lane_bit(uint64_t mask, int lane) { return (uint32_t)(mask >> lane) & 1u; }

// Word of the lane below (lane 0: `first`).
__device__ __forceinline__ uint32_t lane_up(uint32_t v, uint32_t first) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)v, 0x138 /* wave_shr:1 */, 0xF, 0xF, false);
}

// Word of the lane above (lane 63: `last`).
__device__ __forceinline__ uint32_t lane_down(uint32_t v, uint32_t last) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)last, (int)v, 0x130 /* wave_shl:1 */, 0xF, 0xF, false);
}

// Limbs of sum_l t_l 2^(32 l), every t_l below 2^63; returns the carry out of the
// top lane.
template <int C>
__device__ __forceinline__ uint32_t limbs_of_sums(const uint64_t (&t)[C], uint32_t (&v)[C], int lane) {
    uint32_t below = 0, cin = 0;
#pragma unroll
    for (int c = 0; c < C; c++) {
        const uint32_t lo = (uint32_t)t[c], hi = (uint32_t)(t[c] >> 32);
        const uint32_t u = lo + lane_up(hi, below);
        below = (uint32_t)__builtin_amdgcn_readlane((int)hi, 63);
        const uint64_t cm = limb_carries(__ballot(u < lo), __ballot(u == 0xFFFFFFFFu), cin);
        v[c] = u + lane_bit(cm, lane);
    }
    return below + cin;
}

// v <- v - n when v >= n; over: a carry out of v's top lane that counts to v.
template <int C>
__device__ __forceinline__ void limbs_reduce_once(uint32_t (&v)[C], const uint32_t (&n)[C], int lane, uint32_t over = 0) {
    uint32_t d[C], cin = 1;                                  // v - n = v + ~n + 1
#pragma unroll
    for (int c = 0; c < C; c++) {
        const uint32_t u = v[c] + ~n[c];
        const uint64_t cm = limb_carries(__ballot(u < v[c]), __ballot(u == 0xFFFFFFFFu), cin);
        d[c] = u + lane_bit(cm, lane);
    }
    if (cin | over) {                                        // no borrow
#pragma unroll
        for (int c = 0; c < C; c++) v[c] = d[c];
    }
}

// v <- v + a; returns the carry out of the top lane.
template <int C>
__device__ __forceinline__ uint32_t limbs_add(uint32_t (&v)[C], const uint32_t (&a)[C], int lane) {
    uint32_t cin = 0;
#pragma unroll
    for (int c = 0; c < C; c++) {
        const uint32_t s = v[c] + a[c];
        const uint64_t cm = limb_carries(__ballot(s < a[c]), __ballot(s == 0xFFFFFFFFu), cin);
        v[c] = s + lane_bit(cm, lane);
    }
    return cin;
}

// Limb l (uniform) of a number.
template <int C>
__device__ __forceinline__ uint32_t limb_at(const uint32_t (&v)[C], int l) {
    if constexpr (C == 1) return (uint32_t)__builtin_amdgcn_readlane((int)v[0], l);
    uint32_t r = 0;
#pragma unroll
    for (int c = 0; c < C; c++)
        if (l >> 6 == c) r = (uint32_t)__builtin_amdgcn_readlane((int)v[c], l & 63);
    return r;
}

// Index of the top nonzero limb (0 when there is none).
template <int C>
__device__ __forceinline__ int top_limb(const uint32_t (&v)[C]) {
    int t = 0;
#pragma unroll
    for (int c = 0; c < C; c++) {
        const uint64_t m = __ballot(v[c] != 0);
        if (m) t = 64 * c + 63 - __builtin_clzll(m);
    }
    return t;
}

// n's top two limbs as a double, for limbs_quotient.
template <int C>
__device__ __forceinline__ double limbs_top(const uint32_t (&n)[C], int t) {
    return (double)limb_at(n, t) + (t ? (double)limb_at(n, t - 1) * 0x1p-32 : 0.0);
}

// An estimate of v / n below 2^11 from three limbs of v, the middle one at n's top,
// and n's top two as a double, nd >= 1.  The limbs left out of either change the
// quotient's value by less than 2^11 (2^-31 + 2^-50), so the estimate lowered by
// 2^-19 is below it by less than 2^-18: its integer part is floor(v / n) or one less.
__device__ __forceinline__ double limbs_estimate(uint32_t above, uint32_t top, uint32_t below, double nd) {
    return ((double)above * 0x1p32 + (double)top + (double)below * 0x1p-32) / nd - 0x1p-19;
}

// floor(v / n) or one less, for v / n < 2^11; t = top_limb(n), nd = limbs_top(n, t).
template <int C>
__device__ __forceinline__ uint32_t limbs_quotient(const uint32_t (&v)[C], int t, double nd) {
    const double q = limbs_estimate(limb_at(v, t + 1), limb_at(v, t), t ? limb_at(v, t - 1) : 0u, nd);
    return (uint32_t)__builtin_amdgcn_readfirstlane(q > 0.0 ? (int)q : 0);
}

// Limb 0 of sums.
template <int C>
__device__ __forceinline__ uint32_t low_limb(const uint64_t (&u)[C]) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)u[0]);
}

// One limb step of a product with lazy carries: t <- (v's low words + 2^32 (u's
// high words + v's (TWO) + t's)) / 2^32, v's limb 0 dropped.  t stays below 3 2^32.
template <int C, bool TWO>
__device__ __forceinline__ void shift_step(const uint64_t (&u)[C], const uint64_t (&v)[C], uint64_t (&t)[C]) {
#pragma unroll
    for (int c = 0; c < C; c++) {
        uint32_t last = 0;
        if (c + 1 < C) last = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v[c + 1 < C ? c + 1 : 0]);
        const uint32_t dn = lane_down((uint32_t)v[c], last);
        t[c] = (uint64_t)dn + (uint32_t)(u[c] >> 32) + (TWO ? (uint32_t)(v[c] >> 32) : 0u) + (uint32_t)(t[c] >> 32);
    }
}

// -n^-1 mod 2^32 of odd n: n inverts itself mod 2^3, each step doubles the bits.
__device__ __forceinline__ uint32_t neg_inverse32(uint32_t n) {
    uint32_t inv = n;
#pragma unroll
    for (int i = 0; i < 4; i++) inv *= 2u - n * inv;
    return 0u - inv;
}

// Montgomery product r = a b / 2^(32 L) mod n in [0, n): odd n of at most L <= 64 C
// limbs, a < 2^(32 L), b < n; ninv = neg_inverse32(n's limb 0).  L steps of one limb
// of a times all lanes; a step's chain (multiply-add, lane 0 to the scalar unit,
// multiply-add, the shift by one lane) is about 100 cycles.
template <int C>
__device__ __forceinline__ void limbs_montmul(const uint32_t (&a)[C], const uint32_t (&b)[C], const uint32_t (&n)[C],
                                              uint32_t ninv, int L, int lane, uint32_t (&r)[C]) {
    uint64_t t[C], u[C], v[C];
#pragma unroll
    for (int c = 0; c < C; c++) t[c] = 0;
    for (int i = 0; i < L; i++) {
        const uint32_t x = limb_at(a, i);
#pragma unroll
        for (int c = 0; c < C; c++) u[c] = (uint64_t)x * b[c] + (uint32_t)t[c];
        const uint32_t m = low_limb(u) * ninv;
#pragma unroll
        for (int c = 0; c < C; c++) v[c] = (uint64_t)m * n[c] + (uint32_t)u[c];
        shift_step<C, true>(u, v, t);
    }
    const uint32_t over = limbs_of_sums(t, r, lane);           // below 2 n
    limbs_reduce_once(r, n, lane, over);
}

}  // namespace rnsrsa
