// Wave engine: the matrix-core product with every channel of 16 NT elements
// in ONE wavefront (shapes with W = 1; included by kernels_mfma.hpp).
//
// With all 4 MT slots in one wave the digits never leave its registers: lane
// (g, n) computes the digits of slots 4 mt + g for element n, and because the
// order of the contraction's K index is free, the tables order it so that the
// digit words of tiles 4 ks .. 4 ks + 3 of a lane ARE its 16-byte operand of
// k-step ks (MLayout::word_of).  A product needs no barrier and no exchange
// through LDS, only one lane broadcast per extension (the redundant row).
//
// A workgroup is WAVE_GROUP waves, each with its own elements of one job; they
// share the job's constant tiles of both extensions in LDS (54 KB at k = 33)
// and nothing else.  An extension runs tile by tile: the matrix instructions
// of one tile and the per-channel steps of the tile before it are independent,
// so a single wave keeps both units busy, with two tiles' results in registers
// instead of all of them.
//
// What bounds it: about 290 vector instructions a product at k = 33, multiply-adds
// among them at the full rate, and 54 matrix instructions of 16 cycles.  Issuing both keeps
// the vector unit 63% and the matrix cores 39% busy (16,384 decryptions), which
// together is the whole time: with two waves per SIMD the two units still take turns.
// Three waves with three tiles each, digits exchanged through LDS between two
// barriers, kept them 58% and 28% busy.  RSA-2048 CRT decryptions
// (k = 33): 16,384 in 3.17 -> 2.45 ms, 32,768 in 6.96 -> 4.93 ms; RSA-1024 (k =
// 17) 16,384 in 1.04 -> 0.70 ms.
#pragma once

namespace rnsrsa {

// Second operands of a product: registers (the state itself), or an LDS buffer
// (+ lane) to which a window's table entry was copied ahead of its use.
template <int M, int NT>
struct MRegOperand {
    const MState<M, NT> &s;
    __device__ __forceinline__ uint32_t b(int t, int nt) const { return s.b[t][nt]; }
    __device__ __forceinline__ uint32_t p(int t, int nt) const { return s.p[t][nt]; }
    __device__ __forceinline__ uint32_t r(int nt) const { return s.r[nt]; }
};
template <int M, int NT>
struct MLdsOperand {
    const uint32_t *y;
    __device__ __forceinline__ uint32_t b(int t, int nt) const { return y[(t * NT + nt) * 64]; }
    __device__ __forceinline__ uint32_t p(int t, int nt) const { return y[(M * NT + t * NT + nt) * 64]; }
    __device__ __forceinline__ uint32_t r(int nt) const { return y[(2 * M * NT + nt) * 64]; }
};

// Values of lane groups 2 and 3, in every lane group: two swaps of rows, about 20
// cycles where a read through LDS takes over 100, of which k = 17's short products do
// not hide enough (a lone RSA-1024 decryption 535 -> 514 us).
__device__ __forceinline__ void lane_groups_23(uint32_t v, uint32_t &g2, uint32_t &g3) {
    const auto hi = __builtin_amdgcn_permlane32_swap(v, v, false, false);           // [1]: groups 2 3 2 3
    const auto r = __builtin_amdgcn_permlane16_swap(hi[1], hi[1], false, false);    // [0]: 2 2 2 2, [1]: 3 3 3 3
    g2 = r[0];
    g3 = r[1];
}

// The slots' constants into LDS, [MT][4 lane groups][2][4]: B {m, m^-1 (SQ: -m^-1)
// mod 2^32, nu, c (wide: nu2)}, B' {m, m^-1, H, 0 (ONCE: MLayout::zdig; wide: m 2^OSH)}.
template <int K, int MT, int NT, int F, bool ONCE = false>
__device__ __forceinline__ void wave_constants(const gu32 *__restrict__ mb, const gu32 *__restrict__ mk, uint32_t *c,
                                               int threads) {
    using S = MShp<K, 1, MT, NT>;
    constexpr bool SQ = F != kPlain, WIDE = F == kWide;
    for (int i = threadIdx.x; i < MT * 32; i += threads) {
        const int f = i & 7, mt = i >> 5, ln = 16 * ((i >> 3) & 3);
        uint32_t v = 0;
        if (f < 4) {
            if (f < 2 || !SQ) v = f < 3 ? mb[S::LY.slotB() + (mt * 3 + f) * 64 + ln] : mk[S::LY.slotC() + mt * 64 + ln];
            else v = mk[S::LY.sqB() + (mt * 4 + (f == 2 ? 0 : 3)) * 64 + ln];
            if (SQ && f == 1) v = 0u - v;
        } else if (f < 6 || !WIDE) {
            if (f < 7) v = mb[S::LY.slotP() + (mt * 4 + (f - 4)) * 64 + ln];
            else if (ONCE) v = mk[S::LY.zdig() + mt * 64 + ln];
        } else {
            const uint64_t off = (uint64_t)mb[S::LY.slotP() + mt * 4 * 64 + ln] << S::OSH;
            v = f == 6 ? (uint32_t)off : (uint32_t)(off >> 32);
        }
        c[i] = v;
    }
}

// F: MForm
template <int K, int MT, int NT, int F, bool ONCE = false>
struct WaveEngine {
    using S = MShp<K, 1, MT, NT>;
    static constexpr int KS = S::KSTEPS;
    static_assert(4 * KS > MT, "a digit word for the offset after the last tile");
    static constexpr bool SQ = F != kPlain, WIDE = F == kWide;   // see kWideShift
    static_assert(!WIDE || S::LY.wide(), "a slot for the estimate row");

    const mfma_v4i *A1, *A2;             // LDS: the extensions' tiles [MT][KS][64], + lane
    mfma_v4i R1[MT][KS];                 // A1REG: the first extension's in registers
    // ONCE: a single product, whose tiles of the first extension come from global
    // memory: 29 instead of 76 KB of LDS and 144 instead of 232 registers let three
    // waves share a SIMD (40,000 products at k = 33: 17.9 -> 15.2 us, 65,536: 24.6 -> 22.4)
    static constexpr bool A1GLOBAL = NT == 1 && ONCE, A1REG = NT == 1 && !ONCE;
    gcv4i *A1g;
    const uint32_t *cl;                  // LDS: the slots' constants [MT][4][2][4], + this lane group's
    uint32_t Mpinv_r, Minv_r, N_r;
    int32_t est_r;                       // the wide form's estimate constant
    int32_t kf[4];                       // see mfma_accumulate
    MState<MT, NT> x;
    int lane;

    // Digit words of one group of 16 elements: word j of w[ks] is tile 4 ks + j's.
    struct Digits {
        mfma_v4i w[KS];
        // the offset digit (and words whose columns are zero)
        __device__ __forceinline__ Digits() {
#pragma unroll
            for (int i = MT; i < 4 * KS; i++) w[i / 4][i % 4] = 1;
        }
        __device__ __forceinline__ void set(int mt, uint32_t v) { w[mt / 4][mt % 4] = (int)mfma_pack(v); }
    };

    Digits d2[NT];                       // xi' (WIDE: the kept residues) of the last product

    __device__ __forceinline__ uint4 cB(int mt) const { return *(const uint4 *)(cl + 32 * mt); }
    __device__ __forceinline__ uint4 cP(int mt) const { return *(const uint4 *)(cl + 32 * mt + 4); }
    __device__ __forceinline__ MSlotB slotB(int mt) const {
        const uint4 v = cB(mt);
        return MSlotB{v.x, SQ ? 0u - v.y : v.y, v.z, v.w};
    }
    __device__ __forceinline__ MSlotP slotP(int mt) const {
        const uint4 v = cP(mt);
        return MSlotP{v.x, v.y, v.z, 0u};
    }

    // The tiles and the slots' constants into LDS, by all waves of the
    // workgroup (a barrier follows before their first use).
    __device__ __forceinline__ void setup(const gu32 *__restrict__ mb, const gu32 *__restrict__ mk, uint32_t *lds, int l) {
        lane = l;
        constexpr int NQ = MT * KS * 64;
        gcv4i *a1 = (gcv4i *)(mk + S::LY.a1()), *a2 = (gcv4i *)(SQ ? mk + S::LY.a2s() : mb + S::LY.a2());
        mfma_v4i *t = (mfma_v4i *)lds;
        for (int i = threadIdx.x; i < NQ; i += 64 * S::WAVE_GROUP) {
            t[i] = a2[i];
            if (!A1GLOBAL) t[NQ + i] = a1[i];
        }
        A2 = t + lane;
        A1 = t + NQ + lane;
        A1g = a1 + lane;
        uint32_t *c = lds + (A1GLOBAL ? 1 : 2) * NQ * 4;
        wave_constants<K, MT, NT, F, ONCE>(mb, mk, c, 64 * S::WAVE_GROUP);
        cl = c + 8 * (lane >> 4);
        Mpinv_r = mb[S::LY.bscal() + 0];
        Minv_r = mb[S::LY.bscal() + 1];
        N_r = mk[S::LY.kscal() + 0];
        est_r = (int32_t)mk[S::LY.kscal() + 1];
#pragma unroll
        for (int b = 0; b < 4; b++) {
            kf[b] = 1 << (8 * b);
            asm volatile("" : "+s"(kf[b]));
        }
    }

    // An extension of every group's digits in steps of G tiles, the redundant
    // row's tile first.  use(mt, D) takes tile mt's results; each step holds
    // the matrix instructions of its tiles, use() of the step before and the
    // LDS reads of the step after it, and the scheduling barriers keep the
    // compiler from moving work across the steps (it would start the vector
    // work of every tile early and spill it).  A vector step is a chain of
    // about 16 dependent multiplications and additions, each a few cycles
    // longer than its issue, so G NT chains are interleaved.
    // Steps of one tile with the first extension's tiles in registers measured
    // best for 16 elements (16,384 decryptions: 2.53 ms; two tiles and every tile
    // from LDS 2.66 ms); two tiles for 32 (k <= 9), whose registers hold none.
    static constexpr int G = NT == 1 ? 1 : 2;
    __device__ __forceinline__ void load_tiles() {
        if (A1REG)
#pragma unroll
            for (int mt = 0; mt < MT; mt++)
#pragma unroll
                for (int ks = 0; ks < KS; ks++) R1[mt][ks] = A1[(mt * KS + ks) * 64];
    }
    template <bool FIRST>
    __device__ __forceinline__ mfma_v4i tile(const mfma_v4i *A, int mt, int ks) const {
        if constexpr (FIRST && A1REG) return R1[mt][ks];
        else if constexpr (FIRST && A1GLOBAL) return A1g[(mt * KS + ks) * 64];
        else return A[(mt * KS + ks) * 64];
    }
    template <bool FIRST, class L, class U>
    __device__ __forceinline__ void extension(const mfma_v4i *A, const Digits (&d)[NT], L load, U use) const {
        // an opaque zero: the tiles never change, and without it the compiler
        // reads all of them ahead of the exponent loop and spills them
        int zo;
        asm volatile("s_mov_b32 %0, 0" : "=s"(zo));
        A += zo;
        constexpr auto order = [](int i) { return i == 0 ? MT - 1 : i - 1; };
        constexpr int STEPS = (MT + G - 1) / G;
        mfma_v4i D[2][G][NT], a[2][G][KS];
        decltype(load(0)) c[2][G];
#pragma unroll
        for (int t = 0; t < G && t < MT; t++)
#pragma unroll
            for (int ks = 0; ks < KS; ks++) a[0][t][ks] = tile<FIRST>(A, order(t), ks);
#pragma unroll
        for (int i = 0; i <= STEPS; i++) {
#pragma unroll
            for (int t = 0; t < G; t++)
                if ((i + 1) * G + t < MT)
#pragma unroll
                    for (int ks = 0; ks < KS; ks++)
                        a[(i + 1) & 1][t][ks] = tile<FIRST>(A, order((i + 1) * G + t), ks);
#pragma unroll
            for (int t = 0; t < G; t++)
                if (i * G + t < MT) c[i & 1][t] = load(order(i * G + t));
#pragma unroll
            for (int t = 0; t < G; t++)
#pragma unroll
                for (int nt = 0; nt < NT; nt++) D[i & 1][t][nt] = mfma_v4i{0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < KS; ks++)
#pragma unroll
                for (int t = 0; t < G; t++)
#pragma unroll
                    for (int nt = 0; nt < NT; nt++)
                        if (i * G + t < MT)
                            D[i & 1][t][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[i & 1][t][ks], d[nt].w[ks],
                                                                                   D[i & 1][t][nt], 0, 0, 0);
#pragma unroll
            for (int t = 0; t < G; t++)
                if (i > 0 && (i - 1) * G + t < MT) use(order((i - 1) * G + t), c[(i - 1) & 1][t], D[(i - 1) & 1][t]);
            if (i < STEPS) __builtin_amdgcn_sched_barrier(0);
        }
    }
    // the redundant row's low word, in every lane of its element
    __device__ __forceinline__ uint32_t redundant(const mfma_v4i &D) const {
        // one tile: few instructions, so the copies that the swaps need count (300,000
        // powers at k = 3 236 us with them, 213 us through LDS; a lone one 56 us either way)
        if constexpr (MT == 1)
            return (uint32_t)__builtin_amdgcn_ds_bpermute(((lane & 15) + 48) * 4, (int)mfma_combine_lo(D));
        uint32_t g2, g3;
        lane_groups_23(mfma_combine_lo(D), g2, g3);
        return g3;
    }

    // Step (i): digits xi of x y.
    template <class Y>
    __device__ __forceinline__ void step1(const Y &y, Digits (&d)[NT]) const {
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
            const uint4 c = cB(mt);
#pragma unroll
            for (int nt = 0; nt < NT; nt++) {
                if constexpr (WIDE) {
                    d[nt].set(mt, redc_any((uint64_t)x.b[mt][nt] * y.b(mt, nt), c.x, c.y));
                } else if constexpr (SQ) {
                    // below the prime: the narrow offset is one m_i M_i, so a digit above m_i
                    // with sigma_i = -1 could make the quotient, and the result, negative
                    d[nt].set(mt, mulredc(x.b[mt][nt], y.b(mt, nt), c.x, 0u - c.y));
                } else {
                    uint32_t xi = mulredc(mulredc(x.b[mt][nt], y.b(mt, nt), c.x, c.y), c.w, c.x, c.y);
                    if (ONCE && xi == 0) xi = cP(mt).w;
                    d[nt].set(mt, xi);
                }
            }
        }
    }
    // One product x <- x y M^-1 (y may be x).  FULL = false stops after the
    // B' residues and, without scaled B residues, leaves the digits xi' in d2.
    //
    // With the wide second extension (WIDE) its digits are the kept B' residues, which saves the
    // multiplication by H and its reduction; step (iv)'s sum is small, so
    // that its reduction needs no correction (but in the first tile, where the
    // primes are closest to 2^32); B residues may exceed their prime.
    template <bool FULL, class Y>
    __device__ __forceinline__ void product(const Y &y) {
        Digits d1[NT];
        step1(y, d1);
        uint32_t xr[NT];
#pragma unroll
        for (int nt = 0; nt < NT; nt++) xr[nt] = x.r[nt] * y.r(nt);
        struct LoadP {
            uint4 c;
            uint32_t y[NT];
        };
        auto loadP = [&](int mt) {
            LoadP l;
            l.c = cP(mt);
#pragma unroll
            for (int nt = 0; nt < NT; nt++) l.y[nt] = y.p(mt, nt);
            return l;
        };
        extension<true>(A1, d1, loadP, [&](int mt, const LoadP &l, const mfma_v4i (&D)[NT]) {   // (ii), (iii)
            const uint32_t m = l.c.x, u = l.c.y;
            const uint64_t off = WIDE ? ((uint64_t)l.c.w << 32) | l.c.z : (uint64_t)m << S::OSH;
#pragma unroll
            for (int nt = 0; nt < NT; nt++) {
                if (mt == MT - 1) x.r[nt] = (xr[nt] + redundant(D[nt]) * N_r) * Minv_r;
                const uint64_t T = mfma_accumulate<S::PAIR_I32>(D[nt], (uint64_t)x.p[mt][nt] * l.y[nt] + off, kf);
                const uint32_t r = redc((uint32_t)T, (uint32_t)(T >> 32), m, u);
                x.p[mt][nt] = r;
                d2[nt].set(mt, WIDE ? r : mulredc(r, l.c.z, m, u));
            }
        });
        if constexpr (!FULL) return;
        uint32_t alpha[NT], alpha_h[NT];
        extension<false>(A2, d2, [&](int mt) { return cB(mt); }, [&](int mt, const uint4 &c, const mfma_v4i (&D)[NT]) {   // (iv)
            const uint32_t m = c.x;
#pragma unroll
            for (int nt = 0; nt < NT; nt++) {
                if (mt == MT - 1) {
                    if constexpr (WIDE) {
                        // the redundant row is lane group 3's, the estimate group 2's
                        uint32_t est, red;
                        lane_groups_23(lane < 48 ? (uint32_t)D[nt][0] : mfma_combine_lo(D[nt]), est, red);
                        const uint32_t lo = (red - x.r[nt]) * Mpinv_r;
                        const int32_t h = ((int32_t)est + est_r - (int32_t)(lo >> 18)) >> 14;
                        alpha_h[nt] = ((uint32_t)h << (32 - kWideShift)) + (lo >> kWideShift);
                        alpha[nt] = lo & ((1u << kWideShift) - 1);
                    } else {
                        alpha[nt] = (redundant(D[nt]) - x.r[nt]) * Mpinv_r;
                    }
                }
                if constexpr (WIDE) {
                    const uint64_t T = mfma_accumulate<S::PAIR_I32>(
                        D[nt], (uint64_t)alpha[nt] * c.z + (uint64_t)alpha_h[nt] * c.w, kf);
                    x.b[mt][nt] = mt == 0 ? redc_any(T, m, c.y) : redc_small(T, m, c.y);
                } else {
                    const uint64_t T = mfma_accumulate<S::PAIR_I32>(
                        D[nt], (uint64_t)alpha[nt] * c.z + ((uint64_t)m << S::OSH), kf);
                    x.b[mt][nt] = redc((uint32_t)T, (uint32_t)(T >> 32), m, SQ ? 0u - c.y : c.y);
                }
            }
        });
    }
};

// The same product with the tiles of 16 elements split over WV waves (the same
// tables; MT = WV * TW): for launches too small to give every SIMD two waves,
// where a product's latency counts.  A wave owns tiles [TW wave, TW wave + TW),
// keeps its share of both extensions' tiles in registers and passes its digit
// words on through LDS, [word][lane], so that every access is 64 consecutive
// words.  The last wave owns the redundant row; it publishes the redundant
// residue with its digits xi', and the other waves compute the second
// extension's last tile (redundant and estimate rows) too, so a product has
// two barriers.  A product's chain (two contractions, two reductions, two
// exchanges) bounds it, 0.75 us alone on its SIMDs; a lone RSA-2048 decryption
// takes 0.91 ms here and 1.6 ms on one wave.
template <int K, int MT, int WV, int F>
struct SplitEngine {
    static constexpr int NT = 1, TW = MT / WV;
    static constexpr bool SQ = F != kPlain, WIDE = F == kWide;
    using S = MShp<K, 1, MT, 1>;
    static constexpr int KS = S::KSTEPS;
    static_assert(S::LY.wide() && MT == WV * TW && 4 * KS > MT, "whole tiles per wave, a digit word for the offset");

    mfma_v4i A1[TW][KS], A2[TW][KS], AR[KS];   // AR: second extension's last tile
    uint4 cb[TW], cp[TW];                      // slot constants as in WaveEngine
    uint32_t Mpinv_r, Minv_r, N_r;
    int32_t est_r, kf[4];
    MState<TW, 1> x;
    int lane, wave;
    uint32_t *buf;                             // [2][MT + 1][64] digit words (and the redundant residue), + lane

    __device__ __forceinline__ MSlotB slotB(int t) const { return MSlotB{cb[t].x, SQ ? 0u - cb[t].y : cb[t].y, cb[t].z, cb[t].w}; }
    __device__ __forceinline__ MSlotP slotP(int t) const { return MSlotP{cp[t].x, cp[t].y, cp[t].z, 0u}; }

    __device__ __forceinline__ void setup(const gu32 *__restrict__ mb, const gu32 *__restrict__ mk, uint32_t *lds, int wv, int l) {
        lane = l;
        wave = wv;
        buf = lds + lane;
#pragma unroll
        for (int t = 0; t < TW; t++) {
            const int mt = wave * TW + t;
            cb[t].x = mb[S::LY.slotB() + (mt * 3 + 0) * 64 + lane];
            const uint32_t u = mb[S::LY.slotB() + (mt * 3 + 1) * 64 + lane];
            cb[t].y = SQ ? 0u - u : u;
            cb[t].z = SQ ? mk[S::LY.sqB() + (mt * 4 + 0) * 64 + lane] : mb[S::LY.slotB() + (mt * 3 + 2) * 64 + lane];
            cb[t].w = WIDE ? mk[S::LY.sqB() + (mt * 4 + 3) * 64 + lane] : mk[S::LY.slotC() + mt * 64 + lane];
            cp[t].x = mb[S::LY.slotP() + (mt * 4 + 0) * 64 + lane];
            cp[t].y = mb[S::LY.slotP() + (mt * 4 + 1) * 64 + lane];
            cp[t].z = mb[S::LY.slotP() + (mt * 4 + 2) * 64 + lane];
        }
        Mpinv_r = mb[S::LY.bscal() + 0];
        Minv_r = mb[S::LY.bscal() + 1];
        N_r = mk[S::LY.kscal() + 0];
        est_r = (int32_t)mk[S::LY.kscal() + 1];
#pragma unroll
        for (int b = 0; b < 4; b++) {
            kf[b] = 1 << (8 * b);
            asm volatile("" : "+s"(kf[b]));
        }
    }
    __device__ __forceinline__ void load_tiles(const gu32 *__restrict__ mb, const gu32 *__restrict__ mk) {
        gcv4i *a1 = (gcv4i *)(mk + S::LY.a1()), *a2 = (gcv4i *)(SQ ? mk + S::LY.a2s() : mb + S::LY.a2());
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
#pragma unroll
            for (int t = 0; t < TW; t++) {
                A1[t][ks] = mfma_tile_load(a1, (wave * TW + t) * KS + ks, 16u * lane);
                A2[t][ks] = mfma_tile_load(a2, (wave * TW + t) * KS + ks, 16u * lane);
            }
            AR[ks] = mfma_tile_load(a2, (MT - 1) * KS + ks, 16u * lane);
        }
    }
    // All digit words of this lane, as the operands of the k-steps.
    __device__ __forceinline__ void gather(int which, mfma_v4i (&w)[KS]) const {
#pragma unroll
        for (int i = 0; i < 4 * KS; i++) w[i / 4][i % 4] = i < MT ? (int)buf[(which * (MT + 1) + i) * 64] : 1;
    }
    __device__ __forceinline__ void publish(int which, int t, uint32_t v) const {
        buf[(which * (MT + 1) + wave * TW + t) * 64] = mfma_pack(v);
    }
    // last: the exit product, which leaves the digits xi' in the second buffer
    template <bool FULL, class Y>
    __device__ __forceinline__ void product(const Y &y) {
#pragma unroll
        for (int t = 0; t < TW; t++) {
            uint32_t xi;
            if constexpr (WIDE) xi = redc_any((uint64_t)x.b[t][0] * y.b(t, 0), cb[t].x, cb[t].y);
            else if constexpr (SQ) xi = mulredc(x.b[t][0], y.b(t, 0), cb[t].x, 0u - cb[t].y);
            else xi = mulredc(mulredc(x.b[t][0], y.b(t, 0), cb[t].x, cb[t].y), cb[t].w, cb[t].x, cb[t].y);
            publish(0, t, xi);
        }
        __syncthreads();
        mfma_v4i w[KS], D[TW], R;
        gather(0, w);
#pragma unroll
        for (int t = 0; t < TW; t++) D[t] = mfma_v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
#pragma unroll
            for (int t = 0; t < TW; t++) D[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A1[t][ks], w[ks], D[t], 0, 0, 0);
        uint32_t lo1 = 0;
        if (wave == WV - 1) lo1 = (uint32_t)__builtin_amdgcn_ds_bpermute(((lane & 15) + 48) * 4, (int)mfma_combine_lo(D[TW - 1]));
#pragma unroll
        for (int t = 0; t < TW; t++) {
            const uint32_t m = cp[t].x, u = cp[t].y;
            const uint64_t T = mfma_accumulate<S::PAIR_I32>(
                D[t], (uint64_t)x.p[t][0] * y.p(t, 0) + ((uint64_t)m << S::OSH), kf);
            const uint32_t r = redc((uint32_t)T, (uint32_t)(T >> 32), m, u);
            x.p[t][0] = r;
            publish(1, t, WIDE && FULL ? r : mulredc(r, cp[t].z, m, u));
        }
        if (wave == WV - 1) {
            x.r[0] = (x.r[0] * y.r(0) + lo1 * N_r) * Minv_r;
            buf[(2 * (MT + 1) - 1) * 64] = x.r[0];
        }
        __syncthreads();
        if constexpr (!FULL) return;
        gather(1, w);
        const uint32_t rr = buf[(2 * (MT + 1) - 1) * 64];
        R = mfma_v4i{0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < TW; t++) D[t] = mfma_v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ks++) R = __builtin_amdgcn_mfma_i32_16x16x64_i8(AR[ks], w[ks], R, 0, 0, 0);
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
#pragma unroll
            for (int t = 0; t < TW; t++) D[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A2[t][ks], w[ks], D[t], 0, 0, 0);
        const uint32_t lo =
            ((uint32_t)__builtin_amdgcn_ds_bpermute(((lane & 15) + 48) * 4, (int)mfma_combine_lo(R)) - rr) * Mpinv_r;
        uint32_t al = lo, ah = 0;
        if constexpr (WIDE) {
            const int32_t est = __builtin_amdgcn_ds_bpermute(((lane & 15) + 32) * 4, R[0]);
            const int32_t h = (est + est_r - (int32_t)(lo >> 18)) >> 14;
            ah = ((uint32_t)h << (32 - kWideShift)) + (lo >> kWideShift);
            al = lo & ((1u << kWideShift) - 1);
        }
#pragma unroll
        for (int t = 0; t < TW; t++) {
            const uint32_t m = cb[t].x;
            if constexpr (WIDE) {
                const uint64_t T = mfma_accumulate<S::PAIR_I32>(D[t], (uint64_t)al * cb[t].z + (uint64_t)ah * cb[t].w, kf);
                x.b[t][0] = t == 0 ? redc_any(T, m, cb[t].y) : redc_small(T, m, cb[t].y);
            } else {
                const uint64_t T = mfma_accumulate<S::PAIR_I32>(D[t], (uint64_t)al * cb[t].z + ((uint64_t)m << S::OSH), kf);
                x.b[t][0] = redc((uint32_t)T, (uint32_t)(T >> 32), m, SQ ? 0u - cb[t].y : cb[t].y);
            }
        }
    }
};

// The product on a team of 8 waves (k = 65 and 66), for bases whose tiles do not fit
// one wave's share of LDS: a wave has MT / 8 tiles, the first MT % 8 one more, so
// that at k = 65 a SIMD's two waves hold at most five of the 17 (six waves of three,
// as before, left two SIMDs with six).  Tiles are in registers but, at three per
// wave, L1 + L2 of the wave's and, for every wave, the redundant one, which all
// compute: those are in LDS.  Digit words pass through LDS as [k-step][lane][4],
// the layout of the operands.  Otherwise as SplitEngine.
//
// With both extensions' tiles split over six waves of 11 channels and a redundant
// row each, without the wide form -> this: RSA-4096, one decryption 3.05 -> 2.48 ms,
// 4,096 in 4.98 -> 4.37 ms; 10,007 RSA-2048 encryptions 145 -> 130 us.
template <int K, int MT, int NT, int F, int TW, bool ONCE = false>
struct TeamEngine {
    using S = MShp<K, 1, MT, NT>;
    static constexpr bool SQ = F != kPlain, WIDE = F == kWide;
    static constexpr int KS = S::KSTEPS, WV = S::TEAM_WAVES;
    // tiles of the first and second extension kept in LDS, not in registers
    static constexpr int L1 = TW == 3 ? S::TEAM_L1 : 0, L2 = TW == 3 ? S::TEAM_L2 : 0;
    static constexpr int T1 = TW - L1, T2 = TW - L2;
    static_assert(S::LY.wide() && 4 * KS > MT, "a digit word for the offset");

    mfma_v4i A1[T1][KS], A2[T2][KS];
    const mfma_v4i *lt;                        // LDS tiles: the second extension's last, the first wave's L2, its L1; + lane
    uint4 cb[TW], cp[TW];                      // slot constants (wave_constants)
    uint32_t Mpinv_r, Minv_r, N_r;
    int32_t est_r, kf[4];
    MState<TW, NT> x;
    int lane, wave, tile0;
    uint32_t *buf;                             // [2][NT][KS][64][4] digit words, [NT][64] redundant residues, + 4 lane

    __device__ __forceinline__ MSlotB slotB(int t) const {
        return MSlotB{cb[t].x, SQ ? 0u - cb[t].y : cb[t].y, cb[t].z, cb[t].w};
    }
    __device__ __forceinline__ MSlotP slotP(int t) const { return MSlotP{cp[t].x, cp[t].y, cp[t].z, 0u}; }

    // lds: the constants and tiles, then the exchange buffer; a barrier and
    // load_constants follow.
    __device__ __forceinline__ void setup(const gu32 *__restrict__ mb, const gu32 *__restrict__ mk, uint32_t *lds, int wv, int l) {
        lane = l;
        wave = wv;
        tile0 = S::team_tile0(wv);
        wave_constants<K, MT, NT, F, ONCE>(mb, mk, lds, 64 * WV);
        mfma_v4i *t = (mfma_v4i *)(lds + 32 * MT);
        lt = t + lane;
        gcv4i *a1 = (gcv4i *)(mk + S::LY.a1()), *a2 = (gcv4i *)(SQ ? mk + S::LY.a2s() : mb + S::LY.a2());
        for (int i = threadIdx.x; i < S::TEAM_TILES * KS * 64; i += 64 * WV) {
            const int z = i / (KS * 64), r = i % (KS * 64);
            t[i] = z == 0              ? a2[(MT - 1) * KS * 64 + r]
                   : z <= S::TEAM_L2 ? a2[(3 - S::TEAM_L2 + z - 1) * KS * 64 + r]
                                      : a1[(3 - S::TEAM_L1 + z - 1 - S::TEAM_L2) * KS * 64 + r];
        }
        buf = lds + 32 * MT + S::TEAM_TILES * KS * 256 + 4 * lane;
        hp = mb + S::LY.slotP() + (tile0 * 4 + 2) * 64 + lane;
        for (int i = threadIdx.x; i < 2 * NT * (4 * KS - MT) * 64; i += 64 * WV) {   // the offset digit
            const int z = i / 64, wd = MT + z % (4 * KS - MT), h = z / (4 * KS - MT);
            (buf - 4 * lane)[(h * KS + wd / 4) * 256 + (i % 64) * 4 + wd % 4] = 1u;
        }
        Mpinv_r = mb[S::LY.bscal() + 0];
        Minv_r = mb[S::LY.bscal() + 1];
        N_r = mk[S::LY.kscal() + 0];
        est_r = (int32_t)mk[S::LY.kscal() + 1];
#pragma unroll
        for (int b = 0; b < 4; b++) {
            kf[b] = 1 << (8 * b);
            asm volatile("" : "+s"(kf[b]));
        }
    }
    __device__ __forceinline__ void load_constants(const uint32_t *lds) {
#pragma unroll
        for (int t = 0; t < TW; t++) {
            const uint32_t *c = lds + 32 * (tile0 + t) + 8 * (lane >> 4);
            cb[t] = *(const uint4 *)c;
            cp[t] = *(const uint4 *)(c + 4);
        }
    }
    __device__ __forceinline__ void load_tiles(const gu32 *__restrict__ mb, const gu32 *__restrict__ mk) {
        gcv4i *a1 = (gcv4i *)(mk + S::LY.a1()), *a2 = (gcv4i *)(SQ ? mk + S::LY.a2s() : mb + S::LY.a2());
#pragma unroll
        for (int ks = 0; ks < KS; ks++) {
#pragma unroll
            for (int t = 0; t < TW; t++) {
                if (t < T1) A1[t < T1 ? t : 0][ks] = mfma_tile_load(a1, (tile0 + t) * KS + ks, 16u * lane);
                if (t < T2) A2[t < T2 ? t : 0][ks] = mfma_tile_load(a2, (tile0 + t) * KS + ks, 16u * lane);
            }
        }
    }
    // All digit words of this lane, as the operands of the k-steps.
    __device__ __forceinline__ void gather(int which, mfma_v4i (&w)[NT][KS]) const {
#pragma unroll
        for (int nt = 0; nt < NT; nt++)
#pragma unroll
            for (int ks = 0; ks < KS; ks++) w[nt][ks] = *(const mfma_v4i *)(buf + ((which * NT + nt) * KS + ks) * 256);
    }
    __device__ __forceinline__ void publish(int which, int t, int nt, uint32_t v) const {
        const int mt = tile0 + t;
        buf[((which * NT + nt) * KS + mt / 4) * 256 + mt % 4] = mfma_pack(v);
    }
    __device__ __forceinline__ uint32_t *shared_r(int nt) const { return buf - 3 * lane + (2 * KS * NT * 4 + nt) * 64; }
    // FULL = false: the exit product, which leaves the digits xi' in the second buffer
    template <bool FULL, class Y>
    __device__ __forceinline__ void product(const Y &y) {
        int zo;                                  // see WaveEngine::extension
        asm volatile("s_mov_b32 %0, 0" : "=s"(zo));
        const mfma_v4i *lz = lt + zo;
#pragma unroll
        for (int t = 0; t < TW; t++) {
            const uint4 c = cb[t];
#pragma unroll
            for (int nt = 0; nt < NT; nt++) {
                uint32_t xi;
                if constexpr (WIDE) xi = redc_any((uint64_t)x.b[t][nt] * y.b(t, nt), c.x, c.y);
                else if constexpr (SQ) xi = mulredc(x.b[t][nt], y.b(t, nt), c.x, 0u - c.y);
                else xi = mulredc(mulredc(x.b[t][nt], y.b(t, nt), c.x, c.y), c.w, c.x, c.y);
                if (ONCE && xi == 0) xi = cp[t].w;
                publish(0, t, nt, xi);
            }
        }
        __syncthreads();
        mfma_v4i w[NT][KS], D[TW][NT], R[NT];
        gather(0, w);
#pragma unroll
        for (int t = 0; t < TW; t++)
#pragma unroll
            for (int nt = 0; nt < NT; nt++) D[t][nt] = mfma_v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
#pragma unroll
            for (int t = 0; t < TW; t++) {
                const mfma_v4i a = t < T1 ? A1[t < T1 ? t : 0][ks] : lz[((1 + L2 + t - T1) * KS + ks) * 64];
#pragma unroll
                for (int nt = 0; nt < NT; nt++)
                    D[t][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, w[nt][ks], D[t][nt], 0, 0, 0);
            }
        uint32_t lo1[NT];
        if (wave == WV - 1)
#pragma unroll
            for (int nt = 0; nt < NT; nt++)
                lo1[nt] = (uint32_t)__builtin_amdgcn_ds_bpermute(((lane & 15) + 48) * 4, (int)mfma_combine_lo(D[TW - 1][nt]));
#pragma unroll
        for (int t = 0; t < TW; t++) {
            const uint4 c = cp[t];
            const uint64_t off = WIDE ? ((uint64_t)c.w << 32) | c.z : (uint64_t)c.x << S::OSH;
            uint32_t H = c.z;
            // the exit takes xi' = r H, whose factor the wide form has no place for
            if (WIDE && !FULL) H = ((const gu32 *)hp)[t * 4 * 64];
#pragma unroll
            for (int nt = 0; nt < NT; nt++) {
                const uint64_t T = mfma_accumulate<S::PAIR_I32>(D[t][nt], (uint64_t)x.p[t][nt] * y.p(t, nt) + off, kf);
                const uint32_t r = redc((uint32_t)T, (uint32_t)(T >> 32), c.x, c.y);
                x.p[t][nt] = r;
                publish(1, t, nt, WIDE && FULL ? r : mulredc(r, H, c.x, c.y));
            }
        }
        if (wave == WV - 1)
#pragma unroll
            for (int nt = 0; nt < NT; nt++) {
                x.r[nt] = (x.r[nt] * y.r(nt) + lo1[nt] * N_r) * Minv_r;
                *shared_r(nt) = x.r[nt];
            }
        __syncthreads();
        if constexpr (!FULL) return;
        gather(1, w);
#pragma unroll
        for (int nt = 0; nt < NT; nt++) R[nt] = mfma_v4i{0, 0, 0, 0};
#pragma unroll
        for (int t = 0; t < TW; t++)
#pragma unroll
            for (int nt = 0; nt < NT; nt++) D[t][nt] = mfma_v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
#pragma unroll
            for (int nt = 0; nt < NT; nt++)
                R[nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(lz[ks * 64], w[nt][ks], R[nt], 0, 0, 0);
#pragma unroll
        for (int ks = 0; ks < KS; ks++)
#pragma unroll
            for (int t = 0; t < TW; t++) {
                const mfma_v4i a = t < T2 ? A2[t < T2 ? t : 0][ks] : lz[((1 + t - T2) * KS + ks) * 64];
#pragma unroll
                for (int nt = 0; nt < NT; nt++)
                    D[t][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, w[nt][ks], D[t][nt], 0, 0, 0);
            }
        uint32_t al[NT], ah[NT];
#pragma unroll
        for (int nt = 0; nt < NT; nt++) {
            const uint32_t rr = *shared_r(nt);
            const uint32_t lo =
                ((uint32_t)__builtin_amdgcn_ds_bpermute(((lane & 15) + 48) * 4, (int)mfma_combine_lo(R[nt])) - rr) * Mpinv_r;
            al[nt] = lo, ah[nt] = 0;
            if constexpr (WIDE) {
                const int32_t est = __builtin_amdgcn_ds_bpermute(((lane & 15) + 32) * 4, R[nt][0]);
                const int32_t h = (est + est_r - (int32_t)(lo >> 18)) >> 14;
                ah[nt] = ((uint32_t)h << (32 - kWideShift)) + (lo >> kWideShift);
                al[nt] = lo & ((1u << kWideShift) - 1);
            }
        }
#pragma unroll
        for (int t = 0; t < TW; t++) {
            const uint4 c = cb[t];
#pragma unroll
            for (int nt = 0; nt < NT; nt++) {
                if constexpr (WIDE) {
                    const uint64_t T = mfma_accumulate<S::PAIR_I32>(
                        D[t][nt], (uint64_t)al[nt] * c.z + (uint64_t)ah[nt] * c.w, kf);
                    x.b[t][nt] = TW > S::TEAM_BASE && t == 0 ? redc_any(T, c.x, c.y) : redc_small(T, c.x, c.y);
                } else {
                    const uint64_t T = mfma_accumulate<S::PAIR_I32>(
                        D[t][nt], (uint64_t)al[nt] * c.z + ((uint64_t)c.x << S::OSH), kf);
                    x.b[t][nt] = redc((uint32_t)T, (uint32_t)(T >> 32), c.x, SQ ? 0u - c.y : c.y);
                }
            }
        }
    }
    const gu32 *hp;                            // H of this lane's slots (base table), [TW][4][64]
};

// The second operand 1 (see mstate_unit) of the tiles from tile0 on, into an
// LDS operand buffer (+ lane).
template <int K, int MT, bool SQ, int M, int NT, class E>
__device__ __forceinline__ void wave_unit(const gu32 *__restrict__ mb, const gu32 *__restrict__ mk, const E &w, int tile0,
                                          int lane, bool entry, uint32_t *y) {
    constexpr MLayout LY{K, 1, MT, NT};
#pragma unroll
    for (int t = 0; t < M; t++) {
        const int mt = tile0 + t;
        const uint32_t kap = mb[LY.slotP() + (mt * 4 + 3) * 64 + lane];
        uint32_t ub = 0u - w.slotB(t).m;
        if (SQ) ub = entry ? mk[LY.slotC() + mt * 64 + lane] : mk[LY.sqB() + (mt * 4 + 1) * 64 + lane];
#pragma unroll
        for (int nt = 0; nt < NT; nt++) {
            y[(t * NT + nt) * 64] = ub;
            y[(M * NT + t * NT + nt) * 64] = kap;
        }
    }
#pragma unroll
    for (int nt = 0; nt < NT; nt++) y[(2 * M * NT + nt) * 64] = 1u;
}

// The exponentiation of one wave's part w.x (M tiles from tile0 on) of a tile
// of job J, from the entry product to the exit product; see modexp_mfma_tile
// for the schedule.  tw: its part of the window table, + lane; yl: its LDS
// operand buffer ([2 M NT + NT][64]), which holds the second operand of every
// product but squarings: the unit, the build's constant operand, the table
// entry of a window, copied while the squarings before it run.  has_r: the wave
// keeps the redundant residue.
template <int K, int MT, bool SQ, int M, int NT, class E>
__device__ __forceinline__ void wave_exponent(const MJob &J, int e0, E &w, int tile0, int lane, gu32 *__restrict__ tw,
                                              uint32_t *yl, bool has_r) {
    constexpr size_t estride = (size_t)(2 * MT + 1) * NT * 64;
    const gu32 *__restrict__ mb = (const gu32 *)J.mb;
    const gu32 *__restrict__ mk = (const gu32 *)J.mk;
    const gu32 *__restrict__ ex = (const gu32 *)J.exp;
    MState<M, NT> &a = w.x;
    const uint32_t *y = yl + lane;
    {
        MState<M, NT> one;
        mstate_one<K, 1, MT, SQ>(mk, tile0, lane, one);
        mstate_store<M, NT>(tw, one, has_r);                     // T[0] = M mod N
    }
    const int wd = mexp_width(ex, J);
    const bool shared_exp = J.exp_stride == 0;
    const int nd = (32 * J.exp_limbs + wd - 1) / wd;
    auto dig_of = [&](int i) {
        MDigits<NT> r;
#pragma unroll
        for (int nt = 0; nt < NT; nt++) {
            const int m = e0 + 16 * nt + (lane & 15);
            r.d[nt] = mexp_digit(ex + (size_t)(m < J.batch ? m : 0) * J.exp_stride, J.exp_limbs, nd, wd, i);
        }
        return r;
    };
    enum { ENTRY, SQX, BUILD, MAIN, EXIT };
    int phase = ENTRY, j = 2, bitpos = -1, sq = 0, di = 0;
    uint32_t dm = 0;
    wave_unit<K, MT, SQ, M, NT>(mb, mk, w, tile0, lane, true, yl + lane);
    for (;;) {
        vmem_drain();                                            // a copied entry has landed
        if (phase == EXIT) {
            w.template product<false>(MLdsOperand<M, NT>{y});
            break;
        }
        w.template product<true>(MLdsOperand<M, NT>{y});
        if (phase == ENTRY) {
            mstate_store<M, NT>(tw + estride, a, has_r);         // T[1] = x
            if (wd > 1) {
                mstate_store_lds<M, NT>(yl + lane, a);
                phase = shared_exp ? SQX : BUILD;
                continue;
            }
        } else if (phase == SQX) {
            mstate_store_lds<M, NT>(yl + lane, a);               // x^2, the build's constant operand
            mstate_load<M, NT>(tw + estride, a, has_r);
            phase = BUILD;
            j = 3;
            continue;
        } else if (phase == BUILD) {
            mstate_store<M, NT>(tw + (size_t)j * estride, a, has_r);   // T[j] = T[j - step] * (x^2 or x)
            j += shared_exp ? 2 : 1;
            if (j < (1 << wd)) continue;
        }
        if (phase != MAIN) {
            phase = MAIN;
            vmem_drain();
            if (shared_exp) {
                bitpos = mexp_top_bit(ex, J.exp_limbs);
                int low = 0;
                const uint32_t t = bitpos < 0 ? 0u : mexp_window(ex, J.exp_limbs, bitpos, wd, &low);
                if (t != 1 || wd > 1) mstate_load<M, NT>(tw + (size_t)t * estride, a, has_r);   // e = 0: the result is 1
                bitpos = low - 1;
            } else {
                mstate_load_elems<M, NT>(tw, estride, dig_of(0), a, has_r);
                di = 1;
            }
            vmem_drain();
        }
        // squarings up to the next multiplication; its operand's copy starts
        // with them
        for (;;) {
            if (sq == 0) {
                if (dm) break;
                if (shared_exp) {
                    if (bitpos < 0) break;
                    if (mexp_bit(ex, bitpos)) {
                        int low;
                        dm = mexp_window(ex, J.exp_limbs, bitpos, wd, &low);
                        const gu32 *src = tw + (size_t)dm * estride;
#pragma unroll
                        for (int r = 0; r < 2 * M * NT; r++) lds_dma_row(src + r * 64, yl + r * 64);
                        if (has_r)
#pragma unroll
                            for (int r = 2 * M * NT; r < (2 * M + 1) * NT; r++) lds_dma_row(src + r * 64, yl + r * 64);
                        sq = bitpos - low + 1;
                        bitpos = low - 1;
                    } else {
                        sq = 1;
                        bitpos--;
                    }
                } else {
                    if (di >= nd) break;
                    const MDigits<NT> t = dig_of(di);
#pragma unroll
                    for (int nt = 0; nt < NT; nt++) {
                        const gu32 *src = tw + (size_t)t.d[nt] * estride;
#pragma unroll
                        for (int r = 0; r < 2 * M; r++) lds_dma_row(src + (r * NT + nt) * 64, yl + (r * NT + nt) * 64);
                        if (has_r) lds_dma_row(src + (2 * M * NT + nt) * 64, yl + (2 * M * NT + nt) * 64);
                    }
                    di++;
                    dm = 1;
                    sq = wd;
                }
            }
            w.template product<true>(MRegOperand<M, NT>{a});
            sq--;
        }
        if (dm) {
            dm = 0;
            continue;
        }
        phase = EXIT;
        wave_unit<K, MT, SQ, M, NT>(mb, mk, w, tile0, lane, false, yl + lane);
    }
}

// One tile of exponentiation job J on one wave.  lds: the workgroup's tiles; wl:
// this wave's part, for the inputs, the operands and the exit.
template <int K, int MT, int NT, int F>
__device__ __forceinline__ void modexp_wave_tile(const MJob &J, int e0, uint32_t *__restrict__ lds, uint32_t *__restrict__ wl,
                                                 uint32_t *__restrict__ table, size_t slot, int max_window) {
    using S = MShp<K, 1, MT, NT>;
    const gu32 *__restrict__ mb = (const gu32 *)J.mb;
    const gu32 *__restrict__ mk = (const gu32 *)J.mk;
    const int lane = threadIdx.x & 63;
    WaveEngine<K, MT, NT, F> w;
    w.setup(mb, mk, lds, lane);
    __syncthreads();
    const int te = mjob_tile_elems(J, S::NM);
    if (e0 >= J.batch) return;                                   // no barrier follows
    MState<MT, NT> &a = w.x;
    wave_entry<K, MT, NT>(J, e0, wl, lane, w, a);
    w.load_tiles();
    wave_exponent<K, MT, F != kPlain, MT, NT>(J, e0, w, 0, lane, (gu32 *)table + (slot << max_window) * (S::SLOTS * 64) + lane, wl, true);

    // leave the RNS (see mfma_exit)
    if constexpr (decltype(w)::WIDE) {                           // the digits xi' = r (M'_t)^-1
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
            const MSlotP sp = w.slotP(mt);
            const uint32_t H = mb[S::LY.slotP() + (mt * 4 + 2) * 64 + lane];
#pragma unroll
            for (int nt = 0; nt < NT; nt++) w.d2[nt].set(mt, mulredc(a.p[mt][nt], H, sp.m, sp.u));
        }
    }
    gcv4i *xt = (gcv4i *)(mb + S::LY.xt());
    uint64_t *tsum = (uint64_t *)wl;
    uint32_t *rl = wl + 2 * S::NM * S::XSLOTS;
    mfma_v4i D[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
        mfma_v4i t[S::KSTEPS];
#pragma unroll
        for (int ks = 0; ks < S::KSTEPS; ks++) t[ks] = mfma_tile_load(xt, mt * S::KSTEPS + ks, 16u * lane);
#pragma unroll
        for (int nt = 0; nt < NT; nt++) {
            D[mt][nt] = mfma_v4i{0, 0, 0, 0};
#pragma unroll
            for (int ks = 0; ks < S::KSTEPS; ks++)
                D[mt][nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(t[ks], w.d2[nt].w[ks], D[mt][nt], 0, 0, 0);
        }
    }
    wave_sync();
#pragma unroll
    for (int nt = 0; nt < NT; nt++) {
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
            tsum[(16 * nt + (lane & 15)) * S::XSLOTS + 4 * mt + (lane >> 4)] =
                mfma_accumulate<S::PAIR_I32>(D[mt][nt], kExitOffset, w.kf);
        if (lane < 16) rl[16 * nt + lane] = a.r[nt];
    }
    wave_sync();
    const int left = J.batch - e0, ne = left < te ? left : te;
    if constexpr (S::EXIT_LANES)
        mfma_exit_lanes<K, 1, MT, NT>(mb, mk, tsum, rl, w.Mpinv_r, lane, J, e0, ne);
    else
        mfma_exit_limbs<K, 1, MT, NT>(mb, mk, tsum, rl, w.Mpinv_r, 0, 1, lane, J, e0, ne);
}

// The same over the WV waves of a workgroup (16 elements).
template <int K, int MT, int WV, int F>
__device__ __forceinline__ void modexp_split_tile(const MJob &J, int e0, uint32_t *__restrict__ lds,
                                                  uint32_t *__restrict__ table, size_t slot, int max_window) {
    using S = MShp<K, 1, MT, 1>;
    constexpr int TW = MT / WV;
    const gu32 *__restrict__ mb = (const gu32 *)J.mb;
    const gu32 *__restrict__ mk = (const gu32 *)J.mk;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    uint32_t *yl = lds + 2 * (MT + 1) * 64 + wave * (2 * TW + 1) * 64;
    uint32_t *io = lds + 2 * (MT + 1) * 64 + WV * (2 * TW + 1) * 64;
    SplitEngine<K, MT, WV, F> w;
    w.setup(mb, mk, lds, wave, lane);
    mfma_stage_inputs<WV, 16>(J, e0, io, wave, lane);
    __syncthreads();
    {
        uint32_t mB[TW], uB[TW], mP[TW], uP[TW];
#pragma unroll
        for (int t = 0; t < TW; t++) {
            const MSlotB sb = w.slotB(t);
            const MSlotP sp = w.slotP(t);
            mB[t] = sb.m, uB[t] = sb.u, mP[t] = sp.m, uP[t] = sp.u;
        }
        mfma_entry<S::ECOLS, 4 * MT, TW, 1>(J, io, wave * TW, lane, mB, uB, mP, uP, w.x);
    }
    w.load_tiles(mb, mk);
    wave_exponent<K, MT, F != kPlain, TW, 1>(J, e0, w, wave * TW, lane,
                                    (gu32 *)table + (slot << max_window) * (S::SLOTS * 64) + wave * 2 * TW * 64 + lane,
                                    yl, wave == WV - 1);

    // leave the RNS: the last product's digits xi' are in the exchange buffer
    mfma_v4i d[S::KSTEPS], D[TW];
    w.gather(1, d);
    gcv4i *xt = (gcv4i *)(mb + S::LY.xt());
    uint64_t *tsum = (uint64_t *)io;
    uint32_t *rl = io + 2 * 16 * S::XSLOTS;
#pragma unroll
    for (int t = 0; t < TW; t++) {
        D[t] = mfma_v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < S::KSTEPS; ks++)
            D[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(mfma_tile_load(xt, (wave * TW + t) * S::KSTEPS + ks, 16u * lane),
                                                         d[ks], D[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < TW; t++)
        tsum[(lane & 15) * S::XSLOTS + 4 * (wave * TW + t) + (lane >> 4)] =
            mfma_accumulate<S::PAIR_I32>(D[t], kExitOffset, w.kf);
    if (wave == WV - 1 && lane < 16) rl[lane] = w.x.r[0];
    __syncthreads();
    const int left = J.batch - e0, te = mjob_tile_elems(J, 16);
    mfma_exit_limbs<K, 1, MT, 1>(mb, mk, tsum, rl, w.Mpinv_r, wave, WV, lane, J, e0, left < te ? left : te);
}

// One tile of exponentiation job J on a team: the part of a wave with TW tiles.
template <int K, int MT, int NT, int F, int TW>
__device__ __forceinline__ void modexp_team_tile(const MJob &J, int e0, uint32_t *__restrict__ lds,
                                                  uint32_t *__restrict__ table, size_t slot, int max_window) {
    using S = MShp<K, 1, MT, NT>;
    constexpr int WV = S::TEAM_WAVES;
    const gu32 *__restrict__ mb = (const gu32 *)J.mb;
    const gu32 *__restrict__ mk = (const gu32 *)J.mk;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    uint32_t *yl = lds + S::TEAM_OPERANDS + (2 * S::team_tile0(wave) + wave) * NT * 64;
    uint32_t *io = lds + S::TEAM_IO;
    TeamEngine<K, MT, NT, F, TW> w;
    w.setup(mb, mk, lds, wave, lane);
    mfma_stage_inputs<WV, 16 * NT>(J, e0, io, wave, lane);
    __syncthreads();
    w.load_constants(lds);
    {
        uint32_t mB[TW], uB[TW], mP[TW], uP[TW];
#pragma unroll
        for (int t = 0; t < TW; t++) {
            const MSlotB sb = w.slotB(t);
            const MSlotP sp = w.slotP(t);
            mB[t] = sb.m, uB[t] = sb.u, mP[t] = sp.m, uP[t] = sp.u;
        }
        mfma_entry<S::ECOLS, 4 * MT, TW, NT>(J, io, w.tile0, lane, mB, uB, mP, uP, w.x);
    }
    w.load_tiles(mb, mk);
    wave_exponent<K, MT, F != kPlain, TW, NT>(J, e0, w, w.tile0, lane,
                                     (gu32 *)table + (slot << max_window) * (S::SLOTS * 64) + w.tile0 * 2 * NT * 64 + lane,
                                     yl, wave == WV - 1);

    // leave the RNS: the last product's digits xi' are in the exchange buffer
    mfma_v4i d[NT][S::KSTEPS];
    w.gather(1, d);
    gcv4i *xt = (gcv4i *)(mb + S::LY.xt());
    uint64_t *tsum = (uint64_t *)io;
    uint32_t *rl = io + 2 * 16 * NT * S::XSLOTS;
#pragma unroll
    for (int t = 0; t < TW; t++) {
        mfma_v4i D[NT];
#pragma unroll
        for (int nt = 0; nt < NT; nt++) D[nt] = mfma_v4i{0, 0, 0, 0};
#pragma unroll
        for (int ks = 0; ks < S::KSTEPS; ks++) {
            const mfma_v4i a = mfma_tile_load(xt, (w.tile0 + t) * S::KSTEPS + ks, 16u * lane);
#pragma unroll
            for (int nt = 0; nt < NT; nt++) D[nt] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a, d[nt][ks], D[nt], 0, 0, 0);
        }
#pragma unroll
        for (int nt = 0; nt < NT; nt++)
            tsum[(16 * nt + (lane & 15)) * S::XSLOTS + 4 * (w.tile0 + t) + (lane >> 4)] =
                mfma_accumulate<S::PAIR_I32>(D[nt], kExitOffset, w.kf);
    }
    if (wave == WV - 1 && lane < 16)
#pragma unroll
        for (int nt = 0; nt < NT; nt++) rl[16 * nt + lane] = w.x.r[nt];
    __syncthreads();
    const int left = J.batch - e0, te = mjob_tile_elems(J, 16 * NT);
    mfma_exit_limbs<K, 1, MT, NT>(mb, mk, tsum, rl, w.Mpinv_r, wave, WV, lane, J, e0, left < te ? left : te);
}

}  // namespace rnsrsa
