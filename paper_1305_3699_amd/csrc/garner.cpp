// Garner recombination m = m_q + q ((m_p - m_q) qinv mod p) in limbs, for odd p:
// one element per wave, one limb per lane (limbs.hpp).
//
// A Montgomery product of m_p - m_q by qinv 2^(32 L) mod p and a product by q,
// each L steps of one multiplier limb times all lanes.  A step's chain of about
// 100 cycles (multiply-add, lane 0 to the scalar unit, multiply-add, the shift by
// one lane) bounds a lone element, the vector issue a batch.  The same through
// the RNS (kernels_impl.hpp: 64 elements per workgroup, one lane each for the
// entry, the limbs and the reductions) -> this: RSA-2048, one element 88 -> 4.9 us,
// 16,384 95 -> 31 us; RSA-4096, 4,096 elements 265 -> 18 us; RSA-8192, one element
// 554 -> 22 us, 1,000 600 -> 28 us.
#include "kernels.hpp"
#include "limbs.hpp"

namespace rnsrsa {

namespace {

constexpr int kGarnerWaves = 4;

template <int C>
__device__ __forceinline__ void garner_element(const GarnerLaunch &G, int e, int lane) {
    const int L = G.L;
    const uint32_t *__restrict__ lk = G.lk;
    const uint32_t *__restrict__ src = G.in + (size_t)e * (2 * L);
    uint32_t a[C], mq[C], p[C], q[C], B[C];
#pragma unroll
    for (int c = 0; c < C; c++) {
        const int l = 64 * c + lane;
        const bool in = l < L;
        a[c] = in ? src[l] : 0u;
        mq[c] = in ? src[L + l] : 0u;
        p[c] = in ? lk[l] : 0u;
        q[c] = in ? lk[L + l] : 0u;
        B[c] = in ? lk[2 * L + l] : 0u;
    }
    // a <- m_p - m_q mod 2^(32 L); no borrow leaves the carry 1 (the lanes from L
    // on hold ones and pass it)
    uint32_t nb = 1;
#pragma unroll
    for (int c = 0; c < C; c++) {
        const uint32_t u = a[c] + ~mq[c];
        const uint64_t cm = limb_carries(__ballot(u < a[c]), __ballot(u == 0xFFFFFFFFu), nb);
        a[c] = u + lane_bit(cm, lane);
    }
    uint32_t h[C];
    limbs_montmul(a, B, p, lk[4 * L], L, lane, h);
    if (!nb) {                                               // minus 2^(32 L) qinv = B
        uint32_t d[C];
#pragma unroll
        for (int c = 0; c < C; c++) d[c] = 64 * c + lane < L ? lk[3 * L + 64 * c + lane] : 0u;   // p - B
        const uint32_t over = limbs_add(h, d, lane);
        limbs_reduce_once(h, p, lane, over);
    }
    // m = m_q + h q, its low limbs one per step
    uint32_t lo[C];
    uint64_t t[C], u[C];
#pragma unroll
    for (int c = 0; c < C; c++) {
        t[c] = mq[c];
        lo[c] = 0;
    }
#pragma unroll
    for (int k = 0; k < C; k++)
        for (int i = 0; i < 64 && 64 * k + i < L; i++) {
            const uint32_t x = (uint32_t)__builtin_amdgcn_readlane((int)h[k], i);
#pragma unroll
            for (int c = 0; c < C; c++) u[c] = (uint64_t)x * q[c] + (uint32_t)t[c];
            const uint32_t w = low_limb(u);
            if (lane == i) lo[k] = w;
            shift_step<C, false>(u, u, t);
        }
    uint32_t hi[C];
    limbs_of_sums(t, hi, lane);
    uint32_t *__restrict__ out = G.out + (size_t)e * G.out_stride;
#pragma unroll
    for (int c = 0; c < C; c++) {
        const int l = 64 * c + lane;
        if (l < L && l < G.out_limbs) out[l] = lo[c];
        if (l < L && L + l < G.out_limbs) out[L + l] = hi[c];
    }
}

template <int C>
__global__ __launch_bounds__(64 * kGarnerWaves) void garner_limbs_kernel(GarnerLaunch G) {
    const int e = (int)blockIdx.x * kGarnerWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (e < G.batch) garner_element<C>(G, e, threadIdx.x & 63);
}

// Grouped: workgroup t serves the job j with jobs[j].tile0 <= t < jobs[j+1].tile0.
template <int C>
__global__ __launch_bounds__(64 * kGarnerWaves) void garner_limbs_jobs_kernel(const GJob *__restrict__ jobs, int njobs) {
    const int t = blockIdx.x;
    int lo = 0, hi = njobs - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (jobs[mid].tile0 <= t) lo = mid; else hi = mid - 1;
    }
    const GJob J = jobs[lo];
    const int e = (t - J.tile0) * kGarnerWaves + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (e < J.g.batch) garner_element<C>(J.g, e, threadIdx.x & 63);
}

}  // namespace

int garner_limbs_tiles(size_t elements) { return (int)((elements + kGarnerWaves - 1) / kGarnerWaves); }

hipError_t launch_garner_limbs(const GarnerLaunch &a, hipStream_t s) {
    const dim3 g((unsigned)garner_limbs_tiles((size_t)a.batch)), b(64 * kGarnerWaves);
    if (a.batch <= 0) return hipSuccess;
    if (a.L <= 64) hipLaunchKernelGGL(garner_limbs_kernel<1>, g, b, 0, s, a);
    else if (a.L <= 128) hipLaunchKernelGGL(garner_limbs_kernel<2>, g, b, 0, s, a);
    else if (a.L <= kGarnerLimbs) hipLaunchKernelGGL(garner_limbs_kernel<4>, g, b, 0, s, a);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_garner_limbs_jobs(int max_limbs, const GJob *jobs, int njobs, int tiles, hipStream_t s) {
    const dim3 g((unsigned)tiles), b(64 * kGarnerWaves);
    if (tiles <= 0) return hipSuccess;
    if (max_limbs <= 64) hipLaunchKernelGGL(garner_limbs_jobs_kernel<1>, g, b, 0, s, jobs, njobs);
    else if (max_limbs <= 128) hipLaunchKernelGGL(garner_limbs_jobs_kernel<2>, g, b, 0, s, jobs, njobs);
    else if (max_limbs <= kGarnerLimbs) hipLaunchKernelGGL(garner_limbs_jobs_kernel<4>, g, b, 0, s, jobs, njobs);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

}  // namespace rnsrsa
