// Primality steps of key generation on the GPU (include/rnsrsa.h): trial
// division by the first small primes (Sec. 4.3) and Miller-Rabin tests whose
// exponentiations run in RNS in the Montgomery domain (Sec. 3.2), one
// modulus per candidate, all candidates in grouped launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <thread>
#include <tuple>
#include <vector>

#include "bn_host.hpp"
#include "jobs.hpp"
#include "kernels_impl.hpp"
#include "mr_gpu.hpp"

using namespace rnsrsa;
using namespace rnsrsa::api;

namespace {

constexpr int kMaxSmallPrimes = 10000;   // the 10,000th prime is 104729
constexpr int kMaxRounds = 64;

// The first `count` primes, sieve of Eratosthenes below 104730.
std::vector<uint32_t> first_primes(int count) {
    const uint32_t bound = 104730;
    std::vector<uint8_t> composite(bound, 0);
    std::vector<uint32_t> out;
    for (uint32_t i = 2; i < bound && (int)out.size() < count; i++) {
        if (composite[i]) continue;
        out.push_back(i);
        for (uint64_t j = (uint64_t)i * i; j < bound; j += i) composite[j] = 1;
    }
    return out;
}

constexpr int kTdThreads = 256;
constexpr int kTdBlock = 32;        // limbs whose powers the table holds
constexpr int kTdGroup = 8;         // candidates that share one read of the table
constexpr int kTdMaxList = 512;     // most candidates of a second-pass workgroup
constexpr int kTdPad = (kMaxSmallPrimes + kTdThreads - 1) / kTdThreads * kTdThreads;

// Tables of the small primes p, [kTdPad] per row (padding never read back):
// a value x is divisible by p exactly when x inv mod 2^64 <= lim, with inv =
// p^-1 mod 2^64 and lim = (2^64 - 1) / p for odd p, and inv = 2^63, lim = 0 for 2.
struct SmallPrimes {
    uint32_t *p = nullptr;     // the primes
    uint32_t *pw = nullptr;    // [kTdBlock][kTdPad] 2^(32 l) mod p
    uint32_t *blk = nullptr;   // 2^(32 kTdBlock) mod p
    uint64_t *inv = nullptr, *lim = nullptr;
};

// One set per device, kept for the life of the process.
int small_primes(int dev, SmallPrimes *out) {
    static std::mutex mu;
    static std::map<int, SmallPrimes> tables;
    std::lock_guard<std::mutex> lk(mu);
    auto it = tables.find(dev);
    if (it == tables.end()) {
        const std::vector<uint32_t> pr = first_primes(kMaxSmallPrimes);
        std::vector<uint32_t> words((size_t)kTdPad * (kTdBlock + 2), 0u);
        std::vector<uint64_t> wide((size_t)kTdPad * 2, 0u);
        for (size_t i = 0; i < pr.size(); i++) {
            const uint32_t p = pr[i];
            words[i] = p;
            uint64_t v = 1;
            for (int l = 0; l <= kTdBlock; l++) {
                words[(size_t)(l + 1) * kTdPad + i] = (uint32_t)v;
                v = (v << 32) % p;
            }
            uint64_t inv = p;                       // p p = 1 mod 8: three bits, doubled by each step
            for (int k = 0; k < 5; k++) inv *= 2 - p * inv;
            wide[i] = p == 2 ? 1ull << 63 : inv;
            wide[(size_t)kTdPad + i] = p == 2 ? 0 : ~0ull / p;
        }
        uint32_t *dw = nullptr;
        uint64_t *dd = nullptr;
        hipError_t e = hipMalloc((void **)&dw, words.size() * sizeof(uint32_t));
        if (e == hipSuccess) e = hipMalloc((void **)&dd, wide.size() * sizeof(uint64_t));
        if (e == hipSuccess) e = hipMemcpy(dw, words.data(), words.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipMemcpy(dd, wide.data(), wide.size() * sizeof(uint64_t), hipMemcpyHostToDevice);
        if (e != hipSuccess) {
            if (dw) hipFree(dw);
            if (dd) hipFree(dd);
            return hip_fail(e, "small-prime tables");
        }
        SmallPrimes t;
        t.p = dw;
        t.pw = dw + kTdPad;
        t.blk = dw + (size_t)kTdPad * (kTdBlock + 1);
        t.inv = dd;
        t.lim = dd + kTdPad;
        it = tables.emplace(dev, t).first;
    }
    *out = it->second;
    return RNS_OK;
}

struct TdArgs {
    const uint32_t *cand;
    uint8_t *flags;
    SmallPrimes sp;
    int limbs, count;
    int p0, p1;      // the pass's primes
    int span;        // second pass: candidates per workgroup
};

// Limbs are read through the constant address space at uniform addresses:
// scalar loads, whose results are scalar operands of the multiply-adds.
typedef const __attribute__((address_space(4))) uint32_t td_cu32;

// Bit g: prime number t divides candidate list[g] (of n <= kTdGroup) and
// differs from it.
//
// The sum over the limbs of limb x (2^(32 l) mod p): p < 2^17, so each product
// stays below 2^49 and 32 of them below 2^54, one carry-free multiply-add per
// limb instead of a division step.  Longer rows are taken 32 limbs at a time
// from the top; the sum so far is folded to 33 bits (2^32 mod p is a power of
// the table too) and multiplied by 2^1024 mod p in between.  Eight powers are
// in registers at a time and serve kTdGroup candidates (16 of them spilled
// scalar registers).  Bound by the multiply-adds (35 T/s for the whole GPU) and
// the scalar loads between them: 20,000 random odd 1024-bit candidates and
// 10,000 primes take 79 us, against 3,450 us with a double-precision division
// step per limb and prime and no second pass.
__device__ __forceinline__ uint32_t td_group(const TdArgs &A, int t, const int *list, int n) {
    td_cu32 *row[kTdGroup];
    uint64_t acc[kTdGroup];
#pragma unroll
    for (int g = 0; g < kTdGroup; g++) {
        const int i = __builtin_amdgcn_readfirstlane(list[g < n ? g : 0]);
        row[g] = (td_cu32 *)A.cand + (size_t)i * A.limbs;
        acc[g] = 0;
    }
    const uint32_t *__restrict__ pw = A.sp.pw + t;
    for (int l0 = (A.limbs - 1) / kTdBlock * kTdBlock; l0 >= 0; l0 -= kTdBlock) {
        if (l0 + kTdBlock < A.limbs) {
            const uint32_t c1 = pw[kTdPad], cb = A.sp.blk[t];
#pragma unroll
            for (int g = 0; g < kTdGroup; g++) {
                uint64_t v = acc[g];
                v = (v >> 32) * c1 + (uint32_t)v;        // below 2^44
                v = (v >> 32) * c1 + (uint32_t)v;        // below 2^33
                acc[g] = v * cb;
            }
        }
        const int nl = A.limbs - l0 < kTdBlock ? A.limbs - l0 : kTdBlock;
        int l = 0;
        for (; l + 8 <= nl; l += 8) {
            uint32_t c[8];
#pragma unroll
            for (int z = 0; z < 8; z++) c[z] = pw[(size_t)(l + z) * kTdPad];
#pragma unroll
            for (int g = 0; g < kTdGroup; g++)
#pragma unroll
                for (int z = 0; z < 8; z++) acc[g] += (uint64_t)row[g][l0 + l + z] * c[z];
        }
        for (; l < nl; l++) {
            const uint32_t c = pw[(size_t)l * kTdPad];
#pragma unroll
            for (int g = 0; g < kTdGroup; g++) acc[g] += (uint64_t)row[g][l0 + l] * c;
        }
    }
    const uint64_t inv = A.sp.inv[t], lim = A.sp.lim[t];
    uint32_t mask = 0;
#pragma unroll
    for (int g = 0; g < kTdGroup; g++) mask |= acc[g] * inv <= lim ? 1u << g : 0u;
    mask &= (1u << n) - 1u;
    for (uint32_t left = mask; left; left &= left - 1) {      // rare: is it the prime itself?
        const int g = __builtin_ctz(left);
        const uint32_t *__restrict__ x = A.cand + (size_t)list[g] * A.limbs;
        bool same = x[0] == A.sp.p[t];
        for (int l = 1; same && l < A.limbs; l++) same = x[l] == 0;
        if (same) mask &= ~(1u << g);
    }
    return mask;
}

// Trial division in two passes, in one for few primes.  First pass (blockIdx.x:
// kTdGroup candidates): the first kTdThreads primes (or all), which find a factor in about 85% of random odd
// candidates; writes every flag.  Second pass (blockIdx.x: span candidates,
// blockIdx.y: kTdThreads further primes): only the candidates still flagged,
// compacted in LDS; clears the flags of those it finds a factor of.
__global__ __launch_bounds__(kTdThreads) void trial_first_kernel(TdArgs A) {
    __shared__ int list[kTdGroup];
    __shared__ uint32_t found;
    const int c0 = blockIdx.x * kTdGroup;
    const int n = A.count - c0 < kTdGroup ? A.count - c0 : kTdGroup;
    if (threadIdx.x < kTdGroup) list[threadIdx.x] = c0 + threadIdx.x;
    if (threadIdx.x == 0) found = 0;
    __syncthreads();
    for (int t = A.p0 + (int)threadIdx.x; t < A.p1; t += kTdThreads) {
        const uint32_t mask = td_group(A, t, list, n);
        if (mask) atomicOr(&found, mask);
    }
    __syncthreads();
    if ((int)threadIdx.x < n) A.flags[c0 + threadIdx.x] = (found >> threadIdx.x) & 1u ? 0 : 1;
}

__global__ __launch_bounds__(kTdThreads) void trial_rest_kernel(TdArgs A) {
    __shared__ int list[kTdMaxList];
    __shared__ int n_list;
    if (threadIdx.x == 0) n_list = 0;
    __syncthreads();
    const int c0 = blockIdx.x * A.span;
    for (int i = threadIdx.x; i < A.span; i += kTdThreads)
        if (c0 + i < A.count && A.flags[c0 + i]) list[atomicAdd(&n_list, 1)] = c0 + i;
    __syncthreads();
    const int t = A.p0 + (int)(blockIdx.y * kTdThreads + threadIdx.x), n = n_list;
    if (t >= A.p1) return;
    for (int i = 0; i < n; i += kTdGroup) {
        const int m = n - i < kTdGroup ? n - i : kTdGroup;
        uint32_t mask = td_group(A, t, list + i, m);
        while (mask) {
            A.flags[list[i + __builtin_ctz(mask)]] = 0;
            mask &= mask - 1;
        }
    }
}

struct Candidate {
    std::unique_ptr<rns_ctx> ctx;
    Limbs nm1;       // N - 1
    int s = 0;       // N - 1 = 2^s d, d odd
    Limbs d;
};

// Launch x <- x^e (mod each candidate's N) for the listed candidates, x rows
// of `rounds` elements in place; exponent e: per candidate (exps, L limbs
// each) or the shared `shared_exp` of one limb.
int exponentiate(const std::vector<Candidate> &cs, const std::vector<size_t> &which, uint32_t *d_x,
                 const uint32_t *d_exps, const uint32_t *d_shared_exp, uint32_t shared_exp, int L, int rounds,
                 hipStream_t s, std::vector<std::unique_ptr<Scratch>> &keep,
                 std::vector<std::vector<MJob>> &host_jobs) {
    std::map<std::tuple<int, int, int>, JobGroup> groups;
    for (size_t i : which) {
        const rns_ctx *c = cs[i].ctx.get();
        uint32_t *x = d_x + i * (size_t)rounds * L;
        const bool shared = d_exps == nullptr;
        const uint32_t *exp = shared ? d_shared_exp : d_exps + i * (size_t)L;
        const int exp_limbs = shared ? 1 : L;
        if (c->engine != RNS_ENGINE_MATRIX) {
            int rc = run_modexp(c, nullptr, entry_of(c), nullptr, x, L, exp, nullptr, exp_limbs, 0, x, nullptr, L,
                                (size_t)rounds, s);
            if (rc) return rc;
            continue;
        }
        const MLayout &sh = c->mshape;
        JobGroup &g = groups[std::make_tuple(sh.K, sh.W, sh.MT)];
        if (g.jobs.empty()) {
            g.shape = sh;
            g.device = c->device;
        }
        g.take_form(c->mform);
        const std::vector<uint32_t> eh = shared ? std::vector<uint32_t>{shared_exp} : cs[i].d;
        PlannedJob J{};
        J.j.mb = c->d_mbase;
        J.j.mk = c->d_mkey;
        J.j.E = c->d_mentry;
        J.j.exp = exp;
        J.j.in = x;
        J.j.out = x;
        J.j.batch = rounds;
        J.j.in_limbs = L;
        J.j.in_stride = L;
        J.j.L = c->plan.L;
        J.j.out_stride = L;
        J.j.exp_limbs = exp_limbs;
        J.j.exp_stride = 0;
        J.j.window = best_window(eh, 0);
        J.cost = mm_count(eh, J.j.window);
        g.jobs.push_back(J);
    }
    for (auto &kv : groups) {
        JobGroup &g = kv.second;
        finish_group(g);
        retile_group(g, g.device);
        // the job table's host copy lives until the caller synchronises
        host_jobs.emplace_back();
        std::vector<MJob> &js = host_jobs.back();
        for (const PlannedJob &J : g.jobs) js.push_back(J.j);
        keep.emplace_back(new Scratch);
        Scratch &jt = *keep.back();
        int rc = scratch_alloc(jt, js.size() * sizeof(MJob), s);
        if (rc) return rc;
        hipError_t e = hipMemcpyAsync(jt.p, js.data(), js.size() * sizeof(MJob), hipMemcpyHostToDevice, s);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");
        keep.emplace_back(new Scratch);
        Scratch &tb = *keep.back();
        if ((rc = scratch_alloc(tb, g.table_words() * sizeof(uint32_t), s))) return rc;
        if ((e = launch_group(g, (const MJob *)jt.p, (uint32_t *)tb.p, s)) != hipSuccess)
            return hip_fail(e, "grouped modexp launch");
    }
    return RNS_OK;
}

// Arazi's inversion in RNS (Sec. 3.1): d = (1 + f t) / e with t = -f^-1 mod e
// (a scalar), channel by channel on the owned B' channels and the redundant
// one: d_j = (1 + f_j t) e^-1 mod m'_j, then d in binary through the base's
// exit (CRT over B' with alpha from the redundant channel; exact since
// d < n).  One element per lane (f of fl limbs, d of L limbs).
template <int K, int W>
__global__ __launch_bounds__(64 * W) void arazi_kernel(const uint32_t *__restrict__ bc, const uint32_t *__restrict__ mc,
                                                       const uint32_t *__restrict__ f, int fl, uint32_t t, uint32_t e,
                                                       uint32_t einv32, int L, uint32_t *__restrict__ d, int batch) {
    using S = Shp<K, W>;
    constexpr int KS = S::KS, KP = S::KP;
    constexpr Layout LY{K, KP};
    __shared__ uint32_t lds[2 * KP * 64];
    uint32_t *xip = lds + KP * 64;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    const int msg = blockIdx.x * 64 + lane;
    const bool active = msg < batch;
    const uint32_t *__restrict__ fr = f + (size_t)(active ? msg : 0) * fl;
    for (int c = 0; c < KS; c++) {
        const int j = wave * KS + c;
        if (j >= K) break;
        const uint32_t m = bc[LY.mBp() + j];
        uint64_t r = 0;
        for (int l = fl - 1; l >= 0; l--) r = ((r << 32) | fr[l]) % m;
        // e^-1 mod m' by Fermat (m' prime, e not a multiple of it)
        uint64_t inv = 1, b = e % m;
        for (uint32_t x = m - 2; x; x >>= 1) {
            if (x & 1u) inv = inv * b % m;
            b = b * b % m;
        }
        const uint64_t dj = (1 + r * t % m) % m * inv % m;
        xip[j * 64 + lane] = mulredc((uint32_t)dj, bc[LY.MpInv() + j], m, bc[LY.uBp() + j]);   // d_j (M'_j)^-1
    }
    const uint32_t dr = (1u + fr[0] * t) * einv32;                                               // d mod 2^32
    __syncthreads();
    uint64_t s2 = 0;
    for (int j = 0; j < K; j++) s2 += (uint64_t)xip[j * 64 + lane] * bc[LY.C2() + j * LY.crow() + KP];
    const uint32_t alpha = ((uint32_t)s2 - dr) * bc[LY.scal()];
    __syncthreads();
    if (wave != 0) return;
    rns_exit<K, W>(bc, mc, lds, lds + (L + 1) * 64, xip, alpha, L, lane);
    if (active)
        for (int l = 0; l < L; l++) d[(size_t)msg * L + l] = lds[l * 64 + lane];
}

// d = e^-1 mod f by arazi_kernel on the channel tables of context c (whose
// modulus exceeds f).  Returns RNS_OK or the error code (also recorded for
// rns_last_error).
int arazi_inverse(const rns_ctx *c, const Limbs &f, uint32_t e, Limbs &d, hipStream_t s) {
    const int K = c->plan.base->K, W = c->plan.base->W, L = c->plan.L;
    for (uint32_t m : c->plan.base->Bp)
        if (e % m == 0) return fail(RNS_EUNSUPPORTED, "e is a channel prime");
    const uint32_t fe = bn_mod_word(f, e), fi = invmod32(fe, e);
    if (!fi) return fail(RNS_EINVAL, "e not coprime to (p-1)(q-1)");
    const uint32_t t = (e - fi) % e;
    Limbs fl = f;
    fl.resize((size_t)L, 0u);
    Scratch df, dd;
    int rc = scratch_alloc(df, (size_t)L * sizeof(uint32_t), s);
    if (!rc) rc = scratch_alloc(dd, (size_t)L * sizeof(uint32_t), s);
    if (rc) return rc;
    hipError_t he = hipMemcpyAsync(df.p, fl.data(), (size_t)L * sizeof(uint32_t), hipMemcpyHostToDevice, s);
    if (he != hipSuccess) return hip_fail(he, "hipMemcpyAsync");
    bool launched = false;
#define RNSRSA_SHAPE(k, w)                                                                                        \
    if (!launched && K == k && W == w) {                                                                      \
        hipLaunchKernelGGL((arazi_kernel<k, w>), dim3(1), dim3(64 * w), 0, s, c->d_base, c->d_mod,              \
                           (const uint32_t *)df.p, L, t, e, inv2_32(e), L, (uint32_t *)dd.p, 1);               \
        launched = true;                                                                                          \
    }
#include "kernel_configs.inc"
#undef RNSRSA_SHAPE
    if (!launched) return fail(RNS_EUNSUPPORTED, "no channel kernel for this k");
    if ((he = hipGetLastError()) != hipSuccess) return hip_fail(he, "arazi launch");
    d.assign((size_t)L, 0u);
    if ((he = hipMemcpyAsync(d.data(), dd.p, (size_t)L * sizeof(uint32_t), hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (he = hipStreamSynchronize(s)) != hipSuccess)
        return hip_fail(he, "arazi read-back");
    bn_trim(d);
    return RNS_OK;
}

// a^-1 mod p for odd p > 1 by the binary extended Euclidean algorithm
// (invariants x1 a = u and x2 a = v mod p); false when gcd(a, p) > 1.
bool bn_modinv_odd(const Limbs &a, const Limbs &p, Limbs &out) {
    const Limbs one{1};
    Limbs u = bn_mod(a, p), v = p, x1 = one, x2;
    auto half = [&](Limbs &x) {
        if (bn_low(x) & 1u) x = bn_add(x, p);
        x = bn_shr1(x);
    };
    auto sub_mod = [&](const Limbs &x, const Limbs &y) {
        return bn_cmp(x, y) >= 0 ? bn_sub(x, y) : bn_sub(bn_add(x, p), y);
    };
    if (bn_is_zero(u)) return false;
    while (bn_cmp(u, one) != 0 && bn_cmp(v, one) != 0) {
        while (!(bn_low(u) & 1u)) {
            u = bn_shr1(u);
            half(x1);
        }
        while (!(bn_low(v) & 1u)) {
            v = bn_shr1(v);
            half(x2);
        }
        if (bn_cmp(u, v) >= 0) {
            u = bn_sub(u, v);
            x1 = sub_mod(x1, x2);
        } else {
            v = bn_sub(v, u);
            x2 = sub_mod(x2, x1);
        }
        if (bn_is_zero(u) || bn_is_zero(v)) return false;
    }
    out = bn_cmp(u, one) == 0 ? x1 : x2;
    return true;
}

// 2 <= a <= N - 2, for odd N: a is none of 0, 1 and N - 1 and below N.
bool valid_base(const uint32_t *a, const uint32_t *N, int L) {
    int l = L - 1;
    while (l > 0 && a[l] == N[l]) l--;
    if (l == 0 ? a[0] + (uint64_t)1 >= N[0] : a[l] >= N[l]) return false;   // above it only limb 0 differs
    for (l = L - 1; l > 0; l--)
        if (a[l]) return true;
    return a[0] >= 2;
}

bool rows_equal(const uint32_t *a, const Limbs &b, int L) {
    for (int l = 0; l < L; l++)
        if (a[l] != (l < (int)b.size() ? b[l] : 0u)) return false;
    return true;
}

}  // namespace

extern "C" {

int rsa_trial_division(const uint32_t *cand, size_t count, int limbs, int n_primes, uint8_t *flags,
                       void *hip_stream) {
    if (count == 0) return ok();
    if (!cand || !flags) return fail(RNS_EINVAL, "null buffer");
    if (limbs <= 0 || limbs > 4096) return fail(RNS_EINVAL, "limbs must be in 1..4096");
    if (n_primes <= 0 || n_primes > kMaxSmallPrimes) return fail(RNS_EINVAL, "n_primes must be in 1..10000");
    if (count > (size_t)INT32_MAX) return fail(RNS_EINVAL, "count too large");
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "hipGetDevice");
    SmallPrimes sp;
    int rc = RNS_OK;
    try {
        rc = small_primes(dev, &sp);
    } catch (const std::bad_alloc &) {
        rc = fail(RNS_ENOMEM, "out of host memory");
    }
    if (rc) return rc;
    TdArgs a{};
    a.cand = cand;
    a.flags = flags;
    a.sp = sp;
    a.limbs = limbs;
    a.count = (int)count;
    a.p0 = 0;
    // up to 512 primes in the first pass, two rounds at most (100 1024-bit candidates by
    // 500 primes 8.2 us, with a second pass 11.1; 20,000 22 us; three rounds for 768
    // primes 31 us, with a second pass 26)
    a.p1 = n_primes <= 2 * kTdThreads ? n_primes : kTdThreads;
    hipLaunchKernelGGL(trial_first_kernel, dim3((unsigned)((count + kTdGroup - 1) / kTdGroup)), dim3(kTdThreads), 0,
                       (hipStream_t)hip_stream, a);
    if (a.p1 < n_primes) {
        // about 15% of the candidates are left: 512 per workgroup fill about
        // ten groups of 8; fewer candidates are spread wider instead (128 and 512 per
        // workgroup, 1024-bit candidates: 1,000 17.6 and 31 us, 20,000 72.6 and 76.8,
        // 40,000 131.7 and 130.0, 100,000 303 and 268; the same at 64 to 4,096 bits)
        a.p0 = kTdThreads;
        a.p1 = n_primes;
        a.span = count >= 32768 ? kTdMaxList : 128;
        hipLaunchKernelGGL(trial_rest_kernel,
                           dim3((unsigned)((count + a.span - 1) / a.span),
                                (unsigned)((n_primes - kTdThreads + kTdThreads - 1) / kTdThreads)),
                           dim3(kTdThreads), 0, (hipStream_t)hip_stream, a);
    }
    if ((e = hipGetLastError()) != hipSuccess) return hip_fail(e, "trial division launch");
    return ok();
}

int rsa_miller_rabin(const uint32_t *cand, size_t count, int limbs, const uint32_t *bases, int rounds,
                     uint8_t *verdict, void *hip_stream) {
    if (count == 0) return ok();
    if (!cand || !bases || !verdict) return fail(RNS_EINVAL, "null buffer");
    if (limbs <= 0 || limbs > 4096) return fail(RNS_EINVAL, "limbs must be in 1..4096");
    if (rounds <= 0 || rounds > kMaxRounds) return fail(RNS_EINVAL, "rounds must be in 1..64");
    if (count > (size_t)INT32_MAX / kMaxRounds) return fail(RNS_EINVAL, "count too large");
    hipStream_t s = (hipStream_t)hip_stream;
    const int L = limbs;
    const size_t row = (size_t)rounds * L;
    try {
        for (size_t i = 0; i < count; i++) {
            const uint32_t *N = cand + i * L;
            int n = L;
            while (n > 0 && N[n - 1] == 0) n--;
            if (n == 0 || !(N[0] & 1u) || (n == 1 && N[0] <= 3)) return fail(RNS_EINVAL, "candidates must be odd and > 3");
            for (int r = 0; r < rounds; r++)
                if (!valid_base(bases + i * row + (size_t)r * L, N, L)) return fail(RNS_EINVAL, "bases must lie in [2, N - 2]");
        }
        // every candidate's tables built on the device when its base runs on
        // the matrix engine (the default bases do)
        {
            const int grc = miller_rabin_gpu(cand, count, L, bases, rounds, verdict, s);
            if (grc != RNS_EUNSUPPORTED) return grc ? grc : ok();
        }
        std::vector<Candidate> cs(count);
        for (size_t i = 0; i < count; i++) {
            Limbs N = bn_from_ptr(cand + i * L, (size_t)L);
            bn_trim(N);
            Candidate &c = cs[i];
            c.nm1 = bn_sub(N, Limbs{1});
            c.d = c.nm1;
            while (bn_low(c.d) % 2 == 0) {
                c.d = bn_shr1(c.d);
                c.s++;
            }
            c.d.resize((size_t)L, 0u);
        }
        // otherwise one context per candidate, built on a pool of host
        // threads (each on the caller's device); errors are reported on this
        // thread
        int dev = 0;
        hipError_t de = hipGetDevice(&dev);
        if (de != hipSuccess) return hip_fail(de, "hipGetDevice");
        std::vector<int> crc(count, RNS_OK);
        std::atomic<size_t> next{0};
        auto work = [&] {
            if (hipSetDevice(dev) != hipSuccess) return;
            for (size_t i; (i = next.fetch_add(1)) < count;) {
                Limbs N = bn_from_ptr(cand + i * L, (size_t)L);
                bn_trim(N);
                rns_ctx *ctx = nullptr;
                crc[i] = make_context(N, L, &ctx);
                cs[i].ctx.reset(ctx);
            }
        };
        const unsigned nthreads =
            (unsigned)std::min<size_t>(count, std::min(16u, std::max(1u, std::thread::hardware_concurrency())));
        std::vector<std::thread> pool;
        for (unsigned t = 1; t < nthreads; t++) pool.emplace_back(work);
        work();
        for (std::thread &t : pool) t.join();
        for (size_t i = 0; i < count; i++) {
            if (crc[i] == RNS_OK && !cs[i].ctx) crc[i] = RNS_EDEVICE;
            if (crc[i] != RNS_OK) return fail(crc[i], "context set-up failed for candidate " + std::to_string(i));
        }
        // device: per-candidate exponents d, the rows of x (the bases first)
        std::vector<uint32_t> hd(count * (size_t)L);
        for (size_t i = 0; i < count; i++) std::copy(cs[i].d.begin(), cs[i].d.end(), hd.begin() + i * L);
        Scratch d_exps, d_x, d_two;
        int rc = scratch_alloc(d_exps, hd.size() * sizeof(uint32_t), s);
        if (!rc) rc = scratch_alloc(d_x, count * row * sizeof(uint32_t), s);
        if (!rc) rc = scratch_alloc(d_two, sizeof(uint32_t), s);
        if (rc) return rc;
        const uint32_t two = 2;
        hipError_t e = hipMemcpyAsync(d_exps.p, hd.data(), hd.size() * sizeof(uint32_t), hipMemcpyHostToDevice, s);
        if (e == hipSuccess)
            e = hipMemcpyAsync(d_x.p, bases, count * row * sizeof(uint32_t), hipMemcpyHostToDevice, s);
        if (e == hipSuccess) e = hipMemcpyAsync(d_two.p, &two, sizeof(uint32_t), hipMemcpyHostToDevice, s);
        if (e != hipSuccess) return hip_fail(e, "hipMemcpyAsync");

        // state per (candidate, base): 0 undecided, 1 passed, 2 failed
        std::vector<uint8_t> st(count * (size_t)rounds, 0);
        std::vector<uint32_t> hx(count * row);
        std::vector<std::unique_ptr<Scratch>> keep;
        std::vector<std::vector<MJob>> host_jobs;
        std::vector<size_t> which(count);
        for (size_t i = 0; i < count; i++) which[i] = i;
        for (int j = 0; !which.empty(); j++) {
            // j = 0: x = a^d; j > 0: x = x^2
            rc = j == 0 ? exponentiate(cs, which, (uint32_t *)d_x.p, (const uint32_t *)d_exps.p, nullptr, 0, L,
                                       rounds, s, keep, host_jobs)
                        : exponentiate(cs, which, (uint32_t *)d_x.p, nullptr, (const uint32_t *)d_two.p, 2u, L,
                                       rounds, s, keep, host_jobs);
            if (rc) return rc;
            if ((e = hipMemcpyAsync(hx.data(), d_x.p, hx.size() * sizeof(uint32_t), hipMemcpyDeviceToHost, s)) !=
                    hipSuccess ||
                (e = hipStreamSynchronize(s)) != hipSuccess)
                return hip_fail(e, "miller-rabin read-back");
            keep.clear();
            host_jobs.clear();
            std::vector<size_t> next;
            for (size_t i : which) {
                const Candidate &c = cs[i];
                bool open = false;
                for (int r = 0; r < rounds; r++) {
                    uint8_t &z = st[i * rounds + r];
                    if (z) continue;
                    const uint32_t *x = hx.data() + i * row + (size_t)r * L;
                    if (rows_equal(x, c.nm1, L) || (j == 0 && rows_equal(x, Limbs{1}, L)))
                        z = 1;                                      // a^(2^j d) = -1, or a^d = 1
                    else if (j > 0 && rows_equal(x, Limbs{1}, L))
                        z = 2;                                      // 1 reached without passing -1
                    else if (j + 1 >= c.s)
                        z = 2;                                      // no square left to reach -1
                    if (!z) open = true;
                }
                if (open) next.push_back(i);
            }
            which.swap(next);
        }
        for (size_t i = 0; i < count; i++) {
            uint8_t v = 1;
            for (int r = 0; r < rounds; r++) v &= st[i * rounds + r] == 1;
            verdict[i] = v;
        }
    } catch (const std::bad_alloc &) {
        return fail(RNS_ENOMEM, "out of host memory");
    }
    return ok();
}


}  // extern "C"

namespace {

constexpr size_t kMrChunk = 64;

// The first candidate of a stream (host, count x L limbs, in order) that
// passes trial division on the GPU, has gcd(e, c - 1) = 1, differs from
// `exclude` and passes Miller-Rabin with its bases (chunks of up to 64
// eligible candidates, in order).
int first_prime(const uint32_t *cand, const uint32_t *bases, size_t count, int L, int rounds, uint32_t e,
                const Limbs &exclude, hipStream_t s, Limbs &out) {
    Scratch dc, df;
    int rc = scratch_alloc(dc, count * (size_t)L * sizeof(uint32_t), s);
    if (!rc) rc = scratch_alloc(df, count, s);
    if (rc) return rc;
    hipError_t he = hipMemcpyAsync(dc.p, cand, count * (size_t)L * sizeof(uint32_t), hipMemcpyHostToDevice, s);
    if (he != hipSuccess) return hip_fail(he, "hipMemcpyAsync");
    if ((rc = rsa_trial_division((const uint32_t *)dc.p, count, L, kMaxSmallPrimes, (uint8_t *)df.p, s))) return rc;
    std::vector<uint8_t> flags(count);
    if ((he = hipMemcpyAsync(flags.data(), df.p, count, hipMemcpyDeviceToHost, s)) != hipSuccess ||
        (he = hipStreamSynchronize(s)) != hipSuccess)
        return hip_fail(he, "trial division read-back");
    std::vector<size_t> elig;
    for (size_t i = 0; i < count; i++) {
        if (!flags[i]) continue;
        Limbs c = bn_from_ptr(cand + i * L, (size_t)L);
        bn_trim(c);
        if (!(bn_low(c) & 1u) || bn_cmp(c, Limbs{3}) <= 0 || bn_cmp(c, exclude) == 0) continue;
        const uint32_t cm1 = bn_mod_word(bn_sub(c, Limbs{1}), e);
        uint32_t a = e, b = cm1;
        while (b) {
            const uint32_t t = a % b;
            a = b;
            b = t;
        }
        if (a == 1) elig.push_back(i);
    }
    const size_t row = (size_t)rounds * L;
    for (size_t start = 0; start < elig.size(); start += kMrChunk) {
        const size_t n = std::min(kMrChunk, elig.size() - start);
        std::vector<uint32_t> cc(n * (size_t)L), bb(n * row);
        for (size_t k = 0; k < n; k++) {
            std::copy(cand + elig[start + k] * L, cand + (elig[start + k] + 1) * L, cc.begin() + k * L);
            std::copy(bases + elig[start + k] * row, bases + (elig[start + k] + 1) * row, bb.begin() + k * row);
        }
        std::vector<uint8_t> verdict(n);
        if ((rc = rsa_miller_rabin(cc.data(), n, L, bb.data(), rounds, verdict.data(), s))) return rc;
        for (size_t k = 0; k < n; k++)
            if (verdict[k]) {
                out = bn_from_ptr(cc.data() + k * L, (size_t)L);
                bn_trim(out);
                return RNS_OK;
            }
    }
    return fail(RNS_ERANGE, "no probable prime among the candidates");
}

}  // namespace

extern "C" {

int rsa_keygen(const uint32_t *cand_p, const uint32_t *bases_p, const uint32_t *cand_q, const uint32_t *bases_q,
               size_t count, int half_limbs, int rounds, uint32_t e, const rns_opts *opts, uint32_t *n_out,
               rsa_key **out, void *hip_stream) {
    if (!out) return fail(RNS_EINVAL, "null output handle");
    *out = nullptr;
    if (!cand_p || !bases_p || !cand_q || !bases_q || !n_out || count == 0)
        return fail(RNS_EINVAL, "null buffer or empty candidate streams");
    if (half_limbs <= 0 || half_limbs > 2048) return fail(RNS_EINVAL, "half_limbs must be in 1..2048");
    if (rounds <= 0 || rounds > kMaxRounds) return fail(RNS_EINVAL, "rounds must be in 1..64");
    if (e < 3 || !(e & 1u)) return fail(RNS_EINVAL, "e must be odd and >= 3");
    hipStream_t s = (hipStream_t)hip_stream;
    const int H = half_limbs;
    try {
        Limbs p, q;
        int rc = first_prime(cand_p, bases_p, count, H, rounds, e, Limbs{}, s, p);
        if (!rc) rc = first_prime(cand_q, bases_q, count, H, rounds, e, p, s, q);
        if (rc) return rc;
        const Limbs one{1};
        const Limbs pm1 = bn_sub(p, one), qm1 = bn_sub(q, one);
        const Limbs n = bn_mul(p, q), f = bn_mul(pm1, qm1);
        // d = e^-1 mod f by Arazi's formula in RNS on the GPU, on the channel
        // tables of a context for n (n > f > d), checked on the host
        rns_ctx *nc = nullptr;
        if ((rc = make_context(n, 2 * H, &nc))) return rc;
        std::unique_ptr<rns_ctx> nctx(nc);
        Limbs d;
        if ((rc = arazi_inverse(nc, f, e, d, s))) return rc;
        if (bn_cmp(bn_mod(bn_mul_word(d, e), f), one) != 0)
            return fail(RNS_EVERIFY, "d e != 1 mod (p-1)(q-1)");
        const Limbs dp = bn_mod(d, pm1), dq = bn_mod(d, qm1);
        Limbs qinv;
        if (!bn_modinv_odd(q, p, qinv)) return fail(RNS_EINVAL, "q not invertible mod p");
        auto limbs = [](const Limbs &x, int k) {
            Limbs r = x;
            r.resize((size_t)k, 0u);
            return r;
        };
        const Limbs nl = limbs(n, 2 * H), dl = limbs(d, 2 * H);
        const Limbs pl = limbs(p, H), ql = limbs(q, H), dpl = limbs(dp, H), dql = limbs(dq, H), qil = limbs(qinv, H);
        const uint32_t el[1] = {e};
        if ((rc = rsa_key_load(nl.data(), (size_t)(2 * H), el, 1, dl.data(), pl.data(), ql.data(), dpl.data(),
                               dql.data(), qil.data(), (size_t)H, opts, out)))
            return rc;
        std::copy(nl.begin(), nl.end(), n_out);
    } catch (const std::bad_alloc &) {
        return fail(RNS_ENOMEM, "out of host memory");
    }
    return ok();
}

}  // extern "C"
