// Host-side tables of the matrix-core exponentiation kernel (plan_mfma.hpp).
#include "plan_mfma.hpp"

#include <cmath>
#include <functional>


namespace rnsrsa {

bool mfma_shape_for(int K, MfmaShape &out, int group) {
    // the first shape listed for K with the preferred group, else the first for K
    for (int pass = group ? 0 : 1; pass < 2; pass++) {
#define RNSRSA_MSHAPE(k, w, mt, nt)                                    \
    if (K == k && (pass == 1 || group == 16 * (nt))) {               \
        out = MfmaShape{k, w, mt, nt};                                 \
        return true;                                                   \
    }
#define RNSRSA_MTABLES RNSRSA_MSHAPE
#include "kernel_configs_mfma.inc"
#undef RNSRSA_MSHAPE
    }
    return false;
}

bool mfma_launch_shape(int K, MfmaShape &out, int group) {
    if (!mfma_shape_for(K, out, group)) return false;
#define RNSRSA_MSHAPE(k, w, mt, nt) \
    if (out.K == k && out.W == w && out.MT == mt && out.NT == nt) return true;
#include "kernel_configs_mfma.inc"
#undef RNSRSA_MSHAPE
    return mfma_shape_for(K, out, 16);
}

namespace {

// Representative of v mod m in [kDigitSplit - m, kDigitSplit): four balanced bytes.
int64_t balanced(uint32_t v, uint32_t m) { return v >= kDigitSplit ? (int64_t)v - m : (int64_t)v; }

// Representative of v mod 2^32 in [-0x80808080, 0x7F7F7F7F].
int64_t balanced32(uint32_t v) { return v > 0x7F7F7F7Fu ? (int64_t)v - ((int64_t)1 << 32) : (int64_t)v; }

// Signed byte b of a balanced value V = sum_b d_b 256^b, d_b in [-128, 127].
int8_t digit(int64_t V, int b) {
    uint32_t u = (uint32_t)(V + 0x80808080ll);
    return (int8_t)((int)((u >> (8 * b)) & 0xFFu) - 128);
}

// A square root of a modulo the odd prime p (Tonelli-Shanks; p = 3 mod 4 in
// one step), or false when a is not a square mod p.
bool sqrt_mod(uint32_t a, uint32_t p, uint32_t *root) {
    a %= p;
    if (a == 0) {
        *root = 0;
        return true;
    }
    if (powmod32(a, (p - 1) / 2, p) != 1) return false;   // Euler's criterion
    if (p % 4 == 3) {
        *root = powmod32(a, ((uint64_t)p + 1) / 4, p);
        return true;
    }
    uint32_t q = p - 1;
    int s = 0;
    while (!(q & 1)) {
        q >>= 1;
        s++;
    }
    uint32_t z = 2;
    while (powmod32(z, (p - 1) / 2, p) != p - 1) z++;     // a non-residue
    uint32_t c = powmod32(z, q, p), x = powmod32(a, ((uint64_t)q + 1) / 2, p), t = powmod32(a, q, p);
    int m = s;
    while (t != 1) {
        int i = 0;
        uint32_t t2 = t;
        while (t2 != 1) {
            t2 = mulmod32(t2, t2, p);
            i++;
        }
        uint32_t b = c;
        for (int j = 0; j < m - i - 1; j++) b = mulmod32(b, b, p);
        x = mulmod32(x, b, p);
        c = mulmod32(b, b, p);
        t = mulmod32(t, c, p);
        m = i;
    }
    *root = x;
    return true;
}

// One matrix of A tiles [W][MT][KSTEPS][64 lanes][16 bytes] from a value
// function V(slot channel t (-1: redundant), input channel i (K: offset slot), digit a).
template <class F>
void fill_tiles(const MfmaShape &sh, uint32_t *dst, F value, int extra = -2) {   // extra: a row that is no channel

    const int KS = sh.KSTEPS();
    for (int w = 0; w < sh.W; w++)
        for (int mt = 0; mt < sh.MT; mt++)
            for (int ks = 0; ks < KS; ks++)
                for (int l = 0; l < 64; l++) {
                    uint32_t words[4] = {0, 0, 0, 0};
                    const int row = l % 16, g = row / 4, b = row % 4;
                    const int t = mfma_slot_channel(sh, w, mt, g);
                    for (int j = 0; j < 16; j++) {
                        const int kappa = 64 * ks + 16 * (l / 16) + j;
                        const int ch = sh.channel_of(kappa / 4), a = kappa % 4;
                        int64_t V = 0;
                        if ((t < sh.K || t == extra) && ch <= sh.K && (ch < sh.K || a == 0)) V = value(t, ch, a);
                        words[j / 4] |= (uint32_t)(uint8_t)digit(V, b) << (8 * (j % 4));
                    }
                    uint32_t *p = dst + ((((size_t)w * sh.MT + mt) * KS + ks) * 64 + l) * 4;
                    for (int q = 0; q < 4; q++) p[q] = words[q];
                }
}

// Exit tiles: the matrix whose row 4 s + b, applied to the digits of xi'
// (minus kDigitBias) and the offset digit, gives byte partial b of limb s,
// modulo 2^(32 (K+1)).  Column (j, a) holds the balanced base-256 digits of
// M'_j moved up by a bytes; the offset column those of
// kDigitBias sum_j M'_j - kExitOffset sum_s 2^(32 s).
void fill_exit_tiles(const MfmaShape &sh, const BaseSet &bs, uint32_t *dst) {
    const int K = sh.K, NB = 4 * (K + 1), KS = sh.KSTEPS();
    auto balanced_digits = [&](const Limbs &x, int8_t *d) {
        int c = 0;
        for (int r = 0; r < NB; r++) {
            const size_t l = (size_t)r / 4;
            int v = (int)((l < x.size() ? x[l] : 0u) >> (8 * (r % 4)) & 0xFFu) + c;
            c = v > 127 ? 1 : 0;
            d[r] = (int8_t)(v - 256 * c);
        }
    };
    std::vector<int8_t> D((size_t)(K + 1) * NB);
    Limbs sum{0};
    for (int j = 0; j < K; j++) {
        Limbs Mj{1};
        for (int t = 0; t < K; t++)
            if (t != j) Mj = bn_mul_word(Mj, bs.Bp[t]);
        sum = bn_add(sum, Mj);
        balanced_digits(Mj, D.data() + (size_t)j * NB);
    }
    Limbs off((size_t)K + 1, 0u);
    for (int l = 1; l <= K; l++) off[l] = (uint32_t)(kExitOffset >> 32);   // limb 0 of the offset is 0
    Limbs o = bn_mul_word(sum, kDigitBias);
    o.resize((size_t)K + 1, 0u);
    uint32_t borrow = 0;
    for (int l = 0; l <= K; l++) {                                         // o - off mod 2^(32 (K+1))
        const uint64_t d = (uint64_t)o[l] - off[l] - borrow;
        o[l] = (uint32_t)d;
        borrow = (uint32_t)(d >> 63);
    }
    balanced_digits(o, D.data() + (size_t)K * NB);
    for (int st = 0; st < sh.W * sh.MT; st++)
        for (int ks = 0; ks < KS; ks++)
            for (int l = 0; l < 64; l++) {
                uint32_t words[4] = {0, 0, 0, 0};
                const int r = 16 * st + l % 16;                            // output byte 4 s + b
                for (int j = 0; j < 16; j++) {
                    const int kappa = 64 * ks + 16 * (l / 16) + j;
                    const int ch = sh.channel_of(kappa / 4), a = kappa % 4;
                    int8_t v = 0;
                    if (r < NB && (ch < K || (ch == K && a == 0)) && r >= a) v = D[(size_t)ch * NB + r - a];
                    words[j / 4] |= (uint32_t)(uint8_t)v << (8 * (j % 4));
                }
                uint32_t *p = dst + (((size_t)st * KS + ks) * 64 + l) * 4;
                for (int q = 0; q < 4; q++) p[q] = words[q];
            }
}

// The estimate row's weight of input t (see kEstScale).
int64_t est_weight(uint32_t g, uint32_t m) { return (int64_t)(((uint64_t)g * kEstScale + m / 2) / m); }

// Whether the wide form is exact for this modulus: values stay below c N, c =
// 2K + 1 (q^ <= 2 K M: digits of B may exceed their prime by a little, so the
// offset for sigma_i = -1 is 2 m_i M_i); the estimate of alpha is within half
// of 2^32; step (iv)'s sum is positive and, but in the first tile (whose
// reduction takes any sum below 2^64), small enough to leave a result below
// 2^32 without a correction.
bool wide_fits(const ModPlan &mp, const std::vector<uint32_t> &nu2, long double gsum) {
    const BaseSet &bs = *mp.base;
    const int K = bs.K;
    const Limbs c = bn_from_u64((uint64_t)2 * K + 1);
    if (bn_cmp(bn_mul(bn_mul(c, c), mp.N), bs.M) > 0 || bn_cmp(bn_mul(c, mp.N), bs.Mp) >= 0) return false;
    // estimate: weights rounded by 1/2 (times digits up to 128), the three
    // lower digits left out (half a unit of 2^24 each), in units of 2^18
    if ((long double)K * (0.5L * 128 + 0.51L * kEstScale) + 4 >= (long double)(1 << 13)) return false;
    const long double amax = 4294967296.0L * gsum + 2;
    if (amax >= 1099511627776.0L) return false;                        // 2^40
    const uint64_t ah = (uint64_t)(amax / (1 << kWideShift)) + 1 + kWideOffset;
    const uint64_t smax = mfma_sum_bound(K) + 0x80808080ull;
    for (int i = 0; i < K; i++) {
        if ((uint64_t)kWideOffset * nu2[i] <= smax) return false;
        if (i < 4) continue;
        const uint64_t m = bs.B[i];
        const uint64_t hi = (1ull << kWideShift) + ah + (smax >> 32) + 2;   // bound of the sum over 2^32
        if (m + hi >= 1ull << 32) return false;
    }
    return true;
}

// Per-lane slot table [W][MT][64] of f(channel) (channel -1 or >= K: junk).
template <class F>
void fill_slots(const MfmaShape &sh, uint32_t *dst, size_t field_stride, F f) {
    for (int w = 0; w < sh.W; w++)
        for (int mt = 0; mt < sh.MT; mt++)
            for (int g = 0; g < 4; g++) {
                const uint32_t v = f(mfma_slot_channel(sh, w, mt, g));
                std::fill_n(dst + ((size_t)w * sh.MT + mt) * field_stride + 16 * g, 16, v);
            }
}

}  // namespace

MfmaTables make_mfma_tables(const ModPlan &mp, const MfmaShape &sh, bool with_base, bool allow_scaled) {
    const BaseSet &bs = *mp.base;
    const int K = bs.K;
    const MLayout &ly = sh;
    MfmaTables out;
    out.shape = sh;
    if (with_base) out.base.assign(ly.base_size(), 0);
    out.key.assign(ly.key_size(), 0);
    const Limbs &N = mp.N;

    // c_i = -N^-1 M_i^-1 mod m_i, and for the scaled form a sign sigma_i and
    // a root s_i with s_i^2 = sigma_i c_i R^-1 (mod m_i).  A product's
    // quotient digit x y c_i is then REDC(x R s_i * y R s_i) = sigma_i x y c_i:
    // the digit published for channel i is sigma_i xi_i mod m_i, so the first
    // extension takes sigma_i C_i as input i's constants and adds
    // sum_{sigma_i = -1} m_i C_i through its offset column.  (A zero digit
    // then stands for xi_i = m_i: the extension's q lies in [0, K M] instead
    // of [0, K M), which the bounds on the base already cover.)  For a
    // prime = 3 mod 4 one of c_i R^-1 and -c_i R^-1 is a square; the default
    // bases draw such primes.  Without a root for every channel the key keeps
    // sigma_i = 1 and the unscaled form only.
    std::vector<uint32_t> cB(K), sB(K, 1u);
    std::vector<int> sgn(K, 1);
    for (int i = 0; i < K; i++) {
        const uint32_t m = bs.B[i];
        std::vector<uint32_t> others;                                  // M_i mod m_i: product of the other primes
        for (int j = 0; j < K; j++)
            if (j != i) others.push_back(bs.B[j]);
        cB[i] = mulmod32(m - invmod32(bn_mod_word(N, m), m), invmod32(prod_mod32(others, m), m), m);
    }
    out.scaled = allow_scaled && ly.sq_ok();
    for (int i = 0; i < K && out.scaled; i++) {
        const uint32_t m = bs.B[i];
        const uint32_t a = mulmod32(cB[i], invmod32(pow2_32_mod(m), m), m);   // c_i R^-1
        if (sqrt_mod(a, m, &sB[i])) sgn[i] = 1;
        else if (sqrt_mod(m - a, m, &sB[i])) sgn[i] = -1;
        else out.scaled = false;
    }
    // The wide form (see kWideShift): weights g_t, and the root's sign that
    // makes nu2 at least m / 2.
    bool wide = out.scaled && ly.wide();
    std::vector<uint32_t> g(K), nu2(K);
    long double gsum = 0;                                              // sum of g_t / m'_t, so alpha < 2^32 gsum
    if (wide) {
        for (int t = 0; t < K; t++) {
            const uint32_t m = bs.Bp[t];
            std::vector<uint32_t> others;
            for (int j = 0; j < K; j++)
                if (j != t) others.push_back(bs.Bp[j]);
            const uint32_t lam = mulmod32(pow2_32_mod(m), invmod32(prod_mod32(bs.B, m), m), m);   // R M^-1
            g[t] = mulmod32(invmod32(prod_mod32(others, m), m), invmod32(lam, m), m);
            gsum += (long double)g[t] / m;
        }
        for (int i = 0; i < K; i++) {
            const uint32_t m = bs.B[i], mpm = prod_mod32(bs.Bp, m);
            nu2[i] = mulmod32(mulmod32(mulmod32(m - mpm, pow2_64_mod(m), m), sB[i], m), 1u << kWideShift, m);
            if (nu2[i] < m / 2) {
                sB[i] = m - sB[i];
                nu2[i] = m - nu2[i];
            }
        }
        // a base whose primes lie too close to 2^32 (at k = 65 most draws) keeps the
        // scaled form with the narrow second extension
        out.wide = wide = wide_fits(mp, nu2, gsum);
    }
    if (!out.scaled) {
        std::fill(sgn.begin(), sgn.end(), 1);
        std::fill(sB.begin(), sB.end(), 1u);
    }

    // Values of the two extensions' constant matrices, [t + 1][i][a] for output
    // channel t (-1: the redundant row), input channel i (K: the offset
    // column, digit a = 0 only) and digit a, computed once: the residues of
    // M_i = M / m_i modulo a prime m are products of those before and after m_i,
    // and modulo 2^32 prod(B) times m_i^-1 (m_i odd).
    //
    // The digit words carry xi - kDigitBias; the offset column (input channel K,
    // digit value 1) adds kDigitBias * sum_i C_i back, so each extension is the
    // exact integer sum_i xi_i C_i.
    //
    // BE1 (key table): slot t of B' gets sum_i xi_i M_i * G_t with
    // G_t = N R^2 M^-2 mod m'_t, so that one REDC yields q N M^-1 * (R M^-1);
    // the redundant row gets sum_i xi_i M_i mod 2^32.
    // BE2 (base table): slot i of B gets sum_j xi'_j M'_j R^2 mod m_i; the
    // redundant row sum_j xi'_j M'_j mod 2^32.
    // With input signs sig (the first extension of the scaled form) input i's
    // constants are sig_i C_i and the offset column adds
    // kDigitBias sum_i sig_i C_i + sum_{sig_i = -1} m_i C_i.
    const size_t KK = (size_t)(K + 1) * 4;
    // A wide second extension takes weight wgt_i M_i in place of M_i, and its
    // offset column also cancels add(t) (see kWideOffset).  off_sig: multiples of
    // m_i M_i added for sig_i = -1.
    auto ext_values = [&](const std::vector<uint32_t> &in, const std::vector<uint32_t> &outm, auto scale,
                          const std::vector<int> &sig, uint32_t off_sig = 1, const std::vector<uint32_t> *wgt = nullptr,
                          std::function<uint32_t(int)> sub = nullptr) {
        std::vector<int64_t> V((size_t)(K + 1) * KK, 0);
        uint32_t prod_lo = 1;
        for (uint32_t m : in) prod_lo *= m;
        uint32_t off_lo = 0;
        for (int i = 0; i < K; i++) {
            const uint32_t mi_lo = prod_lo * inv2_32(in[i]) * (wgt ? (*wgt)[i] : 1u);
            const uint32_t ci_lo = sig[i] < 0 ? 0u - mi_lo : mi_lo;
            off_lo += kDigitBias * ci_lo + (sig[i] < 0 ? off_sig * in[i] * mi_lo : 0u);
            for (int a = 0; a < 4; a++) V[(size_t)i * 4 + a] = balanced32(ci_lo << (8 * a));
        }
        V[(size_t)K * 4] = balanced32(off_lo);
        for (int t = 0; t < K; t++) {
            const uint32_t m = outm[t], f = scale(t);
            uint32_t fa[4];                                            // 2^(8 a) f
            for (int a = 0; a < 4; a++) fa[a] = mulmod32((1u << (8 * a)) % m, f, m);
            std::vector<uint32_t> after(K + 1, 1u);                    // products of the inputs from i on
            for (int i = K - 1; i >= 0; i--) after[i] = mulmod32(after[i + 1], in[i] % m, m);
            uint32_t before = 1;
            uint64_t off = 0;
            int64_t *row = V.data() + (size_t)(t + 1) * KK;
            for (int i = 0; i < K; i++) {
                uint32_t mi = mulmod32(before, after[i + 1], m);
                before = mulmod32(before, in[i] % m, m);
                if (wgt) mi = mulmod32(mi, (*wgt)[i] % m, m);
                const uint32_t ci = sig[i] < 0 && mi ? m - mi : mi;
                off = (off + mulmod32(kDigitBias % m, ci, m)) % m;
                if (sig[i] < 0) off = (off + mulmod32(mulmod32(off_sig, in[i] % m, m), mi, m)) % m;
                for (int a = 0; a < 4; a++)
                    row[(size_t)i * 4 + a] = balanced(mulmod32(ci, fa[a], m), m);
            }
            uint32_t o = mulmod32((uint32_t)off, f, m);
            if (sub) o = (uint32_t)(((uint64_t)o + m - sub(t) % m) % m);
            row[(size_t)K * 4] = balanced(o, m);
        }
        return V;
    };
    const std::vector<int> plus(K, 1);
    std::vector<uint32_t> G(K);
    for (int t = 0; t < K; t++) {
        uint32_t m = bs.Bp[t];
        uint32_t minv = invmod32(prod_mod32(bs.B, m), m);
        G[t] = mulmod32(mulmod32(bn_mod_word(N, m), pow2_64_mod(m), m), mulmod32(minv, minv, m), m);
    }
    const std::vector<int64_t> V1 = ext_values(bs.B, bs.Bp, [&](int t) { return G[t]; }, sgn, wide ? 2u : 1u);
    fill_tiles(sh, out.key.data() + ly.a1(),
               [&](int t, int i, int a) -> int64_t { return V1[(size_t)(t + 1) * KK + (size_t)i * 4 + a]; });
    auto okc = [&](int t) { return t >= 0 && t < K; };
    if (with_base) {
    const std::vector<int64_t> V2 = ext_values(bs.Bp, bs.B, [&](int t) { return pow2_64_mod(bs.B[t]); }, plus);
    fill_tiles(sh, out.base.data() + ly.a2(),
               [&](int t, int j, int a) -> int64_t { return V2[(size_t)(t + 1) * KK + (size_t)j * 4 + a]; });
    // per-slot constants; junk slots use a valid modulus and zero constants
    const uint32_t mB0 = bs.B[K - 1], mP0 = bs.Bp[K - 1];
    const size_t fs = (size_t)3 * 64;      // [W][MT][3][64]
    fill_slots(sh, out.base.data() + ly.slotB() + 0 * 64, fs, [&](int t) { return okc(t) ? bs.B[t] : mB0; });
    fill_slots(sh, out.base.data() + ly.slotB() + 1 * 64, fs, [&](int t) { return inv2_32(okc(t) ? bs.B[t] : mB0); });
    fill_slots(sh, out.base.data() + ly.slotB() + 2 * 64, fs, [&](int t) -> uint32_t {
        if (!okc(t)) return 0;
        uint32_t m = bs.B[t], mpm = prod_mod32(bs.Bp, m);
        return mulmod32(mpm ? m - mpm : 0, pow2_64_mod(m), m);   // nu = -M' R^2 mod m_i
    });
    const size_t fp = (size_t)4 * 64;      // [W][MT][4][64]
    fill_slots(sh, out.base.data() + ly.slotP() + 0 * 64, fp, [&](int t) { return okc(t) ? bs.Bp[t] : mP0; });
    fill_slots(sh, out.base.data() + ly.slotP() + 1 * 64, fp, [&](int t) { return inv2_32(okc(t) ? bs.Bp[t] : mP0); });
    fill_slots(sh, out.base.data() + ly.slotP() + 3 * 64, fp, [&](int t) -> uint32_t {
        if (!okc(t)) return 0;
        uint32_t m = bs.Bp[t];
        return mulmod32(pow2_32_mod(m), invmod32(prod_mod32(bs.B, m), m), m);     // kappa = R M^-1
    });
    fill_slots(sh, out.base.data() + ly.slotP() + 2 * 64, fp, [&](int t) -> uint32_t {
        if (!okc(t)) return 0;
        uint32_t m = bs.Bp[t];
        std::vector<uint32_t> others;
        for (int j = 0; j < K; j++)
            if (j != t) others.push_back(bs.Bp[j]);
        return mulmod32(prod_mod32(bs.B, m), invmod32(prod_mod32(others, m), m), m);   // H = M (M'_t)^-1
    });
    fill_exit_tiles(sh, bs, out.base.data() + ly.xt());
    for (int l = 0; l <= K && l < (int)bs.Mp.size(); l++) out.base[ly.MpF() + l] = bs.Mp[l];
    out.base[ly.bscal() + 0] = inv2_32(bn_low(bs.Mp));
    out.base[ly.bscal() + 1] = inv2_32(bn_low(bs.M));
    const size_t fc = (size_t)3 * 64;      // [W][MT][3][64]
    fill_slots(sh, out.base.data() + ly.mmconv() + 0 * 64, fc,
               [&](int t) -> uint32_t { return okc(t) ? pow2_64_mod(bs.B[t]) : 0; });
    fill_slots(sh, out.base.data() + ly.mmconv() + 1 * 64, fc, [&](int t) -> uint32_t {
        if (!okc(t)) return 0;
        const uint32_t m = bs.Bp[t];
        return mulmod32(pow2_64_mod(m), invmod32(prod_mod32(bs.B, m), m), m);
    });
    fill_slots(sh, out.base.data() + ly.mmconv() + 2 * 64, fc,
               [&](int t) -> uint32_t { return okc(t) ? prod_mod32(bs.B, bs.Bp[t]) : 0; });
    }

    // key: sigma_i c_i mod m_i; "one" = M mod N in the kept representation
    fill_slots(sh, out.key.data() + ly.slotC(), 64, [&](int t) -> uint32_t {
        if (!okc(t)) return 0;
        return sgn[t] < 0 && cB[t] ? bs.B[t] - cB[t] : cB[t];
    });
    const size_t os = (size_t)2 * 64;      // [W][MT][2][64]
    fill_slots(sh, out.key.data() + ly.one(), os, [&](int t) -> uint32_t {
        if (!okc(t)) return 0;
        uint32_t m = bs.B[t];
        return mulmod32(bn_mod_word(mp.Mmod, m), pow2_32_mod(m), m);
    });
    fill_slots(sh, out.key.data() + ly.one() + 64, os, [&](int t) -> uint32_t {
        if (!okc(t)) return 0;
        uint32_t m = bs.Bp[t];
        uint32_t kappa = mulmod32(pow2_32_mod(m), invmod32(prod_mod32(bs.B, m), m), m);   // R M^-1
        return mulmod32(bn_mod_word(mp.Mmod, m), kappa, m);
    });
    out.key[ly.one() + (size_t)sh.W * sh.MT * 2 * 64] = bn_low(mp.Mmod);
    for (int l = 0; l < K && l < (int)N.size(); l++) out.key[ly.Nl() + l] = N[l];
    out.key[ly.kscal() + 0] = bn_low(N);
    if (out.scaled) {
        // second extension with row t scaled by s_t (R^2 s_t mod m_t); the
        // wide form's with weights and its estimate row
        const std::vector<int64_t> V2s = ext_values(
            bs.Bp, bs.B, [&](int t) { return mulmod32(pow2_64_mod(bs.B[t]), sB[t], bs.B[t]); }, plus, 1,
            wide ? &g : nullptr,
            wide ? std::function<uint32_t(int)>([&](int t) { return mulmod32(kWideOffset, nu2[t], bs.B[t]); }) : nullptr);
        const int est = 4 * sh.MT - 2;
        fill_tiles(sh, out.key.data() + ly.a2s(),
                   [&](int t, int j, int a) -> int64_t {
                       if (wide && t == est) return j < K && a == 3 ? est_weight(g[j], bs.Bp[j]) : 0;
                       return V2s[(size_t)(t + 1) * KK + (size_t)j * 4 + a];
                   },
                   wide ? est : -2);
        if (wide) {
            // the digits' bias, half a unit of the estimate's rounding, the offset
            const long double bias = (long double)kDigitBias / (1 << 24) * kEstScale * gsum;
            out.key[ly.kscal() + 1] = (uint32_t)(int32_t)llroundl(bias) + (1u << 13) +
                                      ((uint32_t)kWideOffset >> (32 - kWideShift) << 14);
        }
        if (wide) {
            uint32_t t = 0;
            for (int i = 0; i < K; i++) t += sgn[i] < 0 ? 1 : 0;
            const Limbs tN = bn_mul(N, Limbs{t});
            out.key[ly.kscal() + 2] = bn_low(tN);
            fill_slots(sh, out.key.data() + ly.mmfix(), 2 * 64, [&](int c) { return okc(c) ? bn_mod_word(tN, bs.B[c]) : 0u; });
            fill_slots(sh, out.key.data() + ly.mmfix() + 64, 2 * 64,
                       [&](int c) { return okc(c) ? bn_mod_word(tN, bs.Bp[c]) : 0u; });
        }
        fill_slots(sh, out.key.data() + ly.zdig(), 64, [&](int t) { return okc(t) && sgn[t] < 0 ? bs.B[t] : 0u; });
        const size_t fq = (size_t)4 * 64;      // [W][MT][4][64]
        fill_slots(sh, out.key.data() + ly.sqB() + 3 * 64, fq, [&](int t) -> uint32_t { return wide && okc(t) ? nu2[t] : 0; });
        fill_slots(sh, out.key.data() + ly.sqB() + 0 * 64, fq, [&](int t) -> uint32_t {
            if (!okc(t)) return 0;
            const uint32_t m = bs.B[t], mpm = prod_mod32(bs.Bp, m);
            return mulmod32(mulmod32(mpm ? m - mpm : 0, pow2_64_mod(m), m), sB[t], m);   // nu s_t
        });
        fill_slots(sh, out.key.data() + ly.sqB() + 1 * 64, fq, [&](int t) -> uint32_t {
            return okc(t) ? mulmod32(pow2_32_mod(bs.B[t]), sB[t], bs.B[t]) : 0;      // R s_t
        });
        fill_slots(sh, out.key.data() + ly.sqB() + 2 * 64, fq, [&](int t) -> uint32_t {
            if (!okc(t)) return 0;
            const uint32_t m = bs.B[t];
            return mulmod32(mulmod32(bn_mod_word(mp.Mmod, m), pow2_32_mod(m), m), sB[t], m);   // one s_t
        });
    }
    return out;
}

std::vector<uint32_t> make_mfma_entry_table(const ModPlan &mp, const MfmaShape &sh, const std::vector<Limbs> &Y,
                                            int L) {
    const BaseSet &bs = *mp.base;
    const int K = bs.K;
    const MLayout &ly = sh;
    const size_t cols = ly.ecols();
    const int rows = (int)Y.size() * L;
    const int SW = 4 * sh.MT;    // slots per wave
    std::vector<uint32_t> e((size_t)rows * cols, 0);
    // row j holds the residues of v = Y_h 2^(32 (j mod L)), h = j / L: per
    // channel, (Y_h mod m) times (2^32 mod m)^(j mod L), times the channel's
    // constant factor
    for (int w = 0; w < sh.W; w++)
        for (int s = 0; s < SW; s++) {
            const int t = mfma_slot_channel(sh, w, s / 4, s % 4);
            if (t < 0 || t >= K) continue;
            const uint32_t m = bs.B[t], mp2 = bs.Bp[t];
            const uint32_t r3 = mulmod32(pow2_64_mod(m), pow2_32_mod(m), m);
            const uint32_t r3p = mulmod32(mulmod32(pow2_64_mod(mp2), pow2_32_mod(mp2), mp2),
                                          invmod32(prod_mod32(bs.B, mp2), mp2), mp2);
            const uint32_t w32 = pow2_32_mod(m), w32p = pow2_32_mod(mp2);
            for (size_t h = 0; h < Y.size(); h++) {
                uint32_t vm = mulmod32(bn_mod_word(Y[h], m), r3, m);
                uint32_t vp = mulmod32(bn_mod_word(Y[h], mp2), r3p, mp2);
                for (int l = 0; l < L; l++) {
                    const size_t j = h * (size_t)L + l;
                    e[j * cols + (size_t)w * SW + s] = vm;
                    e[j * cols + (size_t)sh.W * SW + (size_t)w * SW + s] = vp;
                    vm = mulmod32(vm, w32, m);
                    vp = mulmod32(vp, w32p, mp2);
                }
            }
        }
    for (int j = 0; j < rows; j++) e[(size_t)j * cols + cols - 1] = (j % L) ? 0u : bn_low(Y[j / L]);
    return e;
}

}  // namespace rnsrsa
