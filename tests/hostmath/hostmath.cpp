// Host build of the library's field / curve headers, exported for CPU-side tests.
// The same inline functions run inside the HIP kernels; compiling them with g++ lets
// the CPU test-suite check them against the oracle without a GPU.
#include <cstring>

#define TC_HOST_EMU 1
#include <vector>

#include "../../paper_2602_12630_amd/csrc/kernels.h"
#include "../../paper_2602_12630_amd/csrc/pairing.h"

using namespace tc;

static fp_t fp_load(const uint8_t* b) { uint32_t w[12]; memcpy(w, b, 48); return fe_from_limbs<FpParams>(w); }
static void fp_store(uint8_t* b, const fp_t& a) { fp_t p = fe_to_plain(a); memcpy(b, p.l, 48); }
static fr_t fr_load(const uint8_t* b) { uint32_t w[8]; memcpy(w, b, 32); return fe_from_limbs<FrParams>(w); }
static void fr_store(uint8_t* b, const fr_t& a) { fr_t p = fe_to_plain(a); memcpy(b, p.l, 32); }
static g1_affine pt_load(const uint8_t* b) { uint32_t w[24]; memcpy(w, b, 96); return affine_from_canonical(w); }
static void pt_store(uint8_t* b, const g1_affine& p) { uint32_t w[24]; affine_to_canonical(p, w); memcpy(b, w, 96); }

// the phases of a cooperative kernel, lane by lane
template <class K>
static void coop_run(const K& k, uint32_t groups) {
    std::vector<uint8_t> lds(K::LDS_BYTES);
    for (uint32_t g = 0; g < groups; ++g)
        for (int ph = 0; ph < K::PHASES; ++ph)
            for (uint32_t lane = 0; lane < (uint32_t)K::BLOCK; ++lane) k.phase(ph, lane, g, lds.data());
}
template <class K>
static void wave_run(const K& k, uint32_t groups) {
    std::vector<uint8_t> lds(K::LDS_BYTES);
    for (uint32_t g = 0; g < groups; ++g)
        for (int ph = 0; ph < K::PHASES; ++ph)
            for (uint32_t wave = 0; wave < (uint32_t)K::WAVES; ++wave) k.phase(ph, wave, g, lds.data());
}

extern "C" {
void hm_fp_mul(const uint8_t* a, const uint8_t* b, uint8_t* o) { fp_store(o, fp_mul(fp_load(a), fp_load(b))); }
void hm_fp_mul_limbs32(const uint8_t* a, const uint8_t* b, uint8_t* o) { fp_store(o, fe_mul<FpParams>(fp_load(a), fp_load(b))); }
void hm_fp_mul_f64(const uint8_t* a, const uint8_t* b, uint8_t* o) { fp_store(o, fp_mul_f64(fp_load(a), fp_load(b))); }
void hm_fp_sqr_f64(const uint8_t* a, const uint8_t*, uint8_t* o) { fp_store(o, fp_sqr_f64(fp_load(a))); }
void hm_fp_add(const uint8_t* a, const uint8_t* b, uint8_t* o) { fp_store(o, fp_add(fp_load(a), fp_load(b))); }
void hm_fp_sub(const uint8_t* a, const uint8_t* b, uint8_t* o) { fp_store(o, fp_sub(fp_load(a), fp_load(b))); }
void hm_fp_inv(const uint8_t* a, uint8_t* o) { fp_store(o, fe_inv_fermat<FpParams>(fp_load(a))); }
void hm_fp_inv_binary(const uint8_t* a, uint8_t* o) { fp_store(o, fe_inv<FpParams>(fp_load(a))); }
void hm_fr_inv_binary(const uint8_t* a, uint8_t* o) { fr_store(o, fe_inv<FrParams>(fr_load(a))); }
void hm_fp_inv_gcd(const uint8_t* a, uint8_t* o) { fp_store(o, fe_inv_gcd<FpParams>(fp_load(a))); }
void hm_fp_inv_wave(const uint8_t* a, uint8_t* o) { fp_store(o, fp28_to_fp(fp28_inv_wave(fp28_mul(fp28_from_fp(fp_load(a)), fp28_one())))); }
// batches of the wave's inversion (-1: the division steps took over), and those steps by themselves
int hm_fp_inv_batches(const uint8_t* a) { int n; fp28_inv_wave(fp28_mul(fp28_from_fp(fp_load(a)), fp28_one()), &n); return n; }
void hm_fp_inv_divsteps(const uint8_t* a, uint8_t* o) { fp_store(o, fp28_to_fp(fp28_inv_divsteps(fp28_mul(fp28_from_fp(fp_load(a)), fp28_one())))); }
void hm_fr_inv_gcd(const uint8_t* a, uint8_t* o) { fr_store(o, fe_inv_gcd<FrParams>(fr_load(a))); }
void hm_fr_mul(const uint8_t* a, const uint8_t* b, uint8_t* o) { fr_store(o, fr_mul(fr_load(a), fr_load(b))); }
void hm_fr_mul_limbs29(const uint32_t* a, const uint32_t* b, uint32_t* o) { fr_t x, y; memcpy(x.l, a, 32); memcpy(y.l, b, 32); fr_t r = fr_mul_limbs29(x, y); memcpy(o, r.l, 32); }
void hm_fr_add(const uint8_t* a, const uint8_t* b, uint8_t* o) { fr_store(o, fr_add(fr_load(a), fr_load(b))); }
void hm_fr_sub(const uint8_t* a, const uint8_t* b, uint8_t* o) { fr_store(o, fr_sub(fr_load(a), fr_load(b))); }
void hm_fr_from_i32(int32_t v, uint8_t* o) { fr_store(o, fe_from_i32<FrParams>(v)); }
// a + b through the XYZZ laws: mode 0 = mixed add (a accumulated from affine), 1 = full add
// with both operands pushed away from Z = 1 first (a = (a + g) - g style is avoided: we use 2a - a)
void hm_g1_add(const uint8_t* a, const uint8_t* b, int mode, uint8_t* o) {
    g1_affine A = pt_load(a), B = pt_load(b);
    g1_xyzz r;
    if (mode == 0) {
        r = xyzz_madd(xyzz_from_affine(A), B);
    } else if (mode == 1) {
        r = xyzz_add(xyzz_from_affine(A), xyzz_from_affine(B));
    } else {
        // non-trivial ZZ on both sides: A = 2A + (-A), B = 2B + (-B)
        g1_xyzz A2 = xyzz_madd(xyzz_dbl_affine(A), affine_neg(A));
        g1_xyzz B2 = xyzz_madd(xyzz_dbl(xyzz_from_affine(B)), affine_neg(B));
        r = xyzz_add(A2, B2);
    }
    pt_store(o, xyzz_to_affine(r));
}
void hm_g1_mul(const uint8_t* k, const uint8_t* p, uint8_t* o) {
    uint32_t w[8]; memcpy(w, k, 32);
    pt_store(o, xyzz_to_affine(xyzz_mul_affine(w, 256, pt_load(p))));
}
// sum of n points through the four-wave cooperative reduction, phases run lane by lane
struct ArraySrc {
    const g1_xyzz* in;
    uint32_t n;
    g1_xyzz* out;
    uint32_t count(uint32_t) const { return n; }
    g1_xyzz load(uint32_t, uint32_t i) const { return in[i]; }
    void store(uint32_t, const g1_xyzz& r) const { *out = r; }
};
void hm_coop_reduce(const uint8_t* pts, uint32_t n, int spread, uint8_t* o) {
    std::vector<g1_xyzz> in(n ? n : 1);
    for (uint32_t i = 0; i < n; ++i) {
        g1_affine a = pt_load(pts + 96 * (size_t)i);
        // spread = 1: operands away from ZZ = 1, as sums of sums are (2a - a)
        in[i] = spread ? xyzz_madd(xyzz_dbl_affine(a), affine_neg(a)) : xyzz_from_affine(a);
    }
    g1_xyzz r;
    typedef CoopReduce<ArraySrc> K;
    K k{ArraySrc{in.data(), n, &r}};
    coop_run(k, 1);
    pt_store(o, xyzz_to_affine(r));
}
// sum_k k B_k of windows of 2^lognb buckets bit by bit: the sums per bit, their place values, the total
void hm_window_bits(const uint8_t* pts, uint32_t lognb, uint32_t windows, uint8_t* o) {
    const uint32_t chains = lognb + 1, n = chains * windows;
    std::vector<g1_xyzz> bucket((size_t)windows << lognb), sum(windows);
    for (size_t i = 0; i < bucket.size(); ++i) {
        g1_affine a = pt_load(pts + 96 * i);
        bucket[i] = i % 2 ? xyzz_madd(xyzz_dbl_affine(a), affine_neg(a)) : xyzz_from_affine(a);
    }
    std::vector<uint32_t> pieces((size_t)n * BITSUM_PARTS * WV_POINT_WORDS);
    const WavePoints in{bucket.data(), WAVE_XYZZ};
    std::vector<uint32_t> scaled((size_t)n * WV_POINT_WORDS);
    wave_run(BitSumWave{in, in, 1u << lognb, 1u << lognb, 0u, 0u, lognb, pieces.data()}, n * BITSUM_PARTS);
    wave_run(ScaleWave{pieces.data(), lognb, scaled.data()}, n);
    wave_run(WindowWave{scaled.data(), chains, nullptr, sum.data()}, windows);
    for (uint32_t w = 0; w < windows; ++w) pt_store(o + 96 * (size_t)w, xyzz_to_affine(sum[w]));
}
// 13 limbs of 30 bits, raw: mode 0 a b, 1 a^2, 2 a b - c e, 3 a b - f, 4 a^2 - f - 2 g, 5 balanced a, 6 the cut of an element
void hm_fp30(int mode, const int32_t* in, int32_t* o) {
    fp30 x[4], r{};
    for (int i = 0; i < 4; ++i)
        for (int j = 0; j < 13; ++j) x[i].l[j] = in[13 * i + j];
    if (mode == 0) r = fp30_mul(x[0], x[1]);
    else if (mode == 1) r = fp30_sqr(x[0]);
    else if (mode == 2) r = fp30_mul_sub(x[0], x[1], x[2], x[3]);
    else if (mode == 3) r = fp30_mul_less(x[0], x[1], x[2]);
    else if (mode == 4) r = fp30_mont<FP30_SQR, 2>(x[0], x[0], x[0], x[0], x[2], -1, x[3], -2);
    else if (mode == 5) r = fp30_balance(x[0]);
    for (int j = 0; j < 13; ++j) o[j] = r.l[j];
}
// value (raw limbs) -> canonical coordinate and back, and the zero test
void hm_fp30_to_fp(const int32_t* in, uint8_t* o) { fp30 a; for (int j = 0; j < 13; ++j) a.l[j] = in[j]; fp_store(o, fp30_to_fp(a)); }
int hm_fp30_recut(const uint8_t* a) { fp_t x = fp_load(a); return fe_eq(fp30_recut_to_fp(fp30_from_fp(x)), x) && fe_eq(fp30_to_fp(fp30_from_fp(x)), x); }
int hm_fp30_maybe_zero(const int32_t* in, uint32_t K) { fp30 a; for (int j = 0; j < 13; ++j) a.l[j] = in[j]; return fp30_maybe_zero(a, K) ? 1 : 0; }
// the form spread over lanes: a product of raw limbs (14 words each, four rows), and sums and doublings of points
void hm_wave_mul(const uint32_t* a, const uint32_t* b, uint32_t* o) {
    wv x, y;
    for (int i = 0; i < 64; ++i) { x.l[i] = i % 16 < 14 ? a[14 * (i / 16) + i % 16] : 0; y.l[i] = i % 16 < 14 ? b[14 * (i / 16) + i % 16] : 0; }
    wv r = wv_mul(wv_constants(), x, y);
    for (int i = 0; i < 64; ++i) {
        if (i % 16 < 14) o[14 * (i / 16) + i % 16] = r.l[i];
        else if (r.l[i]) o[0] = 0xFFFFFFFFu;
    }
}
void hm_wave_sum(const uint8_t* pts, uint32_t n, int doublings, int spread, uint8_t* o) {
    const wv_consts k = wv_constants();
    wv_point acc = wv_identity();
    for (uint32_t i = 0; i < n; ++i) {
        g1_affine a = pt_load(pts + 96 * (size_t)i);
        g1_xyzz s = spread ? xyzz_madd(xyzz_dbl_affine(a), affine_neg(a)) : xyzz_from_affine(a);
        wv_point p = wv_load(&s);
        if (spread == 2) { p.v = wv_negate(p.v); p.v = wv_negate(wv_mul(k, p.v, wv_table(W28_ONE))); }
        wv_accumulate(k, acc, p);
    }
    for (int i = 0; i < doublings; ++i)
        if (!acc.inf) acc.v = wv_dbl(k, acc.v);
    g1_xyzz r;
    wv_store(&r, acc);
    pt_store(o, xyzz_to_affine(r));
}
// the verifier's short final exponentiation against the plain one: must be its cube; also x^p, x^(p^2) by powers
int hm_final_exponentiation_forms(const uint8_t* p, uint32_t k) {
    using namespace tc::pairing;
    uint32_t kk[1] = {k};
    g2_affine q = g2_mul(kk, 32, g2_generator());
    fp12 f = miller(pt_load(p), q);
    fp12 e1 = final_exponentiation(f), e3 = final_exponentiation_cubed(f);
    bool cube = f12_eq(f12_mul(f12_sqr(e1), e1), e3);
    // Frobenius maps on an arbitrary element (the Miller value): compare with plain powers by p and p^2
    fp12 xp = f12_one(), base = f;
    for (int i = 0; i < 12 * 32; ++i) {                      // p, bit by bit from the limbs of the modulus
        if ((FpParams::MOD[i >> 5] >> (i & 31)) & 1u) xp = f12_mul(xp, base);
        base = f12_sqr(base);
    }
    bool frob1 = f12_eq(xp, f12_frob1(f));
    bool frob2 = f12_eq(f12_frob1(f12_frob1(f)), f12_frob2(f));
    bool inv = f12_eq(f12_mul(f, f12_inv(f)), f12_one());
    return (cube ? 1 : 0) | (frob1 ? 2 : 0) | (frob2 ? 4 : 0) | (inv ? 8 : 0);
}
void hm_g1_generator(uint8_t* o) { pt_store(o, affine_generator()); }
void hm_phi(const uint8_t* p, uint8_t* o) { fr_t v = phi_map(pt_load(p)); memcpy(o, v.l, 32); }
}
