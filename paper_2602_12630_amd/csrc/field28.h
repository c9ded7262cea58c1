/*
 * A second form of Fp, for the group law: 14 signed limbs of 28 bits, Montgomery radix 2^392.
 *
 * Why: in the 12 x 32-bit form every limb product (v_mad_u64_u32) is followed by an addition that carries into the
 * third word of the column sum, and every modular addition is a carry chain with a conditional subtraction.  With
 * 28-bit limbs a whole column of the product scan -- 14 terms a_i b_j, 14 terms q_i p_j and the carry of the
 * column before -- fits a signed 64-bit accumulator, so a product is 392 multiply-adds (v_mad_i64_i32) and no carry
 * instructions, and an addition or subtraction is 14 independent limb operations: limbs may grow beyond 28 bits
 * and go negative between products, and values need not lie in [0, p).
 *
 * A value is a limb vector l with value(l) = sum_j l_j 2^(28 j), standing for value(l) 2^-392 mod p.
 *   "normal":  limbs 0..12 in [0, 2^28), limb 13 a small signed number (the sign of the value lives there);
 *              what fp28_mul / fp28_sqr / fp28_carry return.
 * Bounds (checked by the host tests on extreme operands): a product is exact as long as
 *   14 max|a_j| max|b_j| + 14 * 2^56 + 2^36 < 2^63, e.g. limbs below 2^29.5 on both sides, or 2^30 against 2^29;
 * its result lies in (a b / 2^392, a b / 2^392 + p), i.e. in (-p, 2 p) whenever |a b| < 2^392 p -- the radix
 * leaves 11 bits of room above p, so sums of a few terms never need a reduction.
 *
 * Elements of the 32-bit form (Montgomery radix 2^384, canonical) enter by a re-cut of their bits moved up by 8
 * places (value 2^8 stands for the same field element under the radix 2^392); they leave through a Montgomery step
 * of those eight bits followed by the one full reduction of the path.
 */
#pragma once
#include "field.h"

namespace tc {

struct fp28 {
    int32_t l[14];
};

static constexpr int32_t FP28_MASK = (1 << 28) - 1;

/* the limbs of a 2^8 for a canonical a: bits 28 j - 8 .. 28 j + 19 of a */
TC_HD fp28 fp28_from_fp(const fp_t& a) {
    fp28 r;
    r.l[0] = (int32_t)((a.l[0] << 8) & (uint32_t)FP28_MASK);
#pragma unroll
    for (int j = 1; j < 14; ++j) {
        const int o = 28 * j - 8, w = o >> 5, sh = o & 31;
        uint32_t lo = a.l[w], hi = w + 1 < 12 ? a.l[w + 1] : 0u;
        uint32_t v = sh ? (lo >> sh) | (hi << (32 - sh)) : lo;
        r.l[j] = (int32_t)(v & (uint32_t)FP28_MASK);
    }
    return r;
}

TC_HD fp28 fp28_one() {
    fp28 r;
#pragma unroll
    for (int j = 0; j < 14; ++j) r.l[j] = Fp28Params::ONE[j];
    return r;
}
TC_HD fp28 fp28_add(const fp28& a, const fp28& b) {
    fp28 r;
#pragma unroll
    for (int j = 0; j < 14; ++j) r.l[j] = a.l[j] + b.l[j];
    return r;
}
TC_HD fp28 fp28_sub(const fp28& a, const fp28& b) {
    fp28 r;
#pragma unroll
    for (int j = 0; j < 14; ++j) r.l[j] = a.l[j] - b.l[j];
    return r;
}
/* same value, normal limbs (limbs of up to 31 bits either sign in, 28-bit limbs and a signed top limb out) */
TC_HD fp28 fp28_carry(const fp28& a) {
    fp28 r;
    int32_t c = 0;
#pragma unroll
    for (int j = 0; j < 13; ++j) {
        int32_t s = a.l[j] + c;
        r.l[j] = s & FP28_MASK;
        c = s >> 28;                       /* arithmetic: floor */
    }
    r.l[13] = a.l[13] + c;
    return r;
}

/* a b 2^-392 (mod p) -- or a^2, or a b - c e -- with normal limbs, in (v / 2^392, v / 2^392 + p) for the integer v
 * that is reduced.  Column k of the product scan collects a_i b_(k-i) (and -c_i e_(k-i)) and q_i p_(k-i); q_k is chosen
 * so that the low 28 bits of the column vanish.  The difference of two products costs one reduction, not two; its
 * column sums must obey the bound above with both products counted. */
enum { FP28_MUL = 0, FP28_SQR = 1, FP28_MUL_SUB = 2 };
/* acc += x y: as one chain per column (mac_chain) in products expanded in place, for kernels of two or three waves per SIMD; as the
 * compiler likes it, a column from zero joined to the carry of the column before with an addition, in those that are calls, whose
 * kernels run a wave alone on its SIMD and would wait for each multiply-add (a lone commitment of 2^21 terms 728 against 740 us). */
template <bool CHAIN>
TC_HD void fp28_mac(int64_t& acc, int32_t x, int32_t y) {
    if (CHAIN) mac_chain(acc, x, y);
    else acc += (int64_t)x * (int64_t)y;
}
template <int MODE, bool CHAIN>
TC_HD fp28 fp28_mont(const fp28& a, const fp28& b, const fp28& c, const fp28& e) {
    int64_t acc = 0;
    int32_t q[14], d[14];
    fp28 r;
    if (MODE == FP28_SQR) {
#pragma unroll
        for (int i = 0; i < 14; ++i) d[i] = a.l[i] + a.l[i];        /* cross terms once, with a doubled operand */
    }
    if (MODE == FP28_MUL_SUB) {
#pragma unroll
        for (int i = 0; i < 14; ++i) d[i] = -c.l[i];
    }
#pragma unroll
    for (int k = 0; k < 27; ++k) {
        const int lo = k < 14 ? 0 : k - 13, hi = k < 14 ? k : 13;
        if (MODE == FP28_SQR) {
#pragma unroll
            for (int i = lo; i < k - i; ++i) fp28_mac<CHAIN>(acc, d[i], a.l[k - i]);
            if ((k & 1) == 0) fp28_mac<CHAIN>(acc, a.l[k / 2], a.l[k / 2]);
        } else {
#pragma unroll
            for (int i = lo; i <= hi; ++i) fp28_mac<CHAIN>(acc, a.l[i], b.l[k - i]);
        }
        if (MODE == FP28_MUL_SUB) {
#pragma unroll
            for (int i = lo; i <= hi; ++i) fp28_mac<CHAIN>(acc, d[i], e.l[k - i]);
        }
        if (k < 14) {
#pragma unroll
            for (int i = 0; i < k; ++i) fp28_mac<CHAIN>(acc, q[i], Fp28Params::MOD[k - i]);
            q[k] = (int32_t)(((uint32_t)acc * (uint32_t)Fp28Params::NINV) & (uint32_t)FP28_MASK);
            fp28_mac<CHAIN>(acc, q[k], Fp28Params::MOD[0]);
        } else {
#pragma unroll
            for (int i = lo; i <= 13; ++i) fp28_mac<CHAIN>(acc, q[i], Fp28Params::MOD[k - i]);
            r.l[k - 14] = (int32_t)((uint32_t)acc & (uint32_t)FP28_MASK);
        }
        acc >>= 28;                        /* arithmetic: the accumulator is signed */
    }
    r.l[13] = (int32_t)acc;
    return r;
}
/* expanded in place: for a kernel whose loop is a handful of products and nothing else (no operand shuffling around
 * calls, and the scheduler sees across products).  The fused difference exists in this form only: the four operands
 * of a call would not fit the 32 registers in which arguments travel. */
TC_HD fp28 fp28_mul_inline(const fp28& a, const fp28& b) { return fp28_mont<FP28_MUL, true>(a, b, a, a); }
TC_HD fp28 fp28_sqr_inline(const fp28& a) { return fp28_mont<FP28_SQR, true>(a, a, a, a); }
TC_HD fp28 fp28_mul_sub_inline(const fp28& a, const fp28& b, const fp28& c, const fp28& e) { return fp28_mont<FP28_MUL_SUB, true>(a, b, c, e); }

#if defined(__HIP_DEVICE_COMPILE__)
/* real functions on the device, as for the 32-bit form: operands and result travel in VGPRs */
typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
typedef int32_t i32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ fp28 fp28_unpack(i32x4 a0, i32x4 a1, i32x4 a2, i32x2 a3) {
    fp28 a;
    a.l[0] = a0.x; a.l[1] = a0.y; a.l[2] = a0.z; a.l[3] = a0.w; a.l[4] = a1.x; a.l[5] = a1.y; a.l[6] = a1.z; a.l[7] = a1.w;
    a.l[8] = a2.x; a.l[9] = a2.y; a.l[10] = a2.z; a.l[11] = a2.w; a.l[12] = a3.x; a.l[13] = a3.y;
    return a;
}
__device__ __attribute__((noinline)) fp28 fp28_mul_call(i32x4 a0, i32x4 a1, i32x4 a2, i32x2 a3, i32x4 b0, i32x4 b1, i32x4 b2, i32x2 b3) {
    const fp28 a = fp28_unpack(a0, a1, a2, a3), b = fp28_unpack(b0, b1, b2, b3);
    return fp28_mont<FP28_MUL, false>(a, b, a, a);
}
__device__ __attribute__((noinline)) fp28 fp28_sqr_call(i32x4 a0, i32x4 a1, i32x4 a2, i32x2 a3) {
    const fp28 a = fp28_unpack(a0, a1, a2, a3);
    return fp28_mont<FP28_SQR, false>(a, a, a, a);
}
#define TC_FP28_ARGS(a) i32x4{a.l[0], a.l[1], a.l[2], a.l[3]}, i32x4{a.l[4], a.l[5], a.l[6], a.l[7]}, i32x4{a.l[8], a.l[9], a.l[10], a.l[11]}, i32x2{a.l[12], a.l[13]}
__device__ __forceinline__ fp28 fp28_mul(const fp28& a, const fp28& b) {
    return fp28_mul_call(i32x4{a.l[0], a.l[1], a.l[2], a.l[3]}, i32x4{a.l[4], a.l[5], a.l[6], a.l[7]}, i32x4{a.l[8], a.l[9], a.l[10], a.l[11]},
                         i32x2{a.l[12], a.l[13]}, i32x4{b.l[0], b.l[1], b.l[2], b.l[3]}, i32x4{b.l[4], b.l[5], b.l[6], b.l[7]},
                         i32x4{b.l[8], b.l[9], b.l[10], b.l[11]}, i32x2{b.l[12], b.l[13]});
}
__device__ __forceinline__ fp28 fp28_sqr(const fp28& a) {
    return fp28_sqr_call(i32x4{a.l[0], a.l[1], a.l[2], a.l[3]}, i32x4{a.l[4], a.l[5], a.l[6], a.l[7]}, i32x4{a.l[8], a.l[9], a.l[10], a.l[11]},
                         i32x2{a.l[12], a.l[13]});
}
#elif defined(__HIPCC__)
__device__ fp28 fp28_mul(const fp28& a, const fp28& b);
__device__ fp28 fp28_sqr(const fp28& a);
__host__ inline fp28 fp28_mul(const fp28& a, const fp28& b) { return fp28_mul_inline(a, b); }
__host__ inline fp28 fp28_sqr(const fp28& a) { return fp28_sqr_inline(a); }
#else
inline fp28 fp28_mul(const fp28& a, const fp28& b) { return fp28_mul_inline(a, b); }
inline fp28 fp28_sqr(const fp28& a) { return fp28_sqr_inline(a); }
#endif

/* 12 words of 32 bits from the bits 8 .. 391 of a non-negative value with normal limbs */
TC_HD fp_t fp28_pack_shr8(const uint32_t (&u)[14]) {
    fp_t r;
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const int o = 32 * i + 8, j = o / 28, sh = o % 28;
        uint32_t w = u[j] >> sh;
        if (j + 1 < 14) w |= u[j + 1] << (28 - sh);
        if (56 - sh < 32 && j + 2 < 14) w |= u[j + 2] << (56 - sh);
        r.l[i] = w;
    }
    return r;
}
/* fp28_from_fp undone: the element whose re-cut `a` is (no arithmetic: the limbs are slices of its bits) */
TC_HD fp_t fp28_recut_to_fp(const fp28& a) {
    uint32_t u[14];
#pragma unroll
    for (int j = 0; j < 14; ++j) u[j] = (uint32_t)a.l[j];
    return fp28_pack_shr8(u);
}
/* The canonical element of the 32-bit form (radix 2^384) for a value v with -256 p <= v < 512 p.  The two radices
 * differ by 2^8, so this is a Montgomery step of eight bits: a multiple q p with v + q p = 0 (mod 2^8), taken from
 * 256 p .. 511 p so that the sum is not negative, then the shift; (v + q p) / 2^8 < 4 p. */
TC_HD fp_t fp28_to_fp(const fp28& a) {
    int32_t q = (int32_t)((((uint32_t)a.l[0] * (uint32_t)Fp28Params::NINV) & 0xFFu) + 256u);
    uint32_t u[14];
    int64_t c = 0;
#pragma unroll
    for (int j = 0; j < 13; ++j) {
        c += (int64_t)q * (int64_t)Fp28Params::MOD[j] + (int64_t)a.l[j];
        u[j] = (uint32_t)c & (uint32_t)FP28_MASK;
        c >>= 28;
    }
    c += (int64_t)q * (int64_t)Fp28Params::MOD[13] + (int64_t)a.l[13];
    u[13] = (uint32_t)c;                   /* below 2^26 */
    fp_t r = fp28_pack_shr8(u);
    return fe_reduce_once<FpParams>(fe_reduce_once<FpParams>(fe_reduce_once<FpParams>(r, 0u), 0u), 0u);
}

/* the same as a real function on the device: for the end of a kernel whose loop must keep its registers */
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __attribute__((noinline)) fp_t fp28_to_fp_call(i32x4 a0, i32x4 a1, i32x4 a2, i32x2 a3) { return fp28_to_fp(fp28_unpack(a0, a1, a2, a3)); }
__device__ __forceinline__ fp_t fp28_to_fp_outlined(const fp28& a) { return fp28_to_fp_call(TC_FP28_ARGS(a)); }
#elif defined(__HIPCC__)
__device__ fp_t fp28_to_fp_outlined(const fp28& a);
__host__ inline fp_t fp28_to_fp_outlined(const fp28& a) { return fp28_to_fp(a); }
#else
inline fp_t fp28_to_fp_outlined(const fp28& a) { return fp28_to_fp(a); }
#endif

/* the first two limbs of that test only: no multiple of p is missed, and of the other values all but about
 * (2 K + 1) 2^-56 are told apart -- for a loop that cannot afford the registers of the full test and has a slower
 * path for whatever passes */
TC_HD bool fp28_maybe_zero(const fp28& a, uint32_t K) {
    uint32_t kk = ((uint32_t)a.l[0] * (uint32_t)Fp28Params::PINV + K) & (uint32_t)FP28_MASK;
    if (kk > 2u * K) return false;
    int32_t k = (int32_t)kk - (int32_t)K;
    int64_t c = ((int64_t)a.l[0] - (int64_t)k * (int64_t)Fp28Params::MOD[0]) >> 28;        /* the low 28 bits are zero by the choice of k */
    c += (int64_t)a.l[1] - (int64_t)k * (int64_t)Fp28Params::MOD[1];
    return ((uint32_t)c & (uint32_t)FP28_MASK) == 0;
}
TC_HD bool fp28_is_zero(const fp28& a, uint32_t K) {
    uint32_t kk = ((uint32_t)a.l[0] * (uint32_t)Fp28Params::PINV + K) & (uint32_t)FP28_MASK;
    if (kk > 2u * K) return false;
    int32_t k = (int32_t)kk - (int32_t)K;
    int64_t c = 0;
    uint32_t low = 0;
#pragma unroll
    for (int j = 0; j < 13; ++j) {
        c += (int64_t)a.l[j] - (int64_t)k * (int64_t)Fp28Params::MOD[j];
        low |= (uint32_t)c & (uint32_t)FP28_MASK;
        c >>= 28;
    }
    c += (int64_t)a.l[13] - (int64_t)k * (int64_t)Fp28Params::MOD[13];
    return low == 0 && c == 0;
}

/* R^2 / x (mod p), R = 2^384, for a canonical x != 0 of the 32-bit form: the inverse of a Montgomery representative,
 * in Montgomery form.  Binary GCD with word-sized batches of steps (Pornin, "Optimized Binary GCD for Modular
 * Inversion", 2020) on 28-bit limbs.  Invariants a = u x, b = v x (mod p), a and b non-negative.  A round runs 28
 * halving / subtracting steps on 64-bit approximations of (a, b) -- their 28 low bits, which decide the parities
 * exactly, and the 36 bits below the top bit of a | b, which decide the comparisons -- while recording the steps
 * as a 2 x 2 integer matrix, then applies the matrix once to (a, b) (an exact division by 2^28: the lowest limb of
 * the sums is zero and is dropped; a negative result is negated together with its matrix row) and to (u, v) (one
 * Montgomery step of a limb, i.e. a division by 2^28 modulo p).  u and v stay unreduced with a signed top limb:
 * a round adds at most p to their magnitude.  After 2 len(p) - 1 steps a = 0 and b = 1, so x^-1 = v; further
 * rounds change nothing.  The product with 2^1168 leaves the 28-bit form of R^2 / x.
 * Signed multiply-adds and no sign or carry bookkeeping in the updates: about 1500 vector instructions a round
 * (700 of them the 28 steps) where the 32-bit version (fe_inv_gcd, kept for Fr and the host) takes 2000.  For one lane
 * that inverts by itself, the end of an update's path; normalisation inverts by whole waves (fp28_inv_wave). */
TC_HD fp_t fp_inv28(const fp_t& x) {
    constexpr int N = 14, K = 28;
    int32_t a[N], b[N], u[N], v[N];
#pragma unroll
    for (int j = 0; j < N; ++j) {
        const int o = 28 * j, w = o >> 5, sh = o & 31;
        uint32_t lo = x.l[w], hi = w + 1 < 12 ? x.l[w + 1] : 0u;
        uint32_t t = sh ? (lo >> sh) | (hi << (32 - sh)) : lo;
        a[j] = (int32_t)(t & (uint32_t)FP28_MASK);
        b[j] = Fp28Params::MOD[j];
        u[j] = 0;
        v[j] = 0;
    }
    u[0] = 1;
    for (int round = 0; round < Fp28Params::GCD_ROUNDS; ++round) {
        /* the three limbs from the highest one in which a | b has a bit, if that lies above limb 1 */
        int32_t ctop = a[N - 1] | b[N - 1];
        int32_t a2 = a[N - 1], a1 = a[N - 2], a0 = a[N - 3], b2 = b[N - 1], b1 = b[N - 2], b0 = b[N - 3];
        bool found = ctop != 0;
#pragma unroll
        for (int i = N - 2; i >= 2; --i) {
            int32_t c = a[i] | b[i];
            bool take = !found && c != 0;
            ctop = take ? c : ctop;
            a2 = take ? a[i] : a2; a1 = take ? a[i - 1] : a1; a0 = take ? a[i - 2] : a0;
            b2 = take ? b[i] : b2; b1 = take ? b[i - 1] : b1; b0 = take ? b[i - 2] : b0;
            found = found || c != 0;
        }
        uint64_t xa, xb;
        if (!found) {                                             /* both fit in 56 bits: exact */
            xa = (uint64_t)(uint32_t)a[0] | ((uint64_t)(uint32_t)a[1] << 28);
            xb = (uint64_t)(uint32_t)b[0] | ((uint64_t)(uint32_t)b[1] << 28);
        } else {
            int s = __builtin_clz((uint32_t)ctop) - 4;            /* leading zeros inside the 28-bit limb */
            uint64_t va = ((uint64_t)(uint32_t)a2 << 36) | ((uint64_t)(uint32_t)a1 << 8) | ((uint32_t)a0 >> 20);
            uint64_t vb = ((uint64_t)(uint32_t)b2 << 36) | ((uint64_t)(uint32_t)b1 << 8) | ((uint32_t)b0 >> 20);
            xa = (uint64_t)(uint32_t)a[0] | ((va >> (28 - s)) << 28);
            xb = (uint64_t)(uint32_t)b[0] | ((vb >> (28 - s)) << 28);
        }
        int32_t f0 = 1, g0 = 0, f1 = 0, g1 = 1;
        for (int j = 0; j < K; ++j) {
            bool odd = (xa & 1ull) != 0;
            bool swap = odd && xa < xb;
            uint64_t ta = swap ? xb : xa, tb = swap ? xa : xb;
            int32_t tf0 = swap ? f1 : f0, tf1 = swap ? f0 : f1, tg0 = swap ? g1 : g0, tg1 = swap ? g0 : g1;
            ta -= odd ? tb : 0ull;
            tf0 -= odd ? tf1 : 0;
            tg0 -= odd ? tg1 : 0;
            xa = ta >> 1;
            xb = tb;
            f0 = tf0;
            g0 = tg0;
            f1 = (int32_t)((uint32_t)tf1 << 1);               /* doubling of a possibly negative factor */
            g1 = (int32_t)((uint32_t)tg1 << 1);
        }
        /* (a, b) <- (a f0 + b g0, a f1 + b g1) / 2^28, exact */
        {
            int32_t na[N], nb[N];
            int64_t ca = 0, cb = 0;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                ca += (int64_t)f0 * (int64_t)a[i] + (int64_t)g0 * (int64_t)b[i];
                cb += (int64_t)f1 * (int64_t)a[i] + (int64_t)g1 * (int64_t)b[i];
                if (i > 0) {
                    na[i - 1] = (int32_t)((uint32_t)ca & (uint32_t)FP28_MASK);
                    nb[i - 1] = (int32_t)((uint32_t)cb & (uint32_t)FP28_MASK);
                }
                ca >>= 28;
                cb >>= 28;
            }
            na[N - 1] = (int32_t)ca;
            nb[N - 1] = (int32_t)cb;
            bool nega = na[N - 1] < 0, negb = nb[N - 1] < 0;
            int32_t c1 = 0, c2 = 0;
#pragma unroll
            for (int i = 0; i < N - 1; ++i) {
                int32_t t1 = (nega ? -na[i] : na[i]) + c1, t2 = (negb ? -nb[i] : nb[i]) + c2;
                a[i] = t1 & FP28_MASK;
                b[i] = t2 & FP28_MASK;
                c1 = t1 >> 28;
                c2 = t2 >> 28;
            }
            a[N - 1] = (nega ? -na[N - 1] : na[N - 1]) + c1;
            b[N - 1] = (negb ? -nb[N - 1] : nb[N - 1]) + c2;
            if (nega) { f0 = -f0; g0 = -g0; }
            if (negb) { f1 = -f1; g1 = -g1; }
        }
        /* (u, v) <- (u f0 + v g0, u f1 + v g1) / 2^28 mod p */
        {
            int64_t cu = (int64_t)f0 * (int64_t)u[0] + (int64_t)g0 * (int64_t)v[0];
            int64_t cv = (int64_t)f1 * (int64_t)u[0] + (int64_t)g1 * (int64_t)v[0];
            int32_t qu = (int32_t)(((uint32_t)cu * (uint32_t)Fp28Params::NINV) & (uint32_t)FP28_MASK);
            int32_t qv = (int32_t)(((uint32_t)cv * (uint32_t)Fp28Params::NINV) & (uint32_t)FP28_MASK);
            cu = (cu + (int64_t)qu * (int64_t)Fp28Params::MOD[0]) >> 28;
            cv = (cv + (int64_t)qv * (int64_t)Fp28Params::MOD[0]) >> 28;
            int32_t nu[N], nv[N];
#pragma unroll
            for (int i = 1; i < N; ++i) {
                cu += (int64_t)f0 * (int64_t)u[i] + (int64_t)g0 * (int64_t)v[i] + (int64_t)qu * (int64_t)Fp28Params::MOD[i];
                cv += (int64_t)f1 * (int64_t)u[i] + (int64_t)g1 * (int64_t)v[i] + (int64_t)qv * (int64_t)Fp28Params::MOD[i];
                nu[i - 1] = (int32_t)((uint32_t)cu & (uint32_t)FP28_MASK);
                nv[i - 1] = (int32_t)((uint32_t)cv & (uint32_t)FP28_MASK);
                cu >>= 28;
                cv >>= 28;
            }
            nu[N - 1] = (int32_t)cu;
            nv[N - 1] = (int32_t)cv;
#pragma unroll
            for (int i = 0; i < N; ++i) { u[i] = nu[i]; v[i] = nv[i]; }
        }
    }
    fp28 r, fix;
#pragma unroll
    for (int i = 0; i < N; ++i) { r.l[i] = v[i]; fix.l[i] = Fp28Params::INV_FIX[i]; }
    return fp28_to_fp(fp28_mul(r, fix));
}

/* ---- inversion of one value by a whole wave: the division steps ---------------------------------
 * (what fp28_inv_wave falls back to)
 * Division steps (Bernstein, Yang, "Fast constant-time gcd computation and modular inversion", 2019) in the variant
 * that starts at delta = 1/2; D = delta - 1/2.  A step: if D >= 0 and g odd (f, g, D) <- (g, (g - f) / 2, -D), else
 * (f, g, D) <- (f, (g + (g mod 2) f) / 2, D + 1).  Only the low bits of f and g decide, so 28 steps need the lowest
 * limb alone and their matrix, entries of at most 2^28 in absolute row sum, is applied to the whole numbers
 * afterwards.  Several steps at a time, in the order in which the variable-time inversion of libsecp256k1 (Dettman,
 * Wuille, 2021) takes them: zeros of g are stripped by a count, and while D < 0 no swap can come, so up
 * to six low bits of g are cleared by one multiple of f (-1 / f = f (f f - 2) mod 2^6 for odd f); the start at
 * delta = 1/2 is described there too.
 * About 9.5 passes of the loop per 28 steps, and 28 rounds for a 381-bit modulus (measured on random values). */
TC_HD void fp28_divsteps(int32_t& D, uint32_t f, uint32_t g, int32_t (&m)[4]) {
    uint32_t u = 1, v = 0, q = 0, r = 1;
    int32_t left = 28;
    for (;;) {
        int32_t z = __builtin_ctz(g | (1u << left));
        g >>= z;
        u <<= z;
        v <<= z;
        D += z;
        left -= z;
        if (left == 0) break;
        if (D >= 0) {
            D = -D - 1;
            uint32_t t = f; f = g; g = 0u - t;
            t = u; u = q; q = 0u - t;
            t = v; v = r; r = 0u - t;
        }
        int32_t bits = D > -6 ? -D : 6;
        bits = bits < left ? bits : left;
        uint32_t w = (g * f * (f * f - 2u)) & ((1u << bits) - 1u);
        g += f * w;
        q += u * w;
        r += v * w;
    }
    m[0] = (int32_t)u; m[1] = (int32_t)v; m[2] = (int32_t)q; m[3] = (int32_t)r;
}
/* The loop leaves as soon as the limbs of g are zero, after at most 32 + 14 rounds.
 * 32: from f = p, |g| <= 2 p no more than 881 steps leave a g != 0 (for every D the convex hull of the (f, g) that some
 * sequence of parities reaches, cut at |g| >= 1, until all hulls are empty; the same count for 256 bits and |g| <= f
 * gives 591, one more than published for these steps).
 * 14: g = 0 may stand in limbs that cancel.  The lazily carried limbs are in [-2, 2^28 + 2], so such limbs are
 * l_j = 2^28 k_(j+1) - k_j with k_j in {0, 1}, and each round settles one of them at least. */
static constexpr int FP28_INV_MAX_ROUNDS = 48;
/* The inverse of an element in the form of this header (R^2 / x on the limbs, R = 2^392), x with normal limbs and
 * |x| < 2 p; 0 for 0, and x no other multiple of p.  All lanes of a wave hold the same x and get the same result.
 * Row k = lane / 16 of the wave holds f, g, d, e (k = 0 .. 3), a lane one limb: f = d x, g = e x (mod p).  A round runs
 * the steps once for the wave, on scalar registers (what decides is the same for all lanes), and then spends some
 * thirty vector instructions on the four updates: the limbs of the partner row (permlane16 swap), two
 * multiply-adds, q p for the rows of d and e (a division by 2^28 modulo p), the shift by one limb and one lazy pass of
 * carries (dpp row shifts), limbs staying within [-2, 2^28 + 2] and the sign in limb 13.  d and e grow by at most p a
 * round, 48 p at the end.
 * Bound by the latency of the scalar steps, 30 us. */
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ fp28 fp28_inv_divsteps(const fp28& x) {
    const uint32_t lane = threadIdx.x & 63u, row = lane >> 4, limb = lane & 15u;
    /* selections by mask: written with ?: they become forty branches */
    const int32_t row_f = row == 0 ? -1 : 0, row_g = row == 1 ? -1 : 0, row_d = row == 2 ? -1 : 0, row_e = row == 3 ? -1 : 0;
    int32_t s = 0, p = 0;
#pragma unroll
    for (int j = 0; j < 14; ++j) {
        const int32_t here = limb == (uint32_t)j ? -1 : 0;
        p |= here & Fp28Params::MOD[j];
        s |= here & ((row_g & x.l[j]) | (row_e & Fp28Params::INV_START[j]));
    }
    s |= row_f & p;
    const bool odd_row = (row & 1u) != 0, low = limb < 13u;
    int32_t D = 0;
    for (int round = 0; round < FP28_INV_MAX_ROUNDS; ++round) {
        if ((__ballot(s != 0) & 0xFFFF0000ull) == 0) break;
        int32_t m[4];
        fp28_divsteps(D, (uint32_t)__builtin_amdgcn_readlane(s, 0), (uint32_t)__builtin_amdgcn_readlane(s, 16), m);
        auto pair = __builtin_amdgcn_permlane16_swap((uint32_t)s, (uint32_t)s, false, false);
        int32_t even = (int32_t)pair[0], odd = (int32_t)pair[1];     /* rows (0 0 2 2) and (1 1 3 3) */
        int32_t ma = odd_row ? m[2] : m[0], mb = odd_row ? m[3] : m[1];
        int64_t t = (int64_t)ma * (int64_t)even + (int64_t)mb * (int64_t)odd;
        int32_t qd = (int32_t)(((uint32_t)__builtin_amdgcn_readlane((int32_t)t, 32) * (uint32_t)Fp28Params::NINV) & (uint32_t)FP28_MASK);
        int32_t qe = (int32_t)(((uint32_t)__builtin_amdgcn_readlane((int32_t)t, 48) * (uint32_t)Fp28Params::NINV) & (uint32_t)FP28_MASK);
        int32_t qr = (row_d & qd) | (row_e & qe);
        t += (int64_t)qr * (int64_t)p;
        int32_t lo = (int32_t)((uint32_t)t & (uint32_t)FP28_MASK);
        /* dpp row_shl:1 = 0x101: limb i takes limb i + 1; row_shr:1 = 0x111: limb i takes limb i - 1; zeros enter */
        int32_t n = (int32_t)(t >> 28) + __builtin_amdgcn_update_dpp(0, lo, 0x101, 0xF, 0xF, true);
        int32_t c = low ? n >> 28 : 0;
        s = (low ? n & FP28_MASK : n) + __builtin_amdgcn_update_dpp(0, c, 0x111, 0xF, 0xF, true);
    }
    /* f = +-1 and f = d x: d if f = 1 (mod 4), else -d */
    const bool neg = (__builtin_amdgcn_readlane(s, 0) & 3) == 3;
    fp28 r;
#pragma unroll
    for (int j = 0; j < 14; ++j) {
        int32_t l = __builtin_amdgcn_readlane(s, 32 + j);
        r.l[j] = neg ? -l : l;
    }
    return fp28_carry(r);
}
#elif defined(__HIPCC__)
__device__ fp28 fp28_inv_divsteps(const fp28& x);
#else
/* the same rounds with the lanes of the wave written out as an array (host build of the kernels) */
inline fp28 fp28_inv_divsteps(const fp28& x) {
    int32_t s[4][16] = {}, p[16] = {};
    for (int j = 0; j < 14; ++j) {
        s[0][j] = p[j] = Fp28Params::MOD[j];
        s[1][j] = x.l[j];
        s[3][j] = Fp28Params::INV_START[j];
    }
    int32_t D = 0;
    for (int round = 0; round < FP28_INV_MAX_ROUNDS; ++round) {
        int32_t any = 0;
        for (int j = 0; j < 16; ++j) any |= s[1][j];
        if (!any) break;
        int32_t m[4], n[4][16], c[16];
        fp28_divsteps(D, (uint32_t)s[0][0], (uint32_t)s[1][0], m);
        for (int k = 0; k < 4; ++k) {
            int64_t t[16];
            for (int j = 0; j < 16; ++j) t[j] = (int64_t)m[2 * (k & 1)] * s[k & 2][j] + (int64_t)m[2 * (k & 1) + 1] * s[(k & 2) + 1][j];
            int32_t q = k < 2 ? 0 : (int32_t)(((uint32_t)t[0] * (uint32_t)Fp28Params::NINV) & (uint32_t)FP28_MASK);
            for (int j = 0; j < 16; ++j) t[j] += (int64_t)q * p[j];
            for (int j = 0; j < 16; ++j) n[k][j] = (int32_t)(t[j] >> 28) + (j < 15 ? (int32_t)((uint32_t)t[j + 1] & (uint32_t)FP28_MASK) : 0);
            for (int j = 0; j < 16; ++j) {
                c[j] = j < 13 ? n[k][j] >> 28 : 0;
                n[k][j] = j < 13 ? n[k][j] & FP28_MASK : n[k][j];
            }
            for (int j = 1; j < 16; ++j) n[k][j] += c[j - 1];
        }
        memcpy(s, n, sizeof s);
    }
    const bool neg = (s[0][0] & 3) == 3;
    fp28 r;
    for (int j = 0; j < 14; ++j) r.l[j] = neg ? -s[2][j] : s[2][j];
    return fp28_carry(r);
}
#endif

/* ---- inversion of one value by a whole wave: Euclid's algorithm in batches ----------------------
 * Lehmer's idea (1938): quotients are found on approximations, here doubles of the upper 112 bits of both numbers, and up to a dozen or two of
 * them are collected in a 2 x 2 matrix of 28-bit entries before it is applied to the numbers and their cofactors.  Whatever the quotients are, a
 * matrix of determinant 1 keeps the greatest common divisor and a = s x, b = t x (mod p), so an inexact quotient costs
 * progress at most, no correctness: quotients are rounded products with an approximate reciprocal.  Row k of the wave holds a, b, s, t
 * (k = 0 .. 3; a = p, b = x, s = 0, t = 1 at first), a lane one limb, lazily carried to [-2, 2^28 + 2], the sign in limb 13.  An upper bound of
 * the lengths of a and b says which four limbs to look at; limbs above them only continue the sign.  It ends with one of the
 * two numbers 0 and the other 1 or -1, whose cofactor is the inverse.  Numbers that a batch cannot bring closer (a quotient of more than 27 bits), more
 * than INV_BATCHES of them, or an end other than that: the division steps take over (x = 0 among them).
 * About 16 batches of 10 quotients.  Bound by latency, a chain of four double-precision operations a quotient; a normalisation with one
 * point to a wave 36 -> 22.6 us (one quotient to a comparison and a branch: 27). */
static constexpr int FP28_INV_BATCHES = 30;
TC_HD double fp28_quotient(double A, double B) {
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_rint(A * __builtin_amdgcn_rcp(B));
#else
    return __builtin_rint(A * (1.0 / B));
#endif
}
/* Quotients on (A, B) until a cofactor would pass 2^27, two at a time (a comparison and a branch cost as much as a quotient), then one more if it
 * fits; m = (u0 v0 u1 v1): the numbers become u0 a + v0 b, u1 a + v1 b.  Returns whether they came closer. */
TC_HD bool fp28_euclid_batch(double& A, double& B, int32_t (&m)[4]) {
    constexpr double LIMIT = 134217728.0;
    double u0 = 1.0, v0 = 0.0, u1 = 0.0, v1 = 1.0;
    for (int i = 0; i < 64; ++i) {
        const double q = fp28_quotient(A, B), r = __builtin_fma(-q, B, A), nu = __builtin_fma(-q, u1, u0), nv = __builtin_fma(-q, v1, v0);
        const double p = fp28_quotient(B, r), t = __builtin_fma(-p, r, B), mu = __builtin_fma(-p, nu, u1), mv = __builtin_fma(-p, nv, v1);
        /* (also false for the infinities and the not-a-number that a zero leads to) */
        if (!((__builtin_fabs(nu) + __builtin_fabs(nv)) + (__builtin_fabs(mu) + __builtin_fabs(mv)) <= LIMIT)) break;
        A = r; B = t;
        u0 = nu; v0 = nv; u1 = mu; v1 = mv;
    }
    const double q = fp28_quotient(A, B), nu = __builtin_fma(-q, u1, u0), nv = __builtin_fma(-q, v1, v0);
    if (__builtin_fabs(nu) + __builtin_fabs(nv) <= LIMIT) {
        const double r = __builtin_fma(-q, B, A);
        A = B; B = r;
        u0 = u1; v0 = v1; u1 = nu; v1 = nv;
    }
    m[0] = (int32_t)u0; m[1] = (int32_t)v0; m[2] = (int32_t)u1; m[3] = (int32_t)v1;
    return __builtin_fabs(u0) + __builtin_fabs(v0) + __builtin_fabs(u1) + __builtin_fabs(v1) > 2.0;
}
/* four limbs as a double: h 2^56 + l, h of 56 bits and a sign; with l of the sign of h, so that a small negative number is exact */
TC_HD double fp28_window(int32_t l3, int32_t l2, int32_t l1, int32_t l0) {
    const int64_t h = (int64_t)((uint64_t)((int64_t)l3 * (1 << 28) + l2) << 8) >> 8, l = (int64_t)l1 * (1 << 28) + l0;
    const int64_t up = h < 0 ? 1 : 0;
    return __builtin_fma((double)(h + up), 72057594037927936.0, (double)(l - up * ((int64_t)1 << 56)));
}
/* which limb is the upper one of the four for numbers below 2^bits, and the bound after a batch: what the approximations say, and for their errors
 * 2^27 times a double's rounding of the larger of the numbers before (`was`) and the limbs left out */
TC_HD int fp28_window_top(int bits) {
    const int top = (bits + 29) / 28 - 1;
    return top < 3 ? 3 : top > 13 ? 13 : top;
}
TC_HD int fp28_bits_after(double A, double B, double was, int top) {
    const double bound = __builtin_fmax(__builtin_fabs(A), __builtin_fabs(B)) + was * 5.9604644775390625e-08 + (top > 3 ? 1073741824.0 : 0.0);
    union { double d; uint64_t u; } e;
    e.d = bound;
    return 28 * (top - 3) + (int)(e.u >> 52) - 1022;
}
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __forceinline__ fp28 fp28_inv_wave(const fp28& x) {
    const uint32_t lane = threadIdx.x & 63u, row = lane >> 4, limb = lane & 15u;
    const int32_t row_a = row == 0 ? -1 : 0, row_b = row == 1 ? -1 : 0;
    int32_t s = (row == 3 && limb == 0) ? 1 : 0;
#pragma unroll
    for (int j = 0; j < 14; ++j) {
        const int32_t here = limb == (uint32_t)j ? -1 : 0;
        s |= here & ((row_a & Fp28Params::MOD[j]) | (row_b & x.l[j]));
    }
    const bool odd_row = (row & 1u) != 0, low = limb < 13u;
    int bits = 382;
    double A = 0.0, B = 0.0;
    bool done = false;
    for (int batch = 0; batch < FP28_INV_BATCHES; ++batch) {
        const int top = fp28_window_top(bits);
        A = fp28_window(__builtin_amdgcn_readlane(s, top), __builtin_amdgcn_readlane(s, top - 1), __builtin_amdgcn_readlane(s, top - 2), __builtin_amdgcn_readlane(s, top - 3));
        B = fp28_window(__builtin_amdgcn_readlane(s, 16 + top), __builtin_amdgcn_readlane(s, 15 + top), __builtin_amdgcn_readlane(s, 14 + top), __builtin_amdgcn_readlane(s, 13 + top));
        if (top == 3 && (A == 0.0 || B == 0.0)) { done = true; break; }
        const double was = __builtin_fmax(__builtin_fabs(A), __builtin_fabs(B));
        int32_t m[4];
        if (!fp28_euclid_batch(A, B, m)) break;
        bits = fp28_bits_after(A, B, was, top);
        auto pair = __builtin_amdgcn_permlane16_swap((uint32_t)s, (uint32_t)s, false, false);
        const int32_t even = (int32_t)pair[0], odd = (int32_t)pair[1];
        const int32_t ma = __builtin_amdgcn_readfirstlane(m[0]), mb = __builtin_amdgcn_readfirstlane(m[1]);
        const int32_t mc = __builtin_amdgcn_readfirstlane(m[2]), md = __builtin_amdgcn_readfirstlane(m[3]);
        const int64_t t = (int64_t)(odd_row ? mc : ma) * (int64_t)even + (int64_t)(odd_row ? md : mb) * (int64_t)odd;
        const int32_t hi = low ? (int32_t)(t >> 28) : 0;
        const int32_t n = (low ? (int32_t)((uint32_t)t & (uint32_t)FP28_MASK) : (int32_t)t) + __builtin_amdgcn_update_dpp(0, hi, 0x111, 0xF, 0xF, true);
        const int32_t c = low ? n >> 28 : 0;
        s = (low ? n & FP28_MASK : n) + __builtin_amdgcn_update_dpp(0, c, 0x111, 0xF, 0xF, true);
    }
    if (!done || __builtin_fabs(A + B) != 1.0) return fp28_inv_divsteps(x);
    const bool second = A == 0.0, neg = A + B < 0.0;
    fp28 r, scale;
#pragma unroll
    for (int j = 0; j < 14; ++j) {
        const int32_t l = __builtin_amdgcn_readlane(s, (second ? 48 : 32) + j);
        r.l[j] = neg ? -l : l;
        scale.l[j] = Fp28Params::INV_SCALE[j];
    }
    return fp28_mul(fp28_carry(r), scale);
}
#elif defined(__HIPCC__)
__device__ fp28 fp28_inv_wave(const fp28& x);
#else
/* the same with the lanes of the wave written out as an array (host build of the kernels); `batches` for the tests */
inline fp28 fp28_inv_wave(const fp28& x, int* batches = nullptr) {
    int32_t s[4][14] = {};
    for (int j = 0; j < 14; ++j) {
        s[0][j] = Fp28Params::MOD[j];
        s[1][j] = x.l[j];
    }
    s[3][0] = 1;
    int bits = 382;
    double A = 0.0, B = 0.0;
    bool done = false;
    if (batches) *batches = -1;
    for (int batch = 0; batch < FP28_INV_BATCHES; ++batch) {
        const int top = fp28_window_top(bits);
        A = fp28_window(s[0][top], s[0][top - 1], s[0][top - 2], s[0][top - 3]);
        B = fp28_window(s[1][top], s[1][top - 1], s[1][top - 2], s[1][top - 3]);
        if (top == 3 && (A == 0.0 || B == 0.0)) {
            done = true;
            if (batches) *batches = batch;
            break;
        }
        const double was = __builtin_fmax(__builtin_fabs(A), __builtin_fabs(B));
        int32_t m[4], n[4][14], c[4][14];
        if (!fp28_euclid_batch(A, B, m)) break;
        bits = fp28_bits_after(A, B, was, top);
        for (int k = 0; k < 4; ++k)
            for (int j = 0, hi = 0; j < 14; ++j) {
                const int64_t t = (int64_t)m[2 * (k & 1)] * s[k & 2][j] + (int64_t)m[2 * (k & 1) + 1] * s[(k & 2) + 1][j];
                n[k][j] = (int32_t)((j < 13 ? (uint32_t)t & (uint32_t)FP28_MASK : (uint32_t)t) + (uint32_t)hi);
                hi = (int32_t)(t >> 28);
            }
        for (int k = 0; k < 4; ++k)
            for (int j = 0; j < 14; ++j) {
                c[k][j] = j < 13 ? n[k][j] >> 28 : 0;
                s[k][j] = (j < 13 ? n[k][j] & FP28_MASK : n[k][j]) + (j ? c[k][j - 1] : 0);
            }
    }
    if (!done || __builtin_fabs(A + B) != 1.0) {
        if (batches) *batches = -1;
        return fp28_inv_divsteps(x);
    }
    const int k = A == 0.0 ? 3 : 2;
    fp28 r, scale;
    for (int j = 0; j < 14; ++j) {
        r.l[j] = A + B < 0.0 ? -s[k][j] : s[k][j];
        scale.l[j] = Fp28Params::INV_SCALE[j];
    }
    return fp28_mul(fp28_carry(r), scale);
}
#endif

}  // namespace tc
