/*
 * A third form of Fp, for the loop that adds the points of a bucket: 13 signed limbs of 30 bits, Montgomery radix 2^390.
 *
 * What bounds that loop is the number of vector instructions (a SIMD of the full chip issues one every four clocks whatever it
 * is), and one limb less than the 28-bit form means 338 multiply-adds a product instead of 392 and twenty-four columns instead
 * of twenty-seven.  A column of twelve terms a_i b_j, as many q_i p_j and the carry fits a signed 64-bit sum only if the limbs of one
 * factor and of q and p are balanced, i.e. in [-2^29, 2^29); the limbs of the other may be of 30 bits either sign:
 *   12 2^59 + 2^29 sum |p_j| + 2^35 < 2^63        (and 24 2^58 in place of 12 2^59 for the difference of two balanced products),
 * p cut into balanced limbs having sum |p_j| < 12.41 2^28.  The top limb (below 2^27, values within 64 p) adds little.
 * A product can add multiples of other elements to its result while the digits are taken: a difference "product less known element"
 * costs a multiply-add per limb and comes out balanced.
 *
 * Values are signed: with q balanced a product is within |v| / 2^390 + 0.52 p of zero, and 2^390 = 630 p.
 */
#pragma once
#include "field28.h"

namespace tc {

struct fp30 {
    int32_t l[13];
};
static constexpr uint32_t FP30_MASK = (1u << 30) - 1u;

/* the bits of a canonical a moved up by six places (a 2^6 stands for the same element under the radix 2^390), 30 to a limb */
TC_HD fp30 fp30_from_fp(const fp_t& a) {
    fp30 r;
    r.l[0] = (int32_t)((a.l[0] << 6) & FP30_MASK);
#pragma unroll
    for (int j = 1; j < 13; ++j) {
        const int o = 30 * j - 6, w = o >> 5, sh = o & 31;
        const uint64_t two = ((uint64_t)(w + 1 < 12 ? a.l[w + 1] : 0u) << 32) | a.l[w];
        r.l[j] = (int32_t)((uint32_t)(two >> sh) & FP30_MASK);
    }
    return r;
}
TC_HD fp30 fp30_one() {
    fp30 r;
#pragma unroll
    for (int j = 0; j < 13; ++j) r.l[j] = Fp30Params::ONE[j];
    return r;
}
TC_HD fp30 fp30_sub(const fp30& a, const fp30& b) {
    fp30 r;
#pragma unroll
    for (int j = 0; j < 13; ++j) r.l[j] = a.l[j] - b.l[j];
    return r;
}
TC_HD fp30 fp30_neg(const fp30& a) {
    fp30 r;
#pragma unroll
    for (int j = 0; j < 13; ++j) r.l[j] = -a.l[j];
    return r;
}
/* same value, balanced limbs (limbs within 2^30.5 in) */
TC_HD fp30 fp30_balance(const fp30& a) {
    fp30 r;
    int32_t c = 0;
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        const int32_t s = a.l[j] + c + (1 << 29);
        r.l[j] = (int32_t)((uint32_t)s & FP30_MASK) - (1 << 29);
        c = s >> 30;
    }
    r.l[12] = a.l[12] + c;
    return r;
}
TC_HD int32_t fp30_factor(int32_t m) {
#if defined(__HIP_DEVICE_COMPILE__)
    asm("" : "+s"(m));                 /* a multiply-add each, not three instructions of 64-bit subtraction */
#endif
    return m;
}
/* a b 2^-390 (or a^2, or a b - c e) + m1 f1 + m2 f2, balanced limbs, the columns as chains (mac_chain) */
enum { FP30_MUL = 0, FP30_SQR = 1, FP30_MUL_SUB = 2 };
template <int MODE, int FOLD>
TC_HD fp30 fp30_mont(const fp30& a, const fp30& b, const fp30& c, const fp30& e, const fp30& f1, int32_t m1, const fp30& f2, int32_t m2) {
    int32_t q[13], d[13];
    fp30 r;
    int64_t acc = 0;
    if (MODE == FP30_SQR) {
#pragma unroll
        for (int i = 0; i < 13; ++i) d[i] = a.l[i] + a.l[i];        /* cross terms once, with a doubled operand */
    }
    if (MODE == FP30_MUL_SUB) {
#pragma unroll
        for (int i = 0; i < 13; ++i) d[i] = -c.l[i];
    }
#pragma unroll
    for (int k = 0; k < 25; ++k) {
        const int lo = k < 13 ? 0 : k - 12, hi = k < 13 ? k : 12;
        if (MODE == FP30_SQR) {
#pragma unroll
            for (int i = lo; i < k - i; ++i) mac_chain(acc, d[i], a.l[k - i]);
            if ((k & 1) == 0) mac_chain(acc, a.l[k / 2], a.l[k / 2]);
        } else {
#pragma unroll
            for (int i = lo; i <= hi; ++i) mac_chain(acc, a.l[i], b.l[k - i]);
        }
        if (MODE == FP30_MUL_SUB) {
#pragma unroll
            for (int i = lo; i <= hi; ++i) mac_chain(acc, d[i], e.l[k - i]);
        }
        if (k < 13) {
#pragma unroll
            for (int i = 0; i < k; ++i) mac_chain(acc, q[i], Fp30Params::MOD[k - i]);
            q[k] = (int32_t)(((uint32_t)acc * (uint32_t)Fp30Params::NINV) << 2) >> 2;
            mac_chain(acc, q[k], Fp30Params::MOD[0]);
        } else {
#pragma unroll
            for (int i = lo; i <= 12; ++i) mac_chain(acc, q[i], Fp30Params::MOD[k - i]);
            if (FOLD > 0) mac_chain(acc, f1.l[k - 13], m1);
            if (FOLD > 1) mac_chain(acc, f2.l[k - 13], m2);
            r.l[k - 13] = (int32_t)((uint32_t)acc << 2) >> 2;         /* the digit nearest to the column, and the carry that goes with it */
            acc += (int64_t)1 << 29;
        }
        acc >>= 30;                        /* arithmetic: the sum is signed */
    }
    r.l[12] = (int32_t)acc;
    if (FOLD > 0) r.l[12] += f1.l[12] * m1;
    if (FOLD > 1) r.l[12] += f2.l[12] * m2;
    return r;
}
TC_HD fp30 fp30_mul(const fp30& a, const fp30& b) { return fp30_mont<FP30_MUL, 0>(a, b, a, a, a, 0, a, 0); }
TC_HD fp30 fp30_sqr(const fp30& a) { return fp30_mont<FP30_SQR, 0>(a, a, a, a, a, 0, a, 0); }
TC_HD fp30 fp30_mul_less(const fp30& a, const fp30& b, const fp30& f) { return fp30_mont<FP30_MUL, 1>(a, b, a, a, f, fp30_factor(-1), f, 0); }
TC_HD fp30 fp30_mul_sub(const fp30& a, const fp30& b, const fp30& c, const fp30& e) { return fp30_mont<FP30_MUL_SUB, 0>(a, b, c, e, a, 0, a, 0); }

/* 12 words from the bits 6 .. 389 of non-negative limbs of 30 bits */
TC_HD fp_t fp30_pack_shr6(const uint32_t (&u)[13]) {
    fp_t r;
#pragma unroll
    for (int i = 0; i < 12; ++i) {
        const int o = 32 * i + 6, j = o / 30, sh = o % 30;
        uint32_t w = u[j] >> sh;
        if (j + 1 < 13) w |= u[j + 1] << (30 - sh);
        if (60 - sh < 32 && j + 2 < 13) w |= u[j + 2] << (60 - sh);
        r.l[i] = w;
    }
    return r;
}
/* fp30_from_fp undone */
TC_HD fp_t fp30_recut_to_fp(const fp30& a) {
    uint32_t u[13];
#pragma unroll
    for (int j = 0; j < 13; ++j) u[j] = (uint32_t)a.l[j];
    return fp30_pack_shr6(u);
}
/* The canonical element of the 32-bit form (radix 2^384) for a value within 64 p: a Montgomery step of the six bits between the
 * radices, with a multiple q p, q in 64 .. 127, so that the sum is not negative; (v + q p) / 2^6 < 3 p. */
TC_HD fp_t fp30_to_fp(const fp30& a) {
    const int32_t q = (int32_t)((((uint32_t)a.l[0] * (uint32_t)Fp30Params::NINV) & 63u) + 64u);
    uint32_t u[13];
    int64_t c = 0;
#pragma unroll
    for (int j = 0; j < 12; ++j) {
        c += (int64_t)q * (int64_t)Fp30Params::MOD[j] + (int64_t)a.l[j];
        u[j] = (uint32_t)c & FP30_MASK;
        c >>= 30;
    }
    u[12] = (uint32_t)(int32_t)(c + (int64_t)q * (int64_t)Fp30Params::MOD[12] + (int64_t)a.l[12]);
    return fe_reduce_once<FpParams>(fe_reduce_once<FpParams>(fp30_pack_shr6(u), 0u), 0u);
}
/* as a real function on the device: for the end of a kernel whose loop must keep its registers */
#if defined(__HIP_DEVICE_COMPILE__)
__device__ __attribute__((noinline)) fp_t fp30_to_fp_call(i32x4 a0, i32x4 a1, i32x4 a2, int32_t a3) {
    fp30 a;
    a.l[0] = a0.x; a.l[1] = a0.y; a.l[2] = a0.z; a.l[3] = a0.w; a.l[4] = a1.x; a.l[5] = a1.y; a.l[6] = a1.z; a.l[7] = a1.w;
    a.l[8] = a2.x; a.l[9] = a2.y; a.l[10] = a2.z; a.l[11] = a2.w; a.l[12] = a3;
    return fp30_to_fp(a);
}
__device__ __forceinline__ fp_t fp30_to_fp_outlined(const fp30& a) {
    return fp30_to_fp_call(i32x4{a.l[0], a.l[1], a.l[2], a.l[3]}, i32x4{a.l[4], a.l[5], a.l[6], a.l[7]}, i32x4{a.l[8], a.l[9], a.l[10], a.l[11]}, a.l[12]);
}
#elif defined(__HIPCC__)
__device__ fp_t fp30_to_fp_outlined(const fp30& a);
__host__ inline fp_t fp30_to_fp_outlined(const fp30& a) { return fp30_to_fp(a); }
#else
inline fp_t fp30_to_fp_outlined(const fp30& a) { return fp30_to_fp(a); }
#endif

/* can a value within K p be a multiple of p?  The first two limbs decide: no multiple is missed, and of the other values all but
 * about (2 K + 1) 2^-60 are told apart */
TC_HD bool fp30_maybe_zero(const fp30& a, uint32_t K) {
    const uint32_t kk = ((uint32_t)a.l[0] * (uint32_t)Fp30Params::PINV + K) & FP30_MASK;
    if (kk > 2u * K) return false;
    const int32_t k = (int32_t)kk - (int32_t)K;
    int64_t c = ((int64_t)a.l[0] - (int64_t)k * (int64_t)Fp30Params::MOD[0]) >> 30;         /* its low 30 bits are zero by the choice of k */
    c += (int64_t)a.l[1] - (int64_t)k * (int64_t)Fp30Params::MOD[1];
    return ((uint32_t)c & FP30_MASK) == 0;
}

/* A running sum in this form (balanced limbs). */
struct g1_xyzz30 {
    fp30 X, Y, ZZ, ZZZ;
};
/* a <- a + (x2, y2), both finite, x2 and y2 with limbs of 30 bits either sign and within 64 p; false (a unusable) when the sum may be a
 * doubling or the identity.  In multiples of p: U2, S2 within 0.7, P and R within 65 in the first addition after a was a point as it
 * comes, 14 from then on, PP within 7.3, PPP and Q 1.3, X3 11.1, D 12.4, Y3 2, ZZ3 and ZZZ3 0.6. */
TC_HD bool xyzz30_madd_regular(g1_xyzz30& a, const fp30& x2, const fp30& y2) {
    const fp30 P = fp30_mul_less(x2, a.ZZ, a.X);
    if (fp30_maybe_zero(P, 128u)) return false;
    const fp30 R = fp30_mul_less(y2, a.ZZZ, a.Y);
    const fp30 PP = fp30_sqr(P);
    const fp30 PPP = fp30_mul(P, PP);
    const fp30 Q = fp30_mul(a.X, PP);
    const fp30 X3 = fp30_mont<FP30_SQR, 2>(R, R, R, R, PPP, fp30_factor(-1), Q, fp30_factor(-2));
    a.Y = fp30_mul_sub(R, fp30_balance(fp30_sub(Q, X3)), a.Y, PPP);
    a.ZZ = fp30_mul(a.ZZ, PP);
    a.ZZZ = fp30_mul(a.ZZZ, PPP);
    a.X = X3;
    return true;
}

}  // namespace tc
