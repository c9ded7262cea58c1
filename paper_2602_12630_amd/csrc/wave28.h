/*
 * Fp and the group law with an element spread over a row of sixteen lanes, for chains of dependent group operations
 * that few lanes of the chip take part in.
 *
 * A lane-wide product (field28.h) is some 460 instructions that a wave issues one after the other: 1.1 us, whether one
 * lane needs the result or 64.  Where a launch has a handful of points to add or one point to double a hundred times
 * over, that latency is all of its time.  Here limb j of an element sits in lane j of a row (the 28-bit limbs of field28.h,
 * radix 2^392, lanes 14 and 15 zero): a step of the Montgomery product is two multiply-adds and five other instructions
 * for all limbs at once, a product about 125 instructions, and the four rows of a wave take the up to four independent
 * products of a group operation side by side.  A point (X, Y, ZZ, ZZZ) is one register, a coordinate to a row; rows
 * are exchanged by permlane swaps, limbs by dpp row shifts and broadcasts: no LDS and no barrier inside an operation.
 * The price is throughput: a wave's worth of lane-wide additions costs a fifth as much per addition.
 *
 * Values are never negative.  Limbs are "normal" below 2^28 + 16 (what products and differences return); sums of up to three
 * may enter a product.  Value bounds, with coordinates below 256 p on entry (a re-cut element is below 2^8 p, results
 * are below 180 p): a product of a and b is below a b / 2521 p + 2 p; a difference is a - b + 128 p, for b below 127 p with limbs
 * below 2^30 - 4.
 *
 * On the host (CPU build of the tests) a wave's register is an array of 64 words and the same steps run over it.
 */
#pragma once
#include "g1.h"
#include "rt.h"

namespace tc {

enum { W28_MP = 0, W28_P = 1, W28_128P = 2, W28_512P = 3, W28_ONE = 4, W28_FROM_PLAIN = 5, W28_TO_PLAIN = 6, W28_BETA = 7, W28_ROWS = 8 };
#if defined(__HIPCC__)
static __device__ const uint32_t WAVE28_TABLE[W28_ROWS][16] = {TC_WAVE28_ROWS};
#else
static const uint32_t WAVE28_TABLE[W28_ROWS][16] = {TC_WAVE28_ROWS};
#endif

/* one word per lane of a wave */
struct wv {
#if defined(__HIPCC__)
    uint32_t l;
#else
    uint32_t l[64];
#endif
};
/* what every lane keeps at hand: its limb of the constants of the products and differences */
struct wv_consts {
    wv mp, p, p128;
};

#if defined(__HIPCC__)
#define WV_LANES(...) \
    {                                                             \
        const uint32_t lane = threadIdx.x & 63u;                  \
        (void)lane;                                               \
        __VA_ARGS__;                                                \
    }
#define WV_AT(x) (x).l
/* true in the one lane that writes what the whole wave has worked out */
TC_DEV bool wv_first_lane() { return (threadIdx.x & 63u) == 0u; }
#else
#define WV_LANES(...) \
    for (uint32_t lane = 0; lane < 64u; ++lane) {                 \
        __VA_ARGS__;                                                \
    }
#define WV_AT(x) (x).l[lane]
inline bool wv_first_lane() { return true; }
#endif

TC_DEV wv wv_table(int row) {
    wv r;
    WV_LANES(WV_AT(r) = WAVE28_TABLE[row][lane & 15u])
    return r;
}
TC_DEV wv_consts wv_constants() {
    wv_consts k;
    k.mp = wv_table(W28_MP);
    k.p = wv_table(W28_P);
    k.p128 = wv_table(W28_128P);
    return k;
}
TC_DEV wv wv_zero() {
    wv r;
    WV_LANES(WV_AT(r) = 0u)
    return r;
}
TC_DEV wv wv_add(const wv& a, const wv& b) {
    wv r;
    WV_LANES(WV_AT(r) = WV_AT(a) + WV_AT(b))
    return r;
}
/* the word of a lane of the wave, the same in all lanes */
TC_DEV uint32_t wv_read(const wv& a, int from) {
#if defined(__HIPCC__)
    return (uint32_t)__builtin_amdgcn_readlane((int)a.l, from);
#else
    return a.l[from];
#endif
}
/* is any word of row r set? */
TC_DEV bool wv_row_any(const wv& a, int r) {
#if defined(__HIPCC__)
    return ((__ballot(a.l != 0u) >> (16 * r)) & 0xFFFFull) != 0ull;
#else
    uint32_t any = 0;
    for (int j = 0; j < 16; ++j) any |= a.l[16 * r + j];
    return any != 0;
#endif
}
/* row r of the result: row r of r0, r1, r2, r3 */
TC_DEV wv wv_pick(const wv& r0, const wv& r1, const wv& r2, const wv& r3) {
    wv r;
    WV_LANES(uint32_t even = lane & 16u ? WV_AT(r1) : WV_AT(r0); uint32_t odd = lane & 16u ? WV_AT(r3) : WV_AT(r2); WV_AT(r) = lane & 32u ? odd : even)
    return r;
}
/* out[r]: row r of x in all four rows */
TC_DEV void wv_spread(const wv& x, wv (&out)[4]) {
#if defined(__HIPCC__)
    auto half = __builtin_amdgcn_permlane16_swap(x.l, x.l, false, false);              /* rows 0 0 2 2 and 1 1 3 3 */
    auto even = __builtin_amdgcn_permlane32_swap(half[0], half[0], false, false);
    auto odd = __builtin_amdgcn_permlane32_swap(half[1], half[1], false, false);
    out[0].l = even[0]; out[1].l = odd[0]; out[2].l = even[1]; out[3].l = odd[1];
#else
    for (int r = 0; r < 4; ++r)
        for (int i = 0; i < 64; ++i) out[r].l[i] = x.l[16 * r + (i & 15)];
#endif
}

#if defined(__HIPCC__)
/* dpp: 0x150 + i broadcasts lane i of each row, row_shl:1 = 0x101 (lane j takes j + 1), row_shr:1 = 0x111; zeros enter */
template <int I>
__device__ __forceinline__ uint32_t dpp_broadcast(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + I, 0xF, 0xF, true); }
__device__ __forceinline__ uint32_t dpp_from_above(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x101, 0xF, 0xF, true); }
__device__ __forceinline__ uint32_t dpp_from_below(uint32_t x) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x111, 0xF, 0xF, true); }
template <int I>
__device__ __forceinline__ void wv_mul_step(uint32_t a, uint32_t b, uint32_t mp, uint32_t& n, uint32_t& q) {
    uint64_t acc = (uint64_t)dpp_broadcast<I>(a) * b;
    asm("" : "+v"(acc));               /* a_i b is ready before q is: no multiply-add of its own in the chain from q to q */
    if (I) acc += (uint64_t)q * mp;
    acc += n;
    uint32_t lo = (uint32_t)acc & (uint32_t)FP28_MASK;
    q = dpp_broadcast<0>(lo);
    n = (uint32_t)(acc >> 28) + dpp_from_above(lo);
}
#endif
/* one pass of carries: limbs of up to 32 bits in, below 2^28 + 16 out */
TC_DEV wv wv_carry(const wv& a) {
    wv r;
#if defined(__HIPCC__)
    r.l = (a.l & (uint32_t)FP28_MASK) + dpp_from_below(a.l >> 28);
#else
    for (int i = 0; i < 64; ++i) r.l[i] = (a.l[i] & (uint32_t)FP28_MASK) + ((i & 15) ? a.l[i - 1] >> 28 : 0u);
#endif
    return r;
}
/* a b 2^-392 (mod p) in every row.  Step i adds a_i b, takes the lowest 28 bits q off the sum T and makes up for them:
 *   (T - q) / 2^28 + q (c p + 1) / 2^28 = (T + q c p) / 2^28,  c = -1 / p (mod 2^28),
 * so that q needs no product before it is used; its multiple of (c p + 1) / 2^28, a number below p, is added with the
 * next step's.  The last step divides p itself out (q c mod 2^28 times p), which leaves a value below
 * a b / 2^392 + 2 p.  Between the steps a limb is one word: what is above 28 bits of its own sum and the low 28 bits of the
 * limb above.  Limbs of a and b: a_i b_j below 2^59.3. */
TC_DEV wv wv_mul(const wv_consts& k, const wv& a, const wv& b) {
    wv r;
#if defined(__HIPCC__)
    uint32_t n = 0, q = 0;
    wv_mul_step<0>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<1>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<2>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<3>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<4>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<5>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<6>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<7>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<8>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<9>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<10>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<11>(a.l, b.l, k.mp.l, n, q);
    wv_mul_step<12>(a.l, b.l, k.mp.l, n, q);
    uint64_t acc = (uint64_t)dpp_broadcast<13>(a.l) * b.l;
    asm("" : "+v"(acc));
    acc += (uint64_t)q * k.mp.l;
    acc += n;
    uint32_t last = (dpp_broadcast<0>((uint32_t)acc) * (uint32_t)Fp28Params::NINV) & (uint32_t)FP28_MASK;
    acc += (uint64_t)last * k.p.l;
    r.l = (uint32_t)(acc >> 28) + dpp_from_above((uint32_t)acc & (uint32_t)FP28_MASK);
#else
    for (int row = 0; row < 64; row += 16) {
        uint32_t n[17] = {}, q = 0;
        uint64_t acc[16];
        for (int i = 0; i < 14; ++i) {
            for (int j = 0; j < 16; ++j) acc[j] = (uint64_t)a.l[row + i] * b.l[row + j] + n[j] + (uint64_t)q * k.mp.l[row + j];
            if (i == 13) {
                q = ((uint32_t)acc[0] * (uint32_t)Fp28Params::NINV) & (uint32_t)FP28_MASK;
                for (int j = 0; j < 16; ++j) acc[j] += (uint64_t)q * k.p.l[row + j];
            } else {
                q = (uint32_t)acc[0] & (uint32_t)FP28_MASK;
            }
            for (int j = 0; j < 16; ++j) {
                uint64_t s = (acc[j] >> 28) + (j < 15 ? (uint32_t)acc[j + 1] & (uint32_t)FP28_MASK : 0u);
                n[j] = (uint32_t)s;
                if (s >> 32) abort();                  /* the bound on the limbs */
            }
        }
        for (int j = 0; j < 16; ++j) r.l[row + j] = n[j];
    }
#endif
    return wv_carry(r);
}
/* a - b + 128 p, normal limbs */
TC_DEV wv wv_sub(const wv_consts& k, const wv& a, const wv& b) {
    wv r;
    WV_LANES(WV_AT(r) = WV_AT(a) + (WV_AT(k.p128) - WV_AT(b)))
    return wv_carry(r);
}
/* one bit per lane of the wave */
template <class Each>
TC_DEV uint64_t wv_ballot(const Each& each) {
#if defined(__HIPCC__)
    return __ballot(each(threadIdx.x & 63u));
#else
    uint64_t bits = 0;
    for (uint32_t lane = 0; lane < 64u; ++lane) bits |= (uint64_t)(each(lane) ? 1 : 0) << lane;
    return bits;
#endif
}
/* does row 0 of x (below 256 p, normal limbs) stand for zero?  A multiple of p is told from its lowest limb but for some
 * 2^-20 of the other values; then the limbs are looked at one by one. */
TC_DEV bool wv_is_zero(const wv& x) {
    if (((wv_read(x, 0) * (uint32_t)Fp28Params::PINV) & (uint32_t)FP28_MASK) > 256u) return false;
    fp28 v;
#if defined(__HIPCC__)
#pragma unroll
#endif
    for (int j = 0; j < 14; ++j) v.l[j] = (int32_t)wv_read(x, j);
    return fp28_is_zero(v, 256u);
}

/* ---- points: X, Y, ZZ, ZZZ in the rows 0 .. 3 ------------------------------------------------------------------ */
struct wv_point {
    wv v;
    bool inf;           /* the identity (v then holds nothing); the same in all lanes */
};
TC_DEV wv_point wv_identity() {
    wv_point r;
    r.v = wv_zero();
    r.inf = true;
    return r;
}
/* 2 a for a finite point (none on this curve has Y = 0).  Three levels of products: V = (2 Y)^2, A = X^2 | W = 2 Y V,
 * S = X V, (3 A)^2, V ZZ | 3 A (S - X3), W Y, W ZZZ.  With coordinates below 256 p (Y below 512 p):
 * X3 below 133 p, Y3 below 166 p. */
TC_DEV wv wv_dbl(const wv_consts& k, const wv& a) {
    wv c[4], m[4], n[4];
    wv_spread(a, c);
    const wv U = wv_add(c[1], c[1]);
    const wv l1 = wv_pick(U, c[0], U, c[0]);
    wv_spread(wv_mul(k, l1, l1), m);                                   /* V, A, V, A */
    const wv M = wv_add(wv_add(m[1], m[1]), m[1]);
    wv_spread(wv_mul(k, wv_pick(U, c[0], M, c[2]), wv_pick(m[0], m[0], M, m[0])), n);      /* W, S, M^2, ZZ3 */
    const wv S2 = wv_add(n[1], n[1]);
    const wv X3 = wv_sub(k, n[2], S2), D = wv_sub(k, wv_add(S2, n[1]), n[2]);             /* S - X3 = 3 S - M^2 */
    wv_spread(wv_mul(k, wv_pick(M, n[0], n[0], n[0]), wv_pick(D, c[1], c[3], c[3])), m);    /* M D, W Y, ZZZ3 */
    return wv_pick(X3, wv_sub(k, m[0], m[1]), n[3], m[2]);
}
/* a <- a + b.  Four levels: U1 U2 S1 S2 | PP RR ZZa.ZZb ZZZa.ZZZb | PPP Q ZZ3 | T1 T2 ZZZ3.  Every case of the group
 * law is settled here.  With coordinates below 256 p (Y below 512 p): X3 below 144 p, Y3 below 142 p. */
TC_DEV void wv_accumulate(const wv_consts& k, wv_point& a, const wv_point& b) {
    if (b.inf) return;
    if (a.inf) { a = b; return; }
    wv c[4], d[4], m[4], n[4];
    wv_spread(a.v, c);
    wv_spread(b.v, d);
    wv_spread(wv_mul(k, wv_pick(c[0], d[0], c[1], d[1]), wv_pick(d[2], c[2], d[3], c[3])), m);      /* U1 U2 S1 S2 */
    const wv P = wv_sub(k, m[1], m[0]), R = wv_sub(k, m[3], m[2]);
    if (wv_is_zero(P)) {
        if (wv_is_zero(R)) a.v = wv_dbl(k, b.v);
        else a.inf = true;
        return;
    }
    wv_spread(wv_mul(k, wv_pick(P, R, c[2], c[3]), wv_pick(P, R, d[2], d[3])), n);                    /* PP RR ZZab ZZZab */
    wv e[4], f[4];
    wv_spread(wv_mul(k, n[0], wv_pick(P, m[0], n[2], n[2])), e);                                     /* PPP Q ZZ3 */
    const wv s = wv_add(e[0], wv_add(e[1], e[1]));
    const wv X3 = wv_sub(k, n[1], s), D = wv_sub(k, wv_add(s, e[1]), n[1]);                          /* Q - X3 = Q + s - RR */
    wv_spread(wv_mul(k, wv_pick(R, m[2], n[3], n[3]), wv_pick(D, e[0], e[0], e[0])), f);            /* T1 T2 ZZZ3 */
    a.v = wv_pick(X3, wv_sub(k, f[0], f[1]), e[2], f[2]);
}
/* -b: Y below 512 p (512 p - Y of a Y below 256 p) */
TC_DEV wv wv_negate(const wv& b) {
    wv r, p512 = wv_table(W28_512P);
    WV_LANES(WV_AT(r) = (lane & 48u) == 16u ? WV_AT(p512) - WV_AT(b) : WV_AT(b))
    return wv_carry(r);
}

/* ---- in and out ------------------------------------------------------------------------------------------------- */
/* The form itself, 64 words, for points on their way from one wave to another: word 63 (the last lane of ZZZ's row, no limb) is 1 for a
 * finite point and 0 for the identity. */
constexpr uint32_t WV_POINT_WORDS = 64, WV_FINITE = 63;
TC_DEV void wv_store_raw(uint32_t* to, const wv_point& p) {
    WV_LANES(to[lane] = p.inf ? 0u : lane == WV_FINITE ? 1u : WV_AT(p.v))
}
TC_DEV wv_point wv_from_raw(const wv& words) {
    wv_point r;
    r.inf = wv_read(words, WV_FINITE) == 0u;
    WV_LANES(WV_AT(r.v) = lane == WV_FINITE ? 0u : WV_AT(words))
    return r;
}
TC_DEV wv_point wv_load_raw(const uint32_t* from) {
    wv w;
    WV_LANES(WV_AT(w) = from[lane])
    return wv_from_raw(w);
}
/* An array of points: raw, in the 32-bit form, or affine.  A point is fetched (one or two words a lane) while the one before is
 * being added, and unpacked when its turn comes. */
struct wv_words {
    wv a, b;
};
enum { WAVE_XYZZ = 0, WAVE_RAW = 1, WAVE_AFFINE = 2 };
struct WavePoints {
    const void* base;
    uint32_t kind;
    TC_DEV wv_words fetch(uint64_t i) const {
        wv_words w;
        if (kind == WAVE_RAW) {
            const uint32_t* p = (const uint32_t*)base + i * WV_POINT_WORDS;
            WV_LANES(WV_AT(w.a) = p[lane]; WV_AT(w.b) = 0u)
        } else {
            /* words at and at - 1 of the lane's coordinate (nothing below the lowest and above the highest); an affine point has two */
            const uint32_t words = kind == WAVE_AFFINE ? 24u : 48u;
            const uint32_t* p = (const uint32_t*)base + i * words;
            WV_LANES(const uint32_t o = 28u * (lane & 15u) + 24u; const uint32_t at = (o >> 5) < 12u ? o >> 5 : 12u; const uint32_t c = 12u * (lane >> 4);
                     WV_AT(w.a) = at && c < words ? p[c + at - 1u] : 0u; WV_AT(w.b) = at < 12u && c < words ? p[c + at] : 0u)
        }
        return w;
    }
    TC_DEV wv_point unpack(const wv_words& w) const {
        if (kind == WAVE_RAW) return wv_from_raw(w.a);
        wv_point r;
        WV_LANES(const uint32_t sh = (28u * (lane & 15u) + 24u) & 31u;
                 WV_AT(r.v) = (lane & 15u) < 14u ? (uint32_t)((((uint64_t)WV_AT(w.b) << 32) | WV_AT(w.a)) >> sh) & (uint32_t)FP28_MASK : 0u)
        if (kind == WAVE_AFFINE) {
            r.inf = !wv_row_any(r.v, 0) && !wv_row_any(r.v, 1);
            const wv one = wv_table(W28_ONE);
            WV_LANES(WV_AT(r.v) = lane < 32u ? WV_AT(r.v) : WV_AT(one))
        } else {
            r.inf = !wv_row_any(r.v, 2);
        }
        return r;
    }
    TC_DEV wv_point load(uint64_t i) const { return unpack(fetch(i)); }
    /* by a lane of its own */
    TC_DEV bool empty(uint64_t i) const {
        return kind == WAVE_RAW ? ((const uint32_t*)base)[i * WV_POINT_WORDS + WV_FINITE] == 0u : fe_is_zero(((const g1_xyzz*)base)[i].ZZ);
    }
};
TC_DEV wv_point wv_load(const g1_xyzz* p) { return WavePoints{p, WAVE_XYZZ}.load(0); }
TC_DEV wv_point wv_load_affine(const g1_affine* p) { return WavePoints{p, WAVE_AFFINE}.load(0); }
/* canonical bytes (x, y as plain numbers of 12 words; anything below 2^384 is taken) */
TC_DEV wv_point wv_load_canonical(const wv_consts& k, const uint32_t* w) {
    wv_point r = WavePoints{w, WAVE_AFFINE}.load(0);
    const wv plain = wv_table(W28_FROM_PLAIN), one = wv_table(W28_ONE);
    r.v = wv_mul(k, r.v, wv_pick(plain, plain, one, one));
    return r;
}
/* all limbs of a lane's row */
TC_DEV fp28 wv_row_limbs(const wv& x, uint32_t lane) {
    fp28 v;
#if defined(__HIPCC__)
    (void)lane;
    v.l[0] = (int32_t)dpp_broadcast<0>(x.l); v.l[1] = (int32_t)dpp_broadcast<1>(x.l); v.l[2] = (int32_t)dpp_broadcast<2>(x.l);
    v.l[3] = (int32_t)dpp_broadcast<3>(x.l); v.l[4] = (int32_t)dpp_broadcast<4>(x.l); v.l[5] = (int32_t)dpp_broadcast<5>(x.l);
    v.l[6] = (int32_t)dpp_broadcast<6>(x.l); v.l[7] = (int32_t)dpp_broadcast<7>(x.l); v.l[8] = (int32_t)dpp_broadcast<8>(x.l);
    v.l[9] = (int32_t)dpp_broadcast<9>(x.l); v.l[10] = (int32_t)dpp_broadcast<10>(x.l); v.l[11] = (int32_t)dpp_broadcast<11>(x.l);
    v.l[12] = (int32_t)dpp_broadcast<12>(x.l); v.l[13] = (int32_t)dpp_broadcast<13>(x.l);
#else
    for (int j = 0; j < 14; ++j) v.l[j] = (int32_t)x.l[(lane & 48u) + (uint32_t)j];
#endif
    return v;
}
/* canonical coordinates in the 32-bit form: every row's element reduced by its first lane */
TC_DEV void wv_store(g1_xyzz* to, const wv_point& p) {
    if (p.inf) {
        if (wv_first_lane()) *to = xyzz_identity();
        return;
    }
    WV_LANES(fp28 v = wv_row_limbs(p.v, lane); if ((lane & 15u) == 0u) (&to->X)[lane >> 4] = fp28_to_fp(v))
}

/* an element that every lane holds (normal limbs, within 128 p either way), plus 128 p, in all rows */
TC_DEV wv wv_from_lanes(const wv_consts& k, const fp28& a) {
    wv r;
    WV_LANES(const uint32_t j = lane & 15u; int32_t l = 0;
             for (int i = 0; i < 14; ++i) l |= (j == (uint32_t)i ? -1 : 0) & a.l[i];
             WV_AT(r) = (uint32_t)(l + (int32_t)WV_AT(k.p128)))
    return wv_carry(r);
}
/* x and y of a finite point in the rows 0 and 1 (below 4 p): one inversion, four levels of products */
TC_DEV wv wv_to_affine(const wv_consts& k, const wv& p) {
    wv c[4];
    wv_spread(p, c);
    const wv den = wv_mul(k, wv_mul(k, c[2], c[3]), wv_table(W28_ONE));           /* ZZ ZZZ, below 2.02 p */
    fp28 d = wv_row_limbs(den, 0), mod;
#if defined(__HIPCC__)
#pragma unroll
#endif
    for (int j = 0; j < 14; ++j) mod.l[j] = Fp28Params::MOD[j];
    const wv inv = wv_from_lanes(k, fp28_inv_wave(fp28_carry(fp28_sub(d, mod))));  /* |d - p| < 2 p, as the inversion wants it */
    const wv t = wv_mul(k, inv, wv_pick(c[3], c[2], c[2], c[2]));                  /* 1 / ZZ, 1 / ZZZ */
    return wv_mul(k, t, wv_pick(c[0], c[1], c[1], c[1]));
}

}  // namespace tc
