"""The library's field / curve headers, compiled for the host with g++, against the oracle.

The HIP kernels inline these same functions; this CPU test finds arithmetic mistakes
(carry handling, exceptional cases of the group law, the G1 -> Fr map) without a GPU."""
import ctypes
import os
import random
import subprocess

import pytest

from oracle import bls12_381 as ec
from oracle import terkle
from oracle.bls12_381 import P, R

HERE = os.path.dirname(os.path.abspath(__file__))
SRC = os.path.join(HERE, "hostmath", "hostmath.cpp")
LIB = os.path.join(HERE, "hostmath", "libhostmath.so")


@pytest.fixture(scope="module")
def hm():
    hdrs = [os.path.join(HERE, "..", "paper_2602_12630_amd", "csrc", h) for h in ("field.h", "field28.h", "field30.h", "g1.h", "constants.h", "kernels.h", "wave28.h", "rt.h", "pairing.h")]
    newest = max(os.path.getmtime(f) for f in [SRC] + hdrs)
    if not os.path.exists(LIB) or os.path.getmtime(LIB) < newest:
        subprocess.check_call(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", "-o", LIB, SRC])
    return ctypes.CDLL(LIB)


def _b(x, n):
    return (ctypes.c_uint8 * n).from_buffer_copy(int(x).to_bytes(n, "little"))


def _call2(fn, a, b, n):
    out = (ctypes.c_uint8 * n)()
    fn(_b(a, n), _b(b, n), out)
    return int.from_bytes(bytes(out), "little")


def test_fp64_product_columns_stay_exact():
    """The FP64 form of the Fp product sums whole columns of 24-bit limb products in a double: the largest
    column any two operands below the modulus can produce, with the reduction terms and the carry, must stay
    below 2^53."""
    top = P >> 360                                   # the 16th limb of an operand is at most that of the modulus
    limb = (1 << 24) - 1
    p24 = [(P >> (24 * j)) & limb for j in range(16)]
    worst, carry = 0, 0
    for k in range(31):
        lo, hi = max(0, k - 15), min(k, 15)
        ab = sum((top if i == 15 else limb) * (top if k - i == 15 else limb) for i in range(lo, hi + 1))
        mp = sum(limb * p24[k - i] for i in range(lo, hi + 1))
        column = ab + mp + carry
        worst = max(worst, column)
        carry = column >> 24
    assert worst < 1 << 53


@pytest.mark.parametrize("group", ["edges", "powers", "random"])
def test_inversion_by_division_steps(hm, group):
    """The wave's inversion (rows of limbs, lazily carried updates)."""
    rng = random.Random(3)
    vals = {"edges": [0, 1, 2, 3, P - 1, P - 2, (P - 1) // 2, (P + 1) // 2, (1 << 28) - 1, P >> 28],
            "powers": [1 << k for k in range(0, 381, 7)] + [P - (1 << k) for k in range(0, 380, 7)],
            "random": [rng.randrange(P) for _ in range(200)]}[group]
    out = (ctypes.c_uint8 * 48)()
    for a in vals:
        hm.hm_fp_inv_wave(_b(a, 48), out)
        assert int.from_bytes(bytes(out), "little") == (pow(a, -1, P) if a else 0), a


def test_inversion_in_batches_of_quotients(hm):
    """What the wave's inversion does before it falls back on division steps: random values take 15 to 17 batches and never fall
    back, plain values so small that the first quotient has more than 27 bits always do; the division steps by themselves."""
    rng = random.Random(16)
    small = [k * pow(2, -392, P) % P for k in (1, 2, 3, -1, -2, 1 << 100, (1 << 353) - 1)]           # their form's limbs are k's
    out = (ctypes.c_uint8 * 48)()
    for a in small + [0]:
        assert hm.hm_fp_inv_batches(_b(a, 48)) == -1
    for a in [rng.randrange(1, P) for _ in range(2000)]:
        assert 15 <= hm.hm_fp_inv_batches(_b(a, 48)) <= 17
    for a in small + [0, 1, P - 1] + [rng.randrange(P) for _ in range(200)]:
        for f in (hm.hm_fp_inv_wave, hm.hm_fp_inv_divsteps):
            f(_b(a, 48), out)
            assert int.from_bytes(bytes(out), "little") == (pow(a, -1, P) if a else 0), a


def test_rounds_of_the_wave_inversion():
    """What the 48 rounds of that inversion rest on: no operand takes more than 881 division steps (32 rounds of 28), and a
    g = 0 that stands in limbs that cancel, in whichever of the 2^13 ways, is all zeros after at most 14 rounds more."""
    rng = random.Random(9)
    edges = [1, 2, P - 1, P + 1, 2 * P - 1, (P + 1) // 2, (1 << 381) - 1] + [1 << k for k in range(0, 381, 20)]
    for x in edges + [rng.randrange(1, 2 * P) for _ in range(200)]:
        for g in (x, -x):
            f, D, steps = P, 0, 0
            while g:
                if D >= 0 and g & 1:
                    f, g, D = g, (g - f) >> 1, -D
                else:
                    g, D = (g + (g & 1) * f) >> 1, D + 1
                steps += 1
            assert abs(f) == 1 and steps <= 881, x
    assert 881 <= 32 * 28
    mask = (1 << 28) - 1
    for ways in range(1 << 13):
        k = [0] + [ways >> j & 1 for j in range(13)] + [0]
        limbs = [(k[j + 1] << 28) - k[j] for j in range(14)]
        assert sum(l << 28 * j for j, l in enumerate(limbs)) == 0
        rounds = 0
        while any(limbs):
            n = [(limbs[j] >> 28) + (limbs[j + 1] & mask if j < 13 else 0) for j in range(14)]
            limbs = [(n[j] & mask if j < 13 else n[j]) + (n[j - 1] >> 28 if j else 0) for j in range(14)]
            rounds += 1
        assert rounds <= 14


def test_fp_fr_arithmetic(hm):
    rng = random.Random(1)
    edge_p = [0, 1, 2, P - 1, P - 2, (P - 1) // 2, (1 << 380), 0xFFFFFFFF, (1 << 352) - 1, (1 << 380) - 1]
    vals = edge_p + [rng.randrange(P) for _ in range(60)]
    for a in vals:
        for b in edge_p + [rng.randrange(P) for _ in range(4)]:
            assert _call2(hm.hm_fp_mul, a, b, 48) == a * b % P                   # 64-bit limbs (host code)
            assert _call2(hm.hm_fp_mul_limbs32, a, b, 48) == a * b % P           # the 32-bit-limb form of the kernels
            assert _call2(hm.hm_fp_mul_f64, a, b, 48) == a * b % P               # 24-bit limbs in doubles (doubling chains)
            assert _call2(hm.hm_fp_sqr_f64, a, b, 48) == a * a % P
            assert _call2(hm.hm_fp_add, a, b, 48) == (a + b) % P
            assert _call2(hm.hm_fp_sub, a, b, 48) == (a - b) % P
    edge_r = [0, 1, 2, R - 1, R - 2, (1 << 254), 0xFFFFFFFF]
    for a in edge_r + [rng.randrange(R) for _ in range(60)]:
        for b in edge_r + [rng.randrange(R) for _ in range(4)]:
            assert _call2(hm.hm_fr_mul, a, b, 32) == a * b % R
            assert _call2(hm.hm_fr_add, a, b, 32) == (a + b) % R
            assert _call2(hm.hm_fr_sub, a, b, 32) == (a - b) % R
    for a in (1, 2, P - 1, rng.randrange(1, P)):
        out = (ctypes.c_uint8 * 48)()
        hm.hm_fp_inv(_b(a, 48), out)
        assert int.from_bytes(bytes(out), "little") * a % P == 1
    for a in (1, 2, 3, P - 1, P - 2, (P - 1) // 2, 1 << 380, rng.randrange(1, P), rng.randrange(1, P)):
        out = (ctypes.c_uint8 * 48)()
        hm.hm_fp_inv_binary(_b(a, 48), out)
        assert int.from_bytes(bytes(out), "little") == pow(a, -1, P)
    for a in (1, 2, R - 1, 1 << 254, rng.randrange(1, R), rng.randrange(1, R)):
        out = (ctypes.c_uint8 * 32)()
        hm.hm_fr_inv_binary(_b(a, 32), out)
        assert int.from_bytes(bytes(out), "little") == pow(a, -1, R)
    for fn_p, fn_r in ((hm.hm_fp_inv_gcd, hm.hm_fr_inv_gcd),):
        edge = [1, 2, 3, (1 << 32), (1 << 62) + 1, (1 << 63) + 5, (1 << 64) - 1, 1 << 64]
        for a in edge + [P - 1, P - 2, (P - 1) // 2, 1 << 380] + [rng.randrange(1, P) for _ in range(300)] + \
                [rng.randrange(1, 1 << rng.randrange(1, 381)) for _ in range(300)]:
            out = (ctypes.c_uint8 * 48)()
            fn_p(_b(a, 48), out)
            assert int.from_bytes(bytes(out), "little") == pow(a, -1, P)
        for a in edge + [R - 1, R - 2, 1 << 254] + [rng.randrange(1, R) for _ in range(300)] + \
                [rng.randrange(1, 1 << rng.randrange(1, 255)) for _ in range(300)]:
            out = (ctypes.c_uint8 * 32)()
            fn_r(_b(a, 32), out)
            assert int.from_bytes(bytes(out), "little") == pow(a, -1, R)
    for v in (0, 1, -1, 127, -128, 32767, -32768, 2**31 - 1, -(2**31)):
        out = (ctypes.c_uint8 * 32)()
        hm.hm_fr_from_i32(ctypes.c_int32(v), out)
        assert int.from_bytes(bytes(out), "little") == v % R


def _pt(fn, *args):
    out = (ctypes.c_uint8 * 96)()
    fn(*args, out)
    return ec.g1_from_bytes(bytes(out))


def _pb(pt):
    return (ctypes.c_uint8 * 96).from_buffer_copy(ec.g1_to_bytes(pt))


def test_group_law_including_exceptional_cases(hm):
    rng = random.Random(2)
    assert _pt(hm.hm_g1_generator) == ec.G1
    pts = [ec.mul(rng.randrange(1, R), ec.G1) for _ in range(5)]
    for mode in (0, 1, 2):
        for a in pts:
            assert _pt(hm.hm_g1_add, _pb(a), _pb(a), mode) == ec.add_affine(a, a)                 # P + P
            assert _pt(hm.hm_g1_add, _pb(a), _pb(ec.neg(a)), mode) is ec.INF                      # P + (-P)
            assert _pt(hm.hm_g1_add, _pb(a), _pb(ec.INF), mode) == a                              # P + O
            assert _pt(hm.hm_g1_add, _pb(ec.INF), _pb(a), mode) == a                              # O + P
            for b in pts:
                assert _pt(hm.hm_g1_add, _pb(a), _pb(b), mode) == ec.add_affine(a, b)
        assert _pt(hm.hm_g1_add, _pb(ec.INF), _pb(ec.INF), mode) is ec.INF
    for k in (0, 1, 2, 3, R - 1, rng.randrange(R), 1 << 200):
        assert _pt(hm.hm_g1_mul, _b(k, 32), _pb(pts[0])) == ec.mul_affine(k, pts[0])

def test_cooperative_reduction(hm):
    """Sums of up to 256 points through the shared-addition kernel, which adds points i and 64 + i, then 128 + i and
    192 + i, the two sums, and halves of the 64 sums: every length at which another step begins or ends, and the operand
    patterns that leave the regular chord rule, namely identities anywhere, equal points (tangent rule), opposite points
    in the first, second and third step, everything cancelling."""
    rng = random.Random(5)
    base = [ec.mul(rng.randrange(1, R), ec.G1) for _ in range(6)]

    def run(points, spread):
        buf = b"".join(ec.g1_to_bytes(p) for p in points)
        arr = (ctypes.c_uint8 * max(len(buf), 1)).from_buffer_copy(buf or b"\0")
        out = (ctypes.c_uint8 * 96)()
        hm.hm_coop_reduce(arr, len(points), spread, out)
        return ec.g1_from_bytes(bytes(out))

    def want(points):
        acc = ec.INF
        for p in points:
            acc = ec.add_affine(acc, p)
        return acc

    cases = [
        [],
        [base[0]],
        [base[0], base[1]],
        [base[0], base[0]],                                  # tangent rule in the last step
        [base[0], ec.neg(base[0])],                          # opposite points
        [ec.INF, base[2]],
        [base[2], ec.INF],
        [ec.INF, ec.INF, ec.INF],
        [base[0], base[1], base[0], base[1]],                # equal points, then a regular sum of theirs
        [base[0], base[1], ec.neg(base[0]), ec.neg(base[1])],
        [base[i % 6] for i in range(17)],
        [base[rng.randrange(6)] if rng.random() < 0.6 else ec.INF for _ in range(255)],
        [ec.mul(i + 1, base[3]) for i in range(64)] + [ec.neg(ec.mul(i + 1, base[3])) for i in range(64)],
        [base[rng.randrange(6)] for _ in range(256)],
    ]
    many = [ec.mul(i + 2, base[4]) for i in range(64)]
    minus = [ec.neg(p) for p in many]
    cases += [many, many + minus[:1], many + many[:1], many + many, many + minus + many[:1], many + minus + many,
              many + minus + many + minus[:1], many + many + many + many, many + minus + minus + minus,
              many + many + minus + minus, many + [ec.INF] * 64 + many + minus, [ec.INF] * 192 + many,
              many[:33] + [ec.INF] * 95 + minus[:33] + [ec.INF] * 63 + many[:1]]
    for n in (32, 33, 63, 64, 65, 127, 128, 129, 191, 192, 193, 255):
        cases.append([base[rng.randrange(6)] for _ in range(n)])
    for spread in (0, 1):
        for pts in cases:
            got = run(pts, spread)
            w = want(pts)
            assert (got is ec.INF and w is ec.INF) or got == w, (len(pts), spread)


def test_fr_product_in_29_bit_limbs(hm):
    """a b 2^-256 mod r, canonical, for operands up to 2^256 - 1 against operands below r (what the 32-bit form takes)."""
    rng = random.Random(14)
    edge = [0, 1, 2, R - 1, R - 2, (R - 1) // 2, (1 << 255) - 1, (1 << 29) - 1, (1 << 232) - 1, 0xFFFFFFFF << 200] + [1 << k for k in range(0, 255, 29)]
    inv = pow(1 << 256, -1, R)
    for a in edge + [(1 << 256) - 1, R, R + 1, 2 * R] + [rng.randrange(1 << 256) for _ in range(200)]:
        for b in [e % R for e in edge] + [rng.randrange(R) for _ in range(4)]:
            assert _call2(hm.hm_fr_mul_limbs29, a, b, 32) == a * b * inv % R


def test_products_in_30_bit_limbs(hm):
    """Products, squares, differences of products and products less known elements at the bounds of their limbs: balanced
    ones at either end of their range, 30 bits either sign against balanced; results balanced and within the stated value."""
    rng = random.Random(15)
    radix, half = 1 << 390, 1 << 29
    val = lambda l: sum(v << (30 * j) for j, v in enumerate(l))
    bal = lambda: [rng.choice([-half, half - 1, rng.randrange(-half, half)]) for _ in range(12)] + [rng.randrange(-(1 << 26), 1 << 26)]
    wide = lambda: [rng.choice([-2 * half + 1, 2 * half - 1, rng.randrange(-2 * half, 2 * half)]) for _ in range(12)] + [rng.randrange(-(1 << 26), 1 << 26)]
    ends = lambda v: [v] * 12 + [1 << 26]

    def run(mode, *x):
        out = (ctypes.c_int32 * 13)()
        x = list(x) + [[0] * 13] * (4 - len(x))
        hm.hm_fp30(mode, (ctypes.c_int32 * 52)(*sum(x, [])), out)
        return list(out)

    for i in range(300):
        a, b, c, e = (bal() for _ in range(4)) if i > 8 else (ends(rng.choice([-half, half - 1])) for _ in range(4))
        w = wide() if i % 3 else ends(rng.choice([-2 * half + 1, 2 * half - 1]))
        A, B, C, E, W = (val(v) for v in (a, b, c, e, w))
        for mode, args, want, folded in ((0, (w, b), W * B, 0), (0, (a, w), A * W, 0), (1, (a,), A * A, 0), (2, (a, b, c, e), A * B - C * E, 0),
                                         (3, (w, b, c), W * B, -C), (4, (a, b, c, e), A * A, -C - 2 * E)):
            r = run(mode, *args)
            assert (val(r) - folded) * radix % P == want % P, mode
            assert all(-half <= v < half for v in r[:12])
            assert abs(val(r) - folded) <= abs(want) / radix + 0.52 * P, mode
        s = [x - y for x, y in zip(a, b)]
        r = run(5, s)
        assert val(r) == A - B and all(-half <= v < half for v in r[:12])
    for v in [0, 1, -1, P, -P, 63 * P, -63 * P, 64 * P - 1, 1 - 64 * P] + [rng.randrange(-64 * P, 64 * P) for _ in range(200)]:
        l, x = [], v
        for _ in range(12):
            d = (x + half) % (2 * half) - half
            l.append(d)
            x = (x - d) >> 30
        l.append(x)
        out = (ctypes.c_uint8 * 48)()
        hm.hm_fp30_to_fp((ctypes.c_int32 * 13)(*l), out)
        assert int.from_bytes(bytes(out), "little") * radix % P == v % P
        assert hm.hm_fp30_maybe_zero((ctypes.c_int32 * 13)(*l), 128) == (v % P == 0)
    for x in [0, 1, P - 1, (1 << 380) + 5] + [rng.randrange(P) for _ in range(100)]:
        assert hm.hm_fp30_recut(_b(x, 48))


def test_product_spread_over_lanes(hm):
    """a b 2^-392 (mod p) with the limbs at the bounds that the group law relies on: 2^29.6 on both sides, 2^30 - 4 against a normal
    operand; the result's limbs are normal and its value is below a b / 2^392 + 2 p.  (The host form stops on a limb sum that leaves
    its word.)"""
    rng = random.Random(12)
    radix, normal, grown = 1 << 392, (1 << 28) + 15, 3 * ((1 << 28) + 15)
    limits = [(grown, grown), ((1 << 30) - 4, normal), (normal, (1 << 30) - 4), (normal, normal), (0, grown), (1, 1)]
    for la, lb in limits * 8:
        draw = lambda l: [rng.choice([l, rng.randrange(l + 1), 0]) for _ in range(13)] + [rng.randrange(1 << 26) if l else 0]
        a, b = [draw(la) for _ in range(4)], [draw(lb) for _ in range(4)]
        if (la, lb) in limits[:4] and rng.random() < 0.3:
            a[0], b[0] = [la] * 13 + [1 << 26], [lb] * 13 + [1 << 26]
        out = (ctypes.c_uint32 * 56)()
        hm.hm_wave_mul((ctypes.c_uint32 * 56)(*sum(a, [])), (ctypes.c_uint32 * 56)(*sum(b, [])), out)
        for row in range(4):
            x, y, r = (sum(v << (28 * j) for j, v in enumerate(l)) for l in (a[row], b[row], out[14 * row : 14 * row + 14]))
            assert r * radix % P == x * y % P
            assert max(out[14 * row : 14 * row + 14]) <= normal and r < x * y // radix + 2 * P


def test_group_law_spread_over_lanes(hm):
    rng = random.Random(13)
    base = [ec.mul(rng.randrange(1, R), ec.G1) for _ in range(5)]
    cases = [[], [base[0]], [base[0], base[0]], [base[0], ec.neg(base[0])], [ec.INF, base[1]], [base[1], ec.INF], [ec.INF] * 3,
             [base[0], base[1], ec.neg(ec.add_affine(base[0], base[1])), base[2]], [base[0], base[1], ec.add_affine(base[0], base[1])],
             [base[i % 5] for i in range(40)], [rng.choice(base + [ec.INF]) for _ in range(40)]]
    for spread in (0, 1, 2):
        for pts in cases:
            for doublings in (0, 1, 130):
                buf = b"".join(ec.g1_to_bytes(p) for p in pts)
                want = ec.INF
                for p in pts:
                    want = ec.add_affine(want, p)
                got = _pt(hm.hm_wave_sum, (ctypes.c_uint8 * max(len(buf), 1)).from_buffer_copy(buf or b"\0"), len(pts), doublings, spread)
                want = ec.mul(1 << doublings, want)
                assert (got is ec.INF and want is ec.INF) or got == want, (len(pts), spread, doublings)


@pytest.mark.parametrize("lognb,windows", [(7, 1), (7, 9), (8, 1), (8, 2), (8, 8)])
def test_window_bit_by_bit(hm, lognb, windows):
    """sum_k k B_k of a few windows of 128 or 256 buckets through the sums per bit, from one workgroup of chains to more
    than 64 chains; buckets empty, equal and opposite among them, and a window with nothing in it."""
    rng = random.Random(lognb * 100 + windows)
    nb = 1 << lognb
    table = [ec.mul(i + 1, ec.G1) for i in range(40)]
    mult = [[0 if w and w == windows - 1 else rng.choice([0, 0, 1, -1]) * rng.randrange(1, 41) for _ in range(nb)] for w in range(windows)]
    mult[0][nb - 1] = 40
    pts = [ec.INF if not m else table[m - 1] if m > 0 else ec.neg(table[-m - 1]) for row in mult for m in row]
    buf = b"".join(ec.g1_to_bytes(p) for p in pts)
    out = (ctypes.c_uint8 * (96 * windows))()
    hm.hm_window_bits((ctypes.c_uint8 * len(buf)).from_buffer_copy(buf), lognb, windows, out)
    for w, row in enumerate(mult):
        total = sum((k + 1) * m for k, m in enumerate(row)) % R
        assert ec.g1_from_bytes(bytes(out)[96 * w : 96 * (w + 1)]) == (ec.mul(total, ec.G1) if total else ec.INF), w


def test_pairing_building_blocks(hm):
    """Inside the host pairing: the verifier's short final exponentiation is the cube of the plain one, the
    p-power map equals the power by p, applying it twice equals the p^2-power map, inversion inverts."""
    rng = random.Random(8)
    for _ in range(2):
        pt = ec.mul(rng.randrange(1, R), ec.G1)
        assert hm.hm_final_exponentiation_forms(_pb(pt), rng.randrange(1, 1 << 32)) == 15


def test_phi_map(hm):
    rng = random.Random(3)
    for pt in [ec.INF, ec.G1, ec.neg(ec.G1)] + [ec.mul(rng.randrange(1, R), ec.G1) for _ in range(20)]:
        out = (ctypes.c_uint8 * 32)()
        hm.hm_phi(_pb(pt), out)
        assert int.from_bytes(bytes(out), "little") == terkle.phi(pt)
