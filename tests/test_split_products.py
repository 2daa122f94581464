"""The carry-free split products of the kernels, replayed with Python integers at their largest operands: that no accumulator can
pass its 64 (or 128) bits for as many terms as the kernels add, that the recombination weights are right, and that the reductions
behind the sums give the canonical residue.

  Acc50 (inner products, conversions of sources below 2^50): d in two 25-bit halves, w in two 32-bit ones, four accumulators with
    the weights 2^0, 2^32, 2^25, 2^57.  Sums of one item (16 digits at most) also stand the digits just below 2^51 of a lazy
    reduction; the row-pass form of the inner products (RipFp) keeps one sum over all items of an output, RIP_MAX_TERMS terms,
    and relies on canonical digits.
  MacAcc (packed products): both factors in two halves of B bits, three accumulators, the two middle products in one.
  Conversions: up to eight sources, and one term more where a folded last limb joins them."""
import re
from fractions import Fraction
from pathlib import Path

import numpy as np
import pytest

LOW25 = (1 << 25) - 1
M64 = (1 << 64) - 1


def split_sum(ds, ws):
    t00 = t01 = t10 = t11 = 0
    for d, w in zip(ds, ws):
        d0, d1 = d & LOW25, d >> 25
        w0, w1 = w & 0xFFFFFFFF, w >> 32
        t00 += d0 * w0
        t01 += d0 * w1
        t10 += d1 * w0
        t11 += d1 * w1
        assert max(t00, t01, t10, t11) <= M64, "a 64-bit accumulator would wrap"
    total = t00 + (t01 << 32) + (t10 << 25) + (t11 << 57)
    assert total < 1 << 128
    return total


@pytest.mark.parametrize("terms", [1, 6, 8, 16])
def test_split_products_equal_the_plain_sum(terms):
    rng = np.random.default_rng(terms)
    for _ in range(200):
        ds = [int(v) for v in rng.integers(0, 1 << 50, terms, dtype=np.uint64)]
        ws = [int(v) for v in rng.integers(0, 1 << 63, terms, dtype=np.uint64) * 2 + rng.integers(0, 2, terms, dtype=np.uint64)]
        assert split_sum(ds, ws) == sum(d * w for d, w in zip(ds, ws))


@pytest.mark.parametrize("dmax", [(1 << 50) - 1, (1 << 51) - 1])
def test_largest_operands_do_not_overflow(dmax):
    for terms in (8, 16):
        ds, ws = [dmax] * terms, [M64] * terms
        assert split_sum(ds, ws) == terms * dmax * M64


CSRC = Path(__file__).resolve().parents[1] / "paper_2602_11470_amd" / "csrc"


def _define(source, name):
    return int(re.search(rf"#define {name} (\d+)", (CSRC / source).read_text()).group(1))


def _redc(T, q):
    """redc of common.h on 64-bit words: T 2^-64 mod q, in [0, q) where T < q 2^64."""
    assert 0 <= T < 1 << 128
    lo, hi = T & M64, T >> 64
    t = (((lo * pow(q, -1, 1 << 64)) & M64) * q) >> 64
    r = hi - t if hi >= t else hi - t + q
    assert 0 <= r <= M64
    return r


def _redc_raw(T, q):
    """redc_raw of kernels.h: T mod q, also where T is beyond q 2^64, as long as the second product is not."""
    second = _redc(T, q) * ((1 << 128) % q)
    assert second < q << 64
    return _redc(second, q)


def _prime_below(bound):
    for q in range(bound - 1, bound - 4096, -2):
        if all(pow(a, q - 1, q) == 1 for a in (2, 3, 5, 7, 11, 13)):
            return q


Q50, Q60, Q61 = _prime_below(1 << 50), _prime_below(1 << 60), _prime_below(1 << 61)


def test_row_pass_inner_product_sums():
    terms = _define("ntt.hip", "RIP_MAX_TERMS")
    q, inv64 = Q50, pow(1 << 64, -1, Q50)
    d = [q - 1] * terms
    b, a = split_sum(d, [q - 1] * terms), split_sum(d, [M64] * terms)      # key words below q, raw draws
    assert b < q << 64 and _redc(b, q) == b * inv64 % q
    assert _redc_raw(a, q) == a % q
    # digits of a lazy reduction would not do
    with pytest.raises(AssertionError):
        split_sum([2 * q - 1] * terms, [M64] * terms)
    # integer limbs: reduced item by item, up to seven digits and a first component (key half), seven raw draws
    for q in (Q60, Q61):
        b, a = 8 * (q - 1) ** 2, 7 * (q - 1) * M64
        assert b < q << 64 and _redc(b, q) == b * pow(1 << 64, -1, q) % q
        assert a < 1 << 128 and _redc_raw(a, q) == a % q


def _mac_limits():
    text = (CSRC / "kernels.hip").read_text()
    out = {}
    for name in ("MacPacked50", "MacPacked60", "MacWords"):
        m = re.search(rf"struct {name} {{[^}}]*?B = (\d+), TERMS = ([^;]+);", text)
        out[name] = int(m.group(1)), eval(m.group(2))
    return out


@pytest.mark.parametrize("name,q", [("MacPacked50", Q50), ("MacPacked60", Q60), ("MacWords", Q61)])
def test_packed_product_sums(name, q):
    B, terms = _mac_limits()[name]
    mask = (1 << B) - 1
    for w in (q - 1, mask, (q - 1) & ~mask):                   # the largest word, the largest lower and upper half
        for b in (q - 1, mask, (q - 1) & ~mask):
            t0 = terms * (b & mask) * (w & mask)
            t1 = terms * ((b & mask) * (w >> B) + (b >> B) * (w & mask))
            t2 = terms * (b >> B) * (w >> B)
            assert max(t0, t1, t2) <= M64, "a 64-bit accumulator would wrap"
            T = t0 + (t1 << B) + (t2 << (2 * B))
            assert T == terms * b * w and T < q << 64
            assert _redc(T, q) == T * pow(1 << 64, -1, q) % q


@pytest.mark.parametrize("sources", [1, 2, 4, 6, 8])
def test_conversion_sums_with_a_folded_limb(sources):
    terms = sources + 1
    # sources below 2^50: Acc50, whatever the weight
    for q in (Q50, Q61):
        T = split_sum([Q50 - 1] * terms, [q - 1] * terms)
        assert T < q << 64 and _redc(T, q) == T * pow(1 << 64, -1, q) % q
    # sources below 2^60, targets below 2^50: halves of 30 and of 25 bits
    y, w = Q60 - 1, Q50 - 1
    y0, y1, w0, w1 = y & ((1 << 30) - 1), y >> 30, w & LOW25, w >> 25
    parts = [terms * v for v in (y0 * w0, y0 * w1, y1 * w0, y1 * w1)]
    assert max(parts) <= M64
    T = parts[0] + (parts[1] << 25) + (parts[2] << 30) + (parts[3] << 55)
    assert T == terms * y * w < Q50 << 64
    # 128-bit sums of 61-bit sources: seven terms with the folded limb among them, eight sources without
    for q in (Q60, Q61):
        T = min(terms, 7) * (Q61 - 1) * (q - 1)
        assert T < q << 64 and 8 * (Q61 - 1) * (q - 1) < q << 64


def test_conversion_sums_in_doubles_stay_exact():
    """|y w - c q| <= 0.88 q a term (c = rint of y w / q, off by three roundings of a value below 2^50), nine terms below 2^53."""
    q = Q50
    qinv = 1.0 / q
    rng = np.random.default_rng(5)
    worst = Fraction(0)
    pairs = [(q - 1, q - 1), (q - 1, q // 2), (q // 2, q - 1), (q - 1, q // 2 + 1), (q - 2, 3)]
    pairs += [(int(a), int(b)) for a, b in zip(rng.integers(q - (1 << 20), q, 4000), rng.integers(0, q, 4000))]
    for y, w in pairs:
        c = np.rint(float(y) * (float(w) * qinv))
        worst = max(worst, abs(Fraction(y * w) - int(c) * q) / q)
    assert worst <= Fraction(88, 100)
    assert 9 * Fraction(88, 100) * q < 1 << 53


@pytest.mark.parametrize("n", [4096, 65536])
@pytest.mark.parametrize("b", [40, 45, 48, 49, 50, 51, 54, 60, 61])
def test_conversion_sums_from_cut_weights(n, b):
    """ConvNear::sum with the weights as the library cuts them up: the largest y and w, for as many terms as conv_near of ops.hip lets a
    table have (a folded limb among them); nothing passes 64 bits (the products' factors 32), and what is left is the sum, below
    q + q / 16."""
    import ctypes
    from oracle import params
    from paper_2602_11470_amd import binding as B

    class Cut(ctypes.Structure):
        _fields_ = [(name, ctypes.c_uint) for name in ("w0", "w1", "v0", "v1")]
    cut = B.lib._Z8conv_cutmmi
    cut.argtypes, cut.restype = [ctypes.c_ulong, ctypes.c_ulong, ctypes.c_int], Cut
    most = _define("common.h", "CONV_MAX_SRC") + 1
    few = int(re.search(r"o\.q < \(1ULL << 50\) \|\| terms <= (\d+)", (CSRC / "ops.hip").read_text()).group(1))
    assert int(re.search(r"if \(b < (\d+) \|\| c >=", (CSRC / "ops.hip").read_text()).group(1)) == 40
    q = params.scan_primes(b, n, 8)[-1]
    c = (1 << b) - q
    t, z = ((b + 1) // 2, 29 - (b - (b + 1) // 2)) if b <= 50 else (30, 61 - b)
    mlo, mhi = 1 << (t - z), c << (3 if b <= 50 else 1)
    m32, mb = (1 << 32) - 1, (1 << b) - 1
    assert mhi <= m32
    rng = np.random.default_rng(b)
    for s, terms in ((25, most), (30, most if b < 51 else few)):
        ymax = (1 << 50) - 1 if s == 25 else (1 << 60) - 1
        for i in range(300):
            ys = [ymax if i < 2 else int(rng.integers(0, ymax)) for _ in range(terms)]
            ws = [q - 1 if i % 2 else int(rng.integers(0, q)) for _ in range(terms)]
            lo = hi = 0
            for y, w in zip(ys, ws):
                x = cut(q, w, s)
                y0, y1 = y & ((1 << s) - 1), y >> s
                assert max(y0, y1) <= m32
                lo, hi = lo + y0 * x.w0 + y1 * x.v0, hi + y0 * x.w1 + y1 * x.v1
            assert max(lo, hi) <= M64
            T = lo + (hi & m32) * mlo + (hi >> 32) * mhi
            assert T <= M64 and (b > 50 or T < 1 << 63)
            for _ in range(2 if b < 49 else 1):
                T = (T >> b) * c + (T & mb)
            assert T < q + q // 16 and T % q == sum(y * w for y, w in zip(ys, ws)) % q
    # the growth of four FP64 stages that start there, and of the integer stages (at most 4 q asked for)
    bound = 1 + 1 / 16
    for _ in range(4):
        bound += 0.5 + 0.375 * bound
    assert bound < 8
