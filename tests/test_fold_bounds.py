"""Bounds of the short reductions for primes q = 2^54 - delta (delta < 2^22),
checked on the CPU with exact integers and 64-bit two's complement wrap,
step for step as the device code takes them:

* the fold of the 13 int8-digit diagonal sums S_s of the matrix-core
  multiply-accumulate (V = sum_s 256^s S_s, |S_s| < 7 2^21 and 0 <= S_12 <=
  2^19 for d <= 128) into a value below 2^57 congruent to V;
* x mod 2^54 + (x >> 54) delta, one conditional subtraction, for x < 2^60
  (the sums transpose, values below 2^58; the last step of the query
  transform, values below 2^60);
* the Horner step of the circuit-private form's flood residues.

Extreme diagonals (every sum at +bound or -bound, alternating signs, the
largest top sum) and random ones, for every such prime of the ring degrees
and limb counts the library derives.  Host arithmetic only, no GPU."""
import random

import oracle

M64 = (1 << 64) - 1
B = 7 * (1 << 21)   # |S_s| bound, d <= 128 (7 digit pairs x 2^14 x 128)
B12 = 1 << 19       # S_12 = sum of x_6 y_6 with x_6, y_6 in [0, 64]


def _s64(x):
    x &= M64
    return x - (1 << 64) if x >> 63 else x


def _i32(x):
    x &= 0xFFFFFFFF
    return x - (1 << 32) if x >> 31 else x


def fold_short(S, q):
    delta = (1 << 54) - q

    def group(s, base):
        g = base
        for j, k in enumerate((1, 1 << 8, 1 << 16, 1 << 24)):
            assert -(1 << 31) <= S[s + j] < 1 << 31
            g = _s64(g + S[s + j] * k)
        return g

    h = _s64(group(8, 0) + ((S[12] & 0xFFFFFFFF) << 32))
    hh = _i32((h & M64) >> 22)
    assert hh == h >> 22                      # the 32-bit field is the exact shift
    hl = h & 0x3FFFFF
    z = _s64(group(4, 0) + delta * hh + (hl << 32))
    zh = _i32((z & M64) >> 24)
    assert zh == z >> 24
    zl = z & 0xFFFFFF
    r = _s64(group(0, 2 * q) + 4 * delta * zh + (zl << 32))
    assert 0 <= r < 1 << 57
    return r


def reduce_short(x, q):
    delta = (1 << 54) - q
    assert 0 <= x < 1 << 60
    r = (x & ((1 << 54) - 1)) + (x >> 54) * delta
    assert r < 2 * q
    return r - q if r >= q else r


def _short_primes():
    out = set()
    for N in (64, 1024, 4096, 8192, 16384, 32768):
        for q in oracle.rns_primes(N, 6):
            if 0 < (1 << 54) - q < 1 << 22:
                out.add(q)
    return sorted(out)


def _diagonals(rng, mode):
    S = []
    for s in range(13):
        lo, hi = (0, B12) if s == 12 else (-(B - 1), B - 1)
        if mode == 0:
            v = rng.randint(lo, hi)
        elif mode == 1:
            v = hi
        elif mode == 2:
            v = lo
        elif mode == 3:
            v = hi if s % 2 else lo
        else:
            v = lo if s % 2 else hi
        S.append(v)
    return S


def test_short_fold_is_congruent_and_below_2_57():
    primes = _short_primes()
    assert len(primes) >= 10
    for q in primes:
        rng = random.Random(q)
        for it in range(400):
            S = _diagonals(rng, it % 5)
            V = sum(v << (8 * s) for s, v in enumerate(S))
            assert fold_short(S, q) % q == V % q, (q, S)


def test_short_reduction_below_2_60():
    for q in _short_primes():
        rng = random.Random(q + 1)
        xs = [0, 1, q - 1, q, 2 * q - 1, (1 << 54) - 1, 1 << 54, (1 << 58) - 1,
              (1 << 60) - 1] + [rng.randrange(1 << 60) for _ in range(2000)]
        for x in xs:
            assert reduce_short(x, q) == x % q, (q, x)


def test_short_horner_step():
    """The flood's Horner step r -> r 2^32 + w (mod q) of the circuit-private
    form: (r >> 22) delta + (r mod 2^22) 2^32 + w < 2^56, then the short
    reduction."""
    for q in _short_primes():
        delta = (1 << 54) - q
        rng = random.Random(q + 2)
        cases = [(0, 0), (q - 1, (1 << 32) - 1), (q - 1, 0), ((1 << 22) - 1, 1)]
        cases += [(rng.randrange(q), rng.randrange(1 << 32)) for _ in range(2000)]
        for r, w in cases:
            assert (r >> 22) < 1 << 32
            y = (r >> 22) * delta + ((r & 0x3FFFFF) << 32) + w
            assert y < 1 << 56
            assert reduce_short(y, q) == (r * (1 << 32) + w) % q, (q, r, w)


def _pm_join(L, H, q):
    """L + 2^24 H (mod q) as the device forms it: every factor and sum within
    its 32- or 64-bit type."""
    delta = (1 << 54) - q
    assert -(1 << 63) <= L < 1 << 63 and -(1 << 63) <= H < 1 << 63
    h0, h1 = H & 0xFFFFFFFF, H >> 32
    assert -(1 << 31) <= h1 < 1 << 31 and 4 * delta < 1 << 31
    r = L + h0 * (1 << 24)
    assert -(1 << 63) <= r < 1 << 63
    r += h1 * 4 * delta
    assert -(1 << 63) <= r < 1 << 63
    return r


def mul_pm(x, w, q):
    """The transforms' product of a signed x, |x| < 2^62, by a fixed w < q."""
    wp = (w << 32) % q
    x0, x1 = x & 0xFFFFFFFF, x >> 32
    assert -(1 << 31) <= x1 < 1 << 31
    words = [w & 0xFFFFFF, w >> 24, wp & 0xFFFFFF, wp >> 24]
    assert all(0 <= v < 1 << 30 for v in words)
    return _pm_join(x0 * words[0] + x1 * words[2], x0 * words[1] + x1 * words[3], q)


def reduce_signed(x, q):
    delta = (1 << 54) - q
    x += q << 9
    assert 0 <= x < 1 << 64
    r = (x >> 54) * delta + (x & ((1 << 54) - 1))
    assert r < 2 * q
    return r - q if r >= q else r


def mulmod_pm(a, b, q):
    """Product of two residues, folded twice; every 32-bit factor checked."""
    delta = (1 << 54) - q
    a0, a1, b0, b1 = a & 0xFFFFFFFF, a >> 32, b & 0xFFFFFFFF, b >> 32
    p0 = a0 * b0
    m = a0 * b1 + a1 * b0 + (p0 >> 32)
    w = (m >> 22) + ((a1 * b1) << 10)
    assert m < 1 << 64 and w < 1 << 64
    z0 = (w & 0xFFFFFFFF) * delta
    z1 = (w >> 32) * delta + (z0 >> 32)
    assert (z1 >> 22) < 1 << 32
    lo = (p0 & 0xFFFFFFFF) + (z0 & 0xFFFFFFFF)
    hi = (m & 0x3FFFFF) + (z1 & 0x3FFFFF)
    return lo + (hi << 32) + (z1 >> 22) * delta


def test_transform_products():
    """mul_pm over |x| < 2^62 (a butterfly's T, which a stage adds to or
    subtracts from a value: 14 stages stay within 147 2^54 < 2^62), mul_pm32,
    mulmod_pm and the transforms' last reduction."""
    unit = 1 << 54
    lo, hi = -5 * unit // 4, 52 * unit // 5
    assert unit + 14 * hi < 1 << 62 and hi + (1 << 57) + (1 << 55) < 1 << 60
    for q in _short_primes():
        rng = random.Random(q + 3)
        xs = [0, 1, -1, (1 << 62) - 1, -(1 << 62) + 1, (1 << 32) - 1, 1 << 32, -(1 << 32),
              ((1 << 30) - 1) << 32, -((1 << 30) << 32) + 0xFFFFFFFF]
        ws = [0, 1, q - 1, (1 << 24) - 1, q >> 1, q - (1 << 24)]
        xs += [rng.randrange(-(1 << 62) + 1, 1 << 62) for _ in range(300)]
        ws += [rng.randrange(q) for _ in range(30)]
        for w in ws:
            for x in xs:
                r = mul_pm(x, w, q)
                assert lo < r < hi and r % q == x * w % q, (q, x, w)
                assert reduce_signed(x, q) == x % q
            for x in [0, (1 << 31) - 1] + [rng.randrange(1 << 31) for _ in range(20)]:
                H = x * (w >> 24)
                r = x * (w & 0xFFFFFF) + (H & 0xFFFFFFFF) * (1 << 24) + (H >> 32) * 4 * (unit - q)
                assert 0 <= r < 1 << 57 and r % q == x * w % q
        for a in [0, 1, q - 1, (1 << 32) - 1, 1 << 32] + [rng.randrange(q) for _ in range(100)]:
            for b in [0, 1, q - 1, (1 << 32) - 1, 1 << 53] + [rng.randrange(q) for _ in range(20)]:
                r = mulmod_pm(a, b, q)
                assert 0 <= r < 1 << 56 and r % q == a * b % q


def test_product_by_a_word():
    """mul_pm32 over its whole range: below 2^57 + 2^54 for x < 2^32, which a value
    just past 2^57 nearly reaches, below 2^57 for x < 2^31; with the lazy inverse's
    value, 2 q and a flood residue it stays where the reduction holds."""
    unit = 1 << 54
    top = 0
    for q in _short_primes() + [unit - (1 << 17), unit - (1 << 22) + 1]:
        rng = random.Random(q + 4)
        ws = [0, 1, q - 1, (((1 << 29) + 1) << 24) | 0xFFFFFF, ((1 << 30) - 2) << 24 | 0xFFFFFF]
        ws += [rng.randrange(q) for _ in range(30)]
        xs = [0, 1, (1 << 31) - 1, (1 << 31) - 8, (1 << 32) - 1, (1 << 32) - 8]
        xs += [rng.randrange(1 << 32) for _ in range(30)]
        for w in ws:
            for x in xs:
                H = x * (w >> 24)
                r = x * (w & 0xFFFFFF) + (H & 0xFFFFFFFF) * (1 << 24) + (H >> 32) * 4 * (unit - q)
                assert r % q == x * w % q
                assert r < ((1 << 57) if x < 1 << 31 else (1 << 57) + unit), (q, x, w)
                top = max(top, r)
    assert top > 1 << 57
    assert 52 * unit // 5 + (1 << 57) + unit + 3 * unit < 1 << 60


def test_workload_primes_take_the_short_forms():
    """The primes of every workload here (N = 4096 ... 16384, L <= 3) are
    2^54 - delta with delta < 2^22, so the batched schedules run the short
    forms; 50- and 52-bit primes do not."""
    for N in (4096, 8192, 16384):
        for q in oracle.rns_primes(N, 3):
            assert 0 < (1 << 54) - q < 1 << 22, (N, q)
    for bits in (50, 52):
        q = oracle.rns_primes(4096, 1, bits=bits)[0]
        assert (1 << 54) - q >= 1 << 22
