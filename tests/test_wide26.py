"""The latency unit's field product (wide26.hpp), modelled on plain integers:
its constant tables, the bounds of its column sums with every operand at its
largest, and its value lane by lane."""

import random
import re

from oracle import te
from oracle.field import P
from paper_2502_11660_amd import build as B

BITS, N = 26, 16
MASK = (1 << BITS) - 1


def _table(name):
    text = open(B.CSRC + "/wide26.hpp").read()
    body = re.search(r"%s(?:\[\d+\])+ = \{(.*?)\};" % name, text, re.S).group(1)
    return [int(x, 16) for x in re.findall(r"0x([0-9a-f]+)u", body)]


def value(limbs):
    return sum(x << (BITS * i) for i, x in enumerate(limbs))


FOLD = [_table("kFold26")[N * k:N * k + N] for k in range(17)]
OFF = _table("kOff26")


def carries(cols):
    """w26_fold's and w26_limbs' pass: bits 26..51 one lane up, the rest two."""
    out = []
    for i, c in enumerate(cols):
        assert c < 1 << 64
        mid = (cols[i - 1] >> BITS) & MASK if i >= 1 else 0
        top = cols[i - 2] >> 2 * BITS if i >= 2 else 0
        out.append((c & MASK) + mid + top)
    return out


def product(a, b):
    """The lanes' arithmetic; every intermediate within its register."""
    cols = [sum(a[i] * b[j - i] for i in range(N) if 0 <= j - i < N) for j in range(32)]
    t = carries(cols)
    assert cols[31] >> BITS == 0 and cols[30] >> 2 * BITS == 0 and max(t) < 1 << 32
    acc = [(t[j] if j < 15 else 0) + sum(t[15 + k] * FOLD[k][j] for k in range(17)) for j in range(N)]
    r = carries(acc)
    assert acc[15] >> BITS == 0 and acc[14] >> 2 * BITS == 0
    return r


def test_tables():
    for k in range(17):
        assert value(FOLD[k]) == pow(2, BITS * (15 + k), P)
    assert value(OFF) % P == 0
    assert value(_table("kK26")) == te.K_TE


def test_values_of_the_additions_operands():
    rng = random.Random(26)
    for _ in range(50):
        x, y = ([rng.choice([0, MASK, rng.getrandbits(26)]) for _ in range(15)] + [rng.getrandbits(16)]
                for _ in range(2))
        d = [u + o - v for u, o, v in zip(x, OFF, y)]
        assert min(d) >= 0
        for a, b in ((x, y), (d, x), (d, d)):
            assert (value(product(a, b)) - value(a) * value(b)) % P == 0


def test_bounds_close():
    """Limb bounds of a product (a, top) carried through every operand of the
    addition and the doubling give the same bounds again."""
    a, top = MASK, 1 << 17
    om, ot = max(OFF[:15]), OFF[15]
    for _ in range(4):
        lim = lambda m, k: [m * a + k * om] * 15 + [m * top + k * ot]  # noqa: E731
        pairs = [(lim(1, 1), lim(1, 1)),   # (Y1 - X1)(Y2 - X2)
                 (lim(2, 0), lim(2, 0)),   # (Y1 + X1)(Y2 + X2)
                 (lim(2, 1), lim(3, 0)),   # F G: D + off - C, D + C
                 (lim(1, 1), lim(2, 1)),   # E F
                 (lim(3, 0), lim(2, 0)),   # G H
                 (lim(1, 1), lim(2, 0)),   # E H, doubling (Y - X)(Y + X)
                 (lim(2, 0), lim(1, 1)),   # doubling: E F
                 (lim(1, 0), lim(0, 1))]   # doubling: G H
        res = [product(*p) for p in pairs]
        a = max(max(r[:15]) for r in res)
        top = max(r[15] for r in res)
        assert min(OFF[:15]) > 2 * a and OFF[15] > 2 * top
    assert a < 1.01 * 2 ** 27 and top < 2 ** 18.2


def test_quotient_of_the_final_reduction():
    """w26_to_words: the 56-bit quotient estimate leaves [0, 2p)."""
    rng = random.Random(27)
    text = open(B.CSRC + "/wide26.hpp").read()
    scale = 1.0 / float(re.search(r"\(1\.0 / ([0-9.]+)\)", text).group(1))
    for i in range(4000):
        v = rng.getrandbits(rng.randint(370, 408))
        if i % 4 == 0:
            v = max(0, P * rng.getrandbits(rng.randint(1, 31)) + rng.choice([-1, 0, 1]))
        v = min(v, (1 << 408) - 1)
        t = v >> 352
        est = float(t >> 32) * 4294967296.0 + float(t & 0xFFFFFFFF)
        est = est * scale - 2.0 ** -18
        q = int(est) if est > 0 else 0
        assert q < 1 << 32 and 0 <= v - q * P < 2 * P
