"""The signed 29-bit field core (fe29.hpp): its constants and column bounds
against the oracle's integers, its asm blocks' register use, and the batched
PADD's coordinates, whose projective scale is part of the result."""

import re

import numpy as np
import pytest

from oracle import te
from oracle.field import P
from paper_2502_11660_amd import build as B
from tests import helpers as H
from tests import test_asm_hazards as TA

LIMBS, BITS = 13, 29


def _table(name):
    text = open(B.CSRC + "/fe29.hpp").read()
    body = re.search(r"%s\[NL29\] = \{([^}]*)\}" % name, text).group(1)
    return [int(x, 0) for x in body.replace("\n", " ").split(",")]


def test_constants():
    value = lambda limbs: sum(x << (BITS * i) for i, x in enumerate(limbs))  # noqa: E731
    neg_p, k = _table("kNP29"), _table("kK29")
    assert value(neg_p) == -P and neg_p[0] == -1
    assert all(abs(x) <= 1 << 28 for x in neg_p[:-1])
    assert value(k) == te.K_TE * pow(2, 406, P) % P


@pytest.mark.parametrize("digits", [13, 14])
@pytest.mark.parametrize("la,va,lb,vb", [
    (1 << 29, 4.76, 1 << 29, 4.76),       # two operands of class d, top limbs up to 2^31
    (3 << 28, 2.0, 1 << 29, 2.0),         # f29_add_p against a difference or sum of record limbs
])
def test_column_sums_fit(digits, la, va, lb, vb):
    """Largest magnitude of a 64-bit column sum, digits at their largest."""
    neg_p = _table("kNP29")
    top = -neg_p[-1]
    a = [la] * 12 + [int(va * top) + 1]
    b = [lb] * 12 + [int(vb * top) + 1]
    assert max(a[-1], b[-1]) <= 1 << 31
    carry = 0
    for col in range(digits + LIMBS - 1):
        s = carry
        s += sum(a[i] * b[col - i] for i in range(LIMBS) if 0 <= col - i < LIMBS)
        s += sum((1 << BITS) * abs(neg_p[col - j]) for j in range(digits) if 1 <= col - j < LIMBS)
        assert s < 1 << 63
        carry = s >> BITS


def test_carry_out_scanner_on_signed_multiply_adds(monkeypatch, tmp_path):
    """tests/test_asm_hazards.py's scan, for the signed multiply-add."""
    monkeypatch.setattr(TA, "MAD", re.compile(TA.MAD.pattern.replace("u64_u32", "i64_i32")))
    bad = "\n".join([";;#ASMSTART", "v_mad_i64_i32 v[70:71], s[10:11], v107, s7, v[70:71]",
                     "v_mad_i64_i32 v[70:71], s[10:11], v111, s11, v[70:71]", ";;#ASMEND"])
    assert len(TA.hazards(bad)) == 1
    TA.test_no_carry_out_overlaps_an_sgpr_factor(tmp_path)


def _edge_elements(n, seed):
    """Field elements with limbs at the ends of their range, then random ones."""
    rng = np.random.Generator(np.random.PCG64([seed, 29]))
    full = (1 << (BITS * LIMBS)) - 1
    edges = [0, 1, 2, P - 1, P - 2, (P - 1) // 2, (P + 1) // 2, full % P, (1 << 376) - 1, 1 << 376]
    edges += [((1 << (BITS * i)) - 1) % P for i in range(1, LIMBS)]
    edges += [(1 << (BITS * i)) % P for i in range(1, LIMBS)]
    out = [edges[int(rng.integers(len(edges)))] if rng.random() < 0.6 else
           int.from_bytes(rng.bytes(48), "little") % P for _ in range(n)]
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("count", [1, 63, 257])
@pytest.mark.parametrize("form", ["mixed", "complete"])
def test_padd_coordinates_and_scale(count, form):
    """Every coordinate equals the addition formula over the integers, three
    Montgomery reductions by 2^392 in all (the scale of the R = 2^384 form
    with a factor 2^8 per product level); any field elements, so that the
    operands' limbs reach their bounds."""
    from paper_2502_11660_amd import api
    ri = pow(2, -392, P)
    a = [tuple(_edge_elements(4, 1000 * i + 1)) for i in range(count)]
    b = [tuple(_edge_elements(3 if form == "mixed" else 4, 1000 * i + 2)) for i in range(count)]
    nb = 3 if form == "mixed" else 4
    out = api.padd_batch(api.to_device(H.soa(a, 4)), api.to_device(H.soa(b, nb)), count,
                         api.MSM_FORM_XYU if form == "mixed" else api.MSM_FORM_XYTZ)
    rows = H.unsoa(api.to_host(out), 4, count)
    for (x1, y1, t1, z1), q, got in zip(a, b, rows):
        x2, y2 = q[0], q[1]
        u2 = q[2] if form == "mixed" else te.K_TE * q[2]
        z2 = 1 << 384 if form == "mixed" else q[3]
        A, Bv = (y1 - x1) * (y2 - x2) * ri, (y1 + x1) * (y2 + x2) * ri
        C, D = t1 * u2 * ri, 2 * z1 * z2 * ri
        E, F, G, Hh = Bv - A, D - C, D + C, Bv + A
        assert got == tuple(v * ri % P for v in (E * F, G * Hh, E * Hh, F * G))
