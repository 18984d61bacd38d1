"""The measured workloads: what programs built on this library have it do.

A verifier or a test computes MSMs of a few dozen points; a prover's
commitments take 2^10 .. 2^22 points, one at a time, in batches of mixed sizes
or as requests to a server, with the points prepared once; and the point
addition itself is used on arrays of points.  `listed` names twelve such cases,
`draw` makes more of the same ranges.

Every input is made on the GPU from the seed: points P_i = k_i G for uniform
256-bit k_i, scalars uniform below the scalar field's order, or ("sparse") a
prover's witness, half of whose values are 0 or 1.
"""

import math

import torch

from paper_2502_11660_amd import api

ENCODINGS = {"signed": api.MSM_DIGITS_SIGNED, "unsigned": api.MSM_DIGITS_UNSIGNED,
             "glv": api.MSM_DIGITS_GLV}
DIGIT_BITS = {"signed": 254, "unsigned": 253, "glv": 128}
TOP_WORD = 0x12AB655E  # the scalar field order's top word: values with a smaller one are below it

WORD_PRODUCTS = 276    # 32x32-bit products of one field multiplication with its reduction
MULS_MIXED, MULS_COMPLETE = 7, 9
MULS_PREPARE = 12      # per record, the batched inverse's share included

MAX_MSM = 1 << 22


def listed():
    return [
        # a handful of points (a verifier's check, a test): launches and the
        # dependent chain of doublings are all there is
        {"name": "msm_33_signed", "kind": "msm", "n": 33, "encoding": "signed", "c": 0, "sparse": False},
        # the paper's small configuration: plain slices of 8 bits
        {"name": "msm_1024_unsigned_c8", "kind": "msm", "n": 1024, "encoding": "unsigned", "c": 8,
         "sparse": False},
        # a small commitment from a loop that must not allocate
        {"name": "noalloc_4099_glv", "kind": "noalloc", "n": 4099, "encoding": "glv", "c": 0,
         "sparse": False},
        # an ordinary commitment, default width
        {"name": "msm_65536_glv", "kind": "msm", "n": 65536, "encoding": "glv", "c": 0, "sparse": False},
        # a witness commitment: half of the scalars 0 or 1, points without images
        {"name": "msm_300007_signed_sparse", "kind": "msm", "n": 300007, "encoding": "signed", "c": 0,
         "sparse": True},
        # the headline workload
        {"name": "msm_1048576_glv_c16", "kind": "msm", "n": 1 << 20, "encoding": "glv", "c": 16,
         "sparse": False},
        # the largest
        {"name": "msm_4194304_glv", "kind": "msm", "n": MAX_MSM, "encoding": "glv", "c": 0,
         "sparse": False},
        # many independent MSMs of log-uniform sizes planned as one batch
        {"name": "batch_64_glv", "kind": "batch", "jobs": 64, "lo": 10, "hi": 18, "encoding": "glv",
         "sparse": False},
        # a burst of requests through the server
        {"name": "server_24_signed", "kind": "server", "jobs": 24, "lo": 12, "hi": 18,
         "encoding": "signed", "sparse": False},
        # a point set on its way into prepared form, with its images
        {"name": "prepare_1048576_endo", "kind": "prepare", "n": 1 << 20, "endo": True},
        # arrays of point additions: a large one with prepared operands, an
        # odd-sized one with extended operands
        {"name": "padd_4194304_mixed", "kind": "padd", "n": 1 << 22, "form": "mixed"},
        {"name": "padd_300001_complete", "kind": "padd", "n": 300001, "form": "complete"},
    ]


def _log_int(rng, lo, hi):
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, n | 1 if rng.random() < 0.5 else n))


def draw(rng):
    kind = rng.choice(["msm", "msm", "msm", "noalloc", "batch", "server", "prepare", "padd"])
    if kind == "padd":
        return {"kind": kind, "n": _log_int(rng, 64, 1 << 22), "form": rng.choice(["mixed", "complete"])}
    if kind == "prepare":
        return {"kind": kind, "n": _log_int(rng, 64, 1 << 21), "endo": rng.random() < 0.5}
    enc = rng.choice(["signed", "unsigned", "glv", "glv"])
    sparse = rng.random() < 0.25
    if kind in ("batch", "server"):
        lo = rng.randint(6, 13)
        return {"kind": kind, "jobs": rng.randint(2, 64) if kind == "batch" else rng.randint(2, 32),
                "lo": lo, "hi": rng.randint(lo + 1, 17), "encoding": enc, "sparse": sparse}
    top = {"signed": 1 << 20, "unsigned": 1 << 19, "glv": MAX_MSM}[enc]
    if kind == "noalloc":
        top = 1 << 16
    n = _log_int(rng, 1, top)
    # the default width, or one a caller's own tuning picks near it
    c = 0
    if rng.random() < 0.4:
        c = max(6, min(16, int(math.log2(n)) - rng.randint(2, 5)))
    if kind == "noalloc":
        c = 0
    return {"kind": kind, "n": n, "encoding": enc, "c": c, "sparse": sparse}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _sizes(case, seed):
    g = torch.Generator().manual_seed(int(seed) * 2 + 1)
    u = torch.rand(case["jobs"], generator=g, dtype=torch.float64) * (case["hi"] - case["lo"]) + case["lo"]
    return [max(1, int(x)) for x in torch.exp2(u).tolist()]


def _draws(case, seed):
    """(k, s): multipliers of the points and scalars, (N, 8) int32 words on the GPU."""
    n = case["n"] if "n" in case else sum(_sizes(case, seed))
    g = torch.Generator(device="cuda").manual_seed(int(seed))

    def words():
        return torch.randint(-(1 << 31), 1 << 31, (n, 8), generator=g, device="cuda", dtype=torch.int32)

    k, s = words(), words()
    s[:, 7] = torch.randint(0, TOP_WORD, (n,), generator=g, device="cuda", dtype=torch.int32)
    if case.get("sparse"):
        small = torch.randint(0, 4, (n,), generator=g, device="cuda", dtype=torch.int32)  # 0, 1: kept short
        s *= (small >= 2).to(torch.int32)[:, None]
        s[:, 0] = torch.where(small < 2, small, s[:, 0])
    return k, s


def _points(k, endo):
    """(xy, inf, prepared records) of P_i = k_i G."""
    n = k.shape[0]
    xy, inf = api.gen_points(k.reshape(-1), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf, endo=endo)
    return xy, inf, xyu


def prepare(case, seed):
    k, s = _draws(case, seed)
    kind = case["kind"]
    if kind == "prepare":
        n = case["n"]
        xy, inf = api.gen_points(k.reshape(-1), n)
        return {"case": case, "xy": xy, "inf": inf, "n": n,
                "out": api.words(api.XYU_WORDS * n * (2 if case["endo"] else 1)),
                "status": torch.zeros(1, dtype=torch.int32, device="cuda")}
    if kind == "padd":
        n = case["n"]
        xyu = _points(k, False)[2].view(n, 3, 12)
        soa = xyu.permute(1, 2, 0).contiguous()                      # X, Y, U rows
        x, y = soa[0].reshape(-1), soa[1].reshape(-1)
        # a: each point scaled by another point's coordinate (Z != 1)
        lam = torch.roll(soa[0], 1, dims=1).reshape(-1).contiguous()
        mul = lambda u, v: api.fe_mul_batch(u, v, n)                 # noqa: E731
        a = torch.cat([mul(x, lam), mul(y, lam), mul(mul(x, y), lam), lam])
        # b: the points in another order, prepared or extended with their own scale
        rolled = torch.roll(soa, 7, dims=2).contiguous()
        if case["form"] == "mixed":
            return {"case": case, "a": a, "b": rolled.reshape(-1), "n": n, "form": api.MSM_FORM_XYU,
                    "out": api.words(4 * 12 * n)}
        x2, y2 = rolled[0].reshape(-1), rolled[1].reshape(-1)
        mu = torch.roll(soa[1], 3, dims=1).reshape(-1).contiguous()
        b = torch.cat([mul(x2, mu), mul(y2, mu), mul(mul(x2, y2), mu), mu])
        return {"case": case, "a": a, "b": b, "n": n, "form": api.MSM_FORM_XYTZ,
                "out": api.words(4 * 12 * n)}
    enc = ENCODINGS[case["encoding"]]
    glv = case["encoding"] == "glv"
    xyu = _points(k, glv)[2]
    s = s.reshape(-1)
    st = {"case": case, "xyu": xyu, "s": s, "enc": enc}
    if kind in ("msm", "noalloc"):
        st["result"] = api.words(api.MSM_RESULT_WORDS)
        if kind == "msm":
            st["ws"] = api.workspace(case["n"], case["c"], enc)
        return st
    sizes = _sizes(case, seed)
    st["result"] = torch.zeros(len(sizes), api.MSM_RESULT_WORDS, dtype=torch.int32, device="cuda")
    rec = api.XYU_WORDS * (2 if glv else 1)
    jobs, at = [], 0
    for j, n in enumerate(sizes):
        jobs.append((xyu[rec * at:rec * (at + n)], s[8 * at:8 * (at + n)], st["result"][j], n, 0))
        at += n
    st["jobs"] = jobs
    if kind == "batch":
        st["batch"] = api.Batch(jobs, enc)
    else:
        need = max(api.workspace_bytes(n, 0, enc) for n in sizes)
        st["server"] = api.Server(max(2 << 30, need), encoding=enc)
    return st


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "msm":
        return api.msm_run(state["xyu"], state["s"], case["n"], case["c"], state["enc"],
                           result=state["result"], ws=state["ws"])
    if kind == "noalloc":
        return api.msm_run_noalloc(state["xyu"], state["s"], case["n"], case["c"], state["enc"],
                                   result=state["result"])
    if kind == "batch":
        state["batch"].run()
        return state["result"]
    if kind == "server":
        server = state["server"]
        for job in state["jobs"]:
            server.submit(*job)
        server.drain()
        server.progress()
        return state["result"]
    if kind == "prepare":
        return api.points_prepare(state["xy"], state["n"], inf=state["inf"], out=state["out"],
                                  status=state["status"], endo=case["endo"])
    return api.padd_batch(state["a"], state["b"], state["n"], state["form"], out=state["out"])


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------

def _msm_adds(n, encoding, c):
    """Point additions of Pippenger's method at its cheapest width (or the
    caller's): a mixed one per digit, two complete ones per bucket."""
    points = 2 * n if encoding == "glv" else n
    best = None
    for w in ([c] if c else range(2, 21)):
        windows = -(-DIGIT_BITS[encoding] // w)
        buckets = windows << (w if encoding == "unsigned" else w - 1)
        muls = points * windows * MULS_MIXED + 2 * min(buckets, points * windows) * MULS_COMPLETE
        best = muls if best is None else min(best, muls)
    return best


def work(case):
    kind = case["kind"]
    if kind == "padd":
        mixed = case["form"] == "mixed"
        return {"bytes": case["n"] * 48 * (11 if mixed else 12),
                "flops": 2 * WORD_PRODUCTS * case["n"] * (MULS_MIXED if mixed else MULS_COMPLETE)}
    if kind == "prepare":
        rec = 2 if case["endo"] else 1
        return {"bytes": case["n"] * (96 + 4 + 144 * rec),
                "flops": 2 * WORD_PRODUCTS * case["n"] * MULS_PREPARE * rec}
    if "n" in case:
        sizes, c = [case["n"]], case["c"]
    else:  # log-uniform sizes: their mean
        lo, hi = 2.0 ** case["lo"], 2.0 ** case["hi"]
        sizes, c = [int((hi - lo) / math.log(hi / lo))] * case["jobs"], 0
    rec = 288 if case["encoding"] == "glv" else 144
    return {"bytes": sum(n * (rec + 32) + 4 * api.MSM_RESULT_WORDS for n in sizes),
            "flops": sum(2 * WORD_PRODUCTS * _msm_adds(n, case["encoding"], c) for n in sizes)}


# ---------------------------------------------------------------------------
# exact values: sum s_i (k_i G) = ((sum s_i k_i) mod r) G in plain integers
# ---------------------------------------------------------------------------

P = 0x01AE3A4617C510EAC63B05C06CA1493B1A22D9F300F5138F1EF3622FBA094800170B5D44300000008508C00000000001
R = 0x12AB655E9A2CA55660B44D1E5C37B00159AA76FED00000010A11800000000001
G = (0x008848DEFE740A67C8FC6225BF87FF5485951E2CAA9D41BB188282C8BD37CB5CD5481512FFCD394EEAB9B16EB21BE9EF,
     0x01914A69C5102EFF1F674F5D30AFEEC4BD7FB348CA3E52D96D182AD44FB82305C2FE3D3634A9591AFD82DE55559C8EA6)


def _add(a, b):
    if a is None or b is None:
        return b if a is None else a
    if a[0] == b[0]:
        if (a[1] + b[1]) % P == 0:
            return None
        m = 3 * a[0] * a[0] * pow(2 * a[1], -1, P) % P
    else:
        m = (b[1] - a[1]) * pow(b[0] - a[0], -1, P) % P
    x = (m * m - a[0] - b[0]) % P
    return x, (m * (a[0] - x) - a[1]) % P


def _mul(k, pt):
    acc = None
    for bit in bin(k)[2:] if k else "":
        acc = _add(acc, acc)
        if bit == "1":
            acc = _add(acc, pt)
    return acc


def _digits16(w):
    w = w.to(torch.int64) & 0xFFFFFFFF
    return torch.stack([w & 0xFFFF, w >> 16], dim=2).reshape(w.shape[0], 16).double()


def _dot(s, k):
    """(sum s_i k_i) mod r: 16-bit digits, whose sums of 2^20 products are
    whole numbers below 2^53."""
    total = 0
    for lo in range(0, s.shape[0], 1 << 20):
        d = _digits16(s[lo:lo + (1 << 20)]).t().contiguous() @ _digits16(k[lo:lo + (1 << 20)])
        for a, row in enumerate(d.tolist()):
            total += sum(int(v) << (16 * (a + b)) for b, v in enumerate(row))
    return total % R


def _result_words(pt):
    w = [0] * api.MSM_RESULT_WORDS
    if pt is None:
        w[24] = 1
    else:
        for c in (0, 1):
            w[12 * c:12 * c + 12] = [(pt[c] >> (32 * i)) & 0xFFFFFFFF for i in range(12)]
    return [v - (1 << 32) if v >> 31 else v for v in w]


def exact(case, seed):
    if case["kind"] in ("padd", "prepare"):
        return None  # projective coordinates; a record per point in plain integers takes too long
    k, s = (t.cpu() for t in _draws(case, seed))
    if "n" in case:
        return torch.tensor(_result_words(_mul(_dot(s, k), G)), dtype=torch.int32)
    rows, at = [], 0
    for n in _sizes(case, seed):
        rows.append(_result_words(_mul(_dot(s[at:at + n], k[at:at + n]), G)))
        at += n
    return torch.tensor(rows, dtype=torch.int32)
