"""Windows of small jobs in one block each: the largest jobs, widest buckets and
most windows that it takes and the first beyond, buckets that no, some or all
chunks split, every bucket-bit count, flags, jobs of different sizes."""

import numpy as np
import pytest

from oracle import msm
from oracle.field import R_ORDER
from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

SIGNED, UNSIGNED, GLV = api.MSM_DIGITS_SIGNED, api.MSM_DIGITS_UNSIGNED, api.MSM_DIGITS_GLV


def _points(n, seed, endo):
    kw = inputs.nonzero_scalars_mod_r(seed, n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    return kw, api.points_prepare(xy, n, inf=inf, endo=endo)[0]


def _check(xyu, sw, kw, n, c, enc, flag=0):
    got, flags = api.decode_result(api.to_host(api.msm_run(xyu, api.to_device(sw), n, c, enc)))
    words = sw.copy()
    words[:, 7] &= (1 << 29) - 1
    assert flags == flag and got == msm.closed_form_words(words, kw), (n, c)


@pytest.mark.parametrize("enc", [SIGNED, UNSIGNED, GLV])
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257])
def test_sizes_and_bits(enc, n):
    kw, xyu = _points(n, 40 + n, enc == GLV)
    sw = inputs.scalars_mod_r(40 + n, n, stream=2)
    sw[n // 2] = inputs.ints_to_words([R_ORDER - 1], 8)[0]
    sw[n // 3] = 0
    for c in (2, 3, 4, 5, 6, 7, 8, 9, 10):
        _check(xyu, sw, kw, n, c, enc)


# window 0 holds one bucket of each size, the others nothing
@pytest.mark.parametrize("sizes", [[256], [1, 255], [255, 1], [3, 250, 3], [5] * 51, [4] * 64,
                                   [7, 2, 9, 1, 30, 12, 64, 3, 100], [1] * 250,
                                   [2, 3, 6, 9, 10, 11, 17, 18, 33, 34, 66]])
@pytest.mark.parametrize("enc", [SIGNED, UNSIGNED])
def test_split_buckets(sizes, enc):
    s = np.repeat(np.arange(1, len(sizes) + 1) % 256, sizes).tolist()
    n = len(s)
    kw, xyu = _points(n, 8, False)
    _check(xyu, inputs.ints_to_words(s, 8), kw, n, 9 if enc == SIGNED else 8, enc)


@pytest.mark.parametrize("enc", [SIGNED, UNSIGNED, GLV])
def test_flag_and_batches(enc):
    """Batches below and above one window per compute unit; one job flagged."""
    rec = 36 * (2 if enc == GLV else 1)
    kw, xyu = _points(128, 6, enc == GLV)
    for jobs in (3, 40):
        sizes = [1 + (j * 37) % 128 for j in range(jobs)]
        args, words = [], []
        for j, n in enumerate(sizes):
            sw = inputs.scalars_mod_r(90 + j, n, stream=2)
            words.append(sw.copy())
            if j == 2:
                sw[n - 1, 7] |= np.uint32(1 << 30)
            args.append((xyu[:rec * n], api.to_device(sw), api.words(api.MSM_RESULT_WORDS), n, 6))
        b = api.Batch(args, enc, use_graph=True)
        for _ in range(3):
            b.run()
            for j, n in enumerate(sizes):
                got, flags = api.decode_result(api.to_host(args[j][2]))
                assert flags == (api.MSM_FLAG_RANGE if j == 2 else 0)
                assert got == msm.closed_form_words(words[j], kw[:n]), (jobs, j)
        b.destroy()
