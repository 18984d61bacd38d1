"""A workspace of msm_batch_workspace_bytes for some jobs with c = 0 serves smaller
ones, also where the widths picked for these need more."""

import ctypes

import pytest
import torch

from oracle import msm
from paper_2502_11660_amd import _lib, api, inputs

S, U, G = _lib.MSM_DIGITS_SIGNED, _lib.MSM_DIGITS_UNSIGNED, _lib.MSM_DIGITS_GLV

CASES = [(G, [513], [512]), (G, [15000], [14423]), (S, [930], [927]),
         (U, [1025], [1024]), (G, [11168, 11059], [10832, 11059]),
         (S, [702, 9277], [631, 8998])]


def _need(sizes, enc, c=0):
    arr = (_lib.MsmJob * len(sizes))(*[_lib.MsmJob(256, 256, 256, n, c) for n in sizes])
    return _lib.lib().msm_batch_workspace_bytes(arr, len(sizes), enc), arr


@pytest.mark.skipif(torch.cuda.is_available(), reason="would copy to made-up pointers")
@pytest.mark.parametrize("enc,larger,sizes", CASES)
def test_smaller_jobs_fit(enc, larger, sizes):
    """On a host without GPU: MSM_EHIP once a plan fits."""
    room, (need, arr) = _need(larger, enc)[0], _need(sizes, enc)
    assert room < need
    h, p = ctypes.c_void_p(), ctypes.c_void_p(256)
    create = _lib.lib().msm_batch_create
    assert create(arr, len(sizes), enc, p, room, 0, ctypes.byref(h)) == _lib.MSM_EHIP
    assert create(arr, len(sizes), enc, p, 1000, 0, ctypes.byref(h)) == _lib.MSM_ENOSPC
    assert create(_need(sizes, enc, 21)[1], len(sizes), enc, p, room, 0,
                  ctypes.byref(h)) == _lib.MSM_EINVAL


@pytest.mark.gpu
@pytest.mark.parametrize("enc,larger,sizes", CASES)
def test_smaller_jobs_run(enc, larger, sizes):
    lib, room = _lib.lib(), _need(larger, enc)[0]
    n = max(sizes)
    kw = inputs.nonzero_scalars_mod_r(95, n, stream=1)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf, endo=enc == G)
    rec = 36 * (2 if enc == G else 1)
    sw = [inputs.scalars_mod_r(95 + j, m, stream=2) for j, m in enumerate(sizes)]
    jobs = [(xyu[:rec * m], api.to_device(sw[j]), api.words(api.MSM_RESULT_WORDS), m, 0)
            for j, m in enumerate(sizes)]
    ws = api.words(room // 4 + 64)
    ws.fill_(-1)
    h = ctypes.c_void_p()
    assert lib.msm_batch_create(api._job_array(jobs, enc), len(jobs), enc, api._ptr(ws), room, 0,
                                ctypes.byref(h)) == _lib.MSM_OK
    assert lib.msm_batch_run(h, api._stream()) == _lib.MSM_OK
    for j, m in enumerate(sizes):
        got, flags = api.decode_result(api.to_host(jobs[j][2]))
        assert flags == 0 and got == msm.closed_form_words(sw[j], kw[:m]), j
    lib.msm_batch_destroy(h)
    assert bool((ws[room // 4:] == -1).all())
