"""A workspace of msm_workspace_bytes(n, 0, encoding) serves every smaller MSM with
c = 0, also where the picked width needs more for fewer points."""

import ctypes

import pytest
import torch

from oracle import msm
from paper_2502_11660_amd import _lib, api, inputs

S, U, G = _lib.MSM_DIGITS_SIGNED, _lib.MSM_DIGITS_UNSIGNED, _lib.MSM_DIGITS_GLV


def _host_status(n, enc, ws_bytes, c=0):
    """msm_run's status on a host without GPU: MSM_EHIP once a plan fits."""
    p = ctypes.c_void_p(256)
    return _lib.lib().msm_run(p, p, n, c, enc, p, p, ws_bytes, None)


@pytest.mark.skipif(torch.cuda.is_available(), reason="would launch on made-up pointers")
@pytest.mark.parametrize("enc", [S, U, G])
def test_smaller_sizes_fit(enc):
    sizes = sorted({int(round(1.13 ** k)) for k in range(8, 105)} | {512, 513, 927, 930, 1024, 1025,
                                                                    14423, 15000})
    need = [_lib.lib().msm_workspace_bytes(n, 0, enc) for n in sizes]
    fell = 0
    for i, n in enumerate(sizes):
        for j in range(i, len(sizes)):
            if need[j] < need[i]:
                fell += 1
                assert _host_status(n, enc, need[j]) == _lib.MSM_EHIP, (n, sizes[j])
        assert _host_status(n, enc, need[i]) == _lib.MSM_EHIP
        assert _host_status(n, enc, 100) == _lib.MSM_ENOSPC
    assert fell > 0


@pytest.mark.gpu
@pytest.mark.parametrize("enc,n,larger", [(G, 512, 513), (G, 14423, 15000), (S, 927, 930),
                                          (U, 1024, 1025)])
def test_run_in_a_larger_size_s_workspace(enc, n, larger):
    ws = api.workspace(larger, 0, enc)
    assert ws.numel() * 4 < api.workspace_bytes(n, 0, enc)
    kw = inputs.nonzero_scalars_mod_r(90 + n, n, stream=1)
    sw = inputs.scalars_mod_r(90 + n, n, stream=2)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf, endo=enc == G)
    ws.fill_(-1)
    got, flags = api.decode_result(api.to_host(api.msm_run(xyu, api.to_device(sw), n, 0, enc, ws=ws)))
    assert flags == 0 and got == msm.closed_form_words(sw, kw)


@pytest.mark.gpu
def test_server_fits_the_width_to_the_schedule():
    """chunk = 4 takes more workspace at the picked width than the arena holds,
    and less at another."""
    n, sched = 20000, {"chunk": 4}

    def need(c):
        jobs = (_lib.MsmJob * 1)(_lib.MsmJob(16, 16, 16, n, c, 4, 0, 0))
        return _lib.lib().msm_batch_workspace_bytes(jobs, 1, S)

    budget = min(need(c) for c in range(4, 21))
    assert need(api.default_window(n)) > budget > api.workspace_bytes(n, 0, S)
    kw = inputs.nonzero_scalars_mod_r(91, n, stream=1)
    sw = inputs.scalars_mod_r(91, n, stream=2)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf)
    res = api.words(api.MSM_RESULT_WORDS)
    srv = api.Server(budget, streams=1)
    srv.submit(xyu, api.to_device(sw), res, n, 0, sched)
    srv.drain()
    got, flags = api.decode_result(api.to_host(res))
    srv.destroy()
    assert flags == 0 and got == msm.closed_form_words(sw, kw)


# bytes that chunks of at least 16 entries need, on quads and on lanes
COMPACT = [(G, 468, 2, 2766336), (S, 1000, 8, 3049472), (S, 20000, 8, 30170880)]


@pytest.mark.skipif(torch.cuda.is_available(), reason="would launch on made-up pointers")
@pytest.mark.parametrize("enc,n,c,nbytes", COMPACT)
def test_longer_chunks_where_there_is_less(enc, n, c, nbytes):
    lib, p = _lib.lib(), ctypes.c_void_p(256)
    assert nbytes < lib.msm_workspace_bytes(n, c, enc)
    assert _host_status(n, enc, nbytes, c) == _lib.MSM_EHIP
    assert lib.msm_bucket_accumulate(p, p, n, c, enc, p, p, nbytes, None) == _lib.MSM_EHIP
    assert _host_status(n, enc, nbytes // 2, c) == _lib.MSM_ENOSPC
    assert lib.msm_bucket_accumulate(p, p, n, c, enc, p, p, nbytes // 2, None) == _lib.MSM_ENOSPC
    assert lib.msm_bucket_accumulate(p, p, n, 0, enc, p, p, nbytes, None) == _lib.MSM_EINVAL


@pytest.mark.gpu
@pytest.mark.parametrize("ones", [False, True])
@pytest.mark.parametrize("enc,n,c,nbytes", COMPACT)
def test_run_in_longer_chunks(enc, n, c, nbytes, ones):
    """ones: half the scalars are 1, a bucket over many chunks."""
    ws = api.words(nbytes // 4 + 64)
    ws.fill_(-1)
    kw = inputs.nonzero_scalars_mod_r(92 + n, n, stream=1)
    sw = inputs.scalars_mod_r(92 + n, n, stream=2)
    if ones:
        sw[: n // 2] = inputs.ints_to_words([1], 8)
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf, endo=enc == G)
    got, flags = api.decode_result(api.to_host(
        api.msm_run(xyu, api.to_device(sw), n, c, enc, ws=ws[:nbytes // 4])))
    assert flags == 0 and got == msm.closed_form_words(sw, kw)
    assert bool((ws[nbytes // 4:] == -1).all())  # nothing beyond the workspace
