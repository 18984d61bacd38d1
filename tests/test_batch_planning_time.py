"""Picking widths costs little beside planning: a batch of many jobs with c = 0."""

import time

from paper_2502_11660_amd import _lib


def test_picks_are_cheap():
    """Against the same jobs with a given width, whose planning has everything but the
    picks: 16-20 times as long when each pick worked its model out anew, 4.4 now; the
    limit lies half way on a logarithmic scale."""
    k = 5000
    jobs = {c: (_lib.MsmJob * k)(*[_lib.MsmJob(256, 256, 256, 700 + i % 1000, c) for i in range(k)])
            for c in (0, 9)}
    best = {c: 1e9 for c in jobs}
    for _ in range(15):
        for c, arr in jobs.items():
            t = time.perf_counter()
            assert _lib.lib().msm_batch_workspace_bytes(arr, k, _lib.MSM_DIGITS_SIGNED) > 0
            best[c] = min(best[c], time.perf_counter() - t)
    assert best[0] < 9 * best[9], best
