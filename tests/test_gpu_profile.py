"""msm_profile_enable's modes: one "accum" record for every MSM, also where one
kernel does everything up to the window sums."""

import pytest

from paper_2502_11660_amd import api, inputs

pytestmark = pytest.mark.gpu

PHASES = ["sort", "accum", "merge", "agg", "horner"]


@pytest.mark.parametrize("n,enc,one_kernel", [
    (33, api.MSM_DIGITS_SIGNED, True), (256, api.MSM_DIGITS_UNSIGNED, True),
    (300, api.MSM_DIGITS_SIGNED, False), (20000, api.MSM_DIGITS_SIGNED, False)])
def test_records_of_a_call(n, enc, one_kernel):
    kw = inputs.nonzero_scalars_mod_r(96, n, stream=1)
    sd = api.to_device(inputs.scalars_mod_r(96, n, stream=2))
    xy, inf = api.gen_points(api.to_device(kw), n)
    xyu, _ = api.points_prepare(xy, n, inf=inf)
    plain = api.to_host(api.msm_run(xyu, sd, n, 8, enc))
    for mode, phases in ((api.MSM_PROFILE_ACCUM_KERNEL, ["accum"]),
                         (api.MSM_PROFILE_PHASES, ["accum", "horner"] if one_kernel else PHASES)):
        for ph in PHASES:
            api.profile_read(ph)
        api.profile_enable(mode)
        try:
            runs = [api.to_host(api.msm_run(xyu, sd, n, 8, enc)) for _ in range(3)]
        finally:
            api.profile_enable(api.MSM_PROFILE_OFF)
        got = {ph: api.profile_read(ph) for ph in PHASES}
        assert {ph: k for ph, (_, k) in got.items()} == {ph: 3 * (ph in phases) for ph in PHASES}
        assert all(0 < got[ph][0] < 100 for ph in phases)
        assert all((r == plain).all() for r in runs)
