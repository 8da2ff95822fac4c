"""The A/C pass with 1, 2, 3, 4 and 8 knot intervals per wavefront: an interval's
observations enter its sums in the same order whatever the range, so the
updates are the same bit for bit; 1 against the oracle is in
test_gpu_ac_ranges.py."""
import numpy as np
import pytest

import oracle
import synth
import synth.configs as C
from test_gpu_ac_ranges import PATTERNS, _thinned
from test_gpu_parity import agis_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("robust", [False, True])
@pytest.mark.parametrize("n_iv,pattern", [(1, "all"), (7, "remainders"), (8, "all"), (9, "few"), (17, "holes"),
                                          (40, "remainders"), (41, "holes")])
def test_ranges_give_the_same_sums(agis_mod, monkeypatch, n_iv, pattern, robust):  # noqa: F811
    agis = agis_mod
    law, spec = C.workload("tiny", n_src=60000, years=n_iv * 1200.0 / synth.YEAR, min_transits=0, ac_obs=True,
                           robust=robust)
    w = _thinned(synth.make_world(spec, law), n_iv, PATTERNS[pattern])
    eta = oracle.observed_field_angles(w)
    out = {}
    for r in (1, 2, 3, 4, 8):
        monkeypatch.setenv("AGIS_AC_RANGE", str(r))
        ctx = agis.agis_create(w.consts, w.knots)
        try:
            agis.agis_load_observations(ctx, w.t, eta, w.sigma, w.src, w.fov, w.cell, w.src_true.shape[0], w.n_cells)
            agis.agis_set_sources(ctx, w.src_start)
            agis.agis_set_attitude(ctx, w.att_start)
            agis.agis_set_calibration(ctx, w.cal_start)
            agis.agis_attitude_calibration_update(ctx)
            out[r] = agis.agis_get_attitude(ctx, w.n_att).copy(), agis.agis_get_calibration(ctx, w.n_cells).copy()
        finally:
            agis.agis_destroy(ctx)
    for r in out:
        assert np.array_equal(out[r][0], out[1][0]) and np.array_equal(out[r][1], out[1][1]), r
