"""The segments' band solve at its edges: systems of 4 to 43 coefficients (the
forward pass works four coefficients ahead, the backward one eight), segments
of one interval, overlaps that reach past the mission's ends and none, and
more segments than one.

Well-conditioned systems (60,000 stars, across-scan records too: 50 records
and more in every knot interval).  An update may differ from the
extended-precision oracle's by 1e-3 uas, the parity target of every update, or
by ten times the double-precision oracle's own largest deviation from it (two
implementations' rounding of the same system, whose maxima over a few hundred
coefficients scatter)."""
import numpy as np
import pytest

import oracle
import synth
import synth.configs as C
from test_gpu_parity import agis_mod  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_iv,seg_len,overlap", [(1, 240, 12), (2, 1, 0), (4, 3, 1), (5, 240, 12), (6, 2, 12),
                                                  (7, 7, 2), (8, 1, 12), (13, 5, 0), (23, 9, 12), (40, 13, 3),
                                                  (40, 240, 12)])
def test_attitude_update_of_short_segments(agis_mod, n_iv, seg_len, overlap):  # noqa: F811
    agis = agis_mod
    law, spec = C.workload("tiny", n_src=60000, years=n_iv * 1200.0 / synth.YEAR, min_transits=0, ac_obs=True,
                           seg_len=seg_len, seg_overlap=overlap)
    w = synth.make_world(spec, law)
    assert w.n_att == n_iv + 3
    eta = oracle.observed_field_angles(w)
    a = {}
    for precision in ("double", "extended"):
        pr = oracle.problem_from_world(w, eta, precision=precision)
        pr.attitude_update()
        a[precision] = np.array(pr.a, dtype=np.float64)
    ctx = agis.agis_create(w.consts, w.knots)
    try:
        agis.agis_load_observations(ctx, w.t, eta, w.sigma, w.src, w.fov, w.cell, w.src_true.shape[0], w.n_cells)
        agis.agis_set_sources(ctx, w.src_start)
        agis.agis_set_attitude(ctx, w.att_start)
        agis.agis_set_calibration(ctx, w.cal_start)
        st = agis.agis_attitude_update(ctx)
        got = agis.agis_get_attitude(ctx, w.n_att)
    finally:
        agis.agis_destroy(ctx)
    assert st["defect"] == 0
    floor = np.abs(a["double"] - a["extended"]).max()
    assert np.abs(got - a["extended"]).max() <= max(1e-3 * synth.UAS, 10.0 * floor)
