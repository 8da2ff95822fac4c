"""Loading with knot intervals of as many records as the sort by source holds
(2,048), one less and one more, beside empty and single-record ones: every record
keeps its place in the residuals, and the blocks' sums hold each once."""
import numpy as np
import pytest

import oracle
import synth
from test_gpu_parity import agis_mod  # noqa: F401
from test_gpu_time_row import _survey, _updated

pytestmark = pytest.mark.gpu

COUNTS = [2047, 0, 2048, 2049, 1, 2, 5000, 129, 128, 2048, 3, 0]


@pytest.mark.parametrize("n_src", [3, 5000])
def test_intervals_around_the_sorts_limit(agis_mod, n_src):  # noqa: F811
    """Residuals to 1e-3 uas of the extended-precision oracle's, the parity
    target; the calibration's update (a mean over 13,000 residuals) too."""
    rng = np.random.default_rng(31)
    f = np.where(np.arange(n_src) % 2 == 0, 1.0, -1.0)
    phi = f * (53.25 * synth.DEG + rng.uniform(-8e-3, 8e-3, n_src))
    w = _survey(32, synth.knot_sequence(0.0, len(COUNTS) * 1200.0, 1200.0), phi, rng.uniform(-0.05, 0.05, n_src),
                lambda j: COUNTS[j], gamma_c=106.5 * synth.DEG)
    # records in no order, with equal times and noise that tells them apart
    at = rng.permutation(w.t.size)
    for name in ("t", "src", "cell", "fov", "sigma", "eta"):
        setattr(w, name, getattr(w, name)[at])
    w.eta = w.eta + 1e-7 * rng.normal(size=w.t.size)
    pr = oracle.problem_from_world(w, w.eta, state="start", precision="extended")
    want = np.asarray(pr.observe()["R"], dtype=np.float64)
    agis = agis_mod
    ctx = agis.agis_create(w.consts, w.knots)
    try:
        agis.agis_load_observations(ctx, w.t, w.eta, w.sigma, w.src, w.fov, w.cell, w.src_true.shape[0], w.n_cells)
        agis.agis_set_sources(ctx, w.src_start)
        agis.agis_set_attitude(ctx, w.att_start)
        agis.agis_set_calibration(ctx, w.cal_start)
        got = agis.agis_residuals(ctx)
    finally:
        agis.agis_destroy(ctx)
    assert np.abs(np.asarray(got) - want).max() <= 1e-3 * synth.UAS
    _, c, c_got = _updated(agis, w, "calibration")
    assert np.abs(c_got - c).max() <= 1e-3 * synth.UAS
