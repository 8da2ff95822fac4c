"""The A/C pass over ranges of knot intervals: fewer intervals than a wavefront
takes and not a multiple of it, intervals without observations at either end and
in between, numbers of observations around multiples of four and of 64.

The interval sums are seen through what they give, the calibration offsets and
the attitude update.  An update may differ from the extended-precision oracle's
by 1e-3 uas, the parity target of every update, or by ten times the
double-precision oracle's own largest deviation from it (two implementations'
rounding of the same system, whose maxima over a few values scatter)."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
import synth.configs as C
from test_gpu_parity import agis_mod  # noqa: F401

pytestmark = pytest.mark.gpu


def _thinned(w, n_iv, pattern):
    """The world's observations with interval j keeping pattern(j) of them (all: None)."""
    iv = np.clip(np.searchsorted(w.knots, w.t, side="right") - 4, 0, n_iv - 1)
    keep = np.ones(w.t.size, bool)
    for j in range(n_iv):
        want = pattern(j)
        if want is not None:
            keep[np.flatnonzero(iv == j)[want:]] = False
    return dataclasses.replace(w, t=w.t[keep], sigma=w.sigma[keep], src=w.src[keep], fov=w.fov[keep],
                               cell=w.cell[keep])


PATTERNS = {
    "all": lambda j: None,
    "remainders": lambda j: 61 + j % 9,
    "holes": lambda j: 0 if j % 5 == 2 or j in (0, 1) else None,
    "few": lambda j: 17 + j % 4,
}


@pytest.mark.parametrize("robust", [False, True])
@pytest.mark.parametrize("n_iv,pattern", [(1, "all"), (7, "remainders"), (8, "all"), (9, "few"), (17, "holes"),
                                          (40, "remainders"), (41, "holes")])
def test_interval_sums(agis_mod, n_iv, pattern, robust):  # noqa: F811
    agis = agis_mod
    law, spec = C.workload("tiny", n_src=60000, years=n_iv * 1200.0 / synth.YEAR, min_transits=0, ac_obs=True,
                           robust=robust)
    w = _thinned(synth.make_world(spec, law), n_iv, PATTERNS[pattern])
    eta = oracle.observed_field_angles(w)
    for block in ("calibration", "attitude"):
        want = {}
        for precision in ("double", "extended"):
            pr = oracle.problem_from_world(w, eta, state="start", precision=precision)
            getattr(pr, block + "_update")()
            want[precision] = np.array(pr.c if block == "calibration" else pr.a, dtype=np.float64)
        ctx = agis.agis_create(w.consts, w.knots)
        try:
            agis.agis_load_observations(ctx, w.t, eta, w.sigma, w.src, w.fov, w.cell, w.src_true.shape[0], w.n_cells)
            agis.agis_set_sources(ctx, w.src_start)
            agis.agis_set_attitude(ctx, w.att_start)
            agis.agis_set_calibration(ctx, w.cal_start)
            getattr(agis, "agis_" + block + "_update")(ctx)
            got = (agis.agis_get_calibration(ctx, w.n_cells) if block == "calibration"
                   else agis.agis_get_attitude(ctx, w.n_att))
        finally:
            agis.agis_destroy(ctx)
        floor = np.abs(want["double"] - want["extended"]).max()
        assert np.abs(got - want["extended"]).max() <= max(1e-3 * synth.UAS, 10.0 * floor), block
