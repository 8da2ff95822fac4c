"""The source update at its edges: 8 to 64 lanes per source, nine-record
transits and single-record ones, sources without observations and fewer sources
than a block takes (whose sums its first wavefront finishes), across-scan
records, and unequally spaced knots, whose attitude also puts the field angles
beyond the range of their series.

An update may differ from the extended-precision oracle's by 1e-3 uas, the
parity target of every update, or by ten times the double-precision oracle's
own largest deviation from it (two implementations' rounding of the same
5 x 5 systems, whose maxima over a few hundred sources scatter)."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
import synth.configs as C
from test_gpu_parity import agis_mod, src_diff_uas  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("group", [8, 16, 32, 64])
@pytest.mark.parametrize("n_src,ccd,ac,uneven", [(2, 9, False, False), (300, 9, True, False), (300, 1, False, False),
                                                 (37, 1, True, True), (130, 9, False, True)])
def test_source_update_over_all_groups(agis_mod, monkeypatch, group, n_src, ccd, ac, uneven):  # noqa: F811
    agis = agis_mod
    law, spec = C.workload("tiny", n_src=n_src, years=1.0, min_transits=8, ccd_per_transit=ccd, ac_obs=ac)
    w = synth.make_world(spec, law)
    if uneven:
        dt = np.diff(w.knots).max()
        shift = np.random.default_rng(7).uniform(-0.3, 0.3, w.knots.size) * dt
        # the ends and the days' boundaries stay (an interval lies within a day)
        shift[:4] = shift[-4:] = shift[(w.knots - w.knots[0]) % 86400.0 == 0.0] = 0.0
        w = dataclasses.replace(w, knots=w.knots + shift)
    # two sources without observations
    w = dataclasses.replace(w, src_true=np.vstack([w.src_true, w.src_true[:2]]),
                            src_start=np.vstack([w.src_start, w.src_start[:2]]))
    n = w.src_true.shape[0]
    eta = oracle.observed_field_angles(w)
    s = {}
    for precision in ("double", "extended"):
        pr = oracle.problem_from_world(w, eta, state="start", precision=precision)
        pr.source_update()
        s[precision] = np.array(pr.s, dtype=np.float64)
    monkeypatch.setenv("AGIS_S_GROUP", str(group))
    ctx = agis.agis_create(w.consts, w.knots)
    try:
        agis.agis_load_observations(ctx, w.t, eta, w.sigma, w.src, w.fov, w.cell, n, w.n_cells)
        agis.agis_set_sources(ctx, w.src_start)
        agis.agis_set_attitude(ctx, w.att_start)
        agis.agis_set_calibration(ctx, w.cal_start)
        agis.agis_source_update(ctx)
        got = agis.agis_get_sources(ctx, n)
    finally:
        agis.agis_destroy(ctx)
    floor = np.abs(src_diff_uas(s["extended"], s["double"])).max()
    assert np.abs(src_diff_uas(s["extended"], got)).max() <= max(1e-3, 10.0 * floor)
