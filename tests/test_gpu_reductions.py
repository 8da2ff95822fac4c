"""The fixed-order reductions of the frame rotator's fit and of the block
statistics, at sizes around a wavefront, a block and a full grid."""
import dataclasses

import numpy as np
import pytest

import oracle
import synth
import synth.configs as C
from test_gpu_parity import agis_mod  # noqa: F401

pytestmark = pytest.mark.gpu


def _empty_world(n_src, t_fr):
    """n_src sources without observations: 50 mas off the reference."""
    law, spec = C.workload("tiny", n_src=1, years=10 * 1200.0 / synth.YEAR, min_transits=0)
    w = synth.make_world(spec, law)
    rng = np.random.default_rng(n_src)
    ref = np.stack([rng.uniform(0.0, 2.0 * np.pi, n_src), np.arcsin(rng.uniform(-0.9, 0.9, n_src)),
                    rng.exponential(synth.MAS, n_src), rng.normal(0.0, 5 * synth.MAS, n_src),
                    rng.normal(0.0, 5 * synth.MAS, n_src)], axis=1)
    s = ref + rng.normal(0.0, 50 * synth.MAS, (n_src, 5))
    return dataclasses.replace(w, consts=dict(w.consts, t_fr=t_fr)), ref, s


@pytest.mark.parametrize("t_fr", [0.0, 0.5 * synth.YEAR])
@pytest.mark.parametrize("n_src", [3, 63, 64, 65, 255, 257, 131072, 131073])
def test_frame_fit_of_any_number_of_sources(agis_mod, n_src, t_fr):  # noqa: F811
    """Unit weights (no source update yet).  Each right-hand side is a
    difference of unit vectors' components (rounding 2 u each, three of them
    in a product) and the least squares of three sources and more all over the
    sky amplify it at most four-fold: 16 u [rad, rad/yr]; the rounding of the
    sums, relative to the 1e-7 rad result, is far below."""
    w, ref, s = _empty_world(n_src, t_fr)
    z = np.zeros(0)
    ctx = agis_mod.agis_create(w.consts, w.knots)
    try:
        agis_mod.agis_load_observations(ctx, z, z, z.astype(np.float32), z.astype(np.int32), z.astype(np.int8),
                                        z.astype(np.int32), n_src, w.n_cells)
        agis_mod.agis_set_sources(ctx, s)
        agis_mod.agis_set_frame_reference(ctx, ref)
        got = agis_mod.agis_frame_fit(ctx)
    finally:
        agis_mod.agis_destroy(ctx)
    pr = oracle.Problem(w.consts, w.knots, z, z, z.astype(np.float32), z.astype(np.int32), z.astype(np.int8),
                        z.astype(np.int32), s, w.att_start, w.cal_start, precision="extended")
    want = np.asarray(pr.frame_fit(ref), dtype=np.float64)
    assert np.abs(got - want).max() <= 16 * np.finfo(float).eps


@pytest.mark.parametrize("n_iv,days", [(3, 1), (61, 1), (64, 1), (253, 4), (600, 9)])
def test_block_statistics(agis_mod, n_iv, days):  # noqa: F811
    """RMS and largest update of every block against the parameters before and
    after it: these differ from the update by the rounding of the sum, at most
    4 u of the parameter (2 pi for alpha); a cell's update by u of its value."""
    law, spec = C.workload("tiny", n_src=40 * n_iv, years=n_iv * 1200.0 / synth.YEAR, min_transits=0, ac_obs=True)
    w = synth.make_world(spec, law)
    eta = oracle.observed_field_angles(w)
    n_src = w.src_true.shape[0]
    ctx = agis_mod.agis_create(w.consts, w.knots)
    try:
        agis_mod.agis_load_observations(ctx, w.t, eta, w.sigma, w.src, w.fov, w.cell, n_src, w.n_cells)
        agis_mod.agis_set_sources(ctx, w.src_true)
        agis_mod.agis_set_attitude(ctx, w.att_start)
        agis_mod.agis_set_calibration(ctx, w.cal_start)
        a, c = agis_mod.agis_attitude_calibration_update(ctx)
        da = agis_mod.agis_get_attitude(ctx, w.n_att) - w.att_start
        dc = agis_mod.agis_get_calibration(ctx, w.n_cells) - w.cal_start
        before = agis_mod.agis_get_sources(ctx, n_src)
        s = agis_mod.agis_source_update(ctx)
        ds = agis_mod.agis_get_sources(ctx, n_src) - before
    finally:
        agis_mod.agis_destroy(ctx)
    assert w.n_cells == 2 * days and (a["n_units"], c["n_units"], s["n_units"]) == (n_iv + 3, 2 * days, n_src)
    u = np.finfo(float).eps
    for st, d, tol in ((a, da, np.full(4, 4 * u)), (c, dc[:, None], np.full(1, 4 * u * np.abs(w.cal_start).max())),
                       (s, ds[:, 1:], np.full(4, 8 * u))):
        k = 1 if st is s else 0                    # alpha moves by the update over cos delta
        rms = np.array(st["rms_update"][k:k + d.shape[1]])
        big = np.array(st["max_update"][k:k + d.shape[1]])
        scale = np.maximum(1.0, np.abs(before[:, 1:]).max(axis=0)) if st is s else 1.0
        assert np.all(np.abs(rms - np.sqrt((d * d).mean(axis=0))) <= tol * scale + 1e-12 * rms)
        assert np.all(np.abs(big - np.abs(d).max(axis=0)) <= tol * scale + 1e-12 * big)
