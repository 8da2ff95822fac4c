"""The A/C pass's own evaluation of a record (its residual, splines, field angle
and observer's orbit) where it leaves the fast paths: basic angles whose
rounded half has a negative error, field angles far outside the series, knots
that are not equally spaced, and knot intervals over which the observer's
longitude advances by more than the orbit series takes.

The surveys are made for that: a nearly constant attitude, and stars at chosen
places (phi, zeta) of the scanning frame, so that a record's angles are known
beforehand.  The observed angles are the oracle's at the true parameters."""
import math
import types

import numpy as np
import pytest

import oracle
import synth
import synth.configs as C
from test_gpu_parity import agis_mod, _qmul  # noqa: F401

pytestmark = pytest.mark.gpu


def _survey(seed, knots, phi, zeta, per_iv, ac_per_iv=0, gamma_c=None, own_cells=False):
    """Records of stars at (phi, zeta): per_iv(j) along-scan and ac_per_iv
    across-scan ones in knot interval j.  own_cells: a pair of calibration
    cells per interval instead of one."""
    rng = np.random.default_rng(seed)
    law, spec = C.workload("tiny", n_src=1, years=10 * 1200.0 / synth.YEAR, min_transits=0)
    consts = dict(synth.make_world(spec, law).consts)
    if gamma_c is not None:
        consts["gamma_c"] = gamma_c
    n_iv, n_att = knots.size - 7, knots.size - 4
    rot = lambda v: np.concatenate([0.5 * v, np.sqrt(1.0 - 0.25 * (v * v).sum(-1, keepdims=True))], -1)  # noqa: E731
    q0 = rng.normal(size=4)
    q0 /= np.linalg.norm(q0)
    a_true = _qmul(np.tile(q0, (n_att, 1)), rot(1e-3 * rng.normal(size=(n_att, 3))))
    u = np.stack([np.cos(zeta) * np.cos(phi), np.cos(zeta) * np.sin(phi), np.sin(zeta)], 1)
    u = np.stack([oracle.vector_rotate(q0, x) for x in u])
    s_true = np.zeros((phi.size, 5))
    s_true[:, 0], s_true[:, 1] = np.arctan2(u[:, 1], u[:, 0]), np.arcsin(u[:, 2])
    s_true[:, 2:] = 1e-8 * rng.normal(size=(phi.size, 3))
    t, src, cell, ac = [], [], [], []
    for j in range(n_iv):
        n = per_iv(j) + ac_per_iv
        t.append(rng.uniform(knots[j + 3], knots[j + 4], n))
        src.append(rng.integers(0, phi.size, n))
        ac.append(np.arange(n) >= per_iv(j))
        if own_cells:                              # one record of either field of view
            up, down = np.flatnonzero(phi > 0), np.flatnonzero(phi < 0)
            src[-1][:2] = rng.choice(up), rng.choice(down)
        cell.append((2 * j if own_cells else 0) + (phi[src[-1]] < 0))
    t, src, cell, ac = (np.concatenate(x) for x in (t, src, cell, ac))
    w = types.SimpleNamespace(consts=consts, knots=knots, t=t, src=src.astype(np.int32),
                              cell=np.where(ac, -1, cell).astype(np.int32),
                              fov=np.where(phi[src] > 0, 1, -1).astype(np.int8),
                              sigma=np.full(t.size, 0.1 * synth.MAS, np.float32), src_true=s_true, att_true=a_true,
                              cal_true=np.zeros(2 * n_iv if own_cells else 2), eps=np.zeros(t.size), n_att=n_att)
    w.src_start = s_true + 1e-7 * rng.normal(size=s_true.shape) * [1, 1, 0, 0, 0]
    w.att_start = _qmul(a_true, rot(1e-7 * rng.normal(size=(n_att, 3))))
    w.cal_start = np.zeros_like(w.cal_true)
    w.n_cells = w.cal_true.size
    w.eta = oracle.observed_field_angles(w)
    return w


def _updated(agis, w, block):
    """The block's parameters after its update from the start: the double and
    the extended oracle's and the library's."""
    out = []
    for precision in ("double", "extended"):
        pr = oracle.problem_from_world(w, w.eta, state="start", precision=precision)
        getattr(pr, block + "_update")()
        out.append(np.array(pr.c if block == "calibration" else pr.a))
    ctx = agis.agis_create(w.consts, w.knots)
    try:
        agis.agis_load_observations(ctx, w.t, w.eta, w.sigma, w.src, w.fov, w.cell, w.src_true.shape[0], w.n_cells)
        agis.agis_set_sources(ctx, w.src_start)
        agis.agis_set_attitude(ctx, w.att_start)
        agis.agis_set_calibration(ctx, w.cal_start)
        getattr(agis, "agis_" + block + "_update")(ctx)
        out.append(agis.agis_get_calibration(ctx, w.n_cells) if block == "calibration"
                   else agis.agis_get_attitude(ctx, w.n_att))
    finally:
        agis.agis_destroy(ctx)
    return out


def _half_angle_error(gamma):
    """Gamma_c / 2 less the angle of its rounded cosine and sine."""
    h = gamma / 2.0
    L = np.longdouble
    return float(L(h) - np.arctan2(L(math.sin(h)), L(math.cos(h))))


@pytest.mark.parametrize("negative", [True, False])
def test_basic_angle_with_either_rounding(agis_mod, negative):  # noqa: F811
    """The rounded cosine and sine of half the basic angle turn by an angle that
    is off by half_angle_error, which both fields' residuals have to make up
    for in opposite senses.  With one cell per field over all records the
    difference of the fields' mean residuals has the rounding of a record (3e-16
    at most in RMS) divided by the root of their number, 1e-18; the wrong
    sense would show as twice the error."""
    gammas = [(106.5 + 1e-3 * m) * synth.DEG for m in range(-400, 400)]
    gamma = (min if negative else max)(gammas, key=_half_angle_error)
    err = _half_angle_error(gamma)
    assert abs(err) > 4e-17 and (err < 0) == negative
    rng = np.random.default_rng(3)
    f = np.where(np.arange(3000) % 2 == 0, 1.0, -1.0)
    eta = rng.uniform(-8e-3, 8e-3, f.size)
    w = _survey(4, synth.knot_sequence(0.0, 60 * 1200.0, 1200.0), f * (0.5 * gamma + eta),
                rng.uniform(-0.05, 0.05, f.size), lambda j: 2000, gamma_c=gamma)
    _, want, got = _updated(agis_mod, w, "calibration")
    assert np.abs((got - want).astype(float)).max() <= 0.25 * abs(err)


def _uneven(seed, n_iv, dt):
    rng = np.random.default_rng(seed)
    inner = np.concatenate([[0.0], np.cumsum(rng.uniform(0.6, 1.4, n_iv) * dt)])
    return np.concatenate([np.full(3, inner[0]), inner, np.full(3, inner[-1])])


@pytest.mark.parametrize("lo,hi", [(0.02, 0.1), (0.3, 1.2), (1.4, 1.7), (2.6, 3.1)])
def test_field_angles_of_any_size(agis_mod, lo, hi):  # noqa: F811
    """One record of either field in every interval, a pair of cells each: a
    pair's update is half the difference of its two residuals.  A residual's
    rounding is that of the direction, 1.5e-16 in RMS (half the figure for two
    implementations' difference), of an angle up to pi and of its sum with
    the basic angle, ulp(pi) / sqrt(12) = 1.3e-16 each: 2.4e-16 together; 4e-16
    allows for 1.7 times that, and half a difference has 1 / sqrt(2) of it."""
    rng = np.random.default_rng(11)
    f = np.where(np.arange(4000) % 2 == 0, 1.0, -1.0)
    w = _survey(12, synth.knot_sequence(0.0, 3000 * 1200.0, 1200.0), f * rng.uniform(lo, hi, f.size),
                rng.uniform(-0.05, 0.05, f.size), lambda j: 2, gamma_c=0.02, own_cells=True)
    _, want, got = _updated(agis_mod, w, "calibration")
    d = (got - want).astype(float)
    assert np.sqrt((d * d).mean()) <= 4e-16 / math.sqrt(2.0)


# (knots, |phi| beyond half the basic angle, zeta, across-scan records per interval)
REGIMES = {
    "uneven": (_uneven(1, 61, 1200.0), 8e-3, 0.05, 0),
    "uneven_ac": (_uneven(2, 61, 1200.0), 8e-3, 9e-3, 12),
    "wide_ac": (synth.knot_sequence(0.0, 40 * 1200.0, 1200.0), 0.6, 1.0, 12),
    "all_round": (_uneven(3, 24, 2400.0), None, 0.5, 12),
    "day_long": (synth.knot_sequence(0.0, 33 * 60000.0, 60000.0), 0.05, 0.05, 12),
    "months_long": (_uneven(4, 9, 8e6), 0.05, 0.05, 12),
}


@pytest.mark.parametrize("regime", list(REGIMES))
@pytest.mark.parametrize("block", ["attitude", "calibration"])
def test_updates_off_the_fast_paths(agis_mod, regime, block):  # noqa: F811
    """An update may differ from the extended-precision oracle's by 1e-3 uas, the
    parity target of every update, or by ten times the double-precision
    oracle's own largest deviation from it (two implementations' rounding of
    the same system, whose maxima over a few hundred coefficients scatter)."""
    knots, width, tilt, n_ac = REGIMES[regime]
    rng = np.random.default_rng(21)
    gamma = 106.5 * synth.DEG
    f = np.where(np.arange(600) % 2 == 0, 1.0, -1.0)
    beyond = rng.uniform(-1.0, 1.0, f.size) * (width if width is not None else 0.0)
    phi = f * (0.5 * gamma + beyond) if width is not None else f * rng.uniform(0.02, math.pi - 0.02, f.size)
    w = _survey(22, knots, phi, rng.uniform(-tilt, tilt, f.size), lambda j: 61 + j % 9, n_ac, gamma_c=gamma)
    double, want, got = _updated(agis_mod, w, block)
    floor = np.abs(double - want).max()
    assert np.abs(got - want).max() <= max(1e-3 * synth.UAS, 10.0 * floor)
