"""Block times (agis_kernel_times) where a block's time lies between events that
another block also uses: blocks that run by themselves in between must not
change the others' times."""
import pytest

import oracle
import synth.configs as C
from test_gpu_parity import agis_mod  # noqa: F401

pytestmark = pytest.mark.gpu

ALONE = {
    "source": ("agis_source_update", {"source_update"}),
    "attitude": ("agis_attitude_update", {"ac_pass", "band_solve"}),
    "calibration": ("agis_calibration_update", {"ac_pass", "calib_solve"}),
}


@pytest.mark.parametrize("robust", [False, True])
@pytest.mark.parametrize("block", list(ALONE))
def test_a_block_alone_leaves_the_other_times(agis_mod, block, robust):  # noqa: F811
    agis = agis_mod
    w = C.make("tiny_robust" if robust else "tiny", n_src=2000, years=0.25, min_transits=0)
    eta = oracle.observed_field_angles(w)
    ctx = agis.agis_create(w.consts, w.knots)
    try:
        agis.agis_load_observations(ctx, w.t, eta, w.sigma, w.src, w.fov, w.cell, w.src_true.shape[0], w.n_cells)
        agis.agis_set_sources(ctx, w.src_start)
        agis.agis_set_attitude(ctx, w.att_start)
        agis.agis_set_calibration(ctx, w.cal_start)
        agis.agis_set_frame_reference(ctx, w.src_true)
        first = agis.agis_iterate(ctx, 2)
        before = agis.agis_kernel_times(ctx)
        call, own = ALONE[block]
        st = getattr(agis, call)(ctx)
        agis.agis_iterate(ctx, 0)                    # reads the times of the last runs
        after = agis.agis_kernel_times(ctx)
    finally:
        agis.agis_destroy(ctx)
    ran = {k for k in before if k != "excess_noise" or robust}
    assert all(before[k] > 0.0 for k in ran), before
    assert all(after[k] == before[k] for k in ran - own), (before, after)
    assert all(after[k] > 0.0 for k in own) and st["ms"] > 0.0, (after, st)
    # an iteration's time holds its blocks'
    assert first[-1]["ms"] >= 0.999 * sum(before.values()) > 0.0
