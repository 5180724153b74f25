"""Launch shapes of small problems, as the library reports them (host queries of a GPU's occupancy)."""

import pytest

import oracle
from paper_1503_07659_amd import dgvol

pytestmark = pytest.mark.gpu

ORDERS = range(1, 8)


@pytest.mark.parametrize("N", ORDERS)
def test_f32s_grid_has_no_workgroup_without_tiles(N):
    """The split-BF16 staged bodies give neighbouring runs of tiles to a workgroup's waves, so a
    workgroup past the last run would only build its operand table."""
    Np, F = oracle.num_nodes(N), 3
    for v in range(dgvol.variant_count(dgvol.FORM_F32S, Np)):
        info = dgvol.variant_info(dgvol.FORM_F32S, Np, v)
        per = info["tiles"] * (1 if info["body"] == 1 else info["waves"])
        for K in (1, 7, 43, 300, 1431, 5000):
            sh = dgvol.launch_shape(dgvol.OP_FORWARD, dgvol.FORM_F32S, Np, v, K, F)
            ntiles = -(-K * F // 16)
            assert sh["grid"] == min(-(-ntiles // per), sh["resident"]), (v, K, sh)


@pytest.mark.parametrize("N", range(1, 6))
def test_adjoint_min_iters_counts_idle_waves(N):
    """min_iters is that of the least-loaded wave: 0 where fewer 16-column tiles than waves are launched."""
    Np = oracle.num_nodes(N)
    for F in (1, 2, 3, 17):
        for K in (1, 16, 160, 1600, 16000):
            sh = dgvol.launch_shape(dgvol.OP_ADJOINT, dgvol.FORM_F64, Np, 0, K, F)
            if sh["units"] < sh["grid"] * (sh["block"] // 64):
                assert sh["min_iters"] == 0, (K, F, sh)
