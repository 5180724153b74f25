"""The adjoint's runs of whole elements below Np = 84 (gu and gG) at the sizes where the share of
elements a wave takes changes: fewer waves with fuller runs, an element more for the first of them,
none left over, and the limit of four tiles past which the odd elements are spread.  Every output
against the oracle at the suite's 1e-12 pair; an element's bits do not depend on the mesh around it."""

import numpy as np
import pytest
import torch

import oracle
from paper_1503_07659_amd import dgvol, synth
from parity import adjoint_cond_c, check_whole

pytestmark = pytest.mark.gpu


# (5, 4436, 5), (3, 55461, 1), (4, 1400, 17): fuller runs; (5, 6178, 5): an element more for 385 of 1931
# waves; (5, 2048, 5): equal runs; (3, 4100, 48), (3, 6200, 33): either side of 64 columns a run
CASES = [(5, 4436, 5), (5, 6178, 5), (5, 2048, 5), (3, 55461, 1), (4, 1400, 17), (2, 33000, 2), (1, 70000, 1),
         (3, 4100, 48), (3, 6200, 33)]


@pytest.mark.parametrize("N,K,F", CASES)
def test_adjoint_runs(N, K, F):
    print(f"[gpu-case] adjoint runs N={N} K={K} F={F}", flush=True)
    Np = oracle.num_nodes(N)
    D = oracle.derivative_matrices(N)
    G = oracle.geometric_factors(synth.tet_vertices(K, 9400 + N))
    u = synth.fields(K, F, Np, 9410 + N, "uniform")
    gout = synth.fields(3 * K, F, Np, 9420 + N, "normal").reshape(3, K, F, Np)
    Dd, Gd, ud, gd = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (D, G, u, gout))
    gu, gG = dgvol.dg_volume_adjoint(Dd, Gd, ud, gd)
    ref_gu, ref_gG = oracle.volume_adjoint(D, G, u, gout)
    c_gu, c_gG = adjoint_cond_c(D, G, u, gout)
    check_whole(gu.cpu().numpy(), ref_gu, c_gu, what="gu")
    check_whole(gG.cpu().numpy(), ref_gG, c_gG, what="gG")
    half = K // 2 + 1
    part = dgvol.dg_volume_adjoint(Dd, Gd[:half].contiguous(), ud[:half].contiguous(), gd[:, :half].contiguous())
    assert torch.equal(part[0], gu[:half]) and torch.equal(part[1], gG[:half])


@pytest.mark.parametrize("N", range(1, 6))
def test_adjoint_grid_is_whole_rounds_over_the_cus(N):
    """A small call's workgroups are no more than a round over the 256 CUs needs for its tiles."""
    Np = oracle.num_nodes(N)
    for F in (1, 3, 17):
        for K in (1, 40, 300, 3000, 30000):
            sh = dgvol.launch_shape(dgvol.OP_ADJOINT, dgvol.FORM_F64, Np, 0, K, F)
            waves = sh["block"] // 64
            assert sh["grid"] <= min(sh["units"], 256 * -(-sh["units"] // (256 * waves)), sh["resident"]), (K, F, sh)
