"""GPU parity of the D cotangent around 43 and 64 parts of 128 columns, between which order 7 runs a part's
row groups on four workgroups with two column slices each.  Bound: the suite's 1e-12 pair against the
FP64 oracle's full reduction; the workspace of the size asked for is enough, and the fixed-scratch
entry point gives the same bits."""

import numpy as np
import pytest
import torch

import oracle
from paper_1503_07659_amd import dgvol, synth
from parity import check_planes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cols", [42 * 128 + 1, 64 * 128 - 5, 64 * 128, 64 * 128 + 1])
@pytest.mark.parametrize("N", [5, 6, 7])
def test_grad_d_parts(N, cols):
    print(f"[gpu-case] grad_d parts N={N} columns={cols}", flush=True)
    Np = oracle.num_nodes(N)
    G = oracle.geometric_factors(synth.tet_vertices(cols, 9500 + N))
    u = synth.fields(cols, 1, Np, 9510 + N, "normal")
    gout = synth.fields(3 * cols, 1, Np, 9520 + N, "normal").reshape(3, cols, 1, Np)
    Gd, ud, gd = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (G, u, gout))
    words = dgvol.grad_d_workspace_bytes(cols, Np, 1) // 8
    work = torch.full((words + 64,), float("nan"), dtype=torch.float64, device="cuda")
    gD = dgvol.dg_volume_grad_d(Gd, ud, gd, work=work[:words])
    assert torch.isnan(work[words:]).all(), "written past the workspace"
    cond = oracle.volume_grad_d(np.abs(G), np.abs(u), np.abs(gout))
    check_planes(gD.cpu().numpy(), oracle.volume_grad_d(G, u, gout), cond, what="gD")
    assert torch.equal(dgvol.dg_volume_grad_d_noalloc(Gd, ud, gd, torch.empty_like(gD)), gD)
