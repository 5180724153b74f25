"""The loop of dg_volume_adjoint_u below Np = 84: at least three 16-column tiles for every wave that can
be resident, where the waves are numbered within the workgroups first, and a ragged end.  gu bit for
bit what dg_volume_adjoint writes, and against the oracle (the suite's 1e-12 pair); nothing is written
past it; the same through autograd."""

import numpy as np
import pytest
import torch

import oracle
from paper_1503_07659_amd import dgvol, synth
from parity import adjoint_cond_c, check_whole

pytestmark = pytest.mark.gpu

# an upper bound of the resident waves of the kernel on 256 CUs (8 a SIMD where registers are few)
WAVES = {1: 8192, 2: 8192, 3: 5120, 4: 3072, 5: 2048}


@pytest.mark.parametrize("F", [3, 17])
@pytest.mark.parametrize("N", sorted(WAVES))
def test_adjoint_u_three_tiles_a_wave(N, F):
    K = (3 * WAVES[N] * 16 + 21) // F + 1
    print(f"[gpu-case] adjoint_u loop N={N} K={K} F={F}", flush=True)
    Np = oracle.num_nodes(N)
    D = oracle.derivative_matrices(N)
    G = oracle.geometric_factors(synth.tet_vertices(K, 9600 + 10 * N + F))
    u = synth.fields(K, F, Np, 9700 + N + F, "uniform")
    gout = synth.fields(3 * K, F, Np, 9800 + N + F, "normal").reshape(3, K, F, Np)
    Dd, Gd, ud, gd = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (D, G, u, gout))
    full, _ = dgvol.dg_volume_adjoint(Dd, Gd, ud, gd)
    buf = torch.full((u.size + 64,), float("nan"), dtype=torch.float64, device="cuda")
    gu = buf[:u.size].view(u.shape)
    dgvol.dg_volume_adjoint_u(Dd, Gd, gd, gu)
    assert torch.isnan(buf[u.size:]).all(), "written past gu"
    assert torch.equal(gu, full)
    ua = ud.clone().requires_grad_(True)
    (ga,) = torch.autograd.grad(dgvol.volume(ua, Gd, Dd), [ua], gd)
    assert torch.equal(ga, gu)
    check_whole(gu.cpu().numpy(), oracle.volume_adjoint(D, G, u, gout)[0], adjoint_cond_c(D, G, u, gout)[0], what="gu")
