"""GPU parity of the adjoint with respect to u alone (dg_volume_adjoint_u), and of autograd when
only u needs a gradient, at the sizes where the tiling can go wrong: one column, tiles short of
and past 16 columns, fewer tiles than workgroups, several tiles per wave, F around 16 (elements
per column), pointers aligned to 8 bytes only.  Bound: the suite's 1e-12 pair against the FP64
oracle (a sum of 9 Np products); gu is also what dg_volume_adjoint writes, bit for bit, since the
two form W and the products of a column in the same order."""

import numpy as np
import pytest
import torch

import oracle
from paper_1503_07659_amd import dgvol, synth
from parity import adjoint_cond_c, check_whole

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (5, 3), (17, 1), (1, 15), (2, 16), (2, 17), (1, 40), (2001, 5)]


def _inputs(N, K, F):
    Np = oracle.num_nodes(N)
    D = oracle.derivative_matrices(N)
    G = oracle.geometric_factors(synth.tet_vertices(K, 8000 + N))
    u = synth.fields(K, F, Np, 8100 + N, "normal")
    gout = synth.fields(3 * K, F, Np, 8200 + N, "normal").reshape(3, K, F, Np)
    return D, G, u, gout


def _dev(x, shift=0):
    buf = torch.full((x.size + shift + 64,), float("nan"), dtype=torch.float64, device="cuda")
    v = buf[shift:shift + x.size].view(x.shape)
    v.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return v


@pytest.mark.parametrize("K,F", SIZES)
@pytest.mark.parametrize("N", range(1, 8))
def test_adjoint_u_edges(N, K, F):
    print(f"[gpu-case] adjoint_u N={N} K={K} F={F}", flush=True)
    D, G, u, gout = _inputs(N, K, F)
    ref = oracle.volume_adjoint(D, G, u, gout)[0]
    cond = adjoint_cond_c(D, G, u, gout)[0]
    Dd, Gd, ud, gd = _dev(D), _dev(G), _dev(u), _dev(gout)
    full, _ = dgvol.dg_volume_adjoint(Dd, Gd, ud, gd)
    buf = torch.full((u.size + 65,), float("nan"), dtype=torch.float64, device="cuda")
    gu = buf[1:1 + u.size].view(u.shape)
    dgvol.dg_volume_adjoint_u(_dev(D, 1), _dev(G, 1), _dev(gout, 1), gu)
    torch.cuda.synchronize()
    check_whole(gu.cpu().numpy(), ref, cond, what="gu")
    b = buf.cpu().numpy()
    assert np.isnan(b[0]) and np.isnan(b[1 + u.size:]).all(), "written outside gu"
    assert torch.equal(gu, full)


@pytest.mark.parametrize("N", [2, 6])
def test_autograd_gradient_of_u_alone(N):
    D, G, u, gout = _inputs(N, 50, 3)
    Dd, Gd, ud, gd = _dev(D), _dev(G), _dev(u), _dev(gout)
    ua = ud.clone().requires_grad_(True)
    (g1,) = torch.autograd.grad(dgvol.volume(ua, Gd, Dd), [ua], gd)
    Ga = Gd.clone().requires_grad_(True)
    g2, gG = torch.autograd.grad(dgvol.volume(ua, Ga, Dd), [ua, Ga], gd)
    assert torch.equal(g1, g2) and gG.shape == Gd.shape
    check_whole(g1.cpu().numpy(), oracle.volume_adjoint(D, G, u, gout)[0], adjoint_cond_c(D, G, u, gout)[0], what="gu")


def test_adjoint_u_validation():
    lib = dgvol.load_library()
    f, a = lib.dg_volume_adjoint_u, 0x100000
    assert f(a, a, a, a, 10, 36, 1, None) == dgvol.DG_EUNSUPPORTED
    assert f(a, a, a, a, -1, 35, 1, None) == dgvol.DG_EINVAL
    assert f(a, a, a, a, 10, 35, 0, None) == dgvol.DG_EINVAL
    assert f(None, None, None, None, 0, 35, 1, None) == dgvol.DG_OK
    for i in range(4):
        args = [a] * 4
        args[i] = None
        assert f(*args, 10, 35, 1, None) == dgvol.DG_EINVAL
        args[i] = a + 4
        assert f(*args, 10, 35, 1, None) == dgvol.DG_EINVAL
