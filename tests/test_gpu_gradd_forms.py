"""GPU parity of the D cotangent around the sizes where the launch takes another form (a part's row
groups and directions on workgroups of their own up to 42 parts of 128 columns; from order 5, row
groups up to 255, on at most 128 longer parts; whole parts beyond), where the columns end inside a k-step of 4 or a unit
of 16 to 128, and with pointers aligned to 8 bytes only.  Bound: the suite's 1e-12 pair against
the FP64 oracle's full reduction."""

import numpy as np
import pytest
import torch

import oracle
from paper_1503_07659_amd import dgvol, synth
from parity import check_planes

pytestmark = pytest.mark.gpu

PARTS = [42 * 128, 42 * 128 + 1, 128 * 128 - 3, 128 * 128 + 2]
CASES = [(N, c, 1) for N in (4, 5, 6, 7) for c in PARTS]
CASES += [(N, c, 1) for N in (5, 6, 7) for c in (255 * 128, 255 * 128 + 1)]
CASES += [(N, k, F) for N in range(1, 8) for k, F in ((1, 1), (3, 1), (2, 2), (33, 1), (7, 19), (43, 3))]


def _dev(x, shift):
    buf = torch.full((x.size + shift + 64,), float("nan"), dtype=torch.float64, device="cuda")
    v = buf[shift:shift + x.size].view(x.shape)
    v.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return v


@pytest.mark.parametrize("N,K,F", CASES)
def test_grad_d_forms(N, K, F):
    print(f"[gpu-case] grad_d forms N={N} K={K} F={F}", flush=True)
    Np = oracle.num_nodes(N)
    G = oracle.geometric_factors(synth.tet_vertices(K, 9000 + N))
    u = synth.fields(K, F, Np, 9100 + N, "normal")
    gout = synth.fields(3 * K, F, Np, 9200 + N, "normal").reshape(3, K, F, Np)
    gD = torch.full((3, Np, Np), float("nan"), dtype=torch.float64, device="cuda")
    dgvol.dg_volume_grad_d(_dev(G, 1), _dev(u, 1), _dev(gout, 1), gD=gD)
    torch.cuda.synchronize()
    cond = oracle.volume_grad_d(np.abs(G), np.abs(u), np.abs(gout))
    check_planes(gD.cpu().numpy(), oracle.volume_grad_d(G, u, gout), cond, what="gD")
