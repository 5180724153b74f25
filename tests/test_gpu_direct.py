"""GPU parity of the FP64 forward body that stores from its accumulators (orders 5, 6, 7) at the
sizes where it can go wrong: one column, tiles short of and past 16 columns, an odd number of
tiles (the second half of a workgroup empty), F around the 16 and 32 columns of an iteration
(elements per column), several iterations per workgroup, and pointers aligned to 8 bytes only.

The bounds are the suite's: normwise and condition-scaled 1e-12 against the FP64 oracle (a sum of
3 Np products has at most (3 Np + 3) 2^-53 of the condition scale, 4e-14 at Np = 120)."""

import numpy as np
import pytest
import torch

import oracle
from paper_1503_07659_amd import dgvol, synth
from parity import check_planes, forward_cond

pytestmark = pytest.mark.gpu

VARIANT = {5: 1, 6: 0, 7: 0}
SIZES = [(1, 1), (5, 3), (16, 1), (17, 1), (11, 3), (1, 31), (1, 32), (2, 33), (3, 100), (3001, 7)]


def _at_offset(x, words):
    """x on the GPU, starting `words` doubles into an allocation (8-byte aligned only for odd words)."""
    buf = torch.full((x.size + words + 64,), float("nan"), dtype=torch.float64, device="cuda")
    v = buf[words:words + x.size].view(x.shape)
    v.copy_(torch.from_numpy(np.ascontiguousarray(x)))
    return buf, v


@pytest.mark.parametrize("K,F", SIZES)
@pytest.mark.parametrize("N", sorted(VARIANT))
def test_direct_body_edges(N, K, F):
    print(f"[gpu-case] direct N={N} K={K} F={F}", flush=True)
    Np = oracle.num_nodes(N)
    D = oracle.derivative_matrices(N)
    G = oracle.geometric_factors(synth.tet_vertices(K, 7000 + N))
    u = synth.fields(K, F, Np, 7100 + N, "normal")
    ref, cond = oracle.volume(D, G, u), forward_cond(D, G, u)
    results = []
    for shift in (0, 1):
        _, Dd = _at_offset(D, shift)
        _, Gd = _at_offset(G, shift)
        _, ud = _at_offset(u, shift)
        buf, out = _at_offset(np.zeros((3, K, F, Np)), shift)
        dgvol.dg_volume_variant(dgvol.FORM_F64, VARIANT[N], Dd, Gd, ud, out=out)
        torch.cuda.synchronize()
        results.append(out.cpu().numpy())
        check_planes(results[-1], ref, cond)
        b = buf.cpu().numpy()
        assert np.isnan(b[:shift]).all() and np.isnan(b[shift + 3 * K * F * Np:]).all(), "written outside out"
    assert np.array_equal(results[0], results[1])
    batched = dgvol.dg_volume_batched([(Dd, Gd, ud)], variants=[VARIANT[N]])[0].cpu().numpy()
    assert np.array_equal(results[0], batched), "batched launch differs from the single one"
