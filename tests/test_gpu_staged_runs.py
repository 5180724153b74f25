"""FP64 forward at orders 1-3 around the numbers of tile runs where they are dealt otherwise: a workgroup
a run up to 256, whole rounds of workgroups beyond, neighbouring runs from three quarters or seven
eighths of a run a wave on, several runs a wave with the first request before the operand table or after
it.  Every output against the oracle (the suite's 1e-12 pair), nothing written past them."""

import numpy as np
import pytest
import torch

import oracle
from paper_1503_07659_amd import dgvol, synth
from parity import check_planes, forward_cond

pytestmark = pytest.mark.gpu

RUNS = [1, 255, 257, 1530, 1800, 2047, 2049, 2570, 3500, 4097, 5200, 8300]


@pytest.mark.parametrize("runs", RUNS)
@pytest.mark.parametrize("N,F", [(1, 1), (1, 3), (2, 1), (2, 5), (3, 1), (3, 3)])
def test_staged_runs(N, F, runs):
    tiles = dgvol.variant_info(dgvol.FORM_F64, oracle.num_nodes(N), 0)["tiles"]
    K = (runs * 16 * tiles - 5) // F
    print(f"[gpu-case] staged runs N={N} K={K} F={F}", flush=True)
    Np = oracle.num_nodes(N)
    D = oracle.derivative_matrices(N)
    G = oracle.geometric_factors(synth.tet_vertices(K, 9900 + N))
    u = synth.fields(K, F, Np, 9910 + N, "normal")
    buf = torch.full((3 * u.size + 64,), float("nan"), dtype=torch.float64, device="cuda")
    out = buf[:3 * u.size].view(3, K, F, Np)
    dgvol.dg_volume(*(torch.from_numpy(x).cuda() for x in (D, G, u)), out=out)
    assert torch.isnan(buf[3 * u.size:]).all(), "written past out"
    check_planes(out.cpu().numpy(), oracle.volume(D, G, u), forward_cond(D, G, u))
