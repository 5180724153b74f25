"""FP64 forward at order 5, where two bodies serve the sizes: up to 240 000 columns (K F; in a batch, as
many nodal values in all) the body that stores from its accumulators, beyond it the staged one.  An element's outputs must not depend on the
mesh it sits in, so the two sum in the same order: the same bits for a mesh in one call, in pieces,
and in a batch, on both sides of the edge.  Elements at both ends are also checked against the oracle
(the suite's 1e-12 pair)."""

import numpy as np
import pytest
import torch

import oracle
from paper_1503_07659_amd import dgvol, synth
from parity import check_planes, forward_cond

pytestmark = pytest.mark.gpu

N, NP = 5, 56
EDGE = dgvol.ORDER5_DIRECT_MAX_VALUES // NP


def _inputs(K, F, seed):
    D = oracle.derivative_matrices(N)
    G = oracle.geometric_factors(synth.tet_vertices(K, seed))
    u = synth.fields(K, F, NP, seed + 1, "normal")
    return (D, G, u), tuple(torch.from_numpy(x).cuda() for x in (D, G, u))


@pytest.mark.parametrize("K,F", [(1, 1), (5, 3), (37, 1), (1001, 3), (3, 100), (2000, 17)])
def test_bodies_agree_bitwise(K, F):
    print(f"[gpu-case] order-5 bodies K={K} F={F}", flush=True)
    _, (D, G, u) = _inputs(K, F, 9100 + K)
    staged = dgvol.dg_volume_variant(dgvol.FORM_F64, 0, D, G, u)
    direct = dgvol.dg_volume_variant(dgvol.FORM_F64, 1, D, G, u)
    assert torch.equal(staged, direct)


def test_default_at_the_edge():
    K = EDGE + 1
    print(f"[gpu-case] order-5 default K={EDGE} and {K} F=1", flush=True)
    (Dh, Gh, uh), (D, G, u) = _inputs(K, 1, 9200)
    whole = dgvol.dg_volume(D, G, u)
    edge = dgvol.dg_volume(D, G[:EDGE], u[:EDGE])
    assert torch.equal(edge, whole[:, :EDGE])
    half = K // 2
    for lo, hi in ((0, half), (half, K)):
        assert torch.equal(dgvol.dg_volume(D, G[lo:hi], u[lo:hi]), whole[:, lo:hi])
    for n, ref in ((K, whole), (EDGE, edge)):
        assert torch.equal(dgvol.dg_volume_batched([(D, G[:n], u[:n])])[0], ref)
    for lo, hi in ((0, 200), (K - 200, K)):
        check_planes(whole[:, lo:hi].cpu().numpy(), oracle.volume(Dh, Gh[lo:hi], uh[lo:hi]),
                     forward_cond(Dh, Gh[lo:hi], uh[lo:hi]))


@pytest.mark.parametrize("op", [dgvol.OP_FORWARD, dgvol.OP_BATCHED])
@pytest.mark.parametrize("F", [1, 16])
def test_default_variant_at_the_edge(op, F):
    assert EDGE * NP == dgvol.ORDER5_DIRECT_MAX_VALUES and EDGE % 16 == 0
    shape = lambda v, K: dgvol.launch_shape(op, dgvol.FORM_F64, NP, v, K, F)  # noqa: E731
    for K, variant in ((EDGE // F, 1), (EDGE // F + 1, 0)):
        assert shape(0, K) != shape(1, K)
        assert shape(dgvol.VARIANT_AUTO, K) == shape(variant, K)


def test_batch_counts_all_its_groups():
    """A batch past the limit runs order 5 staged whatever its own share; the same bits either way."""
    print("[gpu-case] order-5 default in batches", flush=True)
    _, small = _inputs(3000, 3, 9300)
    _, rest = _inputs(EDGE, 1, 9200)
    (alone,) = dgvol.dg_volume_batched([small])
    rest3 = (rest[0], rest[1][:EDGE // 3], rest[2].view(EDGE // 3, 3, NP))
    both = dgvol.dg_volume_batched([small, rest3])
    assert torch.equal(alone, both[0])
    assert torch.equal(both[1], dgvol.dg_volume(*rest3))
