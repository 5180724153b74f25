"""Timing cases of the DG volume library: what a program does with it, through its public entry points.

``listed()`` names the workloads that are followed from change to change, ``draw(rng)`` gives one more
case of the ranges they stand for.  A case is a dict of plain values:

    op      what is called (below)
    N       order of the elements, 1..7 (Np = (N+1)(N+2)(N+3)/6 nodes)
    K, F    elements and fields per element
    u       distribution of the nodal values, "uniform" (-1, 1) or "normal"
    sizes   (mixed) seed of the element counts per order, orders 1..7; K is not used then
    hi      (mixed) the counts are round(2^U(10, hi))

    fwd     dg_volume, FP64, into a kept output buffer (a solver's right-hand side)
    f32s    dg_volume_f32s, FP32 storage and split-BF16 products, the same
    adj     dg_volume_adjoint, FP64, into kept buffers (a hand-written adjoint solver)
    gradd   dg_volume_grad_d, FP64, with a kept workspace
    step    DGVolume through autograd, FP64: forward, then the gradients of the inputs named in `wrt`
            ("u", "uG" or "uGD"); outputs and gradients allocated by the call, as autograd does
    mixed   dg_volume_batched over orders 1..7, form `form` ("f64" or "f32s"), into kept buffers

Meshes are jittered unit tetrahedra (each vertex coordinate moved by U(-0.2, 0.2)); nothing is read from
files.  Inputs are drawn on the GPU from the seed alone.
"""

import types

import torch

from paper_1503_07659_amd import dgvol, setup_host, synth

ORDERS = range(1, 8)


def listed():
    return [
        # one right-hand side of a small mesh: the call and its launch are what it costs
        {"name": "fwd_small", "op": "fwd", "N": 3, "K": 4096, "F": 1, "u": "uniform"},
        # the benchmark's workload: a large mesh of order-4 elements, five fields
        {"name": "fwd_order4", "op": "fwd", "N": 4, "K": 1 << 20, "F": 5, "u": "normal"},
        # a high-order mesh, where the products and not the memory bound the forward pass
        {"name": "fwd_order6", "op": "fwd", "N": 6, "K": 1 << 17, "F": 3, "u": "normal"},
        # the benchmark's workload in the precision form
        {"name": "f32s_order4", "op": "f32s", "N": 4, "K": 1 << 20, "F": 5, "u": "normal"},
        # the benchmark's differentiation workload: both adjoint outputs of a large order-5 mesh
        {"name": "adj_order5", "op": "adj", "N": 5, "K": 1 << 19, "F": 3, "u": "uniform"},
        # a ragged mid-sized mesh with more fields than a 16-column tile holds, low order
        {"name": "adj_order3_F17", "op": "adj", "N": 3, "K": 13601, "F": 17, "u": "uniform"},
        # the cotangent of D on the differentiation workload's mesh
        {"name": "gradd_order5", "op": "gradd", "N": 5, "K": 1 << 19, "F": 3, "u": "uniform"},
        # autograd, gradient of the field only (mesh and matrices fixed), an ordinary odd-sized mesh
        {"name": "step_u_order4", "op": "step", "wrt": "u", "N": 4, "K": 27991, "F": 3, "u": "normal"},
        # autograd with every gradient (field, mesh, matrices), an odd-sized low-order mesh
        {"name": "step_uGD_order2", "op": "step", "wrt": "uGD", "N": 2, "K": 249741, "F": 3, "u": "normal"},
        # autograd, gradients of the field and the mesh, at the highest order
        {"name": "step_uG_order7", "op": "step", "wrt": "uG", "N": 7, "K": 1 << 16, "F": 3, "u": "normal"},
        # an hp mesh: orders 1 to 7 side by side in one batched call, FP64 and the precision form
        {"name": "mixed_f64", "op": "mixed", "form": "f64", "sizes": synth.MIXED_SEED, "hi": 18.0, "F": 3, "u": "normal"},
        {"name": "mixed_f32s", "op": "mixed", "form": "f32s", "sizes": synth.MIXED_SEED, "hi": 18.0, "F": 3,
         "u": "normal"},
    ]


# nodal values (K F Np) of a drawn case, at most: one pass then costs less than the largest listed one
MOST_DOF = {"fwd": 6.0e7, "f32s": 1.2e8, "adj": 3.0e7, "gradd": 3.0e7, "step": 1.2e7}


def draw(rng):
    op = rng.choice(["fwd", "fwd", "fwd", "f32s", "f32s", "adj", "adj", "gradd", "step", "step", "step", "mixed"])
    u = rng.choice(["uniform", "normal"])
    F = rng.choice([1, 2, 3, 3, 4, 5, 5, 6, 7, 9, 12, 17, 20])
    if op == "mixed":
        return {"op": op, "form": rng.choice(["f64", "f32s"]), "sizes": rng.randrange(1, 1 << 30),
                "hi": rng.choice([12.0, 14.0, 16.0]), "F": min(F, 5), "u": u}
    N = rng.choice(ORDERS)
    Np = synth.tetra_count(N)
    dof = 2.0e4 * (MOST_DOF[op] / 2.0e4) ** rng.random()
    K = max(17, min(1 << 20, int(dof / (F * Np))))
    case = {"op": op, "N": N, "K": K, "F": F, "u": u}
    if op == "step":
        case["wrt"] = rng.choice(["u", "u", "uG", "uGD"])
    return case


# ------------------------------------------------------------------ inputs

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 2654435761 % (1 << 62))
    return g


def _matrices(N):
    return torch.from_numpy(setup_host.reference_matrices(N)).to("cuda")


def _mesh(K, gen):
    """G (K, 9) of K jittered unit tetrahedra: the inverse of J = [v1-v0 | v2-v0 | v3-v0] by rows."""
    v = torch.rand((K, 4, 3), dtype=torch.float64, device="cuda", generator=gen).mul_(0.4).sub_(0.2)
    v += torch.from_numpy(synth.UNIT_TET).to("cuda")
    e = v[:, 1:] - v[:, :1]  # columns of J
    rows = torch.stack([torch.linalg.cross(e[:, 1], e[:, 2]), torch.linalg.cross(e[:, 2], e[:, 0]),
                        torch.linalg.cross(e[:, 0], e[:, 1])], dim=1)
    det = (e[:, 0] * rows[:, 0]).sum(-1)
    return (rows / det[:, None, None]).reshape(K, 9)


def _field(shape, dist, gen):
    if dist == "normal":
        return torch.randn(shape, dtype=torch.float64, device="cuda", generator=gen)
    return torch.rand(shape, dtype=torch.float64, device="cuda", generator=gen).mul_(2.0).sub_(1.0)


def _sizes(case):
    """(order, elements) of every group of the case."""
    if case["op"] != "mixed":
        return [(case["N"], case["K"])]
    return sorted(synth.mixed_order_sizes(case["sizes"], ORDERS, 10.0, case["hi"]).items())


def _inputs(case, seed):
    """Per group (D, G, u, gout or None); the precision form's arrays rounded to FP32."""
    gen = _generator(seed)
    single = case["op"] == "f32s" or case.get("form") == "f32s"
    groups = []
    for N, K in _sizes(case):
        Np, F = synth.tetra_count(N), case["F"]
        D, G, u = _matrices(N), _mesh(K, gen), _field((K, F, Np), case["u"], gen)
        gout = _field((3, K, F, Np), "normal", gen) if case["op"] in ("adj", "gradd", "step") else None
        if single:
            D, G, u = D.float(), G.float(), u.float()
        groups.append((D, G, u, gout))
    return groups


def prepare(case, seed):
    op = case["op"]
    groups = _inputs(case, seed)
    D, G, u, gout = groups[0]
    s = types.SimpleNamespace(op=op, D=D, G=G, u=u, gout=gout)
    if op in ("fwd", "f32s"):
        s.out = torch.empty((3, *u.shape), dtype=u.dtype, device="cuda")
    elif op == "adj":
        s.gu, s.gG = torch.empty_like(u), torch.empty_like(G)
    elif op == "gradd":
        s.gD = torch.empty_like(D)
        s.workspace = torch.empty(max(8, dgvol.grad_d_workspace_bytes(u.shape[0], u.shape[2], u.shape[1])),
                                  dtype=torch.uint8, device="cuda")
    elif op == "step":
        s.wrt = [x.requires_grad_(True) for name, x in (("u", u), ("G", G), ("D", D)) if name in case["wrt"]]
    else:
        s.form = dgvol.FORM_F64 if case["form"] == "f64" else dgvol.FORM_F32S
        s.groups = [g[:3] for g in groups]
        s.outs = [torch.empty((3, *g[2].shape), dtype=g[2].dtype, device="cuda") for g in groups]
    return s


def run(s):
    if s.op == "fwd":
        return dgvol.dg_volume(s.D, s.G, s.u, out=s.out)
    if s.op == "f32s":
        return dgvol.dg_volume_f32s(s.D, s.G, s.u, out=s.out)
    if s.op == "adj":
        return dgvol.dg_volume_adjoint(s.D, s.G, s.u, s.gout, gu=s.gu, gG=s.gG)
    if s.op == "gradd":
        return dgvol.dg_volume_grad_d(s.G, s.u, s.gout, gD=s.gD, work=s.workspace)
    if s.op == "mixed":
        return dgvol.dg_volume_batched(s.groups, form=s.form, outs=s.outs)
    out = dgvol.volume(s.u, s.G, s.D)
    return (out, *torch.autograd.grad(out, s.wrt, s.gout))


# ------------------------------------------------------------------ work and values

def work(case):
    op, F = case["op"], case["F"]
    nbytes = flops = 0
    for N, K in _sizes(case):
        Np = synth.tetra_count(N)
        word = 4 if op == "f32s" or case.get("form") == "f32s" else 8
        dof, Dw, Gw = K * F * Np, 3 * Np * Np, 9 * K
        product, combine = dof * 6 * Np, dof * 15  # three Np x Np products; three 3 x 3 combinations per node
        if op in ("fwd", "f32s", "mixed"):
            words, fl = 4 * dof + Gw + Dw, product + combine
        elif op == "adj":
            words, fl = 5 * dof + 2 * Gw + Dw, 2 * product + combine + 18 * dof
        elif op == "gradd":
            words, fl = 4 * dof + Gw + Dw, product + combine
        else:
            # forward; gout read, gu written; the mesh's gradient needs the products again
            words, fl = 8 * dof + Gw + Dw, 2 * (product + combine)
            if "G" in case["wrt"]:
                words, fl = words + Gw, fl + product + 18 * dof
            if "D" in case["wrt"]:
                words, fl = words + Dw, fl + product
        nbytes += word * words
        flops += fl
    return {"bytes": nbytes, "flops": flops}


def exact(case, seed):
    """The outputs of run() by torch matrix products in FP64 on the same inputs."""
    op = case["op"]
    results = []
    for D, G, u, gout in _inputs(case, seed):
        D, G, u = D.double(), G.double(), u.double()
        K, F, Np = u.shape
        Gm = G.reshape(K, 3, 3)
        cols = u.reshape(K * F, Np)
        need_out = op in ("fwd", "f32s", "mixed", "step")
        need_gG = op == "adj" or "G" in case.get("wrt", "")
        need_gu = op in ("adj", "step")
        need_gD = op == "gradd" or "D" in case.get("wrt", "")
        out = torch.zeros((3, K, F, Np), dtype=torch.float64, device="cuda") if need_out else None
        gG = torch.zeros((K, 3, 3), dtype=torch.float64, device="cuda") if need_gG else None
        gu = torch.zeros((K * F, Np), dtype=torch.float64, device="cuda") if need_gu else None
        gD = torch.zeros((3, Np, Np), dtype=torch.float64, device="cuda") if need_gD else None
        for a in range(3):
            if need_out or need_gG:
                R = torch.mm(cols, D[a].t().contiguous()).reshape(K, F, Np)
                for b in range(3):
                    if need_out:
                        out[b] += Gm[:, a, b].reshape(K, 1, 1) * R
                    if need_gG:
                        gG[:, a, b] = (gout[b] * R).sum((1, 2))
            if need_gu or need_gD:
                W = torch.zeros((K, F, Np), dtype=torch.float64, device="cuda")
                for b in range(3):
                    W += Gm[:, a, b].reshape(K, 1, 1) * gout[b]
                W = W.reshape(K * F, Np)
                if need_gu:
                    gu += torch.mm(W, D[a])
                if need_gD:
                    gD[a] = torch.mm(W.t().contiguous(), cols)
        res = [x for x in (out, None if gu is None else gu.reshape(K, F, Np), None if gG is None else gG.reshape(K, 9),
                           gD) if x is not None]
        results.append(res)
    if op == "mixed":
        return [r[0] for r in results]
    return results[0][0] if len(results[0]) == 1 else tuple(results[0])
