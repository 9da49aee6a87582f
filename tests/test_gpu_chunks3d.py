"""3-D element kernels over z-chunks of several layers, every output, theta <= 1.

The division of a mesh into chunks follows its tiles: small meshes are cut into
chunks of one layer, so that only meshes with many tiles march: 33 x 49 x 41 in
chunks of 2 layers (the last of 1), 70 x 50 x 47 of 4 (the last of 3), 250 x 250 x
37 of 19 and 18.  There the sums carried from layer to layer, the ring of three
staged planes and the perturbed planes of the difference quotient are in use.

Residual, tangent and the parameter sums against the oracle on the whole mesh
(the longest one: on boxes); F is linear in lambda and quadratic in eps4, so
differences of the oracle's residual are its derivatives.  The transposed
products are local: at nodes off the cut faces of a box, on the mesh's edge and
across a tile corner, they are those of the box alone.  The difference quotient
against the quotient of two residual calls at its step.  Tolerances as in the
other tests of these kernels: 1e-12, the quotient 1e-6 norm-wise.
"""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import deriv, fem
from oracle.fem import Mesh, Params
from paper_2006_16764_amd import inputs
from parity import check

pytestmark = pytest.mark.gpu

CASES = [((33, 49, 41), 1.0), ((70, 50, 47), 0.5), ((250, 250, 37), 0.5)]
H = (0.4, 0.5, 0.3)


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(a, dtype=np.float64).reshape(-1))).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().reshape(-1, 2)


def boxes(n, m=(6, 6)):
    """Boxes of m columns over all layers: (mesh, its nodes, its nodes off the cut faces)."""
    for x0, y0 in ((0, 0), (13, 14), (n[0] - m[0], n[1] - m[1])):
        box = np.s_[:, y0:y0 + m[1] + 1, x0:x0 + m[0] + 1]
        inner = np.s_[:, (y0 > 0):m[1] + 1 - (y0 + m[1] < n[1]), (x0 > 0):m[0] + 1 - (x0 + m[0] < n[0])]
        nb = (m[0], m[1], n[2])
        yield (x0, y0), Mesh(3, nb, [H[k] * nb[k] for k in range(3)]), box, inner


@pytest.mark.parametrize("n,theta", CASES, ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else str(x))
def test_outputs(n, theta):
    from paper_2006_16764_amd import binding
    print(f"[case] chunks {n} theta {theta}", flush=True)
    p = Params(dt=0.3, eps4=0.05, lam=1.6, D=2.0, theta=theta)
    mesh = Mesh(3, n, [H[k] * n[k] for k in range(3)])
    U, Up = inputs.random_state(3, n, 1), inputs.random_state(3, n, 2)
    v = inputs.random_vector(mesh.n_nodes, 3)
    pb = binding.Problem(binding.make_params(3, n, [H[k] * n[k] for k in range(3)], p.dt, p.eps4, p.lam, p.D,
                                             theta=theta))
    Ud, Upd, vd = dev(U), dev(Up), dev(v)
    F, Jv, Jfd, G, gU, gP, gU1, gP1 = (pb.new_vector().fill_(float("nan")) for _ in range(8))
    gp, gp1 = (torch.zeros(2, dtype=torch.float64, device="cuda") for _ in range(2))
    pb.pf_residual(Ud, Upd, F)
    pb.pf_jvp(Ud, Upd, vd, Jv)
    pb.pf_jvp(Ud, Upd, vd, Jfd, mode=binding.PF_JV_FD, F0=F)
    pb.pf_vjp(Ud, Upd, vd, gU, gP, gp)
    pb.pf_vjp(Ud, Upd, vd, gU=gU1)
    pb.pf_vjp(Ud, Upd, vd, gUprev=gP1, gparams=gp1)
    eps = 2.0 ** -26 * (1.0 + np.linalg.norm(U)) / np.linalg.norm(v)
    ref = (host(pb.pf_residual(dev(U + eps * v), Upd, G)) - host(F)) / eps
    r = np.linalg.norm(host(Jfd) - ref) / np.linalg.norm(ref)
    print(f"[parity] FD product {n}: {r:.3e}", flush=True)
    assert r <= 1e-6, (n, r)
    if mesh.n_nodes < 300000:
        F0 = fem.residual(mesh, U, Up, p)
        check(host(F), F0, 1e-12, f"residual {n}")
        check(host(Jv), deriv.jvp(mesh, U, Up, v, p), 1e-12, f"jvp {n}")
        at = lambda **kw: fem.residual(mesh, U, Up, dataclasses.replace(p, **kw))  # noqa: E731
        gl = float(np.sum(v * (at(lam=p.lam + 1.0) - F0)))
        ge = float(np.sum(v * (at(eps4=2 * p.eps4) - at(eps4=0.0)))) / (2 * p.eps4)
        for g in (gp, gp1):
            assert np.allclose(g.cpu().numpy(), [ge, gl], rtol=1e-10, atol=1e-12 * float(host(gU).__abs__().sum()))
    shape = (n[2] + 1, n[1] + 1, n[0] + 1, 2)
    for at0, bm, box, inner in boxes(n):
        Ub, Upb, vb = (a.reshape(shape)[box].reshape(-1, 2) for a in (U, Up, v))
        gUb, gPb, _, _ = deriv.vjp(bm, Ub, Upb, vb, p)
        pairs = [("gU", gU, gUb), ("gUprev", gP, gPb), ("gU alone", gU1, gUb), ("gUprev alone", gP1, gPb),
                 ("residual", F, fem.residual(bm, Ub, Upb, p)), ("jvp", Jv, deriv.jvp(bm, Ub, Upb, vb, p))]
        for what, got, ref in pairs:
            bshape = (bm.n[2] + 1, bm.n[1] + 1, bm.n[0] + 1, 2)
            check(host(got).reshape(shape)[box][inner].reshape(-1, 2),
                  np.asarray(ref).reshape(bshape)[inner].reshape(-1, 2), 1e-12, f"{what} at {at0}")
    assert pb.close() == 0


def test_time_of_the_previous_state_product():
    """It forms less than the transposed product at as many wavefronts (0.65 to
    0.75 of its time on other meshes): its z-chunks have to be those of two
    workgroups per compute unit too.  Line: 0.8."""
    from paper_2006_16764_amd import binding
    from test_gpu_strips2d import fastest
    n = (4, 4, 20000)
    print(f"[case] time {n}", flush=True)
    pb = binding.Problem(binding.make_params(3, n, [0.4 * k for k in n], 0.3, 0.05, 1.6, 2.0), 1)
    rng = torch.Generator(device="cuda").manual_seed(1)
    U, Up, v = (torch.randn(pb.n_dof, dtype=torch.float64, device="cuda", generator=rng) for _ in range(3))
    G, gp = pb.new_vector(), torch.zeros(2, dtype=torch.float64, device="cuda")
    full = fastest(lambda: pb.pf_vjp(U, Up, v, gU=G))
    prev = fastest(lambda: pb.pf_vjp(U, Up, v, gUprev=G, gparams=gp))
    print(f"[time] transposed {1e3 * full:.1f} us, previous state {1e3 * prev:.1f} us", flush=True)
    assert prev < 0.8 * full
    assert pb.close() == 0
