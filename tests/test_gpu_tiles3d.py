"""The single-pass 3-D element kernels at the edges of their tiles.

A workgroup evaluates 16 x 16 element columns over a chunk of layers, forms the
linear part of the residual and the tangent at the tile's nodes from
one-dimensional rows, and a second kernel adds the partial sums of up to 8
tiles.  Meshes of one element, one layer, and one less, as many and one more
than a multiple of 16 columns per axis, with a different spacing on every axis,
take every kind of tile side.  They are small and cut into chunks of one layer.  Tolerances as in the 2-D test of the same name: 1e-12
against the oracle, 1e-6 norm-wise for an FD product against the quotient of two
residual calls.
"""
import numpy as np
import pytest
import torch

from oracle import deriv, fem
from oracle.fem import Mesh, Params
from paper_2006_16764_amd import inputs
from parity import check

pytestmark = pytest.mark.gpu

SIZES = [(1, 1, 1), (16, 1, 17), (15, 17, 1), (17, 16, 15), (1, 33, 16), (32, 3, 33)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(a, dtype=np.float64).reshape(-1))).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().reshape(-1, 2)


@pytest.mark.parametrize("n", SIZES, ids=lambda n: "x".join(map(str, n)))
def test_thermal_tiles(n):
    from paper_2006_16764_amd import binding
    print(f"[case] thermal tiles {n}", flush=True)
    L = [0.4 * n[0], 0.5 * n[1], 0.3 * n[2]]
    mesh, p = Mesh(3, n, L), Params(dt=0.3, eps4=0.05, lam=1.6, D=2.0)
    U, Up = inputs.random_state(3, n, 1), inputs.random_state(3, n, 2)
    v = inputs.random_vector(mesh.n_nodes, 3)
    pb = binding.Problem(binding.make_params(3, n, L, p.dt, p.eps4, p.lam, p.D))
    a, b, c = (pb.new_vector().fill_(float("nan")) for _ in range(3))
    gp = torch.zeros(2, dtype=torch.float64, device="cuda")
    pb.pf_residual(dev(U), dev(Up), a)
    check(host(a), fem.residual(mesh, U, Up, p), 1e-12, f"residual {n}")
    pb.pf_jvp(dev(U), dev(Up), dev(v), b)
    check(host(b), deriv.jvp(mesh, U, Up, v, p), 1e-12, f"jvp {n}")
    pb.pf_jvp(dev(U), dev(Up), dev(v), c, mode=binding.PF_JV_FD, F0=a)
    eps = 2.0 ** -26 * (1.0 + np.linalg.norm(U)) / np.linalg.norm(v)
    ref = (host(pb.pf_residual(dev(U + eps * v), dev(Up), b)) - host(a)) / eps
    r = np.linalg.norm(host(c) - ref) / np.linalg.norm(ref)
    print(f"[parity] FD product {n}: {r:.3e}", flush=True)
    assert r <= 1e-6, (n, r)
    gU, gP, ge, gl = deriv.vjp(mesh, U, Up, v, p)
    pb.pf_vjp(dev(U), dev(Up), dev(v), a, b, gp)
    check(host(a), gU, 1e-12, f"vjp gU {n}")
    check(host(b), gP, 1e-12, f"vjp gUprev {n}")
    assert np.allclose(gp.cpu().numpy(), [ge, gl], rtol=1e-10, atol=1e-12 * np.abs(gU).sum())
    pb.pf_vjp(dev(U), dev(Up), dev(v), gU=c)
    check(host(c), gU, 1e-12, f"vjp gU alone {n}")
    pb.pf_vjp(dev(U), dev(Up), dev(v), gUprev=c, gparams=gp)
    check(host(c), gP, 1e-12, f"vjp gUprev alone {n}")
    assert pb.close() == 0


def test_long_chunks():
    """Small meshes are cut into short z-chunks; this one has enough tiles for
    chunks of 19 layers.  The operators are local: on a box of 18 x 18 columns
    the values at nodes off the box's cut faces are those of the box alone."""
    from paper_2006_16764_amd import binding
    n = (250, 250, 37)
    print(f"[case] long chunks {n}", flush=True)
    h = (0.4, 0.5, 0.3)
    p = Params(dt=0.3, eps4=0.05, lam=1.6, D=2.0)
    U, Up = inputs.random_state(3, n, 1), inputs.random_state(3, n, 2)
    v = inputs.random_vector(U.shape[0], 3)
    pb = binding.Problem(binding.make_params(3, n, [h[k] * n[k] for k in range(3)], p.dt, p.eps4, p.lam, p.D))
    F, Jv, gU, gP = (pb.new_vector().fill_(float("nan")) for _ in range(4))
    gp = torch.zeros(2, dtype=torch.float64, device="cuda")
    pb.pf_residual(dev(U), dev(Up), F)
    pb.pf_jvp(dev(U), dev(Up), dev(v), Jv)
    pb.pf_vjp(dev(U), dev(Up), dev(v), gU, gP, gp)
    shape = (n[2] + 1, n[1] + 1, n[0] + 1, 2)
    for x0, y0 in ((0, 0), (5, 102), (232, 232)):
        m = (18, 18, n[2])
        box = np.s_[:, y0:y0 + 19, x0:x0 + 19]
        # off the cut faces: those inside the mesh
        inner = np.s_[:, (y0 > 0):19 - (y0 + 18 < n[1]), (x0 > 0):19 - (x0 + 18 < n[0])]
        mesh = Mesh(3, m, [h[k] * m[k] for k in range(3)])
        Ub, Upb, vb = (a.reshape(shape)[box].reshape(-1, 2) for a in (U, Up, v))
        gUb, gPb, _, _ = deriv.vjp(mesh, Ub, Upb, vb, p)
        for what, got, ref in (("residual", F, fem.residual(mesh, Ub, Upb, p)),
                               ("jvp", Jv, deriv.jvp(mesh, Ub, Upb, vb, p)), ("gU", gU, gUb), ("gUprev", gP, gPb)):
            check(host(got).reshape(shape)[box][inner].reshape(-1, 2),
                  np.asarray(ref).reshape(38, 19, 19, 2)[inner].reshape(-1, 2), 1e-12, f"{what} at {x0}, {y0}")
    assert pb.close() == 0
