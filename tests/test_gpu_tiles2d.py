"""The single-pass 2-D element kernels at the edges of their tiles.

A tile evaluates 16 x 16 elements and owns the 15 x 15 nodes in them, so meshes
with one node less, as many, and one node more than a multiple of 15 per axis,
and meshes of one element across, exercise every kind of partial tile.  All
outputs of the three models against the oracle to 1e-12 (the tolerance of the
other parity tests; node sums run in the order of the former two-pass kernels).
The FD products are compared with the quotient (F(U + eps v) - F(U))/eps of two
residual calls at the step eps that the header documents.  Both round F to
about 1e-16 of its terms and U + eps v to 1e-16 of U, which eps = 1e-8 turns
into 1e-8 of the product times the operator's spread: 1e-6 norm-wise.
"""
import numpy as np
import pytest
import torch

from oracle import alloy, deriv, fem, freegrowth
from oracle.fem import Mesh, Params
from paper_2006_16764_amd import inputs
from parity import check

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (13, 14), (14, 15), (15, 1), (29, 16), (1, 30), (44, 31)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(a, dtype=np.float64).reshape(-1))).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().reshape(-1, 2)


def check_fd(residual, U, v, F, Jfd, what):
    """Jfd against the quotient of residual(U + eps v) and F = residual(U)."""
    eps = 2.0 ** -26 * (1.0 + np.linalg.norm(U)) / np.linalg.norm(v)
    ref = (residual(U + eps * v) - F) / eps
    r = np.linalg.norm(Jfd - ref) / np.linalg.norm(ref)
    print(f"[parity] FD product {what}: {r:.3e}", flush=True)
    assert r <= 1e-6, (what, r)


@pytest.mark.parametrize("n", SIZES, ids=lambda n: f"{n[0]}x{n[1]}")
def test_thermal_tiles(n):
    from paper_2006_16764_amd import binding
    print(f"[case] thermal tiles {n}", flush=True)
    L = [0.4 * k for k in n]
    mesh, p = Mesh(2, n, L), Params(dt=0.3, eps4=0.05, lam=1.6, D=2.0)
    U, Up = inputs.random_state(2, n, 1), inputs.random_state(2, n, 2)
    v = inputs.random_vector(mesh.n_nodes, 3)
    pb = binding.Problem(binding.make_params(2, n, L, p.dt, p.eps4, p.lam, p.D))
    a, b, c = (pb.new_vector().fill_(float("nan")) for _ in range(3))
    gp, gp2 = (torch.zeros(2, dtype=torch.float64, device="cuda") for _ in range(2))
    pb.pf_residual(dev(U), dev(Up), a)
    check(host(a), fem.residual(mesh, U, Up, p), 1e-12, f"residual {n}")
    pb.pf_jvp(dev(U), dev(Up), dev(v), b)
    check(host(b), deriv.jvp(mesh, U, Up, v, p), 1e-12, f"jvp {n}")
    pb.pf_jvp(dev(U), dev(Up), dev(v), c, mode=binding.PF_JV_FD, F0=a)
    check_fd(lambda x: host(pb.pf_residual(dev(x), dev(Up), b)), U, v, host(a), host(c), n)
    gU, gP, ge, gl = deriv.vjp(mesh, U, Up, v, p)
    pb.pf_vjp(dev(U), dev(Up), dev(v), a, b, gp)
    check(host(a), gU, 1e-12, f"vjp gU {n}")
    check(host(b), gP, 1e-12, f"vjp gUprev {n}")
    assert np.allclose(gp.cpu().numpy(), [ge, gl], rtol=1e-10, atol=1e-12 * np.abs(gU).sum())
    pb.pf_vjp(dev(U), dev(Up), dev(v), gU=c)
    check(host(c), gU, 1e-12, f"vjp gU alone {n}")
    pb.pf_vjp(dev(U), dev(Up), dev(v), gUprev=c, gparams=gp2)
    check(host(c), gP, 1e-12, f"vjp gUprev alone {n}")
    pb.pf_vjp(dev(U), dev(Up), dev(v), gparams=gp)
    assert torch.equal(gp, gp2)
    assert pb.close() == 0


@pytest.mark.parametrize("n", SIZES[1:], ids=lambda n: f"{n[0]}x{n[1]}")
def test_alloy_tiles(n):
    from paper_2006_16764_amd import binding
    print(f"[case] alloy tiles {n}", flush=True)
    L = [0.4 * k for k in n]
    p = alloy.AlloyParams(dt=0.05, eps4=0.03, lam=4.0, D=3.0, k=0.2, l_T=6.0, x_iso=0.7, v_pull=1.3,
                          theta=0.5)
    m = Mesh(2, n, L)
    U, Un, Unm1 = (inputs.random_state(2, n, s) for s in (1, 2, 3))
    v = inputs.random_vector(m.n_nodes, 4)
    pb = binding.Problem(binding.make_params(2, n, L, p.dt, p.eps4, p.lam, p.D, p.delta2, p.theta))
    ap = binding.pf_alloy_params()
    ap.k, ap.l_T, ap.x_iso, ap.v_pull = p.k, p.l_T, p.x_iso, p.v_pull
    pb.pf_set_alloy(ap)
    F, Jv, E = (pb.new_vector().fill_(float("nan")) for _ in range(3))
    pb.pf_alloy_residual(dev(U), dev(Un), dev(Unm1), 0.3, F)
    check(host(F), alloy.residual(m, U, Un, Unm1, 0.3, p), 1e-12, f"alloy residual {n}")
    pb.pf_alloy_explicit(dev(Un), 0.25, E)
    check(host(E), alloy.explicit(m, Un, 0.25, p), 1e-12, f"alloy explicit {n}")
    pb.pf_alloy_jvp(dev(U), dev(Un), dev(Unm1), 0.3, dev(v), Jv)
    check(host(Jv), alloy.jvp(m, U, Un, Unm1, 0.3, v, p), 1e-12, f"alloy jvp {n}")
    pb.pf_alloy_jvp(dev(U), dev(Un), dev(Unm1), 0.3, dev(v), Jv, mode=binding.PF_JV_FD, F0=F)
    check_fd(lambda x: host(pb.pf_alloy_residual(dev(x), dev(Un), dev(Unm1), 0.3, E)), U, v, host(F),
             host(Jv), n)
    assert pb.close() == 0


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("n", SIZES, ids=lambda n: f"{n[0]}x{n[1]}")
def test_freegrowth_tiles(n, order):
    from paper_2006_16764_amd import binding
    print(f"[case] free-growth tiles {n} order {order}", flush=True)
    L = [0.4 * k for k in n]
    p = freegrowth.FGParams(dt=1e-3, eps4=0.02, beta=50.0, Gamma=0.02, W=0.5, alpha=4.0, Lcp=1.0,
                            Tm=1.0, theta=0.6)
    m = freegrowth.MeshP(2, n, L, order)
    rng = np.random.default_rng(5)
    U, Un, Unm1 = (np.stack([rng.uniform(0, 1, m.n_nodes), rng.uniform(-1, 1, m.n_nodes)], axis=1)
                   for _ in range(3))
    v = rng.standard_normal((m.n_nodes, 2))
    pb = binding.Problem(binding.make_params(2, n, L, p.dt, p.eps4, 0.0, 1.0, p.delta2, p.theta, order))
    fp = binding.pf_freegrowth_params()
    fp.beta, fp.Gamma, fp.W, fp.alpha, fp.Lcp, fp.Tm = p.beta, p.Gamma, p.W, p.alpha, p.Lcp, p.Tm
    pb.pf_set_freegrowth(fp)
    F, Jv, E = (pb.new_vector().fill_(float("nan")) for _ in range(3))
    pb.pf_fg_residual(dev(U), dev(Un), dev(Unm1), F)
    check(host(F), freegrowth.residual(m, U, Un, Unm1, p), 1e-12, f"free-growth residual {n}")
    pb.pf_fg_explicit(dev(Un), E)
    check(host(E), freegrowth.explicit(m, Un, p), 1e-12, f"free-growth explicit {n}")
    pb.pf_fg_jvp(dev(U), dev(Un), dev(Unm1), dev(v), Jv)
    check(host(Jv), freegrowth.jvp(m, U, Un, Unm1, v, p), 1e-12, f"free-growth jvp {n}")
    pb.pf_fg_jvp(dev(U), dev(Un), dev(Unm1), dev(v), Jv, mode=binding.PF_JV_FD, F0=F)
    check_fd(lambda x: host(pb.pf_fg_residual(dev(x), dev(Un), dev(Unm1), E)), U, v, host(F),
             host(Jv), n)
    assert pb.close() == 0
