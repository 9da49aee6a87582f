"""The two forms of the 3-D alloy and free-growth element kernels.

Up to 512 workgroups (all wavefronts at once, one per SIMD) corners and element
vector stay in registers; above, the corners are read at every Gauss plane.
Meshes on either side of that line (alloy: workgroups per element layer times
layers; free growth: of 128 elements) against the oracle to 1e-12, the FD product
against the quotient of two residual calls to 1e-6 as in the tests of the 2-D
tiles; and the time of a call below the line against one above.
"""
import numpy as np
import pytest
import torch

from oracle import alloy, freegrowth
from oracle.fem import Mesh
from paper_2006_16764_amd import inputs
from parity import check
from test_gpu_strips2d import fastest
from test_gpu_tiles2d import check_fd, dev, host

pytestmark = pytest.mark.gpu

ident = lambda n: "x".join(map(str, n))  # noqa: E731


def alloy_problem(n, L, p):
    from paper_2006_16764_amd import binding
    pb = binding.Problem(binding.make_params(3, n, L, p.dt, p.eps4, p.lam, p.D, p.delta2, p.theta))
    ap = binding.pf_alloy_params()
    ap.k, ap.l_T, ap.x_iso, ap.v_pull = p.k, p.l_T, p.x_iso, p.v_pull
    pb.pf_set_alloy(ap)
    return pb


def freegrowth_problem(n, L, p):
    from paper_2006_16764_amd import binding
    pb = binding.Problem(binding.make_params(3, n, L, p.dt, p.eps4, 0.0, 1.0, p.delta2, p.theta))
    fp = binding.pf_freegrowth_params()
    fp.beta, fp.Gamma, fp.W, fp.alpha, fp.Lcp, fp.Tm = p.beta, p.Gamma, p.W, p.alpha, p.Lcp, p.Tm
    pb.pf_set_freegrowth(fp)
    return pb


ALLOY = alloy.AlloyParams(dt=0.05, eps4=0.03, lam=4.0, D=3.0, k=0.2, l_T=6.0, x_iso=0.7, v_pull=1.3, theta=0.5)
GROWTH = freegrowth.FGParams(dt=1e-3, eps4=0.02, beta=50.0, Gamma=0.02, W=0.5, alpha=4.0, Lcp=1.0, Tm=1.0,
                             theta=0.6)


@pytest.mark.parametrize("n", [(2, 3, 512), (2, 3, 513), (13, 11, 260)], ids=ident)
def test_alloy(n):
    from paper_2006_16764_amd import binding
    print(f"[case] alloy elements {n}", flush=True)
    L = [0.4 * n[0], 0.5 * n[1], 0.3 * n[2]]
    m, p = Mesh(3, n, L), ALLOY
    U, Un, Unm1 = (inputs.random_state(3, n, s) for s in (1, 2, 3))
    v = inputs.random_vector(m.n_nodes, 4)
    pb = alloy_problem(n, L, p)
    F, Jv, E = (pb.new_vector().fill_(float("nan")) for _ in range(3))
    pb.pf_alloy_residual(dev(U), dev(Un), dev(Unm1), 0.3, F)
    check(host(F), alloy.residual(m, U, Un, Unm1, 0.3, p), 1e-12, f"alloy residual {n}")
    pb.pf_alloy_explicit(dev(Un), 0.25, E)
    check(host(E), alloy.explicit(m, Un, 0.25, p), 1e-12, f"alloy explicit {n}")
    pb.pf_alloy_jvp(dev(U), dev(Un), dev(Unm1), 0.3, dev(v), Jv)
    check(host(Jv), alloy.jvp(m, U, Un, Unm1, 0.3, v, p), 1e-12, f"alloy jvp {n}")
    pb.pf_alloy_jvp(dev(U), dev(Un), dev(Unm1), 0.3, dev(v), Jv, mode=binding.PF_JV_FD, F0=F)
    check_fd(lambda x: host(pb.pf_alloy_residual(dev(x), dev(Un), dev(Unm1), 0.3, E)), U, v, host(F), host(Jv), n)
    assert pb.close() == 0


@pytest.mark.parametrize("n", [(9, 7, 11), (64, 32, 32), (41, 40, 40)], ids=ident)
def test_freegrowth(n):
    from paper_2006_16764_amd import binding
    print(f"[case] free-growth elements {n}", flush=True)
    L = [0.4 * n[0], 0.5 * n[1], 0.3 * n[2]]
    m, p = freegrowth.MeshP(3, n, L, 1), GROWTH
    rng = np.random.default_rng(5)
    U, Un, Unm1 = (np.stack([rng.uniform(0, 1, m.n_nodes), rng.uniform(-1, 1, m.n_nodes)], axis=1)
                   for _ in range(3))
    v = rng.standard_normal((m.n_nodes, 2))
    pb = freegrowth_problem(n, L, p)
    F, Jv, E = (pb.new_vector().fill_(float("nan")) for _ in range(3))
    pb.pf_fg_residual(dev(U), dev(Un), dev(Unm1), F)
    check(host(F), freegrowth.residual(m, U, Un, Unm1, p), 1e-12, f"free-growth residual {n}")
    pb.pf_fg_explicit(dev(Un), E)
    check(host(E), freegrowth.explicit(m, Un, p), 1e-12, f"free-growth explicit {n}")
    pb.pf_fg_jvp(dev(U), dev(Un), dev(Unm1), dev(v), Jv)
    check(host(Jv), freegrowth.jvp(m, U, Un, Unm1, v, p), 1e-12, f"free-growth jvp {n}")
    pb.pf_fg_jvp(dev(U), dev(Un), dev(Unm1), dev(v), Jv, mode=binding.PF_JV_FD, F0=F)
    check_fd(lambda x: host(pb.pf_fg_residual(dev(x), dev(Un), dev(Unm1), E)), U, v, host(F), host(Jv), n)
    assert pb.close() == 0


def test_time_below_the_line():
    """33^3 elements (297 and 281 workgroups) take two thirds of the time of 44^3
    with corners in registers, 0.86 reloaded.  Line: 0.77."""
    times = {}
    for n in ((33, 33, 33), (44, 44, 44)):
        L = [0.4 * k for k in n]
        for what, make, p in (("alloy", alloy_problem, ALLOY), ("free growth", freegrowth_problem, GROWTH)):
            print(f"[case] time {what} {n}", flush=True)
            pb = make(n, L, p)
            rng = torch.Generator(device="cuda").manual_seed(1)
            U, Up, U2 = (torch.randn(pb.n_dof, dtype=torch.float64, device="cuda", generator=rng) for _ in range(3))
            F = pb.new_vector()
            times[what, n[0]] = fastest(lambda: pb.pf_alloy_residual(U, Up, U2, 0.3, F) if what == "alloy"
                                        else pb.pf_fg_residual(U, Up, U2, F))
            assert pb.close() == 0
    print("[time] " + " ".join(f"{k}: {1e3 * x:.1f} us" for k, x in times.items()), flush=True)
    for what in ("alloy", "free growth"):
        assert times[what, 33] < 0.77 * times[what, 44], (what, times)
