"""Reductions at the sizes that select their routes.

Vectors of at most 8192 entry pairs are summed by one workgroup per basis
vector, longer ones in two passes: meshes of 8192 and 8256 nodes sit on either
side.  Unpreconditioned Krylov solves without restart take the Gram-Schmidt
products through every accumulator set (up to 2, 4, 8, 16 vectors and beyond).
A dot product rounds each of n terms and partial sums to 2^-53: 1e-13 of
sum |x y| bounds it for these n with room.  A solve to rtol may leave its true
residual above rtol |b| by the rounding of the Krylov recurrence: twice rtol.
"""
import math

import numpy as np
import pytest
import torch

from paper_2006_16764_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (24, 17), (127, 63), (128, 63), (300, 200)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(a, dtype=np.float64).reshape(-1))).cuda()


def problem(n, m):
    from paper_2006_16764_amd import binding
    return binding.Problem(binding.make_params(2, n, [0.4 * k for k in n], 0.5, 0.05, 1.6, 2.0), m)


@pytest.mark.parametrize("n", SIZES, ids=lambda n: f"{n[0]}x{n[1]}")
def test_dot(n):
    print(f"[case] dot {n}", flush=True)
    pb = problem(n, 1)
    x, y = (inputs.random_vector(pb.n_nodes, s).reshape(-1) for s in (1, 2))
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    for a, b in ((x, y), (x, x)):
        da = dev(a)
        db = da if b is a else dev(b)
        got = []
        for _ in range(2):
            pb.pf_dot(da, db, out)
            got.append(float(out.cpu()))
        assert got[0] == got[1]
        assert abs(got[0] - math.fsum(a * b)) <= 1e-13 * float(np.sum(np.abs(a * b)))
    assert pb.close() == 0


@pytest.mark.parametrize("n", SIZES[1:], ids=lambda n: f"{n[0]}x{n[1]}")
def test_krylov_products(n):
    from paper_2006_16764_amd import binding
    print(f"[case] Krylov products {n}", flush=True)
    pb = problem(n, 60)
    U, Up = dev(inputs.random_state(2, n, 3, 0.5)), dev(inputs.random_state(2, n, 4, 0.5))
    b = dev(inputs.random_vector(pb.n_nodes, 5))
    pb.pf_precond_setup(U, binding.PF_PC_NONE)
    rtol = 1e-10
    opts = binding.default_opts(gmres_m=60, gmres_maxit=240, pc=binding.PF_PC_NONE,
                                jv_mode=binding.PF_JV_ANALYTIC)
    x, r = pb.new_vector(), pb.new_vector()
    st = pb.pf_linear_solve(U, Up, b, x, rtol=rtol, opts=opts)
    pb.pf_jvp(U, Up, x, r)
    err = float((r - b).norm() / b.norm())
    print(f"[parity] {st['gmres_its_total']} iterations, true residual {err:.3e}", flush=True)
    assert st["gmres_its_total"] > 17
    assert err <= 2 * rtol
    assert pb.close() == 0


@pytest.mark.parametrize("n", [(1, 1), (2, 1), (2, 2)], ids=lambda n: f"{n[0]}x{n[1]}")
def test_krylov_space_exhausted(n):
    """Meshes of 8 to 18 unknowns: the last vectors of the basis lose their
    digits to the projections (the norm by Pythagoras is replaced by the norm
    itself), and the solve ends within as many iterations as unknowns, plus one."""
    from paper_2006_16764_amd import binding
    print(f"[case] exhausted Krylov space {n}", flush=True)
    pb = problem(n, 30)
    U, Up = dev(inputs.random_state(2, n, 3, 0.5)), dev(inputs.random_state(2, n, 4, 0.5))
    b = dev(inputs.random_vector(pb.n_nodes, 5))
    pb.pf_precond_setup(U, binding.PF_PC_NONE)
    opts = binding.default_opts(pc=binding.PF_PC_NONE, jv_mode=binding.PF_JV_ANALYTIC)
    x, r = pb.new_vector(), pb.new_vector()
    st = pb.pf_linear_solve(U, Up, b, x, rtol=1e-13, opts=opts)
    pb.pf_jvp(U, Up, x, r)
    err = float((r - b).norm() / b.norm())
    print(f"[parity] {st['gmres_its_total']} iterations, true residual {err:.3e}", flush=True)
    assert st["gmres_its_total"] <= pb.n_dof + 1
    assert err <= 1e-12
    assert pb.close() == 0


STEPS = [((40, 40, 40), "gmg", 0), ((40, 40, 40), "gmg", 1), ((33, 35, 17), "gmg", 0), ((64, 64, 72), "gmg", 0),
         ((64, 64), "jacobi", 0), ((20, 18, 16), "jacobi", 0), ((72, 104), "gmg", 1), ((75, 101), "gmg", 0),
         ((16, 16), "gmg", 0)]


@pytest.mark.parametrize("n,pc,prec", STEPS, ids=lambda x: "x".join(map(str, x)) if isinstance(x, tuple) else str(x))
def test_step_with_the_norm_formed_by_the_preconditioner(n, pc, prec):
    """FD steps take |z| from the kernel that writes z (finest sweep, replayed
    cycle's copy, one-level solve, Jacobi) or from a sweep of its own.  Both
    Jacobian products lead to the root of F: Newton steps to 1e-10 |F0| agree to
    1e-8 of the increment, as those of the other step tests with the oracle's."""
    from paper_2006_16764_amd import binding
    print(f"[case] step {n} {pc} {prec}", flush=True)
    dim = len(n)
    pb = binding.Problem(binding.make_params(dim, n, [0.4 * k for k in n], 0.1, 0.05, 1.6, 2.0), 40)
    U0 = dev(inputs.random_state(dim, n, 1))
    got = []
    for mode in (binding.PF_JV_FD, binding.PF_JV_ANALYTIC):
        opts = binding.default_opts(tau_r=1e-10, jv_mode=mode, pc_precision=prec,
                                    pc=binding.PF_PC_GMG if pc == "gmg" else binding.PF_PC_JACOBI)
        U = U0.clone()
        st = pb.pf_newton_step(U0, U, opts)
        assert st["f_final"] <= 1e-10 * st["f0"], st
        got.append(U - U0)
    r = float((got[0] - got[1]).norm() / got[1].norm())
    print(f"[parity] FD and analytic step {n} {pc}: {r:.3e}", flush=True)
    assert r < 1e-8, r
    assert pb.close() == 0
