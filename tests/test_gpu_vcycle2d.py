"""The 2-D V-cycle's launches at the edges of their regions, against the oracle.

Sizes select every route: one workgroup for the whole hierarchy (up to 1024
nodes: one to four levels, a full 32 x 32 grid, long strips), the tail below
one or more split levels, coarsest grids that take 8 or 4 Chebyshev steps per
launch (with and without levels above), and nodes one below, at and above
multiples of the owned tiles (10 fine nodes for the down kernel, 12 for the up
kernel, 16 and 24 for the Chebyshev kernel).  Tolerances are those of the other
V-cycle parity tests: 1e-12 in FP64, 2e-5 in FP32.
"""
import numpy as np
import pytest
import torch

from oracle import precond
from oracle.fem import Mesh, Params
from paper_2006_16764_amd import inputs

pytestmark = pytest.mark.gpu

SIZES = [(1, 1), (4, 4), (24, 24), (31, 31), (31, 32), (4, 203), (120, 8), (30, 48), (38, 40), (40, 58),
         (70, 66), (94, 46), (150, 34), (63, 65), (331, 303)]


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(np.asarray(a, dtype=np.float64).reshape(-1))).cuda()


@pytest.mark.parametrize("n", SIZES, ids=lambda n: f"{n[0]}x{n[1]}")
def test_vcycle2d(n):
    from paper_2006_16764_amd import binding
    print(f"[case] 2-D V-cycle {n}", flush=True)
    L = [0.4 * k for k in n]
    mesh, p = Mesh(2, n, L), Params(dt=0.3, eps4=0.05, lam=1.6, D=2.0)
    U = inputs.random_state(2, n, 1)
    r = inputs.random_vector(mesh.n_nodes, 2)
    ref = precond.BlockPreconditioner(mesh, U, p, "gmg").apply(r)
    pb = binding.Problem(binding.make_params(2, n, L, p.dt, p.eps4, p.lam, p.D), 1)
    for prec, tol in ((binding.PF_FP64, 1e-12), (binding.PF_FP32, 2e-5)):
        pb.pf_precond_setup(dev(U), binding.PF_PC_GMG, prec)
        z = pb.new_vector().fill_(float("nan"))
        for _ in range(2):
            pb.pf_precond_apply(dev(r), z)
        got = z.cpu().numpy().reshape(-1, 2)
        err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
        print(f"[parity] {n} precision {prec}: {err:.3e}", flush=True)
        assert err < tol, (n, prec, err)
    assert pb.close() == 0
