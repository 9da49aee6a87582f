"""2-D meshes a few elements wide or high.

Element tiles and the regions of the coarsest Chebyshev solve are 16 x 16 and
32 x 32 lanes; where a mesh is narrower than they are, they are as wide (high) as
the mesh instead.  Lengths that end with a tile, begin another one, and leave a
remainder, both orientations, against the oracle with the tolerances of the tests of the square tiles; and the time of
a strip against that of a square of as many elements.
"""
import numpy as np
import pytest
import torch

import test_gpu_tiles2d as tiles
import test_gpu_vcycle2d as vcycle

pytestmark = pytest.mark.gpu

# (elements across, elements along)
STRIPS = [(1, 254), (1, 255), (2, 126), (2, 300), (3, 200), (7, 64), (16, 61), (24, 90)]
BOTH = [n for s in STRIPS for n in (s, s[::-1])]
ident = lambda n: f"{n[0]}x{n[1]}"  # noqa: E731


@pytest.mark.parametrize("n", BOTH, ids=ident)
def test_thermal(n):
    tiles.test_thermal_tiles(n)


@pytest.mark.parametrize("n", BOTH[:8], ids=ident)
def test_alloy(n):
    tiles.test_alloy_tiles(n)


@pytest.mark.parametrize("order", [1, 2])
@pytest.mark.parametrize("n", BOTH, ids=ident)
def test_freegrowth(n, order):
    tiles.test_freegrowth_tiles(n, order)


# more than 1024 nodes (no tail); from 100000 nodes on 4 steps per launch instead of 8
CYCLES = [(1, 600), (3, 2500), (17, 99), (55, 61), (6, 4000), (1, 60001), (31, 3201), (100, 1003)]


@pytest.mark.parametrize("n", [n for s in CYCLES for n in (s, s[::-1])], ids=ident)
def test_vcycle(n):
    vcycle.test_vcycle2d(n)


def fastest(f):
    f()
    best = float("inf")
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(10):
            f()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 10)
    return best


def test_time_of_a_strip():
    """One element across: twice the nodes of a square, no element evaluated twice;
    a square tile per 15 rows takes 6 to 12 times as long.  Line: 4."""
    from paper_2006_16764_amd import binding
    times = {}
    for n in ((1000, 1000), (1, 1000000), (1000000, 1)):
        print(f"[case] time {n}", flush=True)
        pb = binding.Problem(binding.make_params(2, n, [0.4 * k for k in n], 0.5, 0.05, 1.6, 2.0), 1)
        rng = torch.Generator(device="cuda").manual_seed(1)
        U, Up, v = (torch.randn(pb.n_dof, dtype=torch.float64, device="cuda", generator=rng) for _ in range(3))
        F, z = pb.new_vector(), pb.new_vector()
        t = {"residual": fastest(lambda: pb.pf_residual(U, Up, F)),
             "jvp": fastest(lambda: pb.pf_jvp(U, Up, v, F)),
             "gU": fastest(lambda: pb.pf_vjp(U, Up, v, gU=F))}
        times[n] = t
        print(f"[time] {n} " + " ".join(f"{k} {x * 1e3:.1f} us" for k, x in t.items()), flush=True)
        assert pb.close() == 0
    for n in ((1, 1000000), (1000000, 1)):
        for k, x in times[n].items():
            assert x < 4 * times[(1000, 1000)][k], (n, k, times)
