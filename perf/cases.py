"""Timed workloads of the library, called through its public Python entry points.

A case names a model (thermal, alloy, freegrowth), an operation and a mesh of
nx x ny (x nz) elements.  Operations:

  residual   F(U), the call of an outer time integrator or a matrix-free solver
  jvp        analytic Jacobian-vector product
  vjp        vector-Jacobian product with all its outputs
  vcycle     FP64 multigrid set-up at a state and one apply
  step       one implicit time step (Newton-Krylov, FD products by default)
  adjoint    one step of the discrete adjoint
  gradient   time steps and their backward pass through torch.autograd

Meshes, parameters and initial states follow paper_2006_16764_amd/inputs.py and
bench.py: thermal seeds at spacing 0.8, the directional-solidification front of
the alloy workloads, the quarter seed of the free-growth workloads on order-1
and order-2 elements.  States between the steps of a run are stood in for by
the same profiles a little later in time plus nodal noise of 1e-3.

The finite-difference product is not a case of its own: its last eight digits
are rounding noise of a difference of residuals.  It runs inside `step`.  The
FP32 V-cycle likewise runs inside `step` and `adjoint`, whose solutions do not
depend on its rounding.
"""
import math
import random

import numpy as np
import torch

from paper_2006_16764_amd import binding, evolve, inputs

H_THERMAL = 0.8
DEVICE = "cuda" if torch.cuda.is_available() else "cpu"
F64 = torch.float64


def _case(model, op, n, **options):
    """Plain values of one case; options: theta, order, pc, bits (of the V-cycle), steps."""
    c = {"model": model, "op": op, "dim": len(n), "nx": n[0], "ny": n[1], "nz": n[2] if len(n) == 3 else 1,
         "theta": 1.0 if model == "thermal" else 0.5, "order": 1, "pc": "gmg", "bits": 64, "steps": 1}
    c.update(options)
    return c


def listed():
    named = {
        # the smallest run: a 2-D benchmark step with the plain Jacobi preconditioner, all latency
        "step2d_64_jacobi": _case("thermal", "step", (64, 64), pc="jacobi"),
        # the paper's free-growth benchmark mesh: one time step of a long sequential run
        "freegrowth_step2d_150": _case("freegrowth", "step", (150, 150)),
        # a residual evaluation on a ragged 2-D mesh under Crank-Nicolson weights
        "residual2d_387x251": _case("thermal", "residual", (387, 251), theta=0.5),
        # the linearised operator at the 2-D benchmark size
        "jvp2d_1024": _case("thermal", "jvp", (1024, 1024)),
        # parameter fitting: two steps forward and their adjoint through autograd
        "gradient2d_512": _case("thermal", "gradient", (512, 512), steps=2),
        # directional solidification in 2-D: one Crank-Nicolson step
        "alloy_step2d_1024x256": _case("alloy", "step", (1024, 256)),
        # biquadratic elements at a throughput size (33.6 M unknowns)
        "freegrowth_jvp2d_2048_q2": _case("freegrowth", "jvp", (2048, 2048), order=2),
        # the flagship residual (33.9 M unknowns)
        "residual3d_256": _case("thermal", "residual", (256, 256, 256)),
        # reverse mode on a ragged 3-D mesh
        "vjp3d_129x97x113": _case("thermal", "vjp", (129, 97, 113)),
        # the alloy tangent in 3-D (16.6 M unknowns)
        "alloy_jvp3d_512x128x128": _case("alloy", "jvp", (512, 128, 128)),
        # an ordinary 3-D step with everything in FP64
        "step3d_128": _case("thermal", "step", (128, 128, 128)),
        # the largest: the flagship mixed-precision step
        "step3d_256_fp32": _case("thermal", "step", (256, 256, 256), bits=32),
    }
    return [dict(c, name=name) for name, c in named.items()]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _even(n, m):
    """n rounded to a multiple of m: solver meshes are chosen so that they coarsen."""
    return max(m, int(round(n / m)) * m)


def draw(rng: random.Random):
    kind = rng.choice(["thermal2d", "thermal3d", "thermal_step2d", "thermal_step3d", "vcycle", "adjoint",
                       "gradient", "alloy2d", "alloy3d", "alloy_step", "freegrowth", "freegrowth_step"])
    theta, bits = rng.choice([1.0, 0.5]), rng.choice([64, 32])
    if kind == "thermal2d":
        return _case("thermal", rng.choice(["residual", "jvp", "vjp"]), (_size(rng, 24, 1400), _size(rng, 24, 1400)),
                     theta=theta)
    if kind == "thermal3d":
        return _case("thermal", rng.choice(["residual", "jvp", "vjp"]),
                     (_size(rng, 12, 256), _size(rng, 12, 256), _size(rng, 12, 256)), theta=theta)
    if kind == "thermal_step2d":
        m = rng.choice([1, 4, 16])
        return _case("thermal", "step", (_even(_size(rng, 32, 1024), m), _even(_size(rng, 32, 1024), m)), theta=theta,
                     bits=bits, pc=rng.choice(["gmg", "gmg", "jacobi"]))
    if kind == "thermal_step3d":
        m = rng.choice([1, 4, 16])
        return _case("thermal", "step", tuple(_even(_size(rng, 16, 160), m) for _ in range(3)), theta=theta, bits=bits)
    if kind == "vcycle":
        m = rng.choice([2, 8, 32])
        n = (tuple(_even(_size(rng, 64, 1024), m) for _ in range(2)) if rng.random() < 0.4 else
             tuple(_even(_size(rng, 32, 256), m) for _ in range(3)))
        return _case("thermal", "vcycle", n)
    if kind == "adjoint":
        n = (tuple(_even(_size(rng, 64, 1024), 8) for _ in range(2)) if rng.random() < 0.5 else
             tuple(_even(_size(rng, 16, 160), 8) for _ in range(3)))
        return _case("thermal", "adjoint", n, bits=bits)
    if kind == "gradient":
        n = _even(_size(rng, 48, 512), 8)
        return _case("thermal", "gradient", (n, n), steps=rng.randint(1, 3), bits=bits)
    if kind == "alloy2d":
        return _case("alloy", rng.choice(["residual", "jvp"]), (_size(rng, 48, 2048), _size(rng, 16, 1024)), theta=theta)
    if kind == "alloy3d":
        return _case("alloy", rng.choice(["residual", "jvp"]),
                     (_size(rng, 32, 512), _size(rng, 16, 160), _size(rng, 16, 160)), theta=theta)
    if kind == "alloy_step":
        n = ((_even(_size(rng, 48, 1024), 8), _even(_size(rng, 16, 256), 8)) if rng.random() < 0.6 else
             (_even(_size(rng, 32, 128), 8), _even(_size(rng, 16, 64), 8), _even(_size(rng, 16, 64), 8)))
        return _case("alloy", "step", n, bits=bits)
    order = rng.choice([1, 2])
    if kind == "freegrowth":
        n = ((_size(rng, 32, 2048 // order), _size(rng, 32, 2048 // order)) if order == 2 or rng.random() < 0.6 else
             (_size(rng, 16, 160), _size(rng, 16, 160), _size(rng, 16, 160)))
        return _case("freegrowth", rng.choice(["residual", "jvp"]), n, order=order, theta=theta)
    return _case("freegrowth", "step", (_size(rng, 32, 400 // order), _size(rng, 32, 400 // order)), order=order, bits=bits)


# ------------------------------------------------------------------ inputs
def _mesh(case):
    return tuple(case[k] for k in ("nx", "ny", "nz")[: case["dim"]])


def _workload(case):
    """The recipe of inputs.py behind a case (thermal: its plain parameters)."""
    n, dim = _mesh(case), case["dim"]
    if case["model"] == "alloy":
        return inputs.AlloyWorkload("case", dim, n, 0.002, case["theta"], 1, 0)
    if case["model"] == "freegrowth":
        return inputs.FreeGrowthWorkload("case", dim, n, case["order"], 1e-4, 1, case["theta"])
    return inputs.Workload("case", dim, n[0], 0.5 * H_THERMAL * n[0], 0.5 if dim == 2 else 0.2, 0.05, 1.6, 2.0,
                           5.0 if dim == 2 else 6.0, 4 if dim == 2 else 8, -0.4, 0, 1)


def _axes(case, w):
    """Node coordinates per axis from the box's corner, shaped to broadcast over (z,) y, x."""
    dim, out = case["dim"], []
    h = H_THERMAL if case["model"] == "thermal" else w.h
    for k, nk in enumerate(_mesh(case)):
        shape = [1] * dim
        shape[dim - 1 - k] = nk * case["order"] + 1
        out.append((torch.arange(shape[dim - 1 - k], dtype=F64, device=DEVICE) * (h / case["order"])).reshape(shape))
    return out


def _states(case, seed):
    """(Uprev2, Uprev, U): three consecutive states, each flat and interleaved, and the vector v."""
    w, dim = _workload(case), case["dim"]
    gen = torch.Generator(device=DEVICE).manual_seed(seed)
    rng = random.Random(seed)
    x = _axes(case, w)
    shape = tuple(a.numel() for a in reversed(x))
    width = [float(a.max()) for a in x]
    noise = 0.0 if case["op"] in ("step", "gradient") else 1e-3
    if case["model"] == "thermal":
        R = min(w.radius, 0.25 * min(width))
        centres = [[rng.uniform(min(2 * R, 0.5 * s), max(s - 2 * R, 0.5 * s)) for s in width] for _ in range(w.n_seeds)]

        def field(k):
            phi = torch.full(shape, -1.0, dtype=F64, device=DEVICE)
            for c in centres:
                r = sum((x[a] - c[a]) ** 2 for a in range(dim)).sqrt()
                phi = torch.maximum(phi, -torch.tanh((r - R - 0.05 * k) / math.sqrt(2.0)))
            return phi
        u0, latent = w.u0, 0.5
    elif case["model"] == "alloy":
        d = w.amp * (2.0 * torch.rand(shape[:-1] + (1,), dtype=F64, device=DEVICE, generator=gen) - 1.0)

        def field(k):
            return -torch.tanh((x[0] - w.x_front - d - 0.02 * k) / math.sqrt(2.0)).expand(shape)
        u0, latent = w.u0, 0.3
    else:
        r0 = w.r0 * rng.uniform(0.9, 1.1)
        rho = sum(a ** 2 for a in x).sqrt()
        ang = torch.atan2(x[1] + 0.0 * rho, x[0] + 0.0 * rho)

        def field(k):
            return 0.5 * (1.0 - torch.tanh((rho - r0 * (1.0 + w.eps4 * torch.cos(4.0 * ang)) - 1e-3 * k) / (2.0 * w.W)))
        u0, latent = w.Tm - w.undercooling, 1.0
    phi = [field(0)] * 3 if case["op"] in ("step", "gradient") else [field(k) for k in range(3)]
    out = []
    for k in range(3):
        U = torch.stack([phi[k], u0 + latent * (phi[k] - phi[0])], dim=-1).reshape(-1)
        if noise:
            U = U + noise * torch.randn(U.shape, dtype=F64, device=DEVICE, generator=gen)
        out.append(U)
    v = torch.randn(out[0].shape, dtype=F64, device=DEVICE, generator=gen)
    return out[0], out[1], out[2], v


def _problem(case, w):
    m = 30 if case["op"] in ("step", "adjoint", "gradient") else 1
    if case["model"] == "alloy":
        return binding.alloy_problem_for(w, gmres_m_max=m)
    if case["model"] == "freegrowth":
        return binding.freegrowth_problem_for(w, gmres_m_max=m)
    n = _mesh(case)
    return binding.Problem(binding.make_params(case["dim"], n, [0.5 * H_THERMAL * k for k in n], w.dt, w.eps4, w.lam, w.D,
                                               w.delta2, case["theta"]), m)


def _target(case, U):
    """Target phase of a misfit: the state's own field, slightly blurred towards the melt."""
    return (0.95 * U.view(-1, 2)[:, 0] - 0.05).contiguous()


def _cotangent(case, U):
    """dL/dU of a phase misfit, nodal mass taken as constant."""
    g = torch.zeros_like(U)
    g.view(-1, 2)[:, 0] = (U.view(-1, 2)[:, 0] - _target(case, U)) * H_THERMAL ** case["dim"]
    return g


def _options(case):
    o = {"pc": binding.PF_PC_GMG if case["pc"] == "gmg" else binding.PF_PC_JACOBI,
         "pc_precision": binding.PF_FP64 if case["bits"] == 64 else binding.PF_FP32}
    if case["op"] in ("adjoint", "gradient"):
        # gradients are compared with difference quotients: tight solves on the exact tangent
        o.update(tau_r=1e-12, jv_mode=binding.PF_JV_ANALYTIC)
    return o


def prepare(case, seed):
    w = _workload(case)
    Upp, Up, U, v = _states(case, seed)
    pb = _problem(case, w)
    s = {"case": case, "pb": pb, "Upp": Upp, "Up": Up, "U": U, "v": v, "t": w.dt, "opts": binding.default_opts(**_options(case)),
         "out": [pb.new_vector(U.device) for _ in range(2)], "gp": torch.zeros(2, dtype=F64, device=U.device)}
    if case["op"] == "adjoint":
        s["mu"] = _cotangent(case, U)
    if case["op"] == "gradient":
        s["target"] = _target(case, U)
        s["leaves"] = [torch.tensor(x, dtype=F64, device=U.device, requires_grad=True) for x in (w.eps4, w.lam)]
        s["leaves"].append(Up.clone().requires_grad_(True))
    return s


def run(state):
    case, pb, Upp, Up, U, v = (state[k] for k in ("case", "pb", "Upp", "Up", "U", "v"))
    model, op, out, opts = case["model"], case["op"], state["out"], state["opts"]
    if op == "residual":
        if model == "alloy":
            return pb.pf_alloy_residual(U, Up, Upp, state["t"], out[0])
        if model == "freegrowth":
            return pb.pf_fg_residual(U, Up, Upp, out[0])
        return pb.pf_residual(U, Up, out[0])
    if op == "jvp":
        if model == "alloy":
            return pb.pf_alloy_jvp(U, Up, Upp, state["t"], v, out[0])
        if model == "freegrowth":
            return pb.pf_fg_jvp(U, Up, Upp, v, out[0])
        return pb.pf_jvp(U, Up, v, out[0])
    if op == "vjp":
        pb.pf_vjp(U, Up, v, out[0], out[1], state["gp"])
        return out[0], out[1], state["gp"]
    if op == "vcycle":
        pb.pf_precond_setup(U)
        return pb.pf_precond_apply(v, out[0])
    if op == "step":
        new = out[0].copy_(Up)
        if model == "alloy":
            pb.pf_alloy_step(Upp, Up, 0.0, new, opts)
        elif model == "freegrowth":
            pb.pf_fg_step(Upp, Up, new, opts)
        elif case["theta"] == 1.0:
            pb.pf_newton_step(Up, new, opts)
        else:
            pb.pf_newton_step_theta(Upp, Up, new, opts)
        return new
    if op == "adjoint":
        gp = state["gp"].zero_()
        pb.pf_adjoint_step(U, Up, state["mu"], out[0], out[1], gp, opts)
        return out[0], out[1], gp
    eps4, lam, U0 = state["leaves"]
    UK = evolve.evolve(eps4, lam, U0, pb, case["steps"], opts)
    loss = evolve.misfit(UK, state["target"], pb)
    return (UK.detach(), loss.detach()) + torch.autograd.grad(loss, (eps4, lam, U0))


# ------------------------------------------------------------------ work
# FP64 operations per element of one residual, tangent and adjoint evaluation (add, multiply = 1) by
# sum factorisation over the 3-point rule
_FLOPS = {("thermal", 2, 1): (751, 1200, 1500), ("thermal", 3, 1): (2913, 4795, 5862),
          ("alloy", 2, 1): (1150, 2300, 0), ("alloy", 3, 1): (5200, 10600, 0),
          ("freegrowth", 2, 1): (1050, 2100, 0), ("freegrowth", 3, 1): (4700, 9600, 0),
          ("freegrowth", 2, 2): (2700, 4200, 0)}


def work(case):
    n, dim, op = _mesh(case), case["dim"], case["op"]
    nodes = math.prod(case["order"] * k + 1 for k in n)
    elems = math.prod(n)
    res, jvp, vjp = (f * elems for f in _FLOPS[case["model"], dim, case["order"]])
    stencil = 4 * 3 ** dim * nodes  # one application of the preconditioner's operator, both blocks
    cycle = (6 if case["pc"] == "gmg" else 0) * stencil
    old = 1 if case["model"] != "thermal" or case["theta"] != 1.0 else 0  # U^(n-1) is read too
    if op == "residual":
        vectors, flops = 3 + (old if case["model"] != "thermal" else 0), res
    elif op == "jvp":
        vectors, flops = 4 + (old if case["model"] != "thermal" else 0), jvp
    elif op == "vjp":
        vectors, flops = 5, vjp
    elif op == "vcycle":
        vectors, flops = 3, cycle
    elif op == "step":
        # states in and out; an inexact Newton solve to 1e-10 takes about four iterations and sixteen products
        vectors, flops = 3 + old, 5 * res + 16 * (res + cycle)
    elif op == "adjoint":
        vectors, flops = 5, 14 * (vjp + cycle) + vjp
    else:
        vectors, flops = 4, case["steps"] * (5 * res + 16 * (jvp + cycle) + 16 * (vjp + cycle))
    return {"bytes": 16 * nodes * vectors, "flops": flops}


# ------------------------------------------------------------------ values in 64 bits, by plain torch
class _Rule:
    """Lagrange elements on the box mesh: values and gradients at the 3^dim Gauss points, and their transposes."""

    def __init__(self, n, h, order):
        self.n, self.h, self.order, self.dim = n, h, order, len(n)
        g = math.sqrt(0.6)
        xi, wt = (-g, 0.0, g), (5 / 9, 8 / 9, 5 / 9)
        if order == 1:
            one = [[((1 - t) / 2, (1 + t) / 2) for t in xi], [(-0.5, 0.5) for _ in xi]]
        else:
            one = [[(t * (t - 1) / 2, 1 - t * t, t * (t + 1) / 2) for t in xi], [(t - 0.5, -2 * t, t + 0.5) for t in xi]]
        grids = np.ndindex(*([3] * self.dim))
        self.points = []
        for q in grids:
            w = math.prod(wt[i] * h[k] / 2 for k, i in enumerate(q))
            corners = []
            for a in np.ndindex(*([order + 1] * self.dim)):
                val = math.prod(one[0][q[k]][a[k]] for k in range(self.dim))
                grad = [math.prod(one[1 if j == k else 0][q[j]][a[j]] for j in range(self.dim)) * 2 / h[k]
                        for k in range(self.dim)]
                where = tuple(slice(a[k], a[k] + order * (n[k] - 1) + 1, order) for k in reversed(range(self.dim)))
                corners.append((where, val, grad))
            self.points.append((w, [(xi[i] + 1) / 2 for i in q], corners))

    def nodal(self, x):
        return x.reshape(tuple(self.order * k + 1 for k in reversed(self.n)) + (-1,))

    def at(self, x, point, gradient=True):
        val, grad = 0.0, [0.0] * (self.dim if gradient else 0)
        for where, v, g in point[2]:
            c = x[where]
            val = val + v * c
            grad = [s + g[k] * c for k, s in enumerate(grad)]
        return val, grad

    def add(self, out, field, point, value, flux=()):
        for where, v, g in point[2]:
            out[where + (field,)] += point[0] * (v * value + sum(g[k] * f for k, f in enumerate(flux)))

    def x0(self, point):
        """First coordinate of the point, from the box's corner."""
        return ((torch.arange(self.n[0], dtype=F64, device=DEVICE) + point[1][0]) * self.h[0])


class _Equations:
    """Weak form of one model: s1 + f1 . grad and s2 + f2 . grad against the test functions, at a point."""

    def __init__(self, case, w):
        self.case, self.w, self.dim = case, w, case["dim"]
        h = H_THERMAL if case["model"] == "thermal" else w.h
        self.rule = _Rule(_mesh(case), [h] * self.dim, case["order"])
        self.dt, self.theta = w.dt, case["theta"]
        if case["model"] == "alloy":
            self.D, self.l_T, self.v_pull = w.scales()

    def point(self, eps4, lam, theta, t, x, hist, phi, u, phin, un, *grads):
        """theta: weight of the spatial terms (0 time terms when theta < 0: the operator of E)."""
        w, d = self.w, self.dim
        g, gu = grads[:d], grads[d:]
        rate = 0.0 if theta < 0 else 1.0 / self.dt
        theta = abs(theta)
        q = sum(k * k for k in g)
        S = sum(k ** 4 for k in g)
        Q = q + w.delta2
        a = 1 - 3 * eps4 + 4 * eps4 * S / Q ** 2
        # J = a^2 g + a q da/dg with da/dg_k = 16 eps4 g_k (g_k^2 - S/Q)/Q^2
        J = [a * a * k + a * q * 16 * eps4 * k * (k * k - S / Q) / Q ** 2 for k in g]
        dphi, du = phi - phin, u - un
        if self.case["model"] == "thermal":
            R = phi - phi ** 3 - lam * (1 - phi ** 2) ** 2 * u
            return ((a * a * dphi * rate - theta * R, *[theta * j for j in J]),
                    (du * rate - theta * 0.5 * dphi * rate, *[theta * w.D * k for k in gu]))
        if self.case["model"] == "alloy":
            cu = 1 + (1 - w.k) * u
            G4 = (x - w.x_front - self.v_pull * t) / self.l_T
            R = phi - phi ** 3 - lam * (1 - phi ** 2) ** 2 * (u + G4)
            ph = theta * dphi * rate + hist
            at = cu * ph / (2 * math.sqrt(2) * Q.sqrt())
            return ((cu * a * a * dphi * rate - theta * R, *[theta * j for j in J]),
                    ((1 + w.k) / 2 * du * rate - ph * cu / 2,
                     *[theta * self.D * (1 - phi) / 2 * gu[k] + at * g[k] for k in range(d)]))
        bG = w.beta * w.Gamma
        G2 = bG * phi * (1 - phi) * (1 - 2 * phi) / w.W ** 2 - 5 * w.beta * (w.Tm - u) * phi ** 2 * (1 - phi) ** 2 / w.W
        ph = theta * dphi * rate + hist
        return ((a * a * dphi * rate + theta * G2, *[theta * bG * j for j in J]),
                (du * rate - w.Lcp * ph, *[theta * w.alpha * k for k in gu]))

    def _primal(self, U, Up, hist, point, explicit):
        r = self.rule
        val, grad = r.at(U, point)
        old = val if explicit else r.at(Up, point, False)[0]
        h = 0.0 if hist is None or explicit else r.at(hist, point, False)[0][..., 0]
        args = [val[..., 0], val[..., 1], old[..., 0], old[..., 1]]
        args += [k[..., 0] for k in grad] + [k[..., 1] for k in grad]
        return h, args

    def history(self, Up, Upp):
        if self.case["model"] == "thermal":
            return None
        n = self.rule.nodal
        return (1 - self.theta) / self.dt * (n(Up)[..., :1] - n(Upp)[..., :1])

    def residual(self, U, Up, hist=None, t=0.0, explicit=False, eps4=None, lam=None):
        r, w = self.rule, self.w
        U, Up = r.nodal(U), r.nodal(Up)
        out = torch.zeros_like(U)
        theta = -1.0 if explicit else self.theta
        for p in r.points:
            h, args = self._primal(U, Up, hist, p, explicit)
            for f, terms in enumerate(self.point(w.eps4 if eps4 is None else eps4, getattr(w, "lam", 0.0) if lam is None else lam,
                                                 theta, t, r.x0(p), h, *args)):
                r.add(out, f, p, terms[0], terms[1:])
        return out.reshape(-1)

    def explicit(self, Up, Upp, t):
        """E: the part of a theta step fixed by the previous states."""
        E = (1 - self.theta) * self.residual(Up, Up, t=t, explicit=True)
        if self.case["model"] == "thermal":
            r, E = self.rule, self.rule.nodal(E)
            d = r.nodal(Up) - r.nodal(Upp)
            for p in r.points:
                r.add(E, 1, p, -(1 - self.theta) / (2 * self.dt) * r.at(d, p, False)[0][..., 0])
        return E.reshape(-1)

    def jvp(self, U, Up, v, hist=None, t=0.0):
        r, w = self.rule, self.w
        U, Up, v = r.nodal(U), r.nodal(Up), r.nodal(v)
        out = torch.zeros_like(U)
        for p in r.points:
            h, args = self._primal(U, Up, hist, p, False)
            val, grad = r.at(v, p)
            zero = torch.zeros_like(val[..., 0])
            tang = [val[..., 0], val[..., 1], zero, zero] + [k[..., 0] for k in grad] + [k[..., 1] for k in grad]

            def flat(*a):
                s = self.point(w.eps4, getattr(w, "lam", 0.0), self.theta, t, r.x0(p), h, *a)
                return tuple(s[0]) + tuple(s[1])
            d = torch.func.jvp(flat, tuple(args), tuple(tang))[1]
            for f in range(2):
                r.add(out, f, p, d[f * (self.dim + 1)], d[f * (self.dim + 1) + 1:(f + 1) * (self.dim + 1)])
        return out.reshape(-1)

    def vjp(self, U, Up, W, eps4=None, lam=None):
        """(dF/dU)^T W, (dF/dUprev)^T W and W . dF/d(eps4, lambda)."""
        r, w, m = self.rule, self.w, self.dim + 1
        U, Up, W = r.nodal(U), r.nodal(Up), r.nodal(W)
        gU, gP, gp = torch.zeros_like(U), torch.zeros_like(U), torch.zeros(2, dtype=F64, device=U.device)
        for p in r.points:
            h, args = self._primal(U, Up, None, p, False)
            val, grad = r.at(W, p)
            par = [torch.tensor(x, dtype=F64, device=U.device, requires_grad=True)
                   for x in (w.eps4 if eps4 is None else eps4, w.lam if lam is None else lam)]
            args = [a.detach().requires_grad_(True) for a in args]
            s = self.point(par[0], par[1], self.theta, 0.0, 0.0, h, *args)
            cot = [[val[..., f]] + [k[..., f] for k in grad] for f in range(2)]
            total = sum((a * b).sum() for f in range(2) for a, b in zip(s[f], cot[f]))
            d = torch.autograd.grad(total, par + args)
            gp += p[0] * torch.stack(d[:2])
            d = d[2:]
            r.add(gU, 0, p, d[0], d[4:4 + self.dim])
            r.add(gU, 1, p, d[1], d[4 + self.dim:])
            r.add(gP, 0, p, d[2])
            r.add(gP, 1, p, d[3])
        return gU.reshape(-1), gP.reshape(-1), gp

    def solve(self, Up, Upp, t=0.0):
        """The new state of one step from U = Uprev, by Newton on the exact tangent."""
        hist = self.history(Up, Upp)
        E = self.explicit(Up, Upp, t - self.dt) if self.theta != 1.0 else 0.0
        U, F = Up, self.residual(Up, Up, hist, t) + E
        f0 = f = float(F.norm())
        for _ in range(12):
            if f <= 1e-14 * f0:
                break
            step = _gmres(lambda x: self.jvp(U, Up, x, hist, t), -F, 1e-5)
            F2 = self.residual(U + step, Up, hist, t) + E
            if float(F2.norm()) >= f:
                break
            U, F, f = U + step, F2, float(F2.norm())
        return U


def _gmres(A, b, rtol, m=80):
    beta = float(b.norm())
    V = torch.empty((m + 1, b.numel()), dtype=F64, device=b.device)
    H = np.zeros((m + 1, m))
    V[0] = b / beta
    for j in range(m):
        x = A(V[j])
        for _ in range(2):
            c = V[: j + 1] @ x
            x = x - V[: j + 1].t() @ c
            H[: j + 1, j] += c.cpu().numpy()
        H[j + 1, j] = float(x.norm())
        V[j + 1] = x / H[j + 1, j]
        e = np.zeros(j + 2)
        e[0] = beta
        y = np.linalg.lstsq(H[: j + 2, : j + 1], e, rcond=None)[0]
        if np.linalg.norm(H[: j + 2, : j + 1] @ y - e) <= rtol * beta:
            break
    return V[: j + 1].t() @ torch.from_numpy(y).to(b.device)


def _exact_gradient(case, eq, U0, target):
    states = [U0]
    for _ in range(case["steps"]):
        states.append(eq.solve(states[-1], states[-1]))
    mass = torch.ones((), dtype=F64, device=U0.device)
    for k in reversed(_mesh(case)):
        line = torch.full((k + 1,), H_THERMAL, dtype=F64, device=U0.device)
        line[0] = line[-1] = H_THERMAL / 2
        mass = mass.unsqueeze(-1) * line
    d = states[-1].view(-1, 2)[:, 0] - target
    mu = torch.zeros_like(U0)
    mu.view(-1, 2)[:, 0] = mass.reshape(-1) * d
    loss, gp = 0.5 * (mass.reshape(-1) * d * d).sum(), torch.zeros(2, dtype=F64, device=U0.device)
    for k in range(case["steps"], 0, -1):
        lam = _gmres(lambda x: eq.vjp(states[k], states[k - 1], x)[0], mu, 1e-14)
        _, gP, p = eq.vjp(states[k], states[k - 1], lam)
        gp, mu = gp - p, -gP
    return states[-1], loss, gp[0], gp[1], mu


def exact(case, seed):
    op, dim = case["op"], case["dim"]
    # the V-cycle is defined by the library's own hierarchy; 3-D solves would take minutes here
    if op == "vcycle" or (dim == 3 and op in ("step", "adjoint")):
        return None
    w = _workload(case)
    eq = _Equations(case, w)
    Upp, Up, U, v = _states(case, seed)
    if op == "residual":
        return eq.residual(U, Up, eq.history(Up, Upp), w.dt)
    if op == "jvp":
        return eq.jvp(U, Up, v, eq.history(Up, Upp), w.dt)
    if op == "vjp":
        return eq.vjp(U, Up, v)
    if op == "step":
        return eq.solve(Up, Upp, w.dt)
    if op == "adjoint":
        lam = _gmres(lambda x: eq.vjp(U, Up, x)[0], _cotangent(case, U), 1e-14)
        _, gP, gp = eq.vjp(U, Up, lam)
        return lam, -gP, -gp
    return _exact_gradient(case, eq, Up, _target(case, U))
