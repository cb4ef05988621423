"""Performance cases of the D3Q19 lattice-Boltzmann library.

Three kinds of work cover what a program does with it, each through the
public Python entry points (lb.Lattice and the differentiable rollouts):

  "step"     advance a lattice by some steps and read its state;
  "report"   the diagnostics a running simulation writes: moment fields,
             statistics, conserved sums and the state at masked sites;
  "rollout"  a differentiable rollout with its backward pass.

listed() holds fixed cases, draw() one more from the same ranges, prepare()
and run() make and run one, work() counts the bytes and operations it cannot
do without, and exact() gives its result in plain FP64 torch.
"""

import math

import torch
from torch.utils.checkpoint import checkpoint

from paper_1405_6162_amd import adjoint, lb

MODELS = {"single": lb.LB_SINGLE, "binary": lb.LB_BINARY}
STORAGES = {"f64": lb.LB_F64, "f32": lb.LB_F32, "f16": lb.LB_F16}
BYTES = {"f64": 8, "f32": 4, "f16": 2}
COLLISIONS = {"bgk": lb.LB_BGK, "trt": lb.LB_TRT, "mrt": lb.LB_MRT}
# relaxation times of f: tau_f, tau_minus, tau_bulk, tau_ghost_even, tau_ghost_odd
TIMES = (0.8, 1.1, 1.3, 0.9, 1.2)
RATES = {"bgk": 1, "trt": 2, "mrt": 5}
A, B, KAPPA, MOBILITY = -0.0625, 0.0625, 0.04, 0.45

VELOCITIES = [(0, 0, 0)] + [(x, y, z) for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1)
                            if x * x + y * y + z * z in (1, 2)]
WEIGHTS = [{0: 1 / 3, 1: 1 / 18, 2: 1 / 36}[x * x + y * y + z * z] for x, y, z in VELOCITIES]
# a drawn case moves at most this many bytes, about what the largest listed one moves
MOST_BYTES = 110e9


def _step(name, model, storage, collision, size, nsteps):
    return {"name": name, "kind": "step", "model": model, "storage": storage, "collision": collision,
            "nx": size[0], "ny": size[1], "nz": size[2], "nsteps": nsteps}


def listed():
    return [
        # the smallest run: a 16^3 lattice of the parity tests, launch latency
        _step("single16_f64", "single", "f64", "bgk", (16, 16, 16), 10),
        # a small two-fluid lattice, as in unit tests and parameter scans
        _step("binary32_f64", "binary", "f64", "bgk", (32, 32, 32), 20),
        # an ordinary box whose extents fit no tile, reduced storage, the five-time collision
        _step("single150x70x90_mrt_f32", "single", "f32", "mrt", (150, 70, 90), 25),
        # the single-fluid throughput workload
        _step("single256_f64", "single", "f64", "bgk", (256, 256, 256), 20),
        # the paper-sized two-fluid benchmark
        _step("binary128_f64", "binary", "f64", "bgk", (128, 128, 128), 20),
        # a two-fluid box with a ragged x extent in reduced storage
        _step("binary200x204x100_f32", "binary", "f32", "bgk", (200, 204, 100), 20),
        # the headline throughput workload
        _step("binary256_f64", "binary", "f64", "bgk", (256, 256, 256), 10),
        # the largest reduced-storage workload
        _step("binary384_f16", "binary", "f16", "bgk", (384, 384, 384), 10),
        # a full-precision lattice whose buffers pass 4 GiB each
        _step("binary320_f64", "binary", "f64", "bgk", (320, 320, 320), 5),
        # what a production run writes between its steps
        {"name": "report256_f64", "kind": "report", "model": "binary", "storage": "f64", "collision": "bgk",
         "nx": 256, "ny": 256, "nz": 256},
        # gradient of a shear wave's decay: forward and backward
        {"name": "rollout_single64", "kind": "rollout", "model": "single", "storage": "f64", "collision": "bgk",
         "nx": 64, "ny": 64, "nz": 64, "nsteps": 40, "every": 20},
        # gradient of a spinodal quench with respect to its fields and parameters
        {"name": "rollout_binary128", "kind": "rollout", "model": "binary", "storage": "f64", "collision": "bgk",
         "nx": 128, "ny": 128, "nz": 128, "nsteps": 20, "every": 10},
    ]


def draw(rng):
    """One more case: a kind, then options, then extents spread over the
    logarithm of 8 .. 384 (rollouts: 12 .. 128), about half of them not a
    multiple of anything, and a step count spread over the logarithm."""
    while True:
        kind = rng.choices(("step", "report", "rollout"), (6, 1, 2))[0]
        case = {"kind": kind, "model": rng.choice(("single", "binary")),
                "storage": "f64" if kind == "rollout" else rng.choice(("f64", "f64", "f32", "f32", "f16")),
                "collision": rng.choice(("bgk", "bgk", "trt", "mrt"))}
        top, low = (128, 12) if kind == "rollout" else (384, 8)
        edge = math.exp(rng.uniform(math.log(low), math.log(top)))
        for k in ("nx", "ny", "nz"):
            n = edge * math.exp(rng.uniform(-0.5, 0.5))
            step = rng.choice((1, 1, 8, 16))
            case[k] = min(max(int(round(n / step)) * step, 8), 400)
        if kind != "report":
            case["nsteps"] = int(round(math.exp(rng.uniform(math.log(2 if kind == "rollout" else 1), math.log(40)))))
        if kind == "rollout":
            case["every"] = rng.choice((0, 5, 10, 20))
        if work(case)["bytes"] <= (20e9 if kind == "rollout" else MOST_BYTES):
            return case


def _nd(case):
    return 1 if case["model"] == "single" else 2


def _fields(case, seed):
    """rho, u and phi (binary) of the initial state on the GPU: uniform
    density and velocity noise (a shear wave for single-fluid rollouts), or
    the spinodal quench rho = 1, u = 0, phi uniform in [-0.05, 0.05]."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    shape = (case["nz"], case["ny"], case["nx"])
    kw = dict(dtype=torch.float64, device="cuda")
    if case["model"] == "binary":
        phi = torch.rand(shape, generator=gen, **kw) * 0.1 - 0.05
        return torch.ones(shape, **kw), torch.zeros((3,) + shape, **kw), phi
    if case["kind"] == "rollout":
        u = (torch.rand((3,) + shape, generator=gen, **kw) * 2 - 1) * 1e-4
        y = torch.arange(case["ny"], **kw).reshape(1, -1, 1)
        u[0] += 0.01 * torch.sin(2 * math.pi * y / case["ny"])
        return torch.ones(shape, **kw), u, None
    rho = 1 + 0.01 * torch.randn(shape, generator=gen, **kw)
    return rho, (torch.rand((3,) + shape, generator=gen, **kw) * 2 - 1) * 0.01, None


def _lattice(case, phi):
    t = TIMES
    return lb.Lattice(case["nx"], case["ny"], case["nz"], model=MODELS[case["model"]],
                      storage=STORAGES[case["storage"]], collision=COLLISIONS[case["collision"]], tau_f=t[0],
                      tau_minus=t[1], tau_bulk=t[2], tau_ghost_even=t[3], tau_ghost_odd=t[4], A=A, B=B, kappa=KAPPA,
                      mobility=MOBILITY, rho0=1.0, phi0=float(phi.mean()) if phi is not None else 0.0)


def _mask(case):
    """A ball around the centre of the box, as a probe region."""
    ax = [torch.linspace(-1, 1, case[k], device="cuda", dtype=torch.float64) for k in ("nz", "ny", "nx")]
    z, y, x = torch.meshgrid(*ax, indexing="ij")
    return x * x + y * y + z * z < 0.09


def prepare(case, seed):
    rho, u, phi = _fields(case, seed)
    lat = _lattice(case, phi)
    if case["kind"] == "step":
        lat.init_equilibrium(rho, u, phi)
        return {"lat": lat, "nsteps": case["nsteps"]}
    if case["kind"] == "report":
        lat.init_equilibrium(rho, u, phi)
        lat.step(2)
        return {"lat": lat, "mask": _mask(case)}
    par = lambda v: torch.tensor(v, dtype=torch.float64, device="cuda", requires_grad=True)
    n = RATES[case["collision"]]
    state = {"lat": lat, "nsteps": case["nsteps"], "every": case["every"],
             "tau": par(list(TIMES[:n]) if n > 1 else TIMES[0])}
    if case["model"] == "single":
        lat.init_equilibrium(rho, u)
        state["f0"] = lat.get_state()[0].requires_grad_(True)
    else:
        state.update(rho=rho.requires_grad_(True), u=u.requires_grad_(True), phi=phi.requires_grad_(True),
                     kappa=par(KAPPA), mobility=par(MOBILITY))
    return state


def run(state):
    lat = state["lat"]
    if "mask" in state:
        index = lat.mask_index(state["mask"])
        return lat.moments(), lat.field_stats(), lat.conserved_sums(), index, lat.get_sites(index)
    if "tau" not in state:
        lat.step(state["nsteps"])
        return lat.get_state()
    if "f0" in state:
        leaves = [state["f0"], state["tau"]]
        out = (adjoint.rollout(leaves[0], leaves[1], lat, state["nsteps"], state["every"]),)
        loss = adjoint.velocity_loss(out[0])
    else:
        leaves = [state[k] for k in ("rho", "u", "phi", "kappa", "mobility", "tau")]
        out = adjoint.rollout_binary(*leaves[:3], lat, state["nsteps"], state["every"], *leaves[3:])
        loss = adjoint.binary_loss(*out)
    return [o.detach() for o in out], loss.detach(), torch.autograd.grad(loss, leaves)


def work(case):
    """A step reads and writes every distribution value once, and handing a
    state out reads and writes it once more; an adjoint step reads the state
    and the adjoint and writes the adjoint (beside the forward step); a
    report reads the state once for its sums and fields and writes them."""
    n, nd, es = case["nx"] * case["ny"] * case["nz"], _nd(case), BYTES[case["storage"]]
    state = 19 * nd * n * es
    flops = n * (250 if nd == 1 else 600)
    if case["kind"] == "step":
        return {"bytes": 2 * state * (case["nsteps"] + 1), "flops": flops * case["nsteps"]}
    if case["kind"] == "report":
        inside = int(n * 0.3 ** 3 * math.pi / 6)
        return {"bytes": state + 8 * n * (3 + nd) + n + inside * (4 + 2 * 19 * nd * es), "flops": n * 60 * nd}
    return {"bytes": 5 * state * case["nsteps"] + 2 * state, "flops": 3 * flops * case["nsteps"]}


# ---- the method in plain FP64 torch -------------------------------------------

def _relaxation(case, taus):
    """The relaxation matrix of f (a number for one time): each part of
    f - f^eq divided by its time.  The parts are the even and the odd
    combinations of opposite velocities and, for five times, the moments of
    the orthogonal D3Q19 basis that relax apart: the energy, three even and
    three odd ghosts."""
    if case["collision"] == "bgk":
        return 1 / taus.reshape(())
    kw = dict(dtype=torch.float64, device=taus.device)
    swap = torch.zeros(19, 19, **kw)
    for i, c in enumerate(VELOCITIES):
        swap[i, VELOCITIES.index(tuple(-k for k in c))] = 1
    eye = torch.eye(19, **kw)
    even, odd = (eye + swap) / 2, (eye - swap) / 2
    parts = [even, odd]
    if case["collision"] == "mrt":
        def onto(*polys):
            total = torch.zeros(19, 19, **kw)
            for p in polys:
                m = torch.tensor([float(p(x, y, z, x * x + y * y + z * z)) for x, y, z in VELOCITIES], **kw)
                total += torch.outer(m, m) / (m * m).sum()
            return total
        bulk = onto(lambda x, y, z, s: 19 * s - 30)
        ghost_even = onto(lambda x, y, z, s: (21 * s * s - 53 * s + 24) / 2,
                          lambda x, y, z, s: (3 * s - 5) * (3 * x * x - s),
                          lambda x, y, z, s: (3 * s - 5) * (y * y - z * z))
        ghost_odd = onto(lambda x, y, z, s: (y * y - z * z) * x, lambda x, y, z, s: (z * z - x * x) * y,
                         lambda x, y, z, s: (x * x - y * y) * z)
        parts = [even - bulk - ghost_even, odd - ghost_odd, bulk, ghost_even, ghost_odd]
    return sum(p / t for p, t in zip(parts, taus))


def _along(c, v):
    total = 0
    for k, a in zip(c, v):
        if k:
            total = total + k * a
    return total


def _stencils(phi):
    plus = [torch.roll(phi, -1, d) for d in (2, 1, 0)]
    minus = [torch.roll(phi, 1, d) for d in (2, 1, 0)]
    return [(p - m) / 2 for p, m in zip(plus, minus)], sum(plus) + sum(minus) - 6 * phi


def _equilibria(rho, u, phi, kappa):
    """f^eq and g^eq (None without phi) by direction."""
    usq = u[0] * u[0] + u[1] * u[1] + u[2] * u[2]
    if phi is not None:
        grad, lap = _stencils(phi)
        gsq = grad[0] * grad[0] + grad[1] * grad[1] + grad[2] * grad[2]
        mu = A * phi + B * phi ** 3 - kappa * lap
        iso = A / 2 * phi ** 2 + 3 * B / 4 * phi ** 4 - kappa * phi * lap - kappa / 2 * gsq
    f, g = [], []
    for c, w in zip(VELOCITIES, WEIGHTS):
        s = sum(k * k for k in c)
        cu = _along(c, u)
        shape = 1 + 3 * cu + 4.5 * cu * cu - 1.5 * usq
        if phi is None:
            f.append(w * rho * shape)
            continue
        cg = _along(c, grad)
        stress = s * iso + kappa * cg * cg - (3 * iso + kappa * gsq) / 3
        f.append(w * (rho * shape + 4.5 * stress))
        g.append(w * (phi * shape + 4.5 * (mu - phi / 3) * (s - 1)))
    return f, g if phi is not None else None


def _exact_step(f, g, omega, mobility, kappa):
    rho = sum(f)
    u = [sum(c[k] * fi for c, fi in zip(VELOCITIES, f) if c[k]) / rho for k in range(3)]
    feq, geq = _equilibria(rho, u, sum(g) if g is not None else None, kappa)
    move = lambda a, c: torch.roll(a, (c[2], c[1], c[0]), (0, 1, 2))
    if omega.dim() == 0:
        f = [move(a - omega * (a - e), c) for a, e, c in zip(f, feq, VELOCITIES)]
    else:
        neq = torch.stack([(a - e).reshape(-1) for a, e in zip(f, feq)])
        f = [move(a - d.reshape(a.shape), c) for a, d, c in zip(f, torch.mm(omega, neq), VELOCITIES)]
    if g is not None:
        g = [move(a - (a - e) / (mobility + 0.5), c) for a, e, c in zip(g, geq, VELOCITIES)]
    return f, g


def exact(case, seed):
    n = case["nx"] * case["ny"] * case["nz"]
    if case["kind"] == "rollout" and n * case["nsteps"] * _nd(case) > 1.2e8:
        return None
    rho, u, phi = _fields(case, seed)
    p0 = float(phi.mean()) if phi is not None else 0.0
    kw = dict(dtype=torch.float64, device="cuda")
    taus = torch.tensor(TIMES[:RATES[case["collision"]]], **kw)
    kappa, mobility = torch.tensor(KAPPA, **kw), torch.tensor(MOBILITY, **kw)

    def stored(values, ref):
        if case["storage"] == "f64":
            ref = 0.0
        return torch.stack([a - w * ref for a, w in zip(values, WEIGHTS)])

    if case["kind"] != "rollout":
        with torch.no_grad():
            omega = _relaxation(case, taus)
            f, g = _equilibria(rho, u, phi, kappa)
            for _ in range(case.get("nsteps", 2)):
                f, g = _exact_step(f, g, omega, mobility, kappa)
            if case["kind"] == "step":
                return stored(f, 1.0), stored(g, p0) if g is not None else None
            rho = sum(f)
            j = torch.stack([sum(c[k] * fi for c, fi in zip(VELOCITIES, f) if c[k]) for k in range(3)])
            u, phi = j / rho, sum(g) if g is not None else None
            uu = (u * u).sum(0)
            zero = torch.zeros((), **kw)
            p = [phi.sum(), phi.min(), phi.max(), (phi * phi).sum()] if phi is not None else [zero] * 4
            sums = [rho.sum(), *j.flatten(1).sum(1), p[0]]
            stats = torch.stack(sums + [(rho * uu).sum(), *p[1:], uu.max()])
            index = _mask(case).flatten().nonzero().flatten()
            sites = [stored(v, r).reshape(19, -1)[:, index] if v is not None else None for v, r in ((f, 1.0), (g, p0))]
            return (rho, u, phi), stats, torch.stack(sums), None, sites

    leaves = [taus.reshape(()) if taus.numel() == 1 else taus]
    if case["model"] == "single":
        with torch.no_grad():
            f0 = torch.stack(_equilibria(rho, u, None, kappa)[0])
        leaves = [f0] + leaves
    else:
        leaves = [rho, u, phi, kappa, mobility] + leaves
    leaves = [v.detach().requires_grad_(True) for v in leaves]
    omega = _relaxation(case, leaves[-1])
    if case["model"] == "single":
        f, g = list(leaves[0]), None
    else:
        f, g = _equilibria(*leaves[:4])
    kap, mob = (kappa, mobility) if g is None else leaves[3:5]
    for _ in range(case["nsteps"]):
        f, g = checkpoint(_exact_step, f, g, omega, mob, kap, use_reentrant=False)
    rho = sum(f)
    uu = sum((sum(c[k] * fi for c, fi in zip(VELOCITIES, f) if c[k]) / rho) ** 2 for k in range(3))
    phi = sum(g) if g is not None else None
    loss = (uu if phi is None else uu + phi * phi).mean()
    grads = torch.autograd.grad(loss, leaves)
    return [torch.stack(v).detach() for v in (f, g) if v is not None], loss.detach(), grads
