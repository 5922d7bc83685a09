"""The work a user of this framework has it do, as cases that can be timed.

A case is one call (or one short sequence of calls) of the public Python API on
inputs that already exist.  Four kinds:

* ``run``: a simulation advanced by ``steps`` steps and its six fields read into
  device tensors, on any scheme, storage and boundary mix; optionally with the
  energy and divergence diagnostics of the new state;
* ``batch``: several independent grids advanced together by ``step_batch``;
* ``adjoint``: one forward run and reverse sweep (``Simulation.adjoint``);
* ``design``: one evaluation of the differentiable objective, forward and
  backward (``design_objective``), as an optimiser calls it.

Materials: ``boxes`` is a background of eps 2.08 with dielectric boxes of
eps 12.25 (the benchmark's maps), ``blocks`` boxes of many permittivities,
``graded`` a permittivity that varies from cell to cell (lenses, designs in
progress), ``vacuum`` eps 1.
"""
import math

import numpy as np
import torch

from paper_2502_20610_amd import fdtd
from paper_2502_20610_amd import workloads as wl

DT, DX = 0.5, 1.0
OMEGA = 2.0 * math.pi / (12.0 * math.sqrt(2.08))


def _run(name, shape, steps, **more):
    c = {"kind": "run", "nx": shape[0], "ny": shape[1], "nz": shape[2], "steps": steps, "scheme": "systolic",
         "bc": "000", "storage": "fp32", "materials": "boxes", "lossy": False, "sources": 1, "monitor": False}
    c.update(more)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest grids of a parameter study: launches and latency
        _run("plain_32", (32, 32, 32), 64, scheme="plain"),
        # the cavity-pulse configuration: 64^3 vacuum, closed walls, 100 steps, no sources
        _run("cavity_64", (64, 64, 64), 100, scheme="plain", materials="vacuum", sources=0),
        # ordinary grid of odd sizes on the one-launch step, mixed boundaries, with the energy
        # and divergence diagnostics that a run logs every so many steps
        _run("fused_diagnostics", (201, 150, 173), 32, scheme="plain_fused", bc="010", monitor=True, sources=2),
        # an ordinary grid of ragged sizes on the systolic scheme
        _run("ragged_box", (131, 117, 150), 48),
        # a periodic unit cell: the 256^3 configuration with periodic x and y
        _run("periodic_256", (256, 256, 256), 128, bc="110"),
        # the largest configuration, in the 20-step calls of the benchmark
        _run("box_1024x1024x512", (1024, 1024, 512), 20, sources=3),
        # the same kind of box with an absorbing conductive shell
        _run("absorbing_shell", (384, 360, 256), 64, lossy=True),
        # FP16 storage, for grids that should take half the memory
        _run("half_storage", (512, 448, 384), 48, storage="fp16"),
        # a permittivity that differs from cell to cell
        _run("graded_index", (320, 290, 272), 40, materials="graded"),
        # a sweep over many small grids, advanced together
        {"name": "batch_16", "kind": "batch", "grids": 16, "lo": 16, "hi": 64, "sizes": 5, "steps": 64},
        # one gradient of the inverse-design configuration (its grid, design block and monitor
        # plane, fewer steps)
        {"name": "adjoint_256x256x128", "kind": "adjoint", "nx": 256, "ny": 256, "nz": 128, "steps": 480,
         "lossy": False},
        # one optimiser iteration of a small design problem, forward and backward, whole call
        {"name": "design_64x64x32", "kind": "design", "nx": 64, "ny": 64, "nz": 32, "steps": 200, "lossy": False},
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choices(["run", "batch", "adjoint", "design"], [8, 1, 1.5, 1.5])[0]
    if kind == "batch":
        return {"kind": "batch", "grids": rng.randint(4, 32), "lo": 16, "hi": rng.choice([48, 64, 96, 128]),
                "sizes": rng.randint(0, 1 << 20), "steps": rng.randint(24, 96)}
    if kind in ("adjoint", "design"):
        # long enough for the pulse to pass the block and reach the monitor
        n = (rng.randint(64, 160), rng.randint(64, 160), rng.randint(48, 96)) if kind == "adjoint" else \
            (rng.randint(40, 96), rng.randint(40, 96), rng.randint(24, 64))
        return {"kind": kind, "nx": n[0], "ny": n[1], "nz": n[2], "steps": 160 + rng.randint(n[0] // 2, (3 * n[0]) // 2),
                "lossy": rng.random() < 0.3}
    scheme = rng.choices(["plain", "plain_fused", "systolic"], [3, 1, 4])[0]
    storage = "fp16" if scheme != "plain_fused" and rng.random() < 0.15 else "fp32"
    lossy = storage == "fp32" and rng.random() < 0.25
    steps = rng.choice([16, 20, 32, 50, 64, 100, 128])
    cells = _log(rng, 2.0 ** 13, min(2.0 ** 27, (3.0e9 if scheme == "systolic" else 1.5e9) / steps))
    cells = min(cells, 2.0 ** 24) if scheme == "plain" else cells
    bc = rng.choice(["000", "000", "000", "110", "010", "100", "001", "011"])
    fx, fy = _log(rng, 0.6, 1.7), _log(rng, 0.6, 1.7)
    edge = cells ** (1.0 / 3.0)
    n = [max(16, int(round(edge * f))) for f in (fx, fy, 1.0 / (fx * fy))]
    n = [min(v, 256) if bc != "000" and bc[a] == "1" else v for a, v in enumerate(n)]
    n = [max(v, 20) if bc[a] == "1" else v for a, v in enumerate(n)]
    return _run(None, n, steps, scheme=scheme, bc=bc, storage=storage, lossy=lossy,
                materials=rng.choice(["boxes", "boxes", "blocks", "graded"]), sources=rng.randint(0, 3),
                monitor=rng.random() < 0.25)


# ---- inputs, from the seed alone


def _shape(case):
    return (case["nx"], case["ny"], case["nz"])


def _eps(kind, shape, rng, gen):
    """A permittivity map on the GPU."""
    if kind == "vacuum":
        return torch.ones(shape, device="cuda")
    if kind == "graded":
        axes = [torch.linspace(0.0, math.pi * float(rng.uniform(1.0, 3.0)), s, device="cuda") for s in shape]
        e = (1.0 + torch.sin(axes[0])[:, None, None] * torch.cos(axes[1])[None, :, None]
             * torch.sin(axes[2] + 0.3)[None, None, :])
        return (2.08 + 4.0 * e + 0.5 * torch.rand(shape, device="cuda", generator=gen)).contiguous()
    eps = torch.full(shape, 2.08, device="cuda")
    cells = shape[0] * shape[1] * shape[2]
    hi = [max(2, min(64, s // 3)) for s in shape]
    lo = [max(1, min(8, h // 2)) for h in hi]
    for _ in range(max(4, int(round(2000 * cells / 2.0 ** 29))) if kind == "boxes" else 40):
        side = [int(rng.integers(lo[a], hi[a] + 1)) for a in range(3)]
        at = [int(rng.integers(0, shape[a] - side[a] + 1)) for a in range(3)]
        v = 12.25 if kind == "boxes" else float(rng.uniform(1.0, 12.25))
        eps[at[0]:at[0] + side[0], at[1]:at[1] + side[1], at[2]:at[2] + side[2]] = v
    return eps


def _shell(shape, sigma_max=0.4):
    """The absorbing layer of workloads.graded_shell, on the GPU."""
    depth = max(2, min(16, min(shape) // 5))
    d = [torch.minimum(torch.arange(s, device="cuda"), s - 1 - torch.arange(s, device="cuda")) for s in shape]
    near = torch.minimum(torch.minimum(d[0][:, None, None], d[1][None, :, None]), d[2][None, None, :])
    x = (depth - near.clamp(max=depth)).float() / depth
    return (sigma_max * x * x).contiguous()


def _inputs(case, seed):
    """Everything that defines a ``run`` case: eps, sigma, fields, sources."""
    shape = _shape(case)
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    eps = _eps(case["materials"], shape, rng, gen)
    sigma = _shell(shape) if case["lossy"] else None
    fields = [torch.rand(shape, device="cuda", generator=gen).mul_(2.0).sub_(1.0) for _ in range(6)]
    sources = []
    for q in range(case["sources"]):
        at = [int(rng.integers(1, s)) for s in shape]
        wave = wl.gaussian_sine(4 * case["steps"], DT, amplitude=float(rng.uniform(0.5, 2.0)))
        sources.append(wl.dipole(wl.EZ if q % 2 == 0 else wl.EX, *at, wave))
    return eps, sigma, fields, sources


def _bc(case):
    return tuple(int(v) for v in case.get("bc", "000"))


def _batch_members(case, seed):
    rng = np.random.default_rng(case["sizes"])
    out = []
    for q in range(case["grids"]):
        shape = [int(rng.integers(case["lo"], case["hi"] + 1)) for _ in range(3)]
        out.append(({"kind": "run", "nx": shape[0], "ny": shape[1], "nz": shape[2], "steps": case["steps"],
                     "materials": "blocks", "lossy": False, "sources": 1}, seed * 1000 + q))
    return out


def _design_setup(case, seed):
    """Permittivity, conductivity, design and monitor boxes and the source of an inverse-design
    run: a block in the middle, a dipole six cells before its -x side, a monitor plane six cells
    behind its +x side."""
    shape = _shape(case)
    rng = np.random.default_rng(seed)
    lo = tuple((3 * s) // 8 for s in shape)
    hi = tuple(max(l + 1, (5 * s) // 8) for l, s in zip(lo, shape))
    design = rng.uniform(2.08, 12.25, [h - l for l, h in zip(lo, hi)]).astype(np.float32)
    eps = np.full(shape, np.float32(2.08), np.float32)
    eps[lo[0]:hi[0], lo[1]:hi[1], lo[2]:hi[2]] = design
    sigma = np.ascontiguousarray(_shell(shape, 0.2).cpu().numpy()) if case["lossy"] else None
    mx = min(shape[0] - 1, hi[0] + 6)
    wave = wl.gaussian_sine(case["steps"], DT, amplitude=float(rng.uniform(0.5, 2.0)))
    source = wl.dipole(wl.EZ, max(1, lo[0] - 6), shape[1] // 2, shape[2] // 2, wave)
    args = dict(nsteps=case["steps"], mon_comp=wl.EZ, mon_lo=(mx, lo[1], shape[2] // 4),
                mon_hi=(mx + 1, hi[1], (3 * shape[2]) // 4), omega=OMEGA, des_lo=lo, des_hi=hi)
    return eps, sigma, design, source, args


# ---- what a program has in hand before the call


def _simulation(case, seed, stream=None):
    eps, sigma, fields, sources = _inputs(case, seed)
    sim = fdtd.Simulation(_shape(case), DT, DX, _bc(case), scheme=case.get("scheme", "systolic"),
                          storage=case.get("storage", "fp32"), stream=stream)
    torch.cuda.synchronize()
    sim.set_materials(eps, sigma=sigma)
    sim.set_fields(fields)
    for s in sources:
        sim.add_source(s["comp"], s["i"], s["j"], s["k"], s["waveform"])
    sim.synchronize()
    return sim


def prepare(case, seed):
    state = {"case": case}
    if case["kind"] == "run":
        state["sim"] = _simulation(case, seed)
        state["sim"].prepare(case["steps"])
        state["fields"] = [torch.empty(_shape(case), device="cuda") for _ in range(6)]
        if case["monitor"]:
            state["sums"] = torch.empty(len(fdtd.INVARIANT_NAMES), dtype=torch.float64, device="cuda")
            state["div"] = [torch.empty(_shape(case), dtype=torch.float64, device="cuda") for _ in range(2)]
    elif case["kind"] == "batch":
        state["stream"] = torch.cuda.Stream()
        state["sims"], state["fields"] = [], []
        for member, s in _batch_members(case, seed):
            state["sims"].append(_simulation(member, s, stream=state["stream"].cuda_stream))
            state["fields"].append(torch.empty((6,) + _shape(member), device="cuda"))
    elif case["kind"] == "adjoint":
        eps, sigma, design, source, args = _design_setup(case, seed)
        sim = fdtd.Simulation(_shape(case), DT, DX, (0, 0, 0), scheme="plain")
        sim.set_materials(eps, sigma=sigma)
        sim.add_source(source["comp"], source["i"], source["j"], source["k"], source["waveform"])
        state.update(sim=sim, args=args, grad=torch.empty((3,) + design.shape, device="cuda"))
        state["zero"] = [torch.zeros(_shape(case), device="cuda") for _ in range(6)]
    else:
        eps, sigma, design, source, args = _design_setup(case, seed)
        state["problem"] = fdtd.DesignProblem(eps, (0, 0, 0), DT, DX, [source], args, sigma=sigma)
        state["x"] = torch.from_numpy(design).cuda()
    torch.cuda.synchronize()
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "run":
        sim = state["sim"]
        sim.step(case["steps"])
        out = {"fields": list(sim.read_fields(out=state["fields"]))}
        if case["monitor"]:
            out["sums"], out["div_e"], out["div_h"] = sim.invariants(device_out=(state["sums"], *state["div"]))
        return out
    if case["kind"] == "batch":
        fdtd.step_batch(state["sims"], case["steps"])
        for sim, f in zip(state["sims"], state["fields"]):
            sim.read_fields(out=list(f))
        return state["fields"]
    if case["kind"] == "adjoint":
        # every evaluation of an objective starts from fields at rest
        state["sim"].set_fields(state["zero"])
        J, grad = state["sim"].adjoint(out=state["grad"], **state["args"])
        return {"J": J, "grad": grad}
    x = state["x"].detach().requires_grad_(True)
    J = fdtd.design_objective(x, state["problem"])
    J.backward()
    return {"J": J.detach(), "grad": x.grad}


# ---- what a pass cannot do without


def work(case):
    if case["kind"] == "batch":
        # the axes are drawn evenly from lo..hi
        cells = case["grids"] * (0.5 * (case["lo"] + case["hi"])) ** 3
        return {"bytes": cells * 84.0, "flops": cells * 36.0 * case["steps"]}
    cells = float(case["nx"]) * case["ny"] * case["nz"]
    if case["kind"] == "run":
        # the state in and out, the coefficients in, and the fields handed to the caller
        b = (12 + 6 + 12 + 24) if case["storage"] == "fp16" else (24 + (24 if case["lossy"] else 12) + 24 + 24)
        if case["monitor"]:
            b += 16
        return {"bytes": cells * b, "flops": cells * case["steps"] * (39.0 if case["lossy"] else 36.0)}
    # coefficients in; the fields and the adjoint fields of the sweep fit on no chip and are
    # not counted; the gradient out
    box = cells / 64.0
    per = (39.0 + 30.0 + 9.0) if case["lossy"] else (36.0 + 30.0)
    return {"bytes": cells * (24 if case["lossy"] else 12) + 12.0 * box, "flops": cells * case["steps"] * per}


# ---- the same in 64 bits, in plain torch


def _coefficients(eps, sigma, bc):
    """ca, cb per component: E = ca E + cb curl H, 1 and 0 on tangential wall entries."""
    ca, cb = [], []
    e = eps.double()
    h = torch.zeros_like(e) if sigma is None else sigma.double() * DT / (2.0 * e)
    a0, b0 = (1.0 - h) / (1.0 + h), DT / (e * DX) / (1.0 + h)
    for c in range(3):
        a, b = a0.clone(), b0.clone()
        for axis in range(3):
            if axis != c and bc[axis] == 0:
                a.select(axis, 0).fill_(1.0)
                b.select(axis, 0).zero_()
        ca.append(a)
        cb.append(b)
    return ca, cb


def _curl_h(H):
    """Backward differences, as the E half-step takes them (indices modulo the grid)."""
    d = lambda f, axis: f - torch.roll(f, 1, axis)  # noqa: E731
    return [d(H[2], 1) - d(H[1], 2), d(H[0], 2) - d(H[2], 0), d(H[1], 0) - d(H[0], 1)]


def _curl_e(E):
    """Forward differences, as the H half-step takes them."""
    d = lambda f, axis: torch.roll(f, -1, axis) - f  # noqa: E731
    return [d(E[2], 1) - d(E[1], 2), d(E[0], 2) - d(E[2], 0), d(E[1], 0) - d(E[0], 1)]


def _step64(E, H, ca, cb, sources, n, lossy):
    """One step in place; returns the curl of the old H."""
    ch = _curl_h(H)
    for c in range(3):
        if lossy:
            E[c].mul_(ca[c])
        E[c].addcmul_(cb[c], ch[c])
    for s in sources:
        if n < len(s["waveform"]):
            E[s["comp"]][s["i"], s["j"], s["k"]] += float(s["waveform"][n])
    ce = _curl_e(E)
    for c in range(3):
        H[c].sub_(ce[c], alpha=DT / DX)
    return ch


def _fields64(case, seed, bc, lossy):
    eps, sigma, fields, sources = _inputs(case, seed)
    ca, cb = _coefficients(eps, sigma, bc)
    f = [v.double() for v in fields]
    del fields
    for c in range(3):
        for axis in range(3):
            if axis != c and bc[axis] == 0:
                f[c].select(axis, 0).zero_()
    E, H = f[:3], f[3:]
    for n in range(case["steps"]):
        _step64(E, H, ca, cb, sources, n, lossy)
    return eps, E, H, ca, cb


def _gradient64(case, seed):
    eps, sigma, design, source, args = _design_setup(case, seed)
    ca, cb = _coefficients(torch.from_numpy(eps).cuda(), None if sigma is None else torch.from_numpy(sigma).cuda(),
                           (0, 0, 0))
    box = tuple(slice(l, h) for l, h in zip(args["des_lo"], args["des_hi"]))
    mon = tuple(slice(l, h) for l, h in zip(args["mon_lo"], args["mon_hi"]))
    zeros = lambda: [torch.zeros(eps.shape, dtype=torch.float64, device="cuda") for _ in range(3)]  # noqa: E731
    E, H, ch, old = zeros(), zeros(), [], []
    F, lossy, c0 = 0.0, bool(case["lossy"]), args["mon_comp"]
    phase = lambda n: (math.cos(OMEGA * n * DT), -math.sin(OMEGA * n * DT))  # noqa: E731
    for n in range(case["steps"]):
        old.append([E[c][box].clone() for c in range(3)])
        curl = _step64(E, H, ca, cb, [source], n, lossy)
        ch.append([curl[c][box].clone() for c in range(3)])
        cr, ci = phase(n + 1)
        F = F + torch.complex(E[c0][mon] * cr, E[c0][mon] * ci)
    J = float((F.real ** 2 + F.imag ** 2).sum())
    lE, lH = zeros(), zeros()
    gA, gB = [torch.zeros_like(old[0][0]) for _ in range(3)], [torch.zeros_like(old[0][0]) for _ in range(3)]
    for n in range(case["steps"], 0, -1):
        cr, ci = phase(n)
        curl = _curl_h(lH)
        for c in range(3):
            if lossy:
                lE[c].mul_(ca[c])
            lE[c].sub_(curl[c], alpha=DT / DX)
        lE[c0][mon] += 2.0 * (F.real * cr + F.imag * ci)
        for c in range(3):
            gB[c].addcmul_(lE[c][box], ch[n - 1][c])
            gA[c].addcmul_(lE[c][box], old[n - 1][c])
        curl = _curl_e([cb[c] * lE[c] for c in range(3)])
        for c in range(3):
            lH[c].add_(curl[c])
    grad = []
    for c in range(3):
        a, b = ca[c][box], cb[c][box]
        grad.append(DX / DT * b * ((1.0 - a) * gA[c] - b * gB[c]))
    return J, torch.stack(grad)


def exact(case, seed):
    if case["kind"] == "run":
        bc = _bc(case)
        eps, E, H, ca, cb = _fields64(case, seed, bc, case["lossy"])
        out = {"fields": E + H}
        if case["monitor"]:
            # the diagnostics are of the stored state, whose rounding decides the divergences:
            # they have no value of their own in 64 bits
            out.update(sums=None, div_e=None, div_h=None)
        return out
    if case["kind"] == "batch":
        out = []
        for member, s in _batch_members(case, seed):
            _, E, H, _, _ = _fields64(member, s, (0, 0, 0), False)
            out.append(torch.stack(E + H))
        return out
    J, grad = _gradient64(case, seed)
    if case["kind"] == "design":
        return {"J": torch.tensor(J, dtype=torch.float64), "grad": grad.sum(0)}
    return {"J": J, "grad": grad}
