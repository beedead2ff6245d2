"""Performance cases of the shear solver: the simulations a program runs through kvs.py.

Each case is one pass of such a program on inputs that are already in hand (medium, time step and force or acoustic
samples resident on the GPU): a whole push (projection and time steps), a window of steps, a batched sweep, a solve on
caller-owned buffers, or a training step of the learned preconditioner.  What a pass returns is what the program reads:
traces and peak maps (in the precision of the state they were taken from), potentials and projected forces on the
device, losses with gradients and updated weights.
"""
import math

import numpy as np
import torch

from paper_2607_28414_amd import kvs, train

DEV = "cuda"

# kind "sim": one context.  project: the projection is part of the pass (else it was done before the steps that are
# timed); source: "push" (separable Gaussian push), "epoch" (modulated push drawn on the device, force on every step,
# flexible PCG with a fixed number of iterations), "curl" (curl-based initial state, no force).
SIM = dict(kind="sim", nx=64, ny=64, nz=64, h=0.25e-3, fp64=False, medium="uniform", viscous=True, steps=100,
           push_steps=8, sponge=8, pml=0, tol=1e-8, project=True, source="push", peaks=False, comp=2, tuned=False,
           fixed_iters=0, state=False)


def sim(name, **over):
    return dict(SIM, name=name, **over)


def listed():
    return [
        # the smallest whole simulation, in parity precision, its final state read back: launches and latency
        sim("push_48_fp64", nx=48, ny=48, nz=48, h=0.5e-3, fp64=True, viscous=False, steps=200, push_steps=2, tol=1e-10,
            state=True),
        # a projection inside another program's loop: caller-owned device buffers, ragged grid, FP64
        dict(name="noalloc_ragged", kind="noalloc", nx=93, ny=70, nz=101, h=0.4e-3, tol=1e-8),
        # the benchmark's own workload (12 inclusions, tuned tile, projection and steps), a quarter of its steps
        sim("inclusions_256", nx=256, ny=256, nz=256, medium="spheres", steps=1000, push_steps=6, tuned=True),
        # the homogeneous elastography phantom on its 240 x 200 x 200 grid, default tuning, all components recorded
        sim("phantom_240", nx=240, ny=200, nz=200, steps=400, push_steps=10, comp=3),
        # steps of a transcranial-like run: rows longer than a tile, layers of strong contrast, peak maps and probes
        sim("skull_384", nx=384, ny=320, nz=352, h=0.2e-3, medium="layers", steps=120, push_steps=20, project=False,
            peaks=True),
        # one epoch of a time-varying force: new pattern, flexible PCG with the network, ten steps with force
        sim("epoch_320", nx=320, ny=320, nz=256, h=0.2e-3, medium="smooth", steps=10, push_steps=10, source="epoch",
            fixed_iters=20),
        # wave-speed validation: curl-based start in a lossless medium, Dirichlet walls, FP32 at its 181^3 size
        sim("curl_181", nx=181, ny=181, nz=181, h=0.2e-3, viscous=False, steps=400, push_steps=0, sponge=0,
            source="curl"),
        # absorbing layer around an inclusion medium, ragged grid
        sim("layer_190", nx=190, ny=161, nz=175, medium="spheres", steps=150, push_steps=8, sponge=0, pml=10,
            project=False),
        # parameter sweep: instances of several sizes advanced together, one projection per distinct grid
        dict(name="sweep_24", kind="batch", count=24, edges="64,96,128,160", steps=300, tol=1e-8),
        # one-dimensional Kelvin-Voigt sweep: 16 viscosities, long harmonic drive
        dict(name="lines_16", kind="lines", count=16, nx=301, steps=16000),
        # radiation force from acoustic samples, strain maps, projection and a short run
        dict(name="arf_160", kind="arf", nx=160, ny=144, nz=208, h=0.2e-3, samples=24, per_call=8, steps=100, tol=1e-8),
        # one optimiser step of the learned preconditioner over a small sample set (forward and backward)
        dict(name="train_64", kind="train", n=64, samples=6),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the same ranges: sizes over their logarithm, odd ones included."""
    pick = rng.choice(["push64", "noalloc", "hetero", "uniform", "wide", "epoch", "curl", "layer", "batch", "lines", "arf",
                       "train"])
    if pick == "push64":
        return {**SIM, "nx": _log(rng, 24, 96), "ny": _log(rng, 24, 96), "nz": _log(rng, 24, 96), "h": 0.5e-3, "fp64": True,
                "viscous": rng.random() < 0.5, "steps": _log(rng, 50, 200), "push_steps": rng.randint(1, 6),
                "tol": rng.choice([1e-8, 1e-10]), "state": True}
    if pick == "noalloc":
        return {"kind": "noalloc", "nx": _log(rng, 20, 120), "ny": _log(rng, 20, 120), "nz": _log(rng, 20, 120),
                "h": 0.4e-3, "tol": rng.choice([1e-6, 1e-8])}
    if pick == "hetero":
        return {**SIM, "nx": _log(rng, 48, 256), "ny": _log(rng, 48, 256), "nz": _log(rng, 48, 256), "medium": "spheres",
                "steps": _log(rng, 100, 600), "push_steps": rng.randint(2, 12), "tuned": rng.random() < 0.5,
                "comp": rng.choice([2, 2, 3])}
    if pick == "uniform":
        return {**SIM, "nx": _log(rng, 48, 256), "ny": _log(rng, 48, 256), "nz": _log(rng, 48, 256),
                "steps": _log(rng, 100, 600), "push_steps": rng.randint(2, 12), "comp": rng.choice([2, 3])}
    if pick == "wide":
        return {**SIM, "nx": _log(rng, 257, 448), "ny": _log(rng, 64, 320), "nz": _log(rng, 64, 320), "h": 0.2e-3,
                "medium": rng.choice(["layers", "uniform"]), "steps": _log(rng, 40, 120), "push_steps": rng.randint(4, 24),
                "project": False, "peaks": rng.random() < 0.6}
    if pick == "epoch":
        return {**SIM, "nx": _log(rng, 96, 320), "ny": _log(rng, 96, 320), "nz": _log(rng, 96, 256), "h": 0.2e-3,
                "medium": "smooth", "steps": 10, "push_steps": 10, "source": "epoch", "fixed_iters": rng.randint(8, 20)}
    if pick == "curl":
        return {**SIM, "nx": _log(rng, 61, 181), "ny": _log(rng, 61, 181), "nz": _log(rng, 61, 181), "h": 0.2e-3,
                "fp64": rng.random() < 0.4, "viscous": False, "steps": _log(rng, 100, 400), "push_steps": 0, "sponge": 0,
                "source": "curl"}
    if pick == "layer":
        return {**SIM, "nx": _log(rng, 64, 200), "ny": _log(rng, 64, 200), "nz": _log(rng, 64, 200), "medium": "spheres",
                "steps": _log(rng, 50, 150), "push_steps": rng.randint(2, 8), "sponge": 0, "pml": rng.randint(6, 12),
                "project": False}
    if pick == "batch":
        edges = ",".join(str(_log(rng, 48, 160)) for _ in range(rng.randint(2, 4)))
        return {"kind": "batch", "count": rng.randint(4, 24), "edges": edges, "steps": _log(rng, 100, 300), "tol": 1e-8}
    if pick == "lines":
        return {"kind": "lines", "count": rng.randint(4, 32), "nx": _log(rng, 101, 401), "steps": _log(rng, 2000, 16000)}
    if pick == "arf":
        return {"kind": "arf", "nx": _log(rng, 64, 176), "ny": _log(rng, 64, 160), "nz": _log(rng, 64, 208), "h": 0.2e-3,
                "samples": 8 * rng.randint(1, 3), "per_call": 8, "steps": _log(rng, 40, 100), "tol": 1e-8}
    return {"kind": "train", "n": rng.choice([32, 40, 48, 56, 64]), "samples": rng.randint(2, 6)}


# ---- inputs ---------------------------------------------------------------------------------------------------


def _axes(case):
    """Node coordinates [m] from the centre node, x, y, z."""
    return [(np.arange(n) - n // 2) * case["h"] for n in (case["nx"], case["ny"], case["nz"])]


def _grid(case):
    return (case["nx"], case["ny"], case["nz"], case["h"], case["h"], case["h"])


def _medium(case, seed):
    """(G, rho, eta): floats for a uniform medium, else [nz][ny][nx] arrays."""
    rng = np.random.default_rng(seed)
    visc = 1.0 if case.get("viscous", True) else 0.0
    if case.get("medium", "uniform") == "uniform":
        return float(rng.uniform(1.5e3, 8e3)), 1000.0, visc * float(rng.uniform(0.3, 1.2))
    x, y, z = _axes(case)
    shape = (len(z), len(y), len(x))
    if case["medium"] == "smooth":
        def wave(a):
            return np.cos(2 * np.pi * a / rng.uniform(4e-3, 12e-3) + rng.uniform(0, 6.28))

        f = (wave(z)[:, None] + wave(y)[None, :])[:, :, None] + wave(x)[None, None, :]
        return 3e3 + 8e2 * f, np.full(shape, 1000.0), visc * (0.75 + 0.2 * f)
    if case["medium"] == "layers":  # a stiff curved sheet over soft tissue
        G, rho, eta = (np.full(shape, v) for v in (1.5e3, 1040.0, visc * 0.8))
        top = z[0] + rng.uniform(0.15, 0.3) * (z[-1] - z[0])
        d = z[:, None, None] - (top + (x[None, None, :] ** 2 + y[None, :, None] ** 2) / 0.14)
        m = (d >= 0) & (d <= rng.uniform(3e-3, 6e-3))
        G[m], rho[m], eta[m] = 1e5, 1900.0, visc * 2.0
        return G, rho, eta
    G, rho, eta = (np.full(shape, v) for v in (2e3, 1000.0, visc * 0.5))  # 12 spherical inclusions
    for _ in range(12):
        c = [rng.uniform(a[0], a[-1]) for a in (x, y, z)]
        r = rng.uniform(1.5e-3, 5e-3)
        box = [np.flatnonzero(np.abs(a - b) <= r) for a, b in zip((x, y, z), c)]
        if any(b.size == 0 for b in box):
            continue
        s = tuple(slice(b[0], b[-1] + 1) for b in box[::-1])
        m = ((z[s[0]] - c[2])[:, None, None] ** 2 + (y[s[1]] - c[1])[None, :, None] ** 2
             + (x[s[2]] - c[0])[None, None, :] ** 2) <= r * r
        G[s][m], rho[s][m], eta[s][m] = rng.uniform(1e3, 1e4), rng.uniform(1000, 1100), visc * rng.uniform(0, 1.5)
    return G, rho, eta


def _push(case, seed):
    """Parameters of the focused Gaussian push (kvs_set_force_pattern)."""
    rng = np.random.default_rng([seed, 1])
    ext = [a[-1] - a[0] for a in _axes(case)]
    p = dict(axis=2, F0=1e4, centre=tuple(float(rng.uniform(-0.1, 0.1) * e) for e in ext),
             sigma_lateral=1e-3, sigma_axial=4e-3)
    if case.get("source") == "epoch":
        k = rng.standard_normal((8, 3))
        k *= (rng.uniform(2 * np.pi / 4e-3, 2 * np.pi / 1e-3, 8) / np.linalg.norm(k, axis=1))[:, None]
        p.update(k=k, phase=rng.uniform(0, 2 * np.pi, 8), mod_amp=0.5 / math.sqrt(8))
    return p


def _push_field(case, seed):
    """The same push as a [3][nz][ny][nx] FP64 device tensor."""
    p = _push(case, seed)
    x, y, z = (torch.from_numpy(a - c).to(DEV) for a, c in zip(_axes(case), p["centre"]))
    lat = torch.exp(-y[:, None] ** 2 / (2 * p["sigma_lateral"] ** 2) - x[None, :] ** 2 / (2 * p["sigma_lateral"] ** 2))
    F = torch.zeros((3, len(z), len(y), len(x)), dtype=torch.float64, device=DEV)
    F[2] = p["F0"] * torch.exp(-z ** 2 / (2 * p["sigma_axial"] ** 2))[:, None, None] * lat
    return F


def _curl_potential(case, seed):
    rng = np.random.default_rng([seed, 2])
    x, y, z = _axes(case)
    s, amp = 3e-3, 1e-6 * rng.uniform(0.5, 2.0)
    A = np.zeros((3, len(z), len(y), len(x)))
    A[1] = amp * np.exp(-z ** 2 / (2 * s * s))[:, None, None] * np.exp(-x ** 2 / (2 * s * s))[None, None, :]
    return A


def _line_probes(case):
    """The lateral line through the centre, as (i, j, k)."""
    return np.array([[i, case["ny"] // 2, case["nz"] // 2] for i in range(case["nx"])], dtype=np.int64)


def _planes(case):
    return [(0, case["nx"] // 2), (1, case["ny"] // 2), (2, case["nz"] // 2)]


def _envelope(case):
    return np.ones(case["push_steps"])


def _net(seed):
    net = kvs.kvs_unet_create()
    train.init_weights(net, np.random.default_rng([seed, 3]))
    return net


class Handles(dict):
    """A state whose contexts, batches and networks are released with it."""

    def __del__(self):
        for c in self.get("ctx", []):
            kvs.kvs_destroy(c)
        if self.get("batch") is not None:
            kvs.kvs_batch_destroy(self["batch"])
        if self.get("net") is not None:
            kvs.kvs_unet_destroy(self["net"])


def prepare(case, seed):
    return {"sim": _prepare_sim, "noalloc": _prepare_noalloc, "batch": _prepare_batch, "lines": _prepare_lines,
            "arf": _prepare_arf, "train": _prepare_train}[case["kind"]](case, seed)


def _prepare_sim(case, seed):
    S = Handles(case=case)
    ctx = kvs.kvs_create(_grid(case), precision=kvs.KVS_FP64 if case["fp64"] else kvs.KVS_FP32,
                         sponge_cells=case["sponge"])
    S["ctx"] = [ctx]
    G, rho, eta = _medium(case, seed)
    if isinstance(G, float):
        kvs.kvs_set_material_uniform(ctx, G, rho, eta)
    else:
        kvs.kvs_set_material(ctx, G, rho, eta)
    kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
    if case["pml"]:
        kvs.kvs_set_pml(ctx, case["pml"])
    kvs.kvs_set_envelope(ctx, _envelope(case))
    kvs.kvs_set_probes(ctx, _line_probes(case), case["comp"])
    if case["tuned"]:
        kvs.kvs_autotune_step(ctx, 10)
    if case["source"] == "curl":
        S["A"] = _curl_potential(case, seed)
    elif case["source"] == "epoch":
        S["pattern"] = _push(case, seed)
        S["net"] = _net(seed)
        kvs.kvs_set_preconditioner(ctx, S["net"])
    else:
        S["F"] = _push_field(case, seed)
        torch.cuda.synchronize()
        kvs.kvs_set_force_device(ctx, S["F"].data_ptr(), 0)
        if not case["project"]:
            kvs.kvs_project(ctx, tol=case["tol"], max_iter=20000)
    if case["peaks"]:
        kvs.kvs_set_peak_planes(ctx, _planes(case))
    return S


def _prepare_noalloc(case, seed):
    F = _push_field(case, seed)
    # a modulated push: sources on every scale of the grid
    g = torch.Generator(device=DEV).manual_seed(seed)
    F *= 1 + 0.2 * torch.randn(F.shape, generator=g, dtype=F.dtype, device=DEV)
    return dict(case=case, F=F, phi=torch.zeros_like(F[0]), FS=torch.zeros_like(F))


def _batch_cases(case, seed):
    rng = np.random.default_rng([seed, 4])
    edges = [int(e) for e in case["edges"].split(",")]
    out = []
    for i in range(case["count"]):
        n = edges[i % len(edges)]
        out.append(dict(nx=n, ny=n, nz=n, h=0.25e-3, G=float(10.0 ** (3 + rng.integers(0, 10) / 9)), rho=1000.0,
                        eta=float(0.1 * rng.integers(0, 16))))
    return out


def _prepare_batch(case, seed):
    inst = _batch_cases(case, seed)
    S = Handles(case=case, inst=inst)
    b = S["batch"] = kvs.kvs_batch_create([_grid(c) for c in inst], precision=kvs.KVS_FP32, sponge_cells=8)
    first = S["first"] = {}
    for i, c in enumerate(inst):
        ctx = kvs.kvs_batch_instance(b, i)
        kvs.kvs_set_material_uniform(ctx, c["G"], c["rho"], c["eta"])
        dt = 0.4 * kvs.kvs_stable_dt(ctx)
        kvs.kvs_set_dt(ctx, dt)
        kvs.kvs_set_envelope(ctx, np.ones(int(round(100e-6 / dt))))
        kvs.kvs_batch_set_probes(b, i, _line_probes(c))
        first.setdefault(c["nx"], i)
    S["F"] = {n: _push_field(inst[i], seed) for n, i in first.items()}
    kvs.kvs_batch_set_component(b, 2)
    torch.cuda.synchronize()
    return S


def _line_inputs(case, seed):
    rng = np.random.default_rng([seed, 5])
    n = case["count"]
    h, G, rho = 0.1e-3, 4e3, 1000.0
    eta = 1.5 * np.arange(n) / max(1, n - 1)
    S = 1 / h ** 2 + 2e-12
    qa, qb = G / rho * S, 2 * eta.max() / rho * S
    dt = 0.3 * (-qb + math.sqrt(qb * qb + 4 * qa)) / (2 * qa)
    t = np.arange(case["steps"]) * dt
    env = []
    for f in rng.uniform(740.0, 800.0, n):
        r = np.minimum(1.0, t * f / 2)
        env.append(0.5 * (1 - np.cos(np.pi * r)) * np.sin(2 * np.pi * f * t))
    return h, G, rho, eta, dt, env


def _prepare_lines(case, seed):
    h, G, rho, eta, dt, env = _line_inputs(case, seed)
    S = Handles(case=case)
    b = S["batch"] = kvs.kvs_batch_create([(case["nx"], 3, 3, h, 1e6, 1e6)] * case["count"], precision=kvs.KVS_FP32)
    FS = np.zeros((3, 3, 3, case["nx"]))
    FS[2, 1, 1, 1] = 1e4
    S["np"] = len(range(6, case["nx"] - 1, 16))
    for i in range(case["count"]):
        ctx = kvs.kvs_batch_instance(b, i)
        kvs.kvs_set_material_uniform(ctx, G, rho, float(eta[i]))
        kvs.kvs_set_dt(ctx, dt)
        kvs.kvs_set_envelope(ctx, env[i])
        kvs.kvs_set_projected_force(ctx, FS)
        kvs.kvs_batch_set_probes(b, i, [[x, 1, 1] for x in range(6, case["nx"] - 1, 16)])
    kvs.kvs_batch_set_component(b, 2)
    return S


ARF = dict(alpha=5.8, c=1540.0, K=1000.0 * 1540.0 ** 2)


def _samples(case, seed):
    """p [samples][N], v [samples][3][N] (FP32): a focused tone burst with speckle, drawn on the device."""
    x, y, z = (torch.from_numpy(a).to(DEV, torch.float32) for a in _axes(case))
    g = torch.Generator(device=DEV).manual_seed(seed)
    amp = 1.5e6 * torch.exp(-(y[:, None] ** 2 + x[None, :] ** 2) / (2 * 2e-3 ** 2))[None] \
        * torch.exp(-(z - 0.1 * z[-1]) ** 2 / (2 * 8e-3 ** 2))[:, None, None]
    amp = amp * (1 + 0.1 * torch.randn(amp.shape, generator=g, device=DEV))
    ph = 2 * math.pi * 1e6 / 1540.0 * z[:, None, None] + 0.2 * torch.randn(amp.shape, generator=g, device=DEV)
    p = torch.empty((case["samples"],) + tuple(amp.shape), device=DEV)
    v = torch.empty((case["samples"], 3) + tuple(amp.shape), device=DEV)
    for s in range(case["samples"]):
        p[s] = amp * torch.sin(2 * math.pi * s / 20 - ph)
        v[s, 2] = p[s] / (1000.0 * 1540.0)
        v[s, 0] = v[s, 2] * (x / 30e-3)[None, None, :]
        v[s, 1] = v[s, 2] * (y / 30e-3)[None, :, None]
    return p, v


def _arf_mask(case):
    m = np.ones((case["nz"], case["ny"], case["nx"]), dtype=np.uint8)
    m[: case["nz"] // 8] = 0
    return m


def _prepare_arf(case, seed):
    S = Handles(case=case)
    ctx = kvs.kvs_create(_grid(case), precision=kvs.KVS_FP32, sponge_cells=8)
    S["ctx"] = [ctx]
    S["p"], S["v"] = _samples(case, seed)
    S["mask"] = _arf_mask(case)
    kvs.kvs_set_material_uniform(ctx, *_medium(case, seed))
    kvs.kvs_set_dt(ctx, 0.4 * kvs.kvs_stable_dt(ctx))
    kvs.kvs_set_envelope(ctx, np.ones(12))
    kvs.kvs_set_probes(ctx, _line_probes(case), 2)
    torch.cuda.synchronize()
    return S


def _prepare_train(case, seed):
    n = case["n"]
    S = Handles(case=case)
    S["net"] = _net(seed)
    S["w0"] = kvs.kvs_unet_get_weights(S["net"])
    g = torch.Generator(device=DEV).manual_seed(seed)
    S["pairs"] = []
    ax = torch.arange(n, dtype=torch.float64, device=DEV) / n
    for q in range(case["samples"]):
        x = torch.zeros((n, n, n), dtype=torch.float64, device=DEV)
        if q % 2:
            f = torch.randn((n - 2,) * 3, generator=g, dtype=torch.float64, device=DEV)
        else:
            c = torch.rand(3, generator=g, dtype=torch.float64, device=DEV)
            e = [torch.exp(-(ax[1:-1] - c[a]) ** 2 / (2 * 0.1 ** 2)) for a in range(3)]
            f = e[0][:, None, None] * e[1][None, :, None] * e[2][None, None, :]
        x[1:-1, 1:-1, 1:-1] = f
        b = torch.zeros_like(x)
        torch.cuda.synchronize()
        kvs.kvs_unet_sample_from_x(x.data_ptr(), b.data_ptr(), (n, n, n))
        S["pairs"].append((b, x))
    torch.cuda.synchronize()
    return S


# ---- one pass --------------------------------------------------------------------------------------------------


def _state_type(case, a):
    """Values of an FP32 state, read back as doubles, are kept as the floats that they are."""
    return a if case.get("fp64") else a.astype(np.float32)


def run(S):
    return {"sim": _run_sim, "noalloc": _run_noalloc, "batch": _run_batch, "lines": _run_lines, "arf": _run_arf,
            "train": _run_train}[S["case"]["kind"]](S)


def _run_sim(S):
    case, ctx = S["case"], S["ctx"][0]
    kvs.kvs_reset_state(ctx)
    if case["source"] == "curl":
        kvs.kvs_set_state_curl(ctx, S["A"])
    elif case["source"] == "epoch":
        kvs.kvs_set_force_pattern(ctx, **S["pattern"])
        kvs.kvs_project(ctx, precond=kvs.KVS_PC_UNET, fixed_iters=case["fixed_iters"])
    elif case["project"]:
        kvs.kvs_set_force_device(ctx, S["F"].data_ptr(), 0)
        kvs.kvs_project(ctx, tol=case["tol"], max_iter=20000)
    kvs.kvs_step(ctx, case["steps"])
    out = {"traces": _state_type(case, kvs.kvs_read_traces(ctx, case["nx"], 3 if case["comp"] == 3 else 1))}
    if case["peaks"]:
        out["peaks"] = [_state_type(case, kvs.kvs_peak_map(ctx, a, i, _grid(case))) for a, i in _planes(case)]
    if case["state"]:
        out["u"], out["w"], _ = kvs.kvs_get_state(ctx, (case["nz"], case["ny"], case["nx"]))
    return out


def _run_noalloc(S):
    c = S["case"]
    kvs.kvs_project_noalloc(_grid(c), S["F"].data_ptr(), S["phi"].data_ptr(), S["FS"].data_ptr(), tol=c["tol"],
                            stream=torch.cuda.current_stream().cuda_stream)
    return {"phi": S["phi"], "FS": S["FS"]}


def _run_batch(S):
    case, b = S["case"], S["batch"]
    kvs.kvs_batch_reset(b)
    for n, i in S["first"].items():
        ctx = kvs.kvs_batch_instance(b, i)
        kvs.kvs_set_force_device(ctx, S["F"][n].data_ptr(), 0)
        kvs.kvs_project(ctx, tol=case["tol"])
    for i, c in enumerate(S["inst"]):
        if S["first"][c["nx"]] != i:
            kvs.kvs_batch_share_projection(b, S["first"][c["nx"]], i)
    kvs.kvs_batch_step(b, case["steps"])
    return [_state_type(case, kvs.kvs_batch_read_traces(b, i, c["nx"])) for i, c in enumerate(S["inst"])]


def _run_lines(S):
    case, b = S["case"], S["batch"]
    kvs.kvs_batch_reset(b)
    kvs.kvs_batch_step(b, case["steps"])
    return [_state_type(case, kvs.kvs_batch_read_traces(b, i, S["np"])) for i in range(case["count"])]


def _run_arf(S):
    case, ctx = S["case"], S["ctx"][0]
    shape = (case["nz"], case["ny"], case["nx"])
    kvs.kvs_reset_state(ctx)
    kvs.kvs_arf_begin(ctx, kvs.KVS_ARF_POYNTING)
    kvs.kvs_strain_begin(ctx, ARF["K"])
    for s in range(0, case["samples"], case["per_call"]):
        kvs.kvs_arf_accumulate_device(ctx, S["p"][s].data_ptr(), S["v"][s].data_ptr(), case["per_call"], 1)
        kvs.kvs_strain_accumulate_device(ctx, S["p"][s].data_ptr(), case["per_call"], 1)
    kvs.kvs_arf_set_force(ctx, ARF["alpha"], ARF["c"], case["samples"], mask=S["mask"])
    kvs.kvs_project(ctx, tol=case["tol"])
    kvs.kvs_step(ctx, case["steps"])
    eps, grad, _ = kvs.kvs_strain_get(ctx, shape)
    return {"traces": _state_type(case, kvs.kvs_read_traces(ctx, case["nx"], 1)), "strain": eps, "gradient": grad}


def _run_train(S):
    n, net = S["case"]["n"], S["net"]
    kvs.kvs_unet_set_weights(net, S["w0"])
    loss = [kvs.kvs_unet_train_sample(net, b.data_ptr(), x.data_ptr(), (n, n, n), q > 0)
            for q, (b, x) in enumerate(S["pairs"])]
    grad = kvs.kvs_unet_get_grad(net)
    kvs.kvs_unet_adam_step(net, 1e-3, len(S["pairs"]))
    return {"loss": np.array(loss, dtype=np.float32), "grad": grad, "weights": kvs.kvs_unet_get_weights(net)}


# ---- what a pass cannot do without -------------------------------------------------------------------------------

STEP_FLOPS = {True: 147, False: 90}  # a viscous and a lossless cell-update, an FMA counted as two
CG_FLOPS = 30                        # per cell and iteration: two stencils, three updates, two sums


def _cg_iters(case):
    """Iterations of CG to the tolerance: about 3.2 per node of the longest edge at 1e-8."""
    return 0.4 * max(case["nx"], case["ny"], case["nz"]) * -math.log10(case["tol"])


def work(case):
    """State read and written once per step (u, w), the medium's maps read once per step; the potential solve's
    potential, residual and direction read and written once per iteration."""
    k = case["kind"]
    if k == "batch":
        inst = _batch_cases(case, 0)
        cells = sum(float(c["nx"]) ** 3 for c in inst)
        edges = {c["nx"]: float(c["nx"]) ** 3 for c in inst}
        its = {n: 3.2 * n for n in edges}
        return {"bytes": 48.0 * cells * case["steps"] + sum(32.0 * edges[n] * its[n] for n in edges),
                "flops": STEP_FLOPS[True] * cells * case["steps"] + sum(CG_FLOPS * edges[n] * its[n] for n in edges)}
    if k == "lines":
        cells = float(case["count"]) * (case["nx"] - 2)
        return {"bytes": 8.0 * case["count"] * case["steps"], "flops": STEP_FLOPS[True] * cells * case["steps"]}
    if k == "train":
        n3 = float(case["n"]) ** 3
        # three convolutions' worth per layer (forward, input and weight gradients), 27 taps
        mac = 27 * (16 + 16 * 32 / 8 + (32 * 64 + 2 * 64 * 64 + 64 * 32) / 64 + 32 * 16 / 8 + 16)
        return {"bytes": case["samples"] * 3 * 8.0 * n3, "flops": case["samples"] * 6.0 * mac * n3}
    cells = float(case["nx"]) * case["ny"] * case["nz"]
    if k == "noalloc":
        return {"bytes": 8.0 * cells * 7, "flops": CG_FLOPS * cells * _cg_iters(case)}
    word = 8.0 if case.get("fp64") else 4.0
    steps = case["steps"]
    maps = 0 if case.get("medium", "uniform") == "uniform" else 3
    flops = STEP_FLOPS[bool(case.get("viscous", True))] * cells * steps
    moved = word * (12 + maps) * cells * steps + 3 * word * cells * case.get("push_steps", 12)
    if k == "arf":
        moved += case["samples"] * 16.0 * cells
    if k == "arf" or (case["project"] and case["source"] == "push"):
        moved += (16.0 + 4 * word) * cells * _cg_iters(case)
        flops += CG_FLOPS * cells * _cg_iters(case)
    if case.get("source") == "epoch":
        mac = 27 * (16 + 16 * 32 / 8 + (32 * 64 + 2 * 64 * 64 + 64 * 32) / 64 + 32 * 16 / 8 + 16)
        moved += 32.0 * cells * case["fixed_iters"]
        flops += (CG_FLOPS + 2 * mac) * cells * case["fixed_iters"]
    return {"bytes": moved, "flops": flops}


# ---- 64-bit values ------------------------------------------------------------------------------------------------


def _project_exact(F, h):
    """F_S and phi of F [3][nz][ny][nx] (equal spacings h) with the discrete sine transform as matrices."""
    b = torch.zeros_like(F[0])
    inner = (slice(1, -1),) * 3
    for a, dim in ((0, 2), (1, 1), (2, 0)):
        b += (torch.roll(F[a], -1, dim) - torch.roll(F[a], 1, dim)) / (2 * h)
    r, lam = b[inner].contiguous(), 0.0
    S = []
    for dim in range(3):
        n = r.shape[dim]
        q = torch.arange(1, n + 1, dtype=torch.float64, device=F.device)
        S.append(math.sqrt(2 / (n + 1)) * torch.sin(math.pi / (n + 1) * q[:, None] * q[None, :]))
        e = -(2 - 2 * torch.cos(math.pi * q / (n + 1))) / h ** 2
        lam = lam + e.reshape([-1 if d == dim else 1 for d in range(3)])

    def dst(v):
        for dim in range(3):
            v = v.movedim(dim, 2).contiguous()
            v = (v.reshape(-1, v.shape[2]) @ S[dim]).reshape(v.shape).movedim(2, dim)
        return v

    phi = torch.zeros_like(b)
    phi[inner] = dst(dst(r) / lam)
    FS = torch.zeros_like(F)
    for a, dim in ((0, 2), (1, 1), (2, 0)):
        v = 0.25 * (torch.roll(F[a], 1, dim) + 2 * F[a] + torch.roll(F[a], -1, dim)) \
            - (torch.roll(phi, -1, dim) - torch.roll(phi, 1, dim)) / (2 * h)
        FS[a][inner] = v[inner]
    return FS, phi


def _stable_dt(G, rho, eta, h):
    S = 3 / h ** 2
    if isinstance(G, float):
        qa, qb = G / rho * S, 2 * eta / rho * S
        return (-qb + math.sqrt(qb * qb + 4 * qa)) / (2 * qa)
    g = torch.zeros_like(G[1:-1, 1:-1, 1:-1])
    c = G[1:-1, 1:-1, 1:-1]
    for dim in range(3):
        for s in (1, -1):
            o = torch.roll(G, s, dim)[1:-1, 1:-1, 1:-1]
            g = torch.maximum(g, 2 * c * o / (c + o))
    inner = (slice(1, -1),) * 3
    qa, qb = g / rho[inner] * S, 2 * eta[inner] / rho[inner] * S
    return float(((-qb + torch.sqrt(qb * qb + 4 * qa)) / (2 * qa)).min())


def _run_exact(case, medium, FS, env, u=None, w=None, dt=None):
    """Traces, peak maps (or None) and final (u, w) of the leapfrog of the package's documentation in FP64."""
    G, rho, eta = medium
    h, L = case["h"], case.get("sponge", 8)
    shape = (case["nz"], case["ny"], case["nx"])
    if not isinstance(G, float):
        G, rho, eta = (torch.from_numpy(a).to(DEV) for a in (G, rho, eta))
    dt = 0.4 * _stable_dt(G, rho, eta, h) if dt is None else dt
    inner = (slice(None),) + (slice(1, -1),) * 3
    shifts = [(1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1)]

    def at(f, s):
        return f[(slice(None),) + tuple(slice(1 + d, f.shape[1 + q] - 1 + d) for q, d in enumerate(s))]

    if isinstance(G, float):
        face, r, e = [G / h ** 2] * 6, rho, eta
        cmax = math.sqrt(G / rho)
    else:
        c = G[None][inner]
        face = [2 * c * at(G[None], s) / (c + at(G[None], s)) / h ** 2 for s in shifts]
        r, e = rho[None][inner], eta[None][inner]
        cmax = float(torch.sqrt(G / rho).max())
    s = 0.0
    if L:
        ramps = []
        for n in shape:
            i = torch.arange(n, dtype=torch.float64, device=DEV)
            ramps.append(torch.clamp(L - torch.minimum(i, n - 1 - i), min=0)[1:-1] / L)
        rmp = torch.maximum(torch.maximum(ramps[0][:, None, None], ramps[1][None, :, None]), ramps[2][None, None, :])
        s = 0.5 * dt * 6 * math.log(10) * cmax / (L * h) * rmp[None]
    a1, a2 = (1 - s) / (1 + s), dt * dt / r / (1 + s)
    u = torch.zeros((3,) + shape, dtype=torch.float64, device=DEV) if u is None else u
    w = torch.zeros_like(u) if w is None else w
    j, k = case["ny"] // 2, case["nz"] // 2
    comp = [0, 1, 2] if case.get("comp", 2) == 3 else [case.get("comp", 2)]
    traces, peaks = [], None
    if case.get("peaks"):
        cut = [(slice(None),) + tuple(i if 2 - a == d else slice(None) for d in range(3)) for a, i in _planes(case)]
        peaks = [torch.zeros_like(u[c][0]) for c in cut]
    visc = not (isinstance(eta, float) and eta == 0.0)
    for n in range(case["steps"]):
        uc, wc = u[inner], w[inner]
        acc = torch.zeros_like(uc)
        for f, sh in zip(face, shifts):
            acc += f * (at(u, sh) - uc)
        if visc:
            lw = -6 * wc
            for sh in shifts:
                lw += at(w, sh)
            acc += (e / (dt * h ** 2)) * lw
        if n < len(env) and env[n] != 0.0:
            acc += env[n] * FS[inner]
        new = a1 * wc + a2 * acc
        w = torch.zeros_like(w)
        w[inner] = new
        u = u + w
        traces.append(torch.stack([u[c, k, j] for c in comp], dim=-1))
        if peaks is not None:
            peaks = [torch.maximum(p, u[c].square().sum(0).sqrt()) for p, c in zip(peaks, cut)]
    tr = torch.stack(traces).cpu().numpy()
    return tr, None if peaks is None else [p.cpu().numpy() for p in peaks], (u, w)


def _curl_state(case, seed, dt):
    A = torch.from_numpy(_curl_potential(case, seed)).to(DEV)

    def d(f, dim):
        return (torch.roll(f, -1, dim) - torch.roll(f, 1, dim)) / (2 * case["h"])

    v = torch.stack([d(A[2], 1) - d(A[1], 0), d(A[0], 0) - d(A[2], 2), d(A[1], 2) - d(A[0], 1)])
    w = torch.zeros_like(v)
    inner = (slice(None),) + (slice(1, -1),) * 3
    w[inner] = dt * v[inner]
    return w


def exact(case, seed):
    k = case["kind"]
    if k == "train":
        return None  # the network's own arithmetic is BF16 with FP32 sums
    if k == "lines":
        return _lines_exact(case, seed)
    if k == "batch":
        return _batch_exact(case, seed)
    cells = case["nx"] * case["ny"] * case["nz"]
    if k == "noalloc":
        FS, phi = _project_exact(_prepare_noalloc(case, seed)["F"], case["h"])
        return {"phi": phi, "FS": FS}
    if cells * case["steps"] > 1.8e10 or case.get("pml") or case.get("source") == "epoch":
        return None  # too long, or (layer, unconverged network solve) without a short plain form
    if k == "arf":
        return _arf_exact(case, seed)
    medium = _medium(case, seed)
    if case["source"] == "curl":
        dt = 0.4 * _stable_dt(*medium, case["h"])
        tr, pk, st = _run_exact(case, medium, None, [], w=_curl_state(case, seed, dt), dt=dt)
    else:
        FS, _ = _project_exact(_push_field(case, seed), case["h"])
        tr, pk, st = _run_exact(case, medium, FS, _envelope(case))
    out = {"traces": tr}
    if pk is not None:
        out["peaks"] = pk
    if case["state"]:
        out["u"], out["w"] = st
    return out


def _batch_exact(case, seed):
    inst, out = _batch_cases(case, seed), []
    if sum(c["nx"] ** 3 for c in inst) * case["steps"] > 1.8e10:
        return None
    first = {}
    for i, c in enumerate(inst):
        first.setdefault(c["nx"], i)
    FS = {n: _project_exact(_push_field(inst[i], seed), 0.25e-3)[0] for n, i in first.items()}
    for c in inst:
        dt = 0.4 * _stable_dt(c["G"], c["rho"], c["eta"], c["h"])
        one = dict(c, steps=case["steps"], sponge=8)
        tr, _, _ = _run_exact(one, (c["G"], c["rho"], c["eta"]), FS[c["nx"]], np.ones(int(round(100e-6 / dt))))
        out.append(tr[:, :, 0])
    return out


def _lines_exact(case, seed):
    h, G, rho, eta, dt, env = _line_inputs(case, seed)
    e = torch.from_numpy(eta / (dt * h * h))[:, None].to(DEV)
    et = torch.from_numpy(eta / dt * 2e-12)[:, None].to(DEV)
    g = torch.from_numpy(np.stack(env)).to(DEV)
    u = torch.zeros((case["count"], case["nx"]), dtype=torch.float64, device=DEV)
    w, a2, rows = torch.zeros_like(u), dt * dt / rho, []
    for n in range(case["steps"]):
        uc, wc = u[:, 1:-1], w[:, 1:-1]
        acc = (u[:, 2:] + u[:, :-2] - 2 * uc) * (G / h ** 2) - 4e-12 * G * uc + (w[:, 2:] + w[:, :-2] - 2 * wc) * e \
            - 2 * et * wc
        acc[:, 0] += 1e4 * g[:, n]
        w[:, 1:-1] = wc + a2 * acc
        u = u + w
        rows.append(u[:, 6:-1:16])
    return list(torch.stack(rows, dim=1).cpu().numpy())


def _arf_exact(case, seed):
    p, v = _samples(case, seed)
    F = torch.zeros((3, case["nz"], case["ny"], case["nx"]), dtype=torch.float64, device=DEV)
    K, h = ARF["K"], case["h"]
    eps = torch.zeros_like(F[0])
    grad = torch.zeros_like(eps)
    inner = (slice(1, -1),) * 3
    for s in range(case["samples"]):
        q = p[s].double()
        F += q[None] * v[s].double()
        st = -q / K
        eps = torch.maximum(eps, st.abs())
        g2 = sum(((torch.roll(st, -1, d) - torch.roll(st, 1, d)) / (2 * h)).square() for d in range(3))
        grad[inner] = torch.maximum(grad[inner], g2.sqrt()[inner])
    F *= 2 * ARF["alpha"] / ARF["c"] / case["samples"]
    F *= torch.from_numpy(_arf_mask(case)).to(DEV)
    FS, _ = _project_exact(F, h)
    tr, _, _ = _run_exact(dict(case, sponge=8), _medium(case, seed), FS, np.ones(12))
    return {"traces": tr, "strain": eps, "gradient": grad}
