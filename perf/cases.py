"""Timed cases of the droplet boxes, their analysis and the shape surrogate.

``listed()`` names the workloads a user of the library runs, from a single small
validation box to the 64-box ensemble that produces the surrogate's training
data; ``draw`` gives further cases of the same ranges.  ``prepare`` builds what a
program holds before the call (context, gradient history, network, inputs made
on the GPU from a seed), ``run`` makes one pass through the public calls,
``work`` counts the bytes and operations a pass cannot do without, and ``exact``
computes the same outputs in plain FP64.
"""
from __future__ import annotations

import math

import numpy as np
import torch

DEV = "cuda:0"

# Model constants of the boxes (tau = 1 for both components): coupling, initial
# densities and interface width, surface tension, and the ghost densities in
# equilibrium with a droplet of radius R.
G_AB = 1.6417
RHO_HI, RHO_LO, WIDTH = 1.0, 0.04, 2.0
SIGMA = 0.089909
MACH = 0.2
CS = 1.0 / math.sqrt(3.0)
STRIDE = 50              # lattice steps between samples of A(t)
TABLE = 2000             # rows of a box's gradient history (repeated when it runs out)

CV = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0), (-1, -1, 0),
      (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1),
      (0, -1, 1)]
WT = [1.0 / 3.0] + [1.0 / 18.0] * 6 + [1.0 / 36.0] * 12

POP_BYTES = {"f64": 8, "f32": 4, "f32d": 4, "f16dev": 2, "bf16dev": 2}
WIDTHS = (576, 512, 512, 512, 3)
MACS = sum(a * b for a, b in zip(WIDTHS[:-1], WIDTHS[1:]))
NPARAM = MACS + sum(WIDTHS[1:])
TRAIN_ROWS = 18872       # windows of the 56 training trajectories of the 64-box ensemble


def listed():
    return [
        # the 32^3 validation box in steady simple shear: 100 steps, droplet shape and fields; launch-bound
        dict(name="shear_32_f64", kind="boxes", nx=32, ny=32, nz=32, nbox=1, bc="ghost", prec="f64", drive="shear",
             steps=100, graph=False),
        # the 128^3 turbulence-driven box of the benchmark: one sample period, moments, a snapshot of the fields
        dict(name="turbulence_128_f32", kind="boxes", nx=128, ny=128, nz=128, nbox=1, bc="ghost", prec="f32",
             drive="ou", steps=50, graph=False),
        # the 64-box ensemble behind the surrogate: one sample period of the captured loop, moments, densities
        dict(name="ensemble_64x64_f32", kind="boxes", nx=64, ny=64, nz=64, nbox=64, bc="ghost", prec="f32",
             drive="ou", steps=50, graph=True),
        # the 256^3 box of the storage-format study in FP16 deviations
        dict(name="study_256_f16", kind="boxes", nx=256, ny=256, nz=256, nbox=1, bc="ghost", prec="f16dev",
             drive="ou", steps=20, graph=False),
        # an odd box elongated along the flow, BF16 deviations, captured loop
        dict(name="channel_150x93x67_bf16", kind="boxes", nx=150, ny=93, nz=67, nbox=1, bc="ghost", prec="bf16dev",
             drive="shear", steps=50, graph=True),
        # an odd periodic box in FP64 (the stationarity and conservation checks run on such boxes)
        dict(name="periodic_100x120x90_f64", kind="boxes", nx=100, ny=120, nz=90, nbox=1, bc="periodic", prec="f64",
             drive="none", steps=20, graph=False),
        # the analysis of a sample: inertia moments, surface area, droplet mass, velocity error, mass reinjection, fields
        dict(name="analysis_128_f32", kind="analysis", nx=128, ny=128, nz=128, nbox=1, prec="f32"),
        # the Maffettone-Minale baseline over the ensemble's 64 histories of 20,000 steps
        dict(name="mm_64x20001", kind="mm", ntraj=64, nrows=20001, substeps=1, every=50),
        # surrogate inference: a serving batch, and a handful of windows where latency counts
        dict(name="predict_8192", kind="predict", n=8192),
        dict(name="predict_7", kind="predict", n=7),
        # surrogate training: 20 mini-batches with gather and symmetry augmentation, then the weights
        dict(name="train_256", kind="train", batch=256, steps=20),
        # gradients of a large batch (what a data-parallel program all-reduces)
        dict(name="gradients_8192", kind="gradients", n=8192),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["boxes", "boxes", "boxes", "analysis", "mm", "predict", "train", "gradients"])
    if kind == "boxes":
        nx, ny, nz = _log(rng, 20, 260), _log(rng, 20, 200), _log(rng, 20, 200)
        nbox = 1 if rng.random() < 0.5 else max(1, min(64, int(_log(rng, 5e4, 6e6) / (nx * ny * nz))))
        bc = "ghost" if rng.random() < 0.75 else "periodic"
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, nbox=nbox, bc=bc,
                    prec=rng.choice(["f64", "f32", "f32", "f32d", "f16dev", "bf16dev"]),
                    drive="none" if bc == "periodic" else rng.choice(["ou", "shear"]), steps=2 * rng.randint(8, 25),
                    graph=rng.random() < 0.5)
    if kind == "analysis":
        nx, ny, nz = _log(rng, 24, 160), _log(rng, 24, 160), _log(rng, 24, 160)
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, nbox=1 if rng.random() < 0.5 else rng.randint(2, 6),
                    prec=rng.choice(["f64", "f32", "f32", "f16dev", "bf16dev"]))
    if kind == "mm":
        ntraj = _log(rng, 1, 4096)
        return dict(kind=kind, ntraj=ntraj, nrows=rng.randint(200, 4000), substeps=rng.choice([1, 1, 2]),
                    every=rng.choice([1, 10, 50]))
    if kind == "predict":
        return dict(kind=kind, n=_log(rng, 1, 21568))
    if kind == "train":
        return dict(kind=kind, batch=_log(rng, 64, 1024), steps=rng.randint(10, 24))
    return dict(kind=kind, n=_log(rng, 64, 8192))


# ---- inputs, shared by prepare and exact -------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _ou(g, m, nsamp, corr=2000.0):
    """m Ornstein-Uhlenbeck histories of traceless 3x3 gradients, unit variance, one sample every STRIDE steps."""
    decay = math.exp(-STRIDE / corr)
    kick = math.sqrt(1.0 - decay * decay)
    xi = torch.randn((nsamp, m, 3, 3), generator=g, device=DEV, dtype=torch.float64)
    out = torch.empty_like(xi)
    out[0] = xi[0]
    for k in range(1, nsamp):
        out[k] = decay * out[k - 1] + kick * xi[k]
    tr = out.diagonal(dim1=-2, dim2=-1).sum(-1)
    out -= tr[..., None, None] / 3.0 * torch.eye(3, device=DEV, dtype=torch.float64)
    return out.transpose(0, 1)


def _per_step(samples, nrows):
    """Samples (m, ns, 3, 3) held every STRIDE steps -> linear rows (m, nrows, 9)."""
    t = torch.arange(nrows, device=DEV, dtype=torch.float64) / STRIDE
    k = t.floor().long().clamp(max=samples.shape[1] - 2)
    f = (t - k)[None, :, None, None]
    return (samples[:, k] * (1.0 - f) + samples[:, k + 1] * f).reshape(samples.shape[0], nrows, 9)


def _radius(case):
    n = min(case["nx"], case["ny"], case["nz"])
    return max(3.0, n * (10.0 / 64.0 if case["nbox"] > 1 else 0.1875 if n <= 32 else 0.125))


def _rho_b(radius):
    """Densities of A and B in the ghost nodes, in equilibrium with a droplet of this radius."""
    return (0.05375933605501905 / radius + 0.04041950406144379, -0.235900760858221 / radius + 1.0375176769822088)


def _history(case, seed):
    """Gradient rows (nbox, rows, 9) of the boxes, numpy; the peak ghost Mach number is spread over the boxes."""
    g = _gen(seed)
    nb, half = case["nbox"], [(case[a] + 1) / 2.0 for a in ("nx", "ny", "nz")]
    machs = torch.linspace(0.5 * MACH if nb > 1 else MACH, MACH, nb, device=DEV, dtype=torch.float64)
    machs = machs * (0.9 + 0.1 * torch.rand(nb, generator=g, device=DEV, dtype=torch.float64))
    if case["drive"] == "shear":
        raw = torch.zeros((nb, TABLE, 9), device=DEV, dtype=torch.float64)
        raw[:, :, 2] = 1.0
        machs = machs * 0.5
    else:
        raw = _per_step(_ou(g, nb, TABLE // STRIDE + 2), TABLE)
    corners = torch.tensor([[a * half[0], b * half[1], c * half[2]] for a in (-1, 1) for b in (-1, 1) for c in (-1, 1)],
                           device=DEV, dtype=torch.float64)
    speed = (raw.reshape(nb, TABLE, 3, 3) @ corners.T).square().sum(2).sqrt().amax((1, 2))
    return (raw * (machs * CS / speed)[:, None, None]).cpu().numpy()


def _center(case, seed):
    """Droplet centre of each box, off the box centre by less than a node."""
    rng = np.random.default_rng(seed)
    c = np.array([(case[a] - 1) / 2.0 for a in ("nx", "ny", "nz")])
    return c + rng.uniform(-0.4, 0.4, (case["nbox"], 3))


def _grid(case):
    z, y, x = torch.meshgrid(*[torch.arange(case[a], device=DEV, dtype=torch.float64) for a in ("nz", "ny", "nx")],
                             indexing="ij")
    return x, y, z


def _analysis_fields(case, seed):
    """Tilted ellipsoidal droplets in a linear flow with a perturbation: rho_a, rho_b (nbox, nz, ny, nx), u (nbox, 3, ...)
    and the gradients (nbox, 3, 3)."""
    rng = np.random.default_rng(seed)
    x, y, z = _grid(case)
    n = min(case["nx"], case["ny"], case["nz"])
    ra, us, As = [], [], []
    for b in range(case["nbox"]):
        q, _ = np.linalg.qr(rng.standard_normal((3, 3)))
        ax = 0.22 * n * np.array([1.3, 1.0, 0.75]) * rng.uniform(0.9, 1.1, 3)
        A = rng.standard_normal((3, 3))
        A -= np.eye(3) * np.trace(A) / 3
        A *= MACH * CS / (2.0 * np.abs(A).sum(1).max() * max(case["nx"], case["ny"], case["nz"]) / 2)
        c = [(case[a] - 1) / 2.0 + rng.uniform(-0.4, 0.4) for a in ("nx", "ny", "nz")]
        d = torch.stack([x - c[0], y - c[1], z - c[2]])
        e = torch.tensordot(torch.tensor(q, device=DEV), d, 1)
        s = sum((e[i] / float(ax[i])).square() for i in range(3)).sqrt()
        ra.append(0.5 * (RHO_HI + RHO_LO) - 0.5 * (RHO_HI - RHO_LO) * torch.tanh((s - 1.0) * float(ax.min()) / WIDTH))
        dc = torch.stack([x - (case["nx"] - 1) / 2.0, y - (case["ny"] - 1) / 2.0, z - (case["nz"] - 1) / 2.0])
        u = torch.tensordot(torch.tensor(A, device=DEV), dc, 1)
        k = 2 * math.pi / n
        u = u + 0.01 * CS * torch.stack([torch.sin(k * y + b), torch.sin(k * z), torch.sin(k * x)])
        us.append(u)
        As.append(A)
    ra = torch.stack(ra)
    return ra, RHO_HI + RHO_LO - ra, torch.stack(us), np.stack(As)


def _target_mass(ra, rb):
    return [1.02 * float(torch.where(ra[b] > rb[b], ra[b], 0.0).sum()) for b in range(ra.shape[0])]


def _mm_inputs(case, seed):
    A = _per_step(_ou(_gen(seed), case["ntraj"], case["nrows"] // STRIDE + 2), case["nrows"])
    return (A * 1e-3).contiguous()


TAU_D = (RHO_HI + RHO_LO) * 0.5 / 3.0 * 10.0 / SIGMA    # eta_s R / sigma at R = 10


def _params(seed):
    rng = np.random.default_rng(seed)
    parts = []
    for a, b in zip(WIDTHS[:-1], WIDTHS[1:]):
        bound = 1.0 / math.sqrt(a)
        parts += [rng.uniform(-bound, bound, a * b), rng.uniform(-bound, bound, b)]
    return np.concatenate(parts).astype(np.float32)


def _windows(seed, n):
    """n windows of 64 samples of A (float32, oldest first) and their semi-axis targets, descending."""
    g = _gen(seed)
    w = (_ou(g, n, 64) * 1e-3).reshape(n, 576).float().contiguous()
    mix = torch.randn((576, 3), generator=g, device=DEV, dtype=torch.float64) / 24.0
    t = 1.0 + 0.04 * torch.tanh(w.double() * 1e3 @ mix)
    return w, t.sort(dim=1, descending=True)[0].float().contiguous()


def _normalization():
    std = np.full(9, 1e-3)
    std[[0, 4, 8]] *= math.sqrt(2.0 / 3.0)
    return np.zeros(576), np.tile(1.0 / std, 64), np.array([1.03, 1.0, 0.97]), np.full(3, 25.0)


def _batches(case, seed):
    rng = np.random.default_rng(seed + 7)
    need = case["batch"] * case["steps"]
    order = np.concatenate([rng.permutation(TRAIN_ROWS) for _ in range(need // TRAIN_ROWS + 1)])[:need].astype(np.int32)
    sym = rng.integers(0, 48, need).astype(np.int32)
    return order, sym


# ---- prepare and run ---------------------------------------------------------------------------

_stream = None


def _side_stream():
    """The stream a program keeps for its boxes (the captured loop needs one that is not the null stream)."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream(device=DEV)
    return _stream


def _make_boxes(case, seed):
    import paper_2112_09972_amd as sc
    ghost, radius = case["bc"] == "ghost", _radius(case)
    lat = sc.Lattice(case["nx"], case["ny"], case["nz"], nbox=case["nbox"], bc=case["bc"], prec=case["prec"],
                     table_len=TABLE if ghost else 1, g_ab=G_AB, rho_b=_rho_b(radius),
                     mach_max=1.05 * MACH if ghost else 0.0, device=DEV, stream=_side_stream())
    rows = _history(case, seed) if ghost else None
    centers = _center(case, seed)
    for b in range(case["nbox"]):
        if ghost:
            lat.set_gradient_table(rows[b], 0, box=b)
        lat.init_droplet(centers[b], radius, WIDTH, RHO_HI, RHO_LO, rows[b, 0] if ghost else None, box=b)
    shape = (case["nbox"], case["nz"], case["ny"], case["nx"])
    st = dict(case=case, lat=lat, rows=rows, upto=TABLE,
              moments=torch.empty((case["nbox"], 10), dtype=torch.float64, device=DEV))
    if case["nbox"] > 1:
        st["rho"] = [torch.empty(shape, dtype=torch.float64, device=DEV) for _ in range(2)]
    return st


def _run_boxes(st):
    import paper_2112_09972_amd as sc
    case, lat = st["case"], st["lat"]
    n = case["steps"]
    with torch.cuda.stream(lat.stream):
        if st["rows"] is not None and lat.step_count + n > st["upto"]:
            for b in range(case["nbox"]):           # the history repeats
                lat.set_gradient_table(st["rows"][b], lat.step_count, box=b)
            st["upto"] = lat.step_count + TABLE
        if case["graph"]:
            lat.step_graph(n)
        else:
            lat.step(n)
        lat.droplet_moments_all(st["moments"])
        if case["nbox"] == 1:
            ra, rb, u = lat.fields()
            return dict(moments=st["moments"], rho_a=ra, rho_b=rb, u=u)
        for b in range(case["nbox"]):               # one array of every box's densities
            sc.sclbm_fields(lat.ctx, b, st["rho"][0][b].data_ptr(), st["rho"][1][b].data_ptr())
        return dict(moments=st["moments"], rho_a=st["rho"][0], rho_b=st["rho"][1])


def _make_analysis(case, seed):
    import paper_2112_09972_amd as sc
    ra, rb, u, A = _analysis_fields(case, seed)
    lat = sc.Lattice(case["nx"], case["ny"], case["nz"], nbox=case["nbox"], bc="ghost", prec=case["prec"], table_len=1,
                     g_ab=G_AB, rho_b=_rho_b(0.22 * min(case["nx"], case["ny"], case["nz"])), device=DEV,
                     stream=_side_stream())
    torch.cuda.synchronize()
    for b in range(case["nbox"]):
        sc.sclbm_init_fields(lat.ctx, b, ra[b].data_ptr(), rb[b].data_ptr(), u[b].data_ptr())
    lat.synchronize()
    nb, shape = case["nbox"], (case["nz"], case["ny"], case["nx"])
    buf = lambda *s: torch.empty(s, dtype=torch.float64, device=DEV)
    return dict(case=case, lat=lat, A=A, target=_target_mass(ra, rb), moments=buf(nb, 10), surface=buf(nb, 2),
                rho_a=buf(nb, *shape), rho_b=buf(nb, *shape), u=buf(nb, 3, *shape))


def _run_analysis(st):
    import paper_2112_09972_amd as sc
    lat, nb = st["lat"], st["case"]["nbox"]
    with torch.cuda.stream(lat.stream):
        lat.droplet_moments_all(st["moments"])
        lat.droplet_surface_all(st["surface"])
        mass = lat.droplet_mass()
        e0 = [lat.velocity_error(st["A"][b], box=b) for b in range(nb)]
        lat.reinject(st["target"])
        for b in range(nb):
            sc.sclbm_fields(lat.ctx, b, st["rho_a"][b].data_ptr(), st["rho_b"][b].data_ptr(), st["u"][b].data_ptr())
    return dict(moments=st["moments"], surface=st["surface"], mass=mass, e0=e0, rho_a=st["rho_a"], rho_b=st["rho_b"],
                u=st["u"])


def _make_net(case, seed, max_batch):
    from paper_2112_09972_amd.mlp import Network
    net = Network(max_batch=max_batch, device=DEV)
    net.set_params(_params(seed))
    net.set_normalization(*_normalization())
    return net


def prepare(case, seed):
    kind = case["kind"]
    if kind == "boxes":
        return _make_boxes(case, seed)
    if kind == "analysis":
        return _make_analysis(case, seed)
    if kind == "mm":
        A = _mm_inputs(case, seed)
        nrec = 1 + (case["nrows"] - 1) // case["every"]
        return dict(case=case, A=A, M=torch.empty((case["ntraj"], nrec, 9), dtype=torch.float64, device=DEV))
    if kind == "predict":
        w, _ = _windows(seed, case["n"])
        return dict(case=case, net=_make_net(case, seed, 8192), w=w)
    if kind == "train":
        w, t = _windows(seed, TRAIN_ROWS)
        order, sym = _batches(case, seed)
        return dict(case=case, net=_make_net(case, seed, max(256, case["batch"])), w=w, t=t,
                    order=torch.from_numpy(order).to(DEV), sym=torch.from_numpy(sym).to(DEV))
    w, t = _windows(seed, case["n"])
    return dict(case=case, net=_make_net(case, seed, max(256, case["n"])), w=w, t=t)


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "boxes":
        return _run_boxes(st)
    if kind == "analysis":
        return _run_analysis(st)
    if kind == "mm":
        import paper_2112_09972_amd as sc
        sc.sclbm_mm_integrate(st["A"].data_ptr(), case["ntraj"], case["nrows"], TAU_D, 1.0, case["substeps"],
                              case["every"], None, st["M"].data_ptr(), torch.cuda.current_stream().cuda_stream)
        return st["M"]
    net = st["net"]
    if kind == "predict":
        return net.predict(st["w"])
    if kind == "train":
        b = case["batch"]
        for s in range(case["steps"]):
            rows = slice(s * b, (s + 1) * b)
            loss = net.train_step(st["w"], st["t"], st["order"][rows], st["sym"][rows], lr=1e-3)
        return dict(loss=loss, params=net.params())
    loss = net.gradients(st["w"], st["t"])
    return dict(loss=loss, grads=net.grads())


# ---- work --------------------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind in ("boxes", "analysis"):
        nodes = case["nx"] * case["ny"] * case["nz"] * case["nbox"]
        dev = case["prec"].endswith("dev")
        state = nodes * (38 * POP_BYTES[case["prec"]] + (4 if dev else 0))   # deviations: and the reference densities
        if kind == "boxes":
            out = nodes * 8 * (5 if case["nbox"] == 1 else 2)
            return dict(bytes=2.0 * state * case["steps"] + state + out, flops=500.0 * nodes * case["steps"])
        return dict(bytes=float(state + nodes * 8 * 5), flops=200.0 * nodes)
    if kind == "mm":
        rows = case["nrows"] - 1
        nrec = 1 + rows // case["every"]
        return dict(bytes=72.0 * case["ntraj"] * (case["nrows"] + nrec),
                    flops=float(case["ntraj"]) * rows * case["substeps"] * 4 * 250)
    weights = 2.0 * MACS
    if kind == "predict":
        return dict(bytes=weights + case["n"] * (576 + 3) * 4.0, flops=2.0 * MACS * case["n"])
    rows = case["n"] if kind == "gradients" else case["batch"]
    once = dict(bytes=weights + rows * (576 + 3) * 4.0 + 4.0 * NPARAM, flops=(6.0 * MACS - 2.0 * 576 * 512) * rows)
    if kind == "gradients":
        return once
    # Adam reads the gradient, the weights and both moments and writes the latter three
    return dict(bytes=case["steps"] * (once["bytes"] + 24.0 * NPARAM), flops=case["steps"] * once["flops"])


# ---- exact: the same outputs in FP64 with plain torch and numpy --------------------------------

def _neighbours(rho, ghost, rb):
    """One layer around (nbox, nz, ny, nx): the ghost density, or the periodic image."""
    if ghost:
        return torch.nn.functional.pad(rho, (1,) * 6, value=rb)
    return torch.nn.functional.pad(rho[:, None], (1,) * 6, mode="circular")[:, 0]


def _stencil(pad, a):
    """sum_i w_i rho(x + c_i) c_ia on the interior of a padded field."""
    nz, ny, nx = (s - 2 for s in pad.shape[1:])
    out = 0.0
    for c, w in zip(CV, WT):
        if c[a]:
            out = out + (w * c[a]) * pad[:, 1 + c[2]:1 + c[2] + nz, 1 + c[1]:1 + c[1] + ny, 1 + c[0]:1 + c[0] + nx]
    return out


def _feq(i, rho, u, usq):
    c = CV[i]
    cu = sum(float(c[a]) * u[a] for a in range(3) if c[a])
    if not any(c):
        return WT[i] * rho * (1.0 - 1.5 * usq)
    return WT[i] * rho * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * usq)


def _stats(ra, rb, case):
    x, y, z = _grid(case)
    d = [x - (case["nx"] - 1) / 2.0, y - (case["ny"] - 1) / 2.0, z - (case["nz"] - 1) / 2.0]
    out = []
    for b in range(ra.shape[0]):
        m = (ra[b] > rb[b]).double()
        md = [m * v for v in d]
        out.append(torch.stack([m.sum()] + [v.sum() for v in md] +
                               [(md[i] * d[j]).sum() for i in range(3) for j in range(i, 3)]))
    return torch.stack(out)


def _barycentric(ra, rb, ja, jb, ghost, rho_b):
    pads = [_neighbours(ra, ghost, rho_b[0]), _neighbours(rb, ghost, rho_b[1])]
    return torch.stack([(ja[a] + jb[a] - 0.5 * G_AB * (ra * _stencil(pads[1], a) + rb * _stencil(pads[0], a))) / (ra + rb)
                        for a in range(3)], 1)


def _exact_boxes(case, seed):
    ghost, radius, nb = case["bc"] == "ghost", _radius(case), case["nbox"]
    rho_b, centers = _rho_b(radius), _center(case, seed)
    rows = torch.tensor(_history(case, seed), device=DEV) if ghost else None
    x, y, z = _grid(case)
    d = [x - (case["nx"] - 1) / 2.0, y - (case["ny"] - 1) / 2.0, z - (case["nz"] - 1) / 2.0]
    col = lambda v: v[:, None, None, None]
    ctr = torch.tensor(centers, device=DEV)
    r = ((x - col(ctr[:, 0])).square() + (y - col(ctr[:, 1])).square() + (z - col(ctr[:, 2])).square()).sqrt()
    ra = 0.5 * (RHO_HI + RHO_LO) - 0.5 * (RHO_HI - RHO_LO) * torch.tanh((r - radius) / WIDTH)
    A0 = rows[:, 0] if ghost else torch.zeros((nb, 9), device=DEV, dtype=torch.float64)
    u = [sum(col(A0[:, 3 * a + k]) * d[k] for k in range(3)) for a in range(3)]
    usq = sum(v * v for v in u)
    f = [[_feq(i, rho, u, usq) for i in range(19)] for rho in (ra, RHO_HI + RHO_LO - ra)]
    del r, u, usq
    mom = lambda fs, a: sum(float(CV[i][a]) * fs[i] for i in range(19) if CV[i][a])
    for t in range(case["steps"]):
        rho = [sum(fs) for fs in f]
        pads = [_neighbours(rho[s], ghost, rho_b[s]) for s in range(2)]
        j = [[mom(fs, a) for a in range(3)] for fs in f]
        up = [(j[0][a] + j[1][a]) / (rho[0] + rho[1]) for a in range(3)]
        del j
        for s in range(2):
            us = [up[a] - G_AB * _stencil(pads[1 - s], a) for a in range(3)]
            usq = sum(v * v for v in us)
            for i in range(19):
                post = _feq(i, rho[s], us, usq)      # tau = 1: the collision gives the equilibrium
                c = CV[i]
                if any(c):
                    post = torch.roll(post, (c[2], c[1], c[0]), (1, 2, 3))
                    if ghost:
                        for axis, n in ((0, case["nx"]), (1, case["ny"]), (2, case["nz"])):
                            if not c[axis]:
                                continue
                            sl = [slice(None)] * 3               # z, y, x
                            sl[2 - axis] = slice(0, 1) if c[axis] > 0 else slice(n - 1, n)
                            sl = tuple(sl)
                            dg = [d[a][sl] - c[a] for a in range(3)]
                            ug = [sum(col(rows[:, t, 3 * a + k]) * dg[k] for k in range(3)) for a in range(3)]
                            post[(slice(None),) + sl] = _feq(i, rho_b[s], ug, sum(v * v for v in ug))
                f[s][i] = post
    rho = [sum(fs) for fs in f]
    out = dict(moments=_stats(rho[0], rho[1], case), rho_a=rho[0], rho_b=rho[1])
    if nb == 1:
        u = _barycentric(rho[0], rho[1], [mom(f[0], a) for a in range(3)], [mom(f[1], a) for a in range(3)], ghost, rho_b)
        out = dict(moments=out["moments"], rho_a=rho[0][0], rho_b=rho[1][0], u=u[0])
    return out


def _surface(phi):
    """Area of {phi = 0} and volume of {phi > 0}, phi linear in the six tetrahedra of each cell along its diagonal."""
    corner = lambda o: phi[o[2]:phi.shape[0] - 1 + o[2], o[1]:phi.shape[1] - 1 + o[1], o[0]:phi.shape[2] - 1 + o[0]]
    offs = [(a, b, c) for a in (0, 1) for b in (0, 1) for c in (0, 1)]
    npos = sum((corner(o) > 0).int() for o in offs)
    vol, area = (npos == 8).sum().double(), 0.0
    cut = (npos > 0) & (npos < 8)
    vals = {o: corner(o)[cut] for o in offs}
    for perm in ((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)):
        o, path = [0, 0, 0], [(0, 0, 0)]
        for a in perm:
            o[a] = 1
            path.append(tuple(o))
        s = torch.stack([vals[p] for p in path], 1)
        p = torch.tensor(path, device=DEV, dtype=torch.float64).expand(s.shape[0], 4, 3)
        s, at = s.sort(dim=1, descending=True)
        p = p.gather(1, at[..., None].expand(-1, -1, 3))
        n = (s > 0).sum(1)
        vol = vol + (n == 4).sum() / 6.0
        cutpt = lambda s, p, a, b: p[:, a] + (s[:, a] / (s[:, a] - s[:, b]))[:, None] * (p[:, b] - p[:, a])
        frac = lambda s, a, b: s[:, a] / (s[:, a] - s[:, b])
        for k, v, rest in ((1, 0, (1, 2, 3)), (3, 3, (0, 1, 2))):
            m = n == k
            ss, pp = s[m], p[m]
            q = [cutpt(ss, pp, v, r) for r in rest]
            area = area + 0.5 * torch.linalg.cross(q[1] - q[0], q[2] - q[0]).norm(dim=1).sum()
            part = (frac(ss, v, rest[0]) * frac(ss, v, rest[1]) * frac(ss, v, rest[2])).sum() / 6.0
            vol = vol + (part if k == 1 else m.sum() / 6.0 - part)
        m = n == 2
        ss, pp = s[m], p[m]
        ac, ad, bc, bd = (cutpt(ss, pp, i, j) for i, j in ((0, 2), (0, 3), (1, 2), (1, 3)))
        area = area + 0.5 * torch.linalg.cross(bd - ac, bc - ad).norm(dim=1).sum()
        al, be, ga, de = (frac(ss, i, j) for i, j in ((0, 2), (0, 3), (1, 2), (1, 3)))
        vol = vol + (al * be + al * de * (1.0 - be) + (1.0 - al) * ga * de).sum() / 6.0
    return torch.stack([torch.as_tensor(area, device=DEV, dtype=torch.float64), vol])


def _exact_analysis(case, seed):
    ra, rb, u, A = _analysis_fields(case, seed)
    nb, rho_b = case["nbox"], _rho_b(0.22 * min(case["nx"], case["ny"], case["nz"]))
    target = _target_mass(ra, rb)
    x, y, z = _grid(case)
    d = torch.stack([x - (case["nx"] - 1) / 2.0, y - (case["ny"] - 1) / 2.0, z - (case["nz"] - 1) / 2.0])
    vel = _barycentric(ra, rb, [ra * u[:, a] for a in range(3)], [rb * u[:, a] for a in range(3)], True, rho_b)
    e0, mass = [], []
    scale = torch.ones_like(ra)
    for b in range(nb):
        lin = torch.tensordot(torch.tensor(A[b], device=DEV), d, 1)
        e0.append(float(((vel[b] - lin).square().sum() / lin.square().sum()).sqrt()))
        inside = ra[b] > rb[b]
        mass.append(float(ra[b][inside].sum()))
        scale[b][inside] = target[b] / mass[b]
    out = dict(moments=_stats(ra, rb, case), surface=torch.stack([_surface(ra[b] - rb[b]) for b in range(nb)]),
               mass=np.array(mass), e0=e0)
    new = ra * scale
    vel = _barycentric(new, rb, [new * u[:, a] for a in range(3)], [rb * u[:, a] for a in range(3)], True, rho_b)
    return dict(out, rho_a=new, rho_b=rb, u=vel)


def _exact_mm(case, seed):
    """Classical RK4 of dM/dt = L M + (L M)^T - (f1 / tau_d)(M - 3 det M / II_M I), L = f2 S + W."""
    if case["nrows"] * case["substeps"] * (1 + case["ntraj"] / 512.0) > 45000:
        return None
    A = _mm_inputs(case, seed).cpu().numpy().reshape(case["ntraj"], case["nrows"], 3, 3).swapaxes(0, 1)
    relax = 80.0 / (5.0 * 35.0) / TAU_D                       # f1 at viscosity ratio 1

    def lmat(G):
        ca = TAU_D * np.abs(G).max((-2, -1))
        f2 = 1.0 + 3.0 * ca * ca / (2.0 + 6.0 * ca * ca)
        T = np.swapaxes(G, -2, -1)
        return 0.5 * (f2[..., None, None] * (G + T) + G - T)

    eye = np.eye(3)

    def rhs(L, M):
        T = L @ M
        m = M.reshape(-1, 9)
        tr = m[:, 0] + m[:, 4] + m[:, 8]
        ii = 0.5 * (tr * tr - (m * m).sum(1))
        det = (m[:, 0] * (m[:, 4] * m[:, 8] - m[:, 5] * m[:, 7]) - m[:, 1] * (m[:, 3] * m[:, 8] - m[:, 5] * m[:, 6])
               + m[:, 2] * (m[:, 3] * m[:, 7] - m[:, 4] * m[:, 6]))
        return T + T.swapaxes(1, 2) - relax * (M - (3.0 * det / ii)[:, None, None] * eye)

    M = np.broadcast_to(eye, (case["ntraj"], 3, 3)).copy()
    rec, h, sub = [M.copy()], 1.0 / case["substeps"], case["substeps"]
    at = [lmat(A[:-1] + (A[1:] - A[:-1]) * (q * 0.5 * h)) for q in range(2 * sub + 1)]
    for n in range(case["nrows"] - 1):
        for s in range(sub):
            La, Lm, Lb = at[2 * s][n], at[2 * s + 1][n], at[2 * s + 2][n]
            k1 = rhs(La, M)
            k2 = rhs(Lm, M + 0.5 * h * k1)
            k3 = rhs(Lm, M + 0.5 * h * k2)
            k4 = rhs(Lb, M + h * k3)
            M = M + (h / 6.0) * (k1 + 2.0 * k2 + 2.0 * k3 + k4)
        if (n + 1) % case["every"] == 0:
            rec.append(M.copy())
    return np.stack(rec, 1).reshape(case["ntraj"], len(rec), 9)


def _unflatten(p):
    out, o = [], 0
    for a, b in zip(WIDTHS[:-1], WIDTHS[1:]):
        out += [p[o:o + a * b].view(b, a), p[o + a * b:o + a * b + b]]
        o += a * b + b
    return out


def _forward(ts, x):
    hs = [x]
    for l in range(4):
        v = hs[-1] @ ts[2 * l].T + ts[2 * l + 1]
        hs.append(v.clamp(min=0.0) if l < 3 else v)
    return hs


def _backward(ts, x, t):
    """Loss (mean squared error of the normalised outputs) and its gradient as one vector."""
    hs = _forward(ts, x)
    e = hs[4] - t
    loss, dz = (e * e).mean(), 2.0 * e / e.numel()
    grads = []
    for l in range(3, -1, -1):
        grads = [(dz.T @ hs[l]).reshape(-1), dz.sum(0)] + grads
        if l:
            dz = (dz @ ts[2 * l]) * (hs[l] > 0)
    return loss, torch.cat(grads)


def _norm_pair(w, t):
    a, b, c, d = (torch.tensor(v, device=DEV).float().double() for v in _normalization())
    return (w.double() - a) * b, (t.double() - c) * d if t is not None else None


def _map_windows(w, sym):
    """P A P^T for every sample, P the signed permutation of each row's symmetry id."""
    perms = [(0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0)]
    P = np.zeros((48, 3, 3))
    for s in range(48):
        for i in range(3):
            P[s, i, perms[s // 8][i]] = -1.0 if (s % 8) >> i & 1 else 1.0
    P = torch.tensor(P, device=DEV)[sym.long()][:, None]
    A = w.double().view(-1, 64, 3, 3)
    return (P @ A @ P.transpose(-1, -2)).reshape(-1, 576)


def exact(case, seed):
    kind = case["kind"]
    if kind == "boxes":
        return _exact_boxes(case, seed)
    if kind == "analysis":
        return _exact_analysis(case, seed)
    if kind == "mm":
        return _exact_mm(case, seed)
    p = torch.tensor(_params(seed), device=DEV, dtype=torch.float64)
    if kind == "predict":
        w, _ = _windows(seed, case["n"])
        y = _forward(_unflatten(p), _norm_pair(w, None)[0])[-1]
        _, _, c, d = _normalization()
        return y / torch.tensor(d, device=DEV) + torch.tensor(c, device=DEV).float().double()
    if kind == "gradients":
        w, t = _windows(seed, case["n"])
        loss, g = _backward(_unflatten(p), *_norm_pair(w, t))
        return dict(loss=loss.reshape(1), grads=g)
    w, t = _windows(seed, TRAIN_ROWS)
    order, sym = (torch.from_numpy(v).to(DEV) for v in _batches(case, seed))
    m, v, b = torch.zeros_like(p), torch.zeros_like(p), case["batch"]
    for s in range(case["steps"]):
        rows = order[s * b:(s + 1) * b].long()
        x, tn = _norm_pair(_map_windows(w[rows], sym[s * b:(s + 1) * b]), t[rows])
        loss, g = _backward(_unflatten(p), x, tn)
        m = 0.9 * m + 0.1 * g
        v = 0.999 * v + 0.001 * g * g
        p = p - 1e-3 * (m / (1.0 - 0.9 ** (s + 1))) / ((v / (1.0 - 0.999 ** (s + 1))).sqrt() + 1e-8)
    return dict(loss=loss.reshape(1), params=p)
