"""The workloads whose speed this framework is held to, through its public entry points.

Kinds of work:

- ``corr``:  one sample's binned correlation: reset, accumulate a trajectory,
  finalize (with ``n_q`` > 0 also S(q, t) and S(q, w) from the bins);
- ``batch``: several samples accumulated in one launch, each finalized;
- ``sq``:    S(q, t) and S(q, w) at arbitrary wave vectors of a point set;
- ``traj``:  a Landau-Lifshitz RK4 trajectory from a given start;
- ``mc``:    Metropolis sweeps (a thermalised start), with their history.

Inputs are made on the GPU from the seed: unit spins that precess about local
axes, the axes partly aligned so that the correlations do not vanish.
``exact`` evaluates each definition in 64 bits with plain torch operations.
"""
import math

import numpy as np
import torch

from paper_2308_07487_amd import inputs, sdc

DEV = "cuda"


def listed():
    return [
        # the smallest sample that is tested and benchmarked: launches and copies decide
        dict(name="sc 8^3 split-BF16", kind="corr", lattice="sc", l0=8, l1=8, l2=8, n_o=32, n_l=64, stride=1,
             prec="split_bf16", connected=False, n_q=0),
        # an ordinary sample of odd edges and counts, the connected correlation of an ordered phase
        dict(name="bcc 13x14x15 split-FP16 connected", kind="corr", lattice="bcc", l0=13, l1=14, l2=15, n_o=75,
             n_l=130, stride=1, prec="split_fp16", connected=True, n_q=0),
        # full single precision with every second frame an origin, and the spectra along a path of wave vectors
        dict(name="sc 21x20x19 FP32 and S(q,w)", kind="corr", lattice="sc", l0=21, l1=20, l2=19, n_o=50, n_l=100,
             stride=2, prec="fp32", connected=False, n_q=40),
        # a 2D square lattice at FP32-level accuracy on the BF16 matrix cores
        dict(name="sc 90x90x1 BF16x3", kind="corr", lattice="sc", l0=90, l1=90, l2=1, n_o=50, n_l=64, stride=1,
             prec="bf16x3", connected=False, n_q=0),
        # the benchmark's default sample: the largest
        dict(name="sc 36^3 split-BF16", kind="corr", lattice="sc", l0=36, l1=36, l2=36, n_o=128, n_l=256, stride=1,
             prec="split_bf16", connected=False, n_q=0),
        # points without a lattice, binned by distance
        dict(name="ball 20011 radial split-BF16", kind="corr", lattice="ball", n=20011, shells=1024, n_o=64, n_l=128,
             stride=1, prec="split_bf16", connected=False, n_q=0),
        # many realizations of different lattices in one launch
        dict(name="batch of 10 samples", kind="batch", n_samples=10, lo=10, hi=22, recipe=5, prec="split_bf16"),
        # q-resolved spectra of a small and of the benchmark's sample
        dict(name="S(q,t) 3001 points 100 q", kind="sq", n=3001, n_q=100, n_o=32, n_l=64, stride=1, connected=True),
        dict(name="S(q,t) 65536 points 1024 q", kind="sq", n=65536, n_q=1024, n_o=64, n_l=128, stride=1,
             connected=False),
        # a trajectory of an antiferromagnet in a field with anisotropy and DMI
        dict(name="RK4 sc 20x22x24, 200 frames", kind="traj", l0=20, l1=22, l2=24, frames=200, J=1.0, D=0.2, A=0.1,
             Hz=0.3, dt=0.02),
        # annealing of the 2D ferromagnet, and sweeps of a large sample at one temperature
        dict(name="MC 32x32x1 anneal", kind="mc", l0=32, l1=32, l2=1, J=-1.0, D=0.0, Hz=0.5, T0=2.0, T1=0.1, cool=0.9,
             per_T=10, final=20),
        dict(name="MC sc 128^3, 20 sweeps", kind="mc", l0=128, l1=128, l2=128, J=-1.0, D=0.0, Hz=0.5, T0=1.0, T1=1.0,
             cool=0.9, per_T=1, final=20),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["corr", "batch", "sq", "traj", "mc"], [6, 1, 2, 1, 2])[0]
    if kind == "batch":
        return dict(kind="batch", n_samples=rng.randint(3, 12), lo=8, hi=rng.randint(12, 22),
                    recipe=rng.randint(0, 10 ** 6), prec=rng.choice(["split_bf16", "split_bf16", "split_fp16", "bf16x3"]))
    if kind == "sq":
        return dict(kind="sq", n=_log_int(rng, 500, 60000), n_q=_log_int(rng, 10, 1000), n_o=rng.randint(8, 100),
                    n_l=rng.randint(16, 160), stride=rng.choice([1, 1, 2]), connected=rng.random() < 0.4)
    if kind == "traj":
        e = [rng.randint(6, 36) for _ in range(3)]
        if rng.random() < 0.3:
            e = [rng.randint(8, 120), rng.randint(8, 120), 1]
        return dict(kind="traj", l0=e[0], l1=e[1], l2=e[2], frames=rng.randint(50, 383), J=rng.choice([1.0, -1.0]),
                    D=rng.choice([0.0, 0.2]), A=rng.choice([0.0, 0.1]), Hz=rng.choice([0.0, 0.3]), dt=0.01)
    if kind == "mc":
        e = [rng.randint(4, 64) for _ in range(3)]
        if rng.random() < 0.4:
            e = [rng.randint(8, 200), rng.randint(8, 200), 1]
        return dict(kind="mc", l0=e[0], l1=e[1], l2=e[2], J=rng.choice([1.0, -1.0]), D=rng.choice([0.0, 0.3]),
                    Hz=rng.choice([0.0, 0.5]), T0=rng.uniform(0.5, 3.0), T1=rng.uniform(0.05, 0.4),
                    cool=rng.uniform(0.7, 0.93), per_T=rng.randint(1, 10), final=rng.randint(5, 40))
    lattice = rng.choice(["sc", "sc", "bcc", "ball"])
    prec = rng.choice(["split_bf16", "split_bf16", "split_bf16", "split_fp16", "bf16x3", "fp32"])
    while True:
        c = dict(kind="corr", lattice=lattice, n_o=rng.randint(8, 128), n_l=rng.randint(8, 256),
                 stride=rng.choice([1, 1, 1, 2, 3]), prec=prec, connected=rng.random() < 0.3, n_q=0)
        if lattice == "ball":
            c.update(n=_log_int(rng, 500, 24000), shells=rng.randint(64, 1024))
        else:
            e = [_log_int(rng, 5, 36) for _ in range(3)]
            if rng.random() < 0.2:
                e = [_log_int(rng, 16, 160), _log_int(rng, 16, 160), 1]
            c.update(l0=e[0], l1=e[1], l2=e[2])
            if rng.random() < 0.3:
                c["n_q"] = rng.randint(3, 60)
        rate = 0.12e15 if prec == "fp32" else 0.9e15  # about what the kernels reach
        if _corr_flops(c) < 0.5 * rate:
            return c


# --- inputs ------------------------------------------------------------------

def _cells(c):
    return (c["l0"], c["l1"], c["l2"])


def _positions(c, seed):
    if c["kind"] == "sq" or c.get("lattice") == "ball":
        n = c["n"]
        return inputs.ball_positions(n, 25.0 * (n / 65536.0) ** (1.0 / 3.0), seed + 77)
    return inputs.bcc_positions(_cells(c)) if c.get("lattice") == "bcc" else inputs.sc_positions(_cells(c))


def _unit(n, gen, bias):
    v = torch.randn(n, 3, generator=gen, device=DEV, dtype=torch.float64)
    v[:, 2] += bias
    return v / v.norm(dim=1, keepdim=True)


def _frames(n, n_frames, seed):
    """[n_frames][n][3] fp32: unit spins precessing about local axes at random rates."""
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    s, ax = _unit(n, gen, 0.7), _unit(n, gen, 1.0)
    w = 0.01 * (3.0 + 2.0 * torch.rand(n, 1, generator=gen, device=DEV, dtype=torch.float64))
    par = ax * (ax * s).sum(1, keepdim=True)
    per, cr = s - par, torch.linalg.cross(ax, s)
    out = torch.empty(n_frames, n, 3, device=DEV, dtype=torch.float32)
    for f in range(n_frames):
        out[f] = (par + torch.cos(w * f) * per + torch.sin(w * f) * cr).float()
    return out


def _t_need(c):
    return (c["n_o"] - 1) * c["stride"] + c["n_l"]


def _samples(c):
    """The samples of a batch as corr cases."""
    out = []
    for s in inputs.batch_samples(c["n_samples"], seed=c["recipe"], edge=(c["lo"], c["hi"])):
        out.append(dict(kind="corr", lattice=s["lattice"], l0=s["cells"][0], l1=s["cells"][1], l2=s["cells"][2],
                        n_o=s["n_origins"], n_l=s["n_lags"], stride=1, prec=c["prec"], connected=False, n_q=0))
    return out


def _m(c):
    """Commensurate wave vectors along Gamma - X - M - R."""
    path = [(0, 0, 0), (1, 0, 0), (1, 1, 0), (1, 1, 1)]
    t = np.linspace(0.0, 3.0, c["n_q"])
    k = np.minimum(t.astype(int), 2)
    p = np.array(path, dtype=float)
    f = p[k] + (t - k)[:, None] * (p[k + 1] - p[k])
    return np.rint(0.5 * f * np.array(_cells(c))).astype(np.int32)


def _q(c, seed):
    return np.concatenate([np.zeros((1, 3)), inputs.powder_wave_vectors(c["n_q"] - 1, 0.05, 3.0, seed + 5)])


def _start(c, seed):
    n = c["l0"] * c["l1"] * c["l2"]
    return _unit(n, torch.Generator(device=DEV).manual_seed(int(seed)), 0.3).float().contiguous()


def _mc_spec(c, seed):
    return sdc.mc_spec(sdc.BINS_SC, cells=_cells(c), J=c["J"], D=c["D"], Hz=c["Hz"], seed=seed, T_start=c["T0"],
                       T_end=c["T1"], cool=c["cool"], sweeps_per_T=c["per_T"], sweeps_final=c["final"])


def _plan(c, seed):
    pos = _positions(c, seed)
    if c["lattice"] == "ball":
        kw = dict(kind=sdc.BINS_RADIAL, n_shells=c["shells"], r_max=_r_max(c))
    else:
        kw = dict(kind=sdc.BINS_BCC if c["lattice"] == "bcc" else sdc.BINS_SC, cells=_cells(c))
    return sdc.Plan(pos, n_origins=c["n_o"], n_lags=c["n_l"], precision=c["prec"], origin_stride=c["stride"],
                    connected=c["connected"], **kw)


def _r_max(c):
    return 50.0 * (c["n"] / 65536.0) ** (1.0 / 3.0)


def _n_sites(c):
    if "n" in c:
        return c["n"]
    return c["l0"] * c["l1"] * c["l2"] * (2 if c.get("lattice") == "bcc" else 1)


def prepare(case, seed):
    c = case
    if c["kind"] == "corr":
        return dict(case=c, plan=_plan(c, seed), frames=_frames(_n_sites(c), _t_need(c), seed),
                    m=_m(c) if c["n_q"] else None)
    if c["kind"] == "batch":
        parts = _samples(c)
        plans = [_plan(p, seed) for p in parts]
        return dict(case=c, plans=plans, batch=sdc.Batch(plans),
                    frames=[_frames(_n_sites(p), _t_need(p), seed + k) for k, p in enumerate(parts)])
    if c["kind"] == "sq":
        acc = sdc.StructureFactor(_positions(c, seed), _q(c, seed), c["n_o"], c["n_l"], origin_stride=c["stride"],
                                  connected=c["connected"])
        return dict(case=c, acc=acc, frames=_frames(c["n"], _t_need(c), seed))
    pos, start = inputs.sc_positions(_cells(c)), _start(c, seed)
    if c["kind"] == "traj":
        return dict(case=c, pos=pos, start=start,
                    frames=torch.empty(c["frames"], pos.shape[0], 3, device=DEV, dtype=torch.float32))
    spec = _mc_spec(c, seed)
    return dict(case=c, mc=sdc.MonteCarlo(pos, spec), spec=spec, start=start, state=torch.empty_like(start))


def run(state):
    s, c = state, state["case"]
    if c["kind"] == "corr":
        p = s["plan"]
        p.reset()
        p.accumulate(s["frames"])
        out = p.finalize()
        if s["m"] is not None:
            out["Sqt"], out["Sqw"] = p.structure_factor(s["m"])
        return out
    if c["kind"] == "batch":
        for p in s["plans"]:
            p.reset()
        s["batch"].accumulate(s["frames"])
        return [p.finalize() for p in s["plans"]]
    if c["kind"] == "sq":
        s["acc"].reset()
        s["acc"].accumulate(s["frames"])
        return s["acc"].finalize()
    if c["kind"] == "traj":
        sdc.traj_generate(s["pos"], sdc.BINS_SC, s["frames"], cells=_cells(c), J=c["J"], dt=c["dt"],
                          init=sdc.INIT_GIVEN, init_state=s["start"], D=c["D"], A=c["A"], Hz=c["Hz"])
        return s["frames"]
    accepted, info = s["mc"].run(s["spec"], s["state"], init_state=s["start"], history=True, info=True)
    return dict(state=s["state"], accepted=accepted, info=info)


# --- the work a pass cannot do without ---------------------------------------

def _corr_flops(c):
    """Matrix-core operations of the precision asked for (its products of 2 flops per pair, origin, component and lag)."""
    products = {"fp32": 1, "split_bf16": 3, "split_fp16": 3, "bf16x3": 6}[c["prec"]]
    return 2.0 * products * 3 * c["n_o"] * c["n_l"] * float(_n_sites(c)) ** 2


def _corr_bytes(c):
    n, n_bins = _n_sites(c), c["shells"] if c["lattice"] == "ball" else _n_sites(c)
    return 12.0 * n * _t_need(c) + 8.0 * n_bins * (c["n_l"] + 1) + 48.0 * c["n_l"] + 32.0 * c["n_q"] * c["n_l"]


def work(case):
    c = case
    if c["kind"] == "corr":
        return dict(bytes=_corr_bytes(c), flops=_corr_flops(c))
    if c["kind"] == "batch":
        return dict(bytes=sum(map(_corr_bytes, _samples(c))), flops=sum(map(_corr_flops, _samples(c))))
    if c["kind"] == "sq":
        # two multiply-adds per wave vector, site and spin column; three complex products per lag and origin
        t = _t_need(c)
        return dict(bytes=12.0 * c["n"] * (t + 1) + 24.0 * c["n_q"] + 32.0 * c["n_q"] * c["n_l"],
                    flops=c["n_q"] * (12.0 * t * c["n"] + 24.0 * c["n_o"] * c["n_l"]))
    n = c["l0"] * c["l1"] * c["l2"]
    if c["kind"] == "traj":
        # four stages per frame: six neighbours (6, with DMI 18 flops each), a cross product and the update
        return dict(bytes=12.0 * n * (c["frames"] + 1), flops=4.0 * n * (c["frames"] - 1) * (6 * (18 if c["D"] else 6) + 21))
    # per update: six neighbours, the trial spin and the energy difference; states read and written once in all
    return dict(bytes=24.0 * n, flops=(36.0 + 80.0) * n * _n_sweeps(c))


# --- 64-bit references -------------------------------------------------------

def _temperatures(c):
    out, t = [], c["T0"]
    while t > c["T1"]:
        out += [t] * c["per_T"]
        t *= c["cool"]
    return out + [c["T1"]] * c["final"]


def _n_sweeps(c):
    return len(_temperatures(c))


def _spectrum(x):
    """One-sided half-Hann windowed transform over the last axis."""
    n = x.shape[-1]
    w = 0.5 * (1.0 + torch.cos(math.pi * torch.arange(n, device=DEV, dtype=torch.float64) / n))
    return torch.fft.fft(x * w)


def _np(x):
    return x.cpu().numpy()


def _exact_corr(c, seed):
    n, n_o, n_l, s = _n_sites(c), c["n_o"], c["n_l"], c["stride"]
    fr = _frames(n, _t_need(c), seed)
    later = fr.double()
    early = later[0:(n_o - 1) * s + 1:s]
    if c["connected"]:
        early = early - early.mean(0, keepdim=True)
    tot_e, tot_l = early.sum(1), later.sum(1)
    csum, cself, sqt = [torch.zeros(n_l, device=DEV, dtype=torch.float64) for _ in range(2)] + [None]
    for t in range(n_l):
        k = slice(t, t + (n_o - 1) * s + 1, s)
        csum[t] = (tot_e * tot_l[k]).sum() / (n * n_o)
        cself[t] = (early * later[k]).sum() / (n * n_o)
    if c["lattice"] == "ball":
        C, counts = _exact_radial(c, seed, early, later)
    else:
        L, N = _cells(c), c["l0"] * c["l1"] * c["l2"]
        sub = 2 if c["lattice"] == "bcc" else 1

        def grids(x):  # [frames][sublattice][3][L0][L1][L2], transformed
            g = x.reshape(x.shape[0], N, sub, 3).permute(0, 2, 3, 1).reshape(x.shape[0], sub, 3, *L)
            return torch.fft.fftn(g, dim=(3, 4, 5))

        ge, gl = grids(early), grids(later)
        H = torch.zeros(n_l, *L, sub, device=DEV, dtype=torch.float64)
        for t in range(n_l):
            g = gl[t:t + (n_o - 1) * s + 1:s]
            for bi in range(sub):
                for bj in range(sub):
                    h = torch.fft.ifftn((ge[:, bi].conj() * g[:, bj]).sum((0, 1))).real
                    if bj < bi:  # the centre of cell k lies half a cell above its corner
                        h = torch.roll(h, (-1, -1, -1), (0, 1, 2))
                    H[t, ..., (bj - bi) % 2] += h
        C = H.reshape(n_l, -1) / (float(n) * n_o)
        counts = torch.full((n,), n, device=DEV, dtype=torch.int64)
        if c["n_q"]:
            m = torch.from_numpy(_m(c)).to(DEV).double()
            ax = [torch.arange(x, device=DEV, dtype=torch.float64) for x in L]
            pos = torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
            if sub == 2:
                pos = torch.stack([pos, pos + 0.5], 1).reshape(-1, 3)
            ph = -2.0 * math.pi * (m / torch.tensor(L, device=DEV, dtype=torch.float64)) @ pos.T
            sqt = torch.polar(torch.ones_like(ph), ph) @ C.T.to(torch.complex128)
    out = dict(C=_np(C), counts=_np(counts), Csum=_np(csum), Cself=_np(cself), Ssum=_np(_spectrum(csum)),
               Sself=_np(_spectrum(cself)))
    if sqt is not None:
        out["Sqt"], out["Sqw"] = _np(sqt), _np(_spectrum(sqt))
    return out


def _exact_radial(c, seed, early, later):
    n, n_o, n_l, s, ns = c["n"], c["n_o"], c["n_l"], c["stride"], c["shells"]
    pos = torch.from_numpy(_positions(c, seed)).to(DEV)
    width = float(np.float32(_r_max(c))) / ns
    e2 = (torch.arange(ns, device=DEV, dtype=torch.float64) * width).square().float()
    # sums of one shell are spread over `lanes` places, so that the adds do not queue on 1024 addresses
    lanes, C, counts = 64, torch.zeros(n_l, ns, device=DEV, dtype=torch.float64), torch.zeros(ns, device=DEV, dtype=torch.int64)
    step = max(1, 200_000_000 // n)
    for i in range(0, n, step):
        p = pos[i:i + step]
        d = p[:, None, :] - pos[None, :, :]
        d2 = (d[..., 0] * d[..., 0] + d[..., 1] * d[..., 1]) + d[..., 2] * d[..., 2]
        del d
        key = torch.bucketize(d2, e2, right=True) - 1
        counts += torch.bincount(key.reshape(-1), minlength=ns)
        place = (key * lanes + torch.arange(n, device=DEV) % lanes).reshape(-1)
        del d2, key
        a = early[:, i:i + step].permute(1, 0, 2).reshape(p.shape[0], -1)
        for t in range(n_l):
            b = later[t:t + (n_o - 1) * s + 1:s].permute(1, 0, 2).reshape(n, -1)
            g = a @ b.T.contiguous()
            C[t] += torch.zeros(ns * lanes, device=DEV, dtype=torch.float64).index_add_(0, place, g.reshape(-1)).reshape(ns, lanes).sum(1)
    return torch.where(counts > 0, C / (n_o * counts.clamp(min=1)), torch.zeros_like(C)), counts


def _exact_sq(c, seed):
    n_o, s = c["n_o"], c["stride"]
    pos = torch.from_numpy(_positions(c, seed)).to(DEV).double()
    q = torch.from_numpy(_q(c, seed)).to(DEV)
    x = _frames(c["n"], _t_need(c), seed).double().permute(1, 0, 2).reshape(c["n"], -1)
    F = torch.zeros(c["n_q"], x.shape[1], device=DEV, dtype=torch.complex128)
    for j in range(0, c["n"], 8192):
        ph = -q @ pos[j:j + 8192].T.contiguous()
        F += torch.complex(torch.cos(ph) @ x[j:j + 8192], torch.sin(ph) @ x[j:j + 8192])
    F = F.reshape(c["n_q"], -1, 3)
    early = F[:, 0:(n_o - 1) * s + 1:s]
    if c["connected"]:
        early = early - early.mean(1, keepdim=True)
    sqt = torch.stack([(early.conj() * F[:, t:t + (n_o - 1) * s + 1:s]).sum((1, 2)) for t in range(c["n_l"])], 1)
    sqt = sqt / (float(c["n"]) * n_o)
    return _np(sqt), _np(_spectrum(sqt))


def _neighbours(L):
    """[6][n] neighbour sites (+x, -x, +y, -y, +z, -z) and [6] whether the bond exists."""
    i = torch.arange(L[0] * L[1] * L[2], device=DEV).reshape(L)
    nb = [torch.roll(i, -d, a).reshape(-1) for a in range(3) for d in (1, -1)]
    return torch.stack(nb), [L[a] > 1 for a in range(3) for _ in (0, 1)]


def _field(c, nb, have, x):
    """sum_j (J x_j + D_ij x x_j) at the sites whose neighbours nb holds."""
    h = torch.zeros(nb.shape[1], 3, device=DEV, dtype=x.dtype)
    for e in range(6):
        if have[e]:
            y, d = x[nb[e]], torch.zeros(3, device=DEV, dtype=x.dtype)
            d[e // 2] = c["D"] * (1.0 if e % 2 == 0 else -1.0)
            h += float(np.float32(c["J"])) * y + torch.linalg.cross(d.float().double().expand_as(y), y)
    return h


def _exact_traj(c, seed):
    nb, have = _neighbours(_cells(c))
    x = _start(c, seed).double()
    dt = c["dt"]

    def rate(y):
        h = _field(c, nb, have, y)
        h[:, 2] -= 2.0 * c["A"] * y[:, 2] + c["Hz"]
        return torch.linalg.cross(h, y)

    out = torch.empty(c["frames"], x.shape[0], 3, device=DEV, dtype=torch.float64)
    out[0] = x
    for f in range(1, c["frames"]):
        k1 = rate(x)
        k2 = rate(x + 0.5 * dt * k1)
        k3 = rate(x + 0.5 * dt * k2)
        k4 = rate(x + dt * k3)
        x = x + dt / 6.0 * (k1 + 2 * k2 + 2 * k3 + k4)
        out[f] = x
    return out


def _philox(c, key):
    """Philox4x32-10 of int64 tensors that hold 32-bit words."""
    low = 0xFFFFFFFF
    k0, k1 = key & low, key >> 32
    for _ in range(10):
        p0, p1 = _mul(c[0], 0xD2511F53), _mul(c[2], 0xCD9E8D57)
        c = [p1[0] ^ c[1] ^ k0, p1[1], p0[0] ^ c[3] ^ k1, p0[1]]
        k0, k1 = (k0 + 0x9E3779B9) & low, (k1 + 0xBB67AE85) & low
    return c


def _mul(a, m):
    """(high, low) 32-bit words of a * m."""
    lo, hi = (a & 0xFFFF) * m, (a >> 16) * m
    hi = hi + (lo >> 16)
    return hi >> 16, ((hi & 0xFFFF) << 16) | (lo & 0xFFFF)


def _exact_mc(c, seed):
    """Checkerboard sweeps; None where the box is not two-coloured or the sample is large."""
    L = _cells(c)
    if any(x % 2 for x in L if x > 1) or min(L[:2]) < 4 or L[2] not in (1, *range(4, 4096)):
        return None
    n = L[0] * L[1] * L[2]
    nb, have = _neighbours(L)
    site = torch.arange(n, device=DEV)
    parity = (site // (L[1] * L[2]) + site // L[2] % L[1] + site % L[2]) % 2
    classes = [torch.nonzero(parity == k).reshape(-1) for k in (0, 1)]
    S = _start(c, seed).double()
    cone, history, T = math.pi, [], c["T0"]
    zero = torch.zeros((), device=DEV, dtype=torch.float64)
    for sweep, T in enumerate(_temperatures(c)):
        accepted, cos_cone = 0, math.cos(cone)
        for i in classes:
            w = _field(c, nb[:, i], have, S)
            o = torch.zeros_like(i)
            r = _philox([i, o + sweep, o, o + 0x80000000], int(seed))
            u = [(v.double() + 0.5) / 4294967296.0 for v in r[:3]]
            s = S[i]
            ca = 1.0 - u[0] * (1.0 - cos_cone)
            sa = torch.sqrt(torch.maximum(zero, 1.0 - ca * ca))
            near = s[:, 2].abs() >= 0.9
            a = torch.zeros_like(s)
            a[:, 0], a[:, 2] = near.double(), 1.0 - near.double()
            e1 = a - (a * s).sum(1, keepdim=True) * s
            e1 = e1 / e1.norm(dim=1, keepdim=True)
            e2 = torch.linalg.cross(s, e1)
            az = 2.0 * math.pi * u[1]
            t = ca[:, None] * s + sa[:, None] * (torch.cos(az)[:, None] * e1 + torch.sin(az)[:, None] * e2)
            t = t / t.norm(dim=1, keepdim=True)
            dE = ((t - s) * w).sum(1) - c["Hz"] * (t[:, 2] - s[:, 2])
            take = (dE <= 0) | (u[2] < torch.exp(-dE / T))
            S[i] = torch.where(take[:, None], t, s)
            accepted += int(take.sum())
        history.append(accepted)
        if accepted / n < 0.2:
            cone = max(1e-3, 0.9 * cone)
        elif accepted / n > 0.4:
            cone = min(math.pi, 1.1 * cone)
    h = _field(c, nb, have, S)
    energy = 0.5 * float((h * S).sum()) - c["Hz"] * float(S[:, 2].sum())
    return dict(state=S, accepted=np.array(history, dtype=np.int64), info=np.array([energy / n, cone, T, 2.0]))


def exact(case, seed):
    c = case
    if c["kind"] == "corr":
        if c["lattice"] == "ball" and float(c["n"]) ** 2 * c["n_l"] > 6e10:
            return None
        return _exact_corr(c, seed)
    if c["kind"] == "batch":
        return [_exact_corr(p, seed + k) for k, p in enumerate(_samples(c))]
    if c["kind"] == "sq":
        return _exact_sq(c, seed)
    if c["kind"] == "traj":
        return _exact_traj(c, seed)
    return _exact_mc(c, seed)
