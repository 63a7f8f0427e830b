"""What this library is used for, as cases that can be timed.

Each case is one call, or one short fixed sequence of calls, that a program
using the library makes again and again: a forward projection (alone, batched
in one graph, with forced detection or its convolution form, for the emission
lines of Tc-99m and Tl-201), the gradient of a projection with respect to the
attenuation map, the response matrix of an acquisition, and the
reconstructions that use it.

Two kinds of maps are used.  "seg": the seeded ellipsoid thorax of this
repository's workloads (a handful of attenuation values, integer activities).
"ct": the same anatomy as a scan and a running image estimate give it: every
voxel has its own attenuation value and its own activity.  "cube": a water
cube with a point source.  Maps, counts and noise are made on the GPU from the
seed alone.
"""
import math
import random

import numpy as np
import torch

import paper_2105_13324_amd as mc

MU_WATER = 0.151
WINDOW = (126.0, 154.0)
ALPHA = math.radians(2.0)
TL201 = ((71.0, 0.9), (167.0, 0.1))
TL201_WINDOWS = ((64.0, 78.0), (150.0, 184.0))

# centre, semi-axes (cm on a 38.4 cm grid), density, activity; painted in order
ORGANS = [
    ((0.0, 0.0, 0.0), (16.0, 11.0, 24.0), 1.0, 1),       # body
    ((8.0, 1.0, 3.0), (5.5, 7.5, 11.0), 0.3, 1),         # lungs
    ((-8.0, 1.0, 3.0), (5.5, 7.5, 11.0), 0.3, 1),
    ((-5.0, -1.0, -11.0), (8.0, 6.0, 5.0), 1.0, 4),      # liver
    ((3.0, -3.5, 0.0), (4.0, 3.5, 5.0), 1.0, 8),         # myocardium
    ((3.0, -3.5, 0.0), (3.0, 2.5, 4.0), 1.0, 1),         # blood pool
    ((0.0, 8.0, 0.0), (1.8, 1.8, 24.0), 1.85, 1),        # spine
]


def listed():
    return [
        # a test-sized call in an outer loop: launches and latency
        dict(name="sim_thorax32", kind="sim", map="seg", n=32, vox=1.2, views=12, arc=180, nu=32, pix=1.2,
             hist=200_000, mode="analog"),
        # the point source in the 64^3 water cube: a calibration call
        dict(name="sim_cube64", kind="sim", map="cube", n=64, vox=0.2, views=1, arc=360, nu=128, pix=0.4,
             hist=1_000_000, mode="analog"),
        # the 128^3 thorax at 60 views: the forward projection of one study
        dict(name="sim_thorax128", kind="sim", map="seg", n=128, vox=0.3, views=60, arc=180, nu=64, pix=0.6,
             hist=100_000_000, mode="analog"),
        # uneven phantoms in one captured launch: a training set, a batch of patients
        dict(name="batch12_graph", kind="batch", map="seg", problems=12, n_lo=96, n_hi=160, views_lo=30,
             views_hi=120, vox=0.3, nu=64, pix=0.6, hist=5_000_000),
        # forced detection of the thorax: low-noise projections
        dict(name="fd_thorax128", kind="sim", map="seg", n=128, vox=0.3, views=60, arc=180, nu=64, pix=0.6,
             hist=10_000_000, mode="fd"),
        # its convolution form
        dict(name="cfd_thorax128", kind="sim", map="seg", n=128, vox=0.3, views=60, arc=180, nu=64, pix=0.6,
             hist=5_000_000, mode="cfd"),
        # one optimisation step on the attenuation map: forward and backward
        dict(name="grad_cube128", kind="grad", map="cube", n=128, vox=0.1, views=1, arc=360, nu=128, pix=0.4,
             hist=10_000_000),
        # a 256^3 study: forced-detection run, its response matrix, a short reconstruction
        dict(name="matrix_thorax256", kind="matrix", map="seg", n=256, vox=0.15, views=120, arc=360, nu=128,
             pix=0.3, hist=10_000_000, factor=4, mode="fd", iters=2),
        # 50 MLEM updates on the sparse matrix of an analog run
        dict(name="mlem_analog256", kind="mlem", map="seg", n=256, vox=0.15, views=120, arc=360, nu=128, pix=0.3,
             hist=1_000_000_000, factor=4, mode="analog", iters=50),
        # 10 MLEM updates on a forced-detection matrix
        dict(name="mlem_fd256", kind="mlem", map="seg", n=256, vox=0.15, views=120, arc=360, nu=128, pix=0.3,
             hist=40_000_000, factor=4, mode="fd", iters=10),
        # OS-EM on the primary matrix with the scatter projection added, 2 x 6 subsets
        dict(name="osem_fd128", kind="osem", map="seg", n=128, vox=0.3, views=60, arc=180, nu=64, pix=0.6,
             hist=10_000_000, factor=2, mode="fd", iters=2, subsets=6),
        # the scatter estimate of an image that is being reconstructed, on a scanned map
        dict(name="scatter_ct128", kind="scatter", map="ct", n=128, vox=0.3, views=60, arc=180, nu=64, pix=0.6,
             hist=3_000_000, factor=2),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng: random.Random):
    kind = rng.choice(["sim", "sim", "sim", "sim", "batch", "grad", "matrix", "mlem", "osem", "scatter"])
    n = int(_log(rng, 24, 176))
    if rng.random() < 0.5:
        n |= 1
    c = dict(kind=kind, map=rng.choice(["seg", "seg", "ct"]), n=n, vox=round(38.4 / n * rng.uniform(0.6, 1.0), 4),
             views=rng.randint(8, 120), arc=rng.choice([180, 360]), nu=rng.randint(24, 128))
    c["pix"] = round(n * c["vox"] / c["nu"], 4)
    if kind == "sim":
        c["mode"] = rng.choice(["analog", "analog", "fd", "cfd", "direction", "interaction"])
        c["hist"] = int(_log(rng, 1e4, 1e8 if c["mode"] == "analog" else 1e7))
        if c["mode"] == "cfd":
            c["nu"] = min(c["nu"], 64)
            c["pix"] = round(n * c["vox"] / c["nu"], 4)
        if c["mode"] == "analog" and rng.random() < 0.3:
            c["lines"] = 2
            c["hist"] = min(c["hist"], 2 * 10 ** 7)
    elif kind == "batch":
        lo = rng.randint(24, 120)
        c = dict(kind=kind, map=c["map"], problems=rng.randint(2, 12), n_lo=lo, n_hi=lo + rng.randint(1, 40),
                 views_lo=rng.randint(1, 30), views_hi=rng.randint(31, 120), vox=0.3, nu=64, pix=0.6,
                 hist=int(_log(rng, 1e5, 5e6)))
    elif kind == "grad":
        if rng.random() < 0.4:
            c.update(map="cube", n=2 * (n // 2), views=1)
        c["hist"] = int(_log(rng, 1e5, 1e7))
    else:
        f = rng.choice([1, 2, 3])
        c["factor"] = f
        c["n"] = max(24, n // f * f) if kind != "scatter" else max(24, n // 6 * 6)
        c["n"] -= c["n"] % f
        c["views"] = rng.randint(16, 90)
        c["hist"] = int(_log(rng, 2e5, 8e6))
        if kind == "scatter":
            c["factor"] = rng.choice([2, 3])
            c["nu"] = 6 * max(4, c["nu"] // 6)
            c["pix"] = round(c["n"] * c["vox"] / c["nu"], 4)
        elif kind == "matrix":
            c["mode"], c["iters"] = rng.choice(["fd", "fd", "analog"]), 2
        else:
            c["mode"] = rng.choice(["fd", "fd", "analog"]) if kind == "mlem" else "fd"
            c["iters"] = rng.randint(4, 40) if kind == "mlem" else rng.randint(1, 3)
            if kind == "osem":
                c["subsets"] = rng.randint(2, 10)
        if c.get("mode") == "analog":
            c["hist"] *= 20
    return c


# ---------------------------------------------------------------------------
# inputs

def _maps(kind, n, vox, seed):
    """mu (float32) and activity (uint32 bits as int32), [n, n, n] on the GPU."""
    if kind == "cube":
        mu = torch.full((n, n, n), MU_WATER, dtype=torch.float32, device="cuda")
        act = torch.zeros((n, n, n), dtype=torch.int32, device="cuda")
        act[n // 2, n // 2, n // 2] = 1
        return mu, act
    rng = np.random.Generator(np.random.PCG64(seed))
    half = 0.5 * n * vox
    s = half / 19.2
    c = -half + (torch.arange(n, dtype=torch.float32, device="cuda") + 0.5) * vox
    z, y, x = c.view(n, 1, 1), c.view(1, n, 1), c.view(1, 1, n)
    rho = torch.zeros((n, n, n), dtype=torch.float32, device="cuda")
    act = torch.zeros((n, n, n), dtype=torch.int32, device="cuda")
    for ctr, axes, dens, a in ORGANS:
        f = rng.uniform(0.85, 1.15, size=3)
        r = [ax * g * s for ax, g in zip(axes, f)]
        inside = (((x - ctr[0] * s) / r[0]) ** 2 + ((y - ctr[1] * s) / r[1]) ** 2
                  + ((z - ctr[2] * s) / r[2]) ** 2) < 1.0
        rho.masked_fill_(inside, dens)
        act.masked_fill_(inside, a)
    mu = MU_WATER * rho
    if kind == "ct":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        mu = mu * (1.0 + 0.03 * torch.randn(mu.shape, generator=g, device="cuda")).clamp_(0.5, 1.5)
        act = (act * 1000.0 * (0.9 + 0.2 * torch.rand(mu.shape, generator=g, device="cuda"))).round_().to(torch.int32)
    return mu.contiguous(), act.contiguous()


def _problem(case, seed, **kw):
    n, vox = kw.get("n", case.get("n")), case["vox"]
    views = kw.get("views", case.get("views"))
    mu, act = _maps(case["map"], n, vox, seed)
    ang = torch.arange(views, dtype=torch.float64, device="cuda") * (math.radians(case.get("arc", 180)) / views)
    cube = case["map"] == "cube"
    return mc.DeviceProblem(
        nx=n, ny=n, nz=n, voxel_cm=vox, mu=mu, activity=act, angles=ang, nu=case["nu"], nv=case["nu"],
        pixel_cm=case["pix"], radius_cm=0.5 * math.sqrt(2.0) * n * vox + 1.0, accept_half_angle_rad=ALPHA,
        e_lo_kev=WINDOW[0], e_hi_kev=WINDOW[1], e_cut_kev=10.0 if cube else WINDOW[0],
        n_histories=case["hist"], seed=seed & 0x7FFFFFFF, problem_id=kw.get("pid", 0),
        source_mode=1 if cube else 0, image_factor=case.get("factor", 0) if case["kind"] != "scatter" else 0)


OPTIONS = {"analog": None, "fd": {"forced_detection": 1}, "cfd": {"forced_detection": 2},
           "direction": {"variance_reduction": 1, "forced_direction_half_angle": ALPHA},
           "interaction": {"variance_reduction": 2}}


def _lines(p, hist):
    """Tl-201: one problem per line and window, histories split by yield."""
    out = []
    for k, (e0, share) in enumerate(TL201):
        for lo, hi in TL201_WINDOWS:
            out.append(p.with_(e0_kev=e0, e_lo_kev=lo, e_hi_kev=hi, e_cut_kev=TL201_WINDOWS[0][0],
                               n_histories=max(1, int(hist * share)), problem_id=k))
    return out


def _forward_with_list(case, p):
    cap = 3 * case["hist"] if case["mode"] == "fd" else max(1 << 14, case["hist"] // 1000)
    return mc.Simulator(p, event_capacity=cap, want_sq=False, options=OPTIONS[case["mode"]])


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        rng = np.random.Generator(np.random.PCG64(3))     # the sizes are the case's, the maps the seed's
        ps = []
        for k in range(case["problems"]):
            n = int(rng.integers(case["n_lo"], case["n_hi"] + 1))
            v = int(rng.integers(case["views_lo"], case["views_hi"] + 1))
            ps.append(_problem(case, seed * 100 + k, n=n, views=v, pid=k))
        sim = mc.Simulator(ps, want_sq=False)
        return dict(case=case, sim=sim, graph=mc.GraphRunner(sim))
    p = _problem(case, seed)
    if kind == "sim":
        ps = _lines(p, case["hist"]) if case.get("lines") else p
        sim = mc.Simulator(ps, want_sq=case["mode"] != "cfd", options=OPTIONS[case["mode"]])
        return dict(case=case, sim=sim)
    if kind == "grad":
        g = torch.Generator(device="cuda")
        g.manual_seed(seed)
        # the gradient of a Poisson loss: 1 - target / expected, per bin
        G = 1.0 - 0.3 * torch.randn(p.tally_shape, dtype=torch.float64, generator=g, device="cuda")
        return dict(case=case, p=p, mu=p.mu.clone().requires_grad_(True), G=G)
    if kind == "scatter":
        return dict(case=case, p=p)
    sim = _forward_with_list(case, p)
    if kind == "matrix":
        n_img = (p.nx // p.image_factor) ** 3
        return dict(case=case, p=p, sim=sim, image=torch.empty(n_img, dtype=torch.float32, device="cuda"))
    sim.run()
    m = mc.system_matrix(p, sim, "all" if kind == "mlem" else "primary")
    st = dict(case=case, m=m, image=torch.empty(m.n_img, dtype=torch.float32, device="cuda"))
    if kind == "mlem":
        st["mlem"] = mc.Mlem(m)
    else:
        st["scatter"] = mc.system_matrix(p, sim, "scatter").proj
        st["proj"] = m.proj + st["scatter"]
        st["bins_per_view"] = p.nu * p.nv
    return st


# ---------------------------------------------------------------------------
# passes

def run(st):
    kind = st["case"]["kind"]
    if kind == "sim":
        s = st["sim"]
        s.run()
        return dict(tally=s.tally, sq=s.tally_sq, fates=s.fates, energy=s.energy, counters=s.counters)
    if kind == "batch":
        st["graph"].replay()
        s = st["sim"]
        return dict(tally=s.tally, fates=s.fates, energy=s.energy, counters=s.counters)
    if kind == "grad":
        lam = mc.MCProject.apply(st["mu"], st["p"], max(1 << 14, st["case"]["hist"] // 500))
        grad, = torch.autograd.grad(lam, st["mu"], st["G"])
        return dict(projection=lam.detach(), grad=grad)
    if kind == "matrix":
        st["sim"].run()
        m = mc.system_matrix(st["p"], st["sim"])
        img = mc.Mlem(m).run(st["image"].fill_(1.0), st["case"]["iters"])
        return dict(T_rowptr=m.T_rowptr, Tt_rowptr=m.Tt_rowptr, proj=m.proj, image=img)
    if kind == "scatter":
        model = mc.ScatterModel(st["p"], st["case"]["hist"], factor=st["case"]["factor"])
        return model.estimate(st["p"].activity)
    img = st["image"].fill_(1.0)
    if kind == "mlem":
        return st["mlem"].run(img, st["case"]["iters"])
    return mc.osem(st["m"], img, st["case"]["iters"], st["case"]["subsets"], st["bins_per_view"],
                   proj=st["proj"], scatter=st["scatter"])


def work(case):
    """Inputs read once, outputs written once; operations of the method: per
    history 2 random blocks, 2.6 flights, 1.4 Kahn attempts and 0.8 scatters
    (about 330), per forced copy its ray (about 8 per voxel crossed)."""
    kind, hist = case["kind"], case["hist"]
    if kind == "batch":
        n3 = ((case["n_lo"] + case["n_hi"]) / 2) ** 3
        tally = 16 * case["nu"] ** 2 * (case["views_lo"] + case["views_hi"]) / 2
        return {"bytes": case["problems"] * (8 * n3 + tally), "flops": 330.0 * hist * case["problems"]}
    n3, bins = float(case["n"]) ** 3, float(case["views"]) * case["nu"] ** 2
    mode = case.get("mode", "fd" if kind == "scatter" else "analog")
    ops = 330.0 * hist + (1.2 * hist * 8 * 0.45 * case["n"] if mode in ("fd", "cfd") else 0.0)
    if kind == "sim":
        return {"bytes": 8 * n3 + 16 * bins * (1 if mode == "cfd" else 2), "flops": ops}
    if kind == "grad":
        return {"bytes": 12 * n3 + 32 * bins, "flops": ops}
    if kind == "scatter":
        return {"bytes": 8 * n3 + 16 * bins, "flops": ops}
    vox = n3 / case["factor"] ** 3
    nnz = 1.0 * hist if mode == "fd" else 1.4e-4 * hist
    if kind == "matrix":
        return {"bytes": 8 * n3 + 16 * nnz * (1 + case["iters"]) + 12 * bins + 8 * vox, "flops": ops + 10 * nnz}
    # each matrix value and column once per sweep, the vectors once
    return {"bytes": case["iters"] * (16 * nnz + 8 * (bins + vox)), "flops": case["iters"] * 4.0 * nnz}


# ---------------------------------------------------------------------------
# the same in 64 bits

def _csr(rowptr, col, val, n, shape):
    return torch.sparse_csr_tensor(rowptr, col[:n].to(torch.int64), val[:n].to(torch.float64), size=shape)


def exact(case, seed):
    """The reconstructions in double precision.  A forward run's outputs are
    whole numbers (fixed-point sums), and what is derived from them follows
    decisions taken along random walks: there is no 64-bit value of those."""
    if case["kind"] not in ("mlem", "osem"):
        return None
    st = prepare(case, seed)
    m = st["m"]
    n = m.nnz
    P = (m.proj if case["kind"] == "mlem" else st["proj"]).to(torch.float64)
    S = torch.ones(m.n_img, dtype=torch.float64, device="cuda")
    T = _csr(m.T_rowptr, m.T_col, m.T_val, n, (m.n_bins, m.n_img))
    Tt = _csr(m.Tt_rowptr, m.Tt_col, m.Tt_val, n, (m.n_img, m.n_bins))
    zero = torch.zeros(m.n_bins, dtype=torch.float64, device="cuda")
    if case["kind"] == "mlem":
        add, subsets = zero, 1
        masks = [torch.ones_like(P)]
    else:
        add, subsets = st["scatter"].to(torch.float64), case["subsets"]
        view = torch.arange(m.n_bins, device="cuda") // st["bins_per_view"]
        masks = [((view % subsets) == k).to(torch.float64) for k in range(subsets)]
    sens = [Tt @ mk for mk in masks]
    S = torch.where(sum(sens) > 0, S, torch.zeros_like(S))
    for _ in range(case["iters"]):
        for mk, se in zip(masks, sens):
            y = T @ S + add
            ratio = torch.where(y > 0, P / y.clamp_min(1e-300), zero) * mk
            S = torch.where(se > 0, S * (Tt @ ratio) / se.clamp_min(1e-300), S)
    return S
