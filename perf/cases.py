"""Measured workloads of the ray tracer and of its proposal network.

Each case is one call, or one short sequence of calls, that a program built on
this package makes through its public entry points: an image of an
instrument, a batch of projections, an error image from replicas, a forward,
a gradient or a training epoch of the proposal network.  Instruments are the
package's own (``workloads``); sizes run from a first look (1e4..1e6 rays) to
the full projection (1e9).
"""
import math

import numpy as np
import torch

import paper_2410_08747_amd as mxr
import workloads

# A projection of the phantom as first set up: 64^3 voxels, a few pixels, a
# ray count that fills no launch evenly.
QUICK = dict(kind="projection", n=64, voxel=1.0, rays=200_003, angle=0.3, strata=64, nx=61, ny=17, ne=33, early_out=False)


def listed():
    return [
        # the plain tracer's first workload: slit, absorber, position-sensitive
        # monitor, 1e6 rays; a call that is mostly launch and latency
        dict(name="basic_1e6", kind="basic", rays=1_000_000),
        # a quick look at a small phantom on a small, odd detector
        dict(name="projection_quick", **QUICK),
        # the full energy-dispersive CT projection: 256^3 phantom, 256 x 64
        # pixels x 128 energy bins, 1e9 rays
        dict(name="projection_256", kind="projection", n=256, voxel=1.0, rays=1_000_000_000, angle=0.0, strata=4096,
             nx=256, ny=64, ne=128, early_out=False),
        # a CT acquisition in small: every phantom size at two angles in one
        # captured batch
        dict(name="ct_batch", kind="batch", sizes="64,128,256,512", angles=2, rays=20_000_000, strata=1024, nx=128, ny=32,
             ne=64, form=2),
        # beamline optics: mirror, two-crystal monochromator, powder plate
        dict(name="beamline_1e8", kind="beamline", rays=100_000_000),
        # focusing instrument: a 16-lens compound refractive lens
        dict(name="crl_1e8", kind="crl", rays=100_000_000, lenses=16),
        # the projection under the paper's own fixed-step model, a third of a
        # voxel per step
        dict(name="stepping_256", kind="stepping", n=256, rays=50_000_000, angle=0.3, strata=1024, nx=256, ny=64, ne=128,
             step=1.0 / 3.0),
        # the photons scattered once in the phantom, aimed at the detector
        dict(name="scatter_256", kind="scatter", n=256, rays=20_000_000, angle=0.3, strata=1024, nx=256, ny=64, ne=128,
             order=1),
        # the error image of an importance-sampled projection: 16 replicas
        # drawn from a proposal mixture and their batch means
        dict(name="replicas_256", kind="replicas", n=256, rays=10_000_000, replicas=16, angle=0.3, strata=1024, nx=256,
             ny=64, ne=128, alpha=0.1),
        # the proposal mixtures of a whole acquisition (360 angles) from one
        # forward of the network
        dict(name="mixtures_360", kind="mixtures", rows=360, batch=4096),
        # the network's loss and gradient over one batch of rows
        dict(name="gradient_64k", kind="gradient", rows=65_536),
        # one epoch of training from the collected rows of eight runs
        dict(name="train_1m", kind="train", rows=1_048_576, batch=65_536, runs=8),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["basic", "projection", "projection", "batch", "beamline", "crl", "stepping", "scatter",
                       "replicas", "mixtures", "gradient", "train"])
    if kind == "basic":
        return dict(kind=kind, rays=_log(rng, 1e4, 1e9))
    if kind == "beamline":
        return dict(kind=kind, rays=_log(rng, 1e5, 3e8))
    if kind == "crl":
        return dict(kind=kind, rays=_log(rng, 1e5, 3e8), lenses=rng.randint(2, 24))
    if kind == "mixtures":
        return dict(kind=kind, rows=_log(rng, 1, 4096), batch=4096)
    if kind == "gradient":
        return dict(kind=kind, rows=_log(rng, 45, 131_072))
    if kind == "train":
        rows = _log(rng, 20_000, 2_000_000)
        return dict(kind=kind, rows=rows, batch=rng.choice([4096, 16_384, 65_536]), runs=rng.randint(1, 8))
    case = dict(kind=kind, n=_log(rng, 40, 256), angle=round(rng.uniform(0.0, 2.0 * math.pi), 3),
                strata=rng.choice([64, 1024, 4096]), nx=rng.randint(40, 256), ny=rng.randint(9, 64),
                ne=rng.randint(16, 128))
    if kind == "projection":
        case.update(rays=_log(rng, 1e5, 5e8), voxel=rng.choice([1.0, 1.0, 0.8]), early_out=rng.random() < 0.25)
    elif kind == "stepping":
        case.update(rays=_log(rng, 1e5, 5e7), step=rng.choice([1.0 / 3.0, 0.5, 1.0]))
    elif kind == "scatter":
        case.update(rays=_log(rng, 1e5, 1e7), order=rng.choice([1, 1, 2]))
    elif kind == "replicas":
        case.update(rays=_log(rng, 1e5, 1e7), replicas=rng.choice([8, 16, 24]), alpha=rng.choice([0.05, 0.1, 0.2]))
    else:
        sizes = rng.choice(["64,96", "64,128,256", "100,200"])
        case = dict(kind="batch", sizes=sizes, angles=rng.randint(2, 4), rays=_log(rng, 1e5, 1e7), strata=1024,
                    nx=rng.randint(40, 160), ny=rng.randint(9, 40), ne=rng.randint(16, 64), form=rng.choice([0, 2]))
    return case


# ------------------------------------------------------------- instruments --

def _volume(n, seed):
    return workloads.make_phantom(n, seed=seed)


def _instrument(case, seed):
    """The case's instrument as a neutral dict (components and arrays)."""
    kind = case["kind"]
    if kind == "basic":
        return workloads.basic_absorber()
    if kind == "beamline":
        return workloads.beamline(d_spacings=workloads.make_d_spacings(seed))
    if kind == "crl":
        return workloads.crl_focusing(n_lenses=case["lenses"])
    mu = workloads.make_mu_tables(seed)
    kw = dict(angle=case["angle"], strata=case["strata"], nx=case["nx"], ny=case["ny"], ne=case["ne"])
    if kind == "scatter":
        mu, kw["scatter_order"] = workloads.make_scatter_tables(mu, seed), case["order"]
    elif kind == "stepping":
        kw["step"] = case["step"]
    elif kind == "projection":
        kw["early_out"] = case["early_out"]
    ins = workloads.edct_projection(_volume(case["n"], seed), mu, **kw)
    for c in ins["components"]:
        if c["type"] == "phantom" and kind == "projection":
            c["voxel"] = case["voxel"]
    return ins


def _mixture(box, seed):
    """A mixture such as the network gives: eight components that cover the
    detector (the inner part of the cone) and the spectrum."""
    lo, hi = (np.array(b) for b in box)
    rng = np.random.default_rng(seed)
    g = np.zeros((8, 7))
    pi = rng.uniform(0.5, 1.5, 8)
    g[:, 0] = pi / pi.sum()
    g[:, 1] = rng.uniform(0.8 * lo[0], 0.8 * hi[0], 8)
    g[:, 2] = rng.uniform(0.2 * lo[1], 0.2 * hi[1], 8)
    g[:, 3] = rng.uniform(35.0, 120.0, 8)
    g[:, 4] = rng.uniform(0.1, 0.4, 8) * hi[0]
    g[:, 5] = rng.uniform(0.08, 0.2, 8) * hi[1]
    g[:, 6] = rng.uniform(15.0, 40.0, 8)
    return g.reshape(56)


# ----------------------------------------------------------------- network --

def _box():
    hi = math.tan(workloads.edct_half_angle())
    return (-hi, -hi, 20.0), (hi, hi, 150.0)


def _parameters(seed):
    rng = np.random.default_rng(seed)
    p = workloads.init_mlp_params(seed)
    return (p + rng.normal(0.0, 0.05, p.shape)).astype(np.float32)


def _contexts(rows, rng):
    """Contexts of projections: angle as cos and sin, phantom size."""
    a = rng.uniform(0.0, 2.0 * math.pi, rows)
    size = np.log2(rng.choice([64.0, 128.0, 256.0, 512.0], rows)) / 9.0
    z = np.zeros(rows)
    return np.stack([z, z, z, np.cos(a), np.sin(a), size], 1).astype(np.float32)


def _targets(rows, rng, lo, hi):
    """Detected rays: directions over the detector, tube energies."""
    y = np.empty((rows, 3))
    y[:, 0] = rng.uniform(0.95 * lo[0], 0.95 * hi[0], rows)
    y[:, 1] = rng.uniform(0.24 * lo[1], 0.24 * hi[1], rows)
    y[:, 2] = np.clip(rng.normal(75.0, 25.0, rows), lo[2] + 0.01, hi[2] - 0.01)
    return y


def _gradient_inputs(case, seed):
    rng = np.random.default_rng(seed)
    lo, hi = _box()
    rows = case["rows"]
    return _parameters(seed), _contexts(rows, rng), _targets(rows, rng, lo, hi), rng.uniform(0.1, 2.0, rows)


# -------------------------------------------------------------------- cases --

def prepare(case, seed):
    kind = case["kind"]
    state = dict(case=case, seed=seed)
    dev = torch.device("cuda", torch.cuda.current_device())
    if kind == "mixtures":
        lo, hi = _box()
        state.update(net=mxr.ProposalNet(_parameters(seed), batch=case["batch"]), lo=lo, hi=hi,
                     ctx=torch.tensor(_contexts(case["rows"], np.random.default_rng(seed + 1)), device=dev))
        return state
    if kind == "gradient":
        lo, hi = _box()
        p, ctx, y, omega = _gradient_inputs(case, seed)
        state.update(net=mxr.ProposalNet(p, batch=case["rows"]), lo=lo, hi=hi, ctx=torch.tensor(ctx, device=dev),
                     y=torch.tensor(y, device=dev), omega=torch.tensor(omega, device=dev))
        return state
    if kind == "train":
        # rows of several collecting runs, each with its monitor image, and
        # a network in the middle of its training (moments and step count)
        rng = np.random.default_rng(seed)
        rows, runs, bins = case["rows"], case["runs"], 256 * 64 * 128
        ins = mxr.Instrument(workloads.edct_projection(_volume(64, seed), workloads.make_mu_tables(seed)))
        lo, hi = ins.proposal_box()
        gen = torch.Generator(device=dev).manual_seed(seed)
        images = [torch.rand(bins, generator=gen, dtype=torch.float64, device=dev) * 1e3 for _ in range(runs)]
        hits = dict(ctx=torch.tensor(_contexts(rows, rng), device=dev),
                    y=torch.tensor(_targets(rows, rng, lo, hi), device=dev),
                    w=torch.rand(rows, generator=gen, dtype=torch.float64, device=dev) + 0.1,
                    bin=torch.randint(0, bins, (rows,), generator=gen, dtype=torch.int64, device=dev))
        net = mxr.ProposalNet(_parameters(seed), batch=case["batch"])
        net.m.normal_(0.0, 1e-3, generator=gen)
        net.v.uniform_(1e-5, 1e-4, generator=gen)
        net.step = 1000
        state.update(ins=ins, hits=hits, images=images, net=net, first=[rows * r // runs for r in range(runs + 1)])
        return state
    if kind == "batch":
        mu = workloads.make_mu_tables(seed)
        shared, jobs = {}, []
        bins = case["nx"] * case["ny"] * case["ne"]
        sizes = [int(x) for x in case["sizes"].split(",")]
        count = torch.zeros(len(sizes) * case["angles"], bins, dtype=torch.int64, device=dev)
        sums = torch.zeros(len(sizes) * case["angles"], 2, bins, dtype=torch.float64, device=dev)
        for s, n in enumerate(sizes):
            volume = _volume(n, seed + s)
            for a in range(case["angles"]):
                ins = workloads.edct_projection(volume, mu, angle=2.0 * math.pi * a / case["angles"] + 0.1 * s,
                                                strata=case["strata"], nx=case["nx"], ny=case["ny"], ne=case["ne"])
                j = len(jobs)
                tallies = [dict(count=count[j], sum_w=sums[j, 0], sum_w2=sums[j, 1])]
                jobs.append((mxr.Instrument(ins, shared=shared), case["rays"], seed, j, tallies))
        state.update(jobs=jobs, batch=mxr.Batch(jobs, schedule=(case["form"], 0, 0, 1)), count=count, sums=sums)
        return state
    ins = mxr.Instrument(_instrument(case, seed))
    state["ins"] = ins
    if kind == "replicas":
        ins.set_proposal(torch.tensor(_mixture(ins.proposal_box(), seed), device=dev), alpha=case["alpha"])
        bins = case["nx"] * case["ny"] * case["ne"]
        state["count"] = torch.zeros(bins, dtype=torch.int64, device=dev)
        state["sum_w2"] = torch.zeros(bins, dtype=torch.float64, device=dev)
        state["sums"] = torch.zeros(case["replicas"], bins, dtype=torch.float64, device=dev)
    return state


def run(state):
    case, seed = state["case"], state["seed"]
    kind = case["kind"]
    if kind == "mixtures":
        out = state["net"].forward(state["ctx"])
        return dict(out=out, gmm=state["net"].mixture(out, state["lo"], state["hi"]))
    if kind == "gradient":
        loss, grad = state["net"].loss_grad(state["ctx"], state["y"], state["omega"], state["lo"], state["hi"])
        return dict(loss=loss, grad=grad)
    if kind == "train":
        net = state["net"]
        steps = -(-case["rows"] // min(case["batch"], case["rows"]))
        log = torch.empty(steps, dtype=torch.float64, device=net.device)
        omega = net.train_from_runs(state["ins"], state["hits"], state["first"], state["images"], epochs=1, lr=1e-4,
                                    seed=7, loss_log=log)
        return dict(omega=omega, loss=log, grad=net.grad, master=net.master, m=net.m, v=net.v)
    if kind == "batch":
        state["count"].zero_()
        state["sums"].zero_()
        state["batch"].run()
        return dict(count=state["count"], sums=state["sums"])
    if kind == "replicas":
        for k in ("count", "sum_w2", "sums"):
            state[k].zero_()
        for r in range(case["replicas"]):
            state["ins"].run(case["rays"], seed=seed, purpose=3 + r,
                             tallies=[dict(count=state["count"], sum_w=state["sums"][r], sum_w2=state["sum_w2"])])
        mean, rel = mxr.batch_means(state["sums"], case["rays"])
        return dict(mean=mean, rel=rel, count=state["count"], sum_w2=state["sum_w2"])
    return state["ins"].run(case["rays"], seed=seed)


def work(case):
    """Operations and bytes of one pass that no implementation can do without.

    Tracing: every emitted ray's draw, source and monitor arithmetic; the walk
    (6 operations a crossing) for the rays that reach the monitor (0.30 of the
    cone); tables and volumes read once, images written once.  Network: its
    products, its rows and parameters."""
    kind = case["kind"]
    per_row = 2 * (6 * 128 + 128 * 128 + 128 * 56)
    if kind == "mixtures":
        return dict(bytes=case["rows"] * (24 + 56 * 12) + 2 * 24632, flops=case["rows"] * per_row)
    if kind == "gradient":
        return dict(bytes=case["rows"] * 56 + 6 * 24632, flops=3.0 * case["rows"] * per_row)
    if kind == "train":
        steps = -(-case["rows"] // min(case["batch"], case["rows"]))
        image = case["runs"] * 256 * 64 * 128 * 8
        return dict(bytes=case["rows"] * (24 + 24 + 16 + 8) + image + steps * 24632 * 26,
                    flops=3.0 * case["rows"] * per_row)
    if kind == "basic":
        return dict(bytes=128 * 128 * 24, flops=120.0 * case["rays"])
    if kind == "beamline":
        return dict(bytes=1024 * 1024 * 24, flops=400.0 * case["rays"])
    if kind == "crl":
        return dict(bytes=(120 * 120 + 130) * 24, flops=case["rays"] * (120.0 + 0.126 * 136.0 * case["lenses"]))
    image = case["nx"] * case["ny"] * case["ne"] * 24
    if kind == "batch":
        sizes = [int(x) for x in case["sizes"].split(",")]
        walk = sum(120.0 + 0.3 * 6.0 * 1.05 * n for n in sizes) * case["angles"] * case["rays"]
        return dict(bytes=sum(n ** 3 for n in sizes) + len(sizes) * case["angles"] * image, flops=walk)
    n = case["n"]
    crossings = 1.05 * n
    if kind == "stepping":
        crossings = n / case["step"]
    elif kind == "scatter":
        crossings = (2 * case["order"] + 1) * 1.05 * n / 0.3
    rays = case["rays"]
    if kind == "replicas":
        rays, image = rays * case["replicas"], image * (case["replicas"] + 4) / 3
        return dict(bytes=n ** 3 + image, flops=rays * (300.0 + 0.85 * 6.0 * crossings))
    return dict(bytes=n ** 3 + image, flops=rays * (120.0 + 0.3 * 6.0 * crossings))


# -------------------------------------------------------------------- exact --

def _uniforms(seed, ray, index):
    """Uniform ``index`` of each ray: Philox4x32-10, key = seed, counter =
    (block, ray low, ray high, 0)."""
    lo32 = np.uint64(0xFFFFFFFF)
    x = [np.full_like(ray, index // 2), ray & lo32, ray >> np.uint64(32), np.zeros_like(ray)]
    k = [seed & 0xFFFFFFFF, (seed >> 32) & 0xFFFFFFFF]
    for _ in range(10):
        a, b = np.uint64(0xD2511F53) * x[0], np.uint64(0xCD9E8D57) * x[2]
        x = [(b >> np.uint64(32)) ^ x[1] ^ np.uint64(k[0]), b & lo32, (a >> np.uint64(32)) ^ x[3] ^ np.uint64(k[1]), a & lo32]
        k = [(k[0] + 0x9E3779B9) & 0xFFFFFFFF, (k[1] + 0xBB67AE85) & 0xFFFFFFFF]
    lo, hi = (x[2], x[3]) if index & 1 else (x[0], x[1])
    return (((hi << np.uint64(32)) | lo) >> np.uint64(12)).astype(np.float64) * 2.0 ** -52 + 2.0 ** -53


def _image(det, x, y, E, w):
    """Histogram sums of weights at the monitor's plane."""
    ix = np.floor((x - det["xmin"]) * (det["nx"] / (det["xmax"] - det["xmin"])))
    iy = np.floor((y - det["ymin"]) * (det["ny"] / (det["ymax"] - det["ymin"])))
    ie = np.floor((E - det["emin"]) * (det["ne"] / (det["emax"] - det["emin"])))
    ok = (ix >= 0) & (ix < det["nx"]) & (iy >= 0) & (iy < det["ny"]) & (ie >= 0) & (ie < det["ne"])
    b = ((iy * det["nx"] + ix) * det["ne"] + ie)[ok].astype(np.int64)
    bins = det["nx"] * det["ny"] * det["ne"]
    return [dict(count=None, sum_w=np.bincount(b, w[ok], bins), sum_w2=np.bincount(b, w[ok] ** 2, bins))]


def _exact_basic(case, seed):
    src, slit, box, det = workloads.basic_absorber()["components"]
    ray = np.arange(case["rays"], dtype=np.uint64)
    u = [_uniforms(seed, ray, i) for i in range(5)]
    x, y = (u[0] - 0.5) * src["wx"], (u[1] - 0.5) * src["wy"]
    sh = np.sqrt(u[2]) * math.sin(0.5 * src["half_angle"])
    st, cz = 2.0 * sh * np.sqrt(1.0 - sh * sh), 1.0 - 2.0 * sh * sh
    dx, dy = st * np.cos(2.0 * math.pi * u[3]), st * np.sin(2.0 * math.pi * u[3])
    E = src["emin"] + (src["emax"] - src["emin"]) * u[4]
    z = slit["pos"][2]
    keep = (np.abs(x + z / cz * dx) <= 0.5 * slit["w"]) & (np.abs(y + z / cz * dy) <= 0.5 * slit["h"])
    x, y, dx, dy, cz, E = (v[keep] for v in (x, y, dx, dy, cz, E))
    near, far = np.zeros(len(x)), np.full(len(x), np.inf)
    for q, d, h, c in ((x, dx, box["hx"], 0.0), (y, dy, box["hy"], 0.0), (np.zeros(len(x)), cz, box["hz"], box["pos"][2])):
        a, b = (c - h - q) / d, (c + h - q) / d
        near, far = np.maximum(near, np.minimum(a, b)), np.minimum(far, np.maximum(a, b))
    L = np.maximum(far - near, 0.0)
    w = np.exp(-(box["mu_a"] / E ** 3 + box["mu_b"]) * L / 10.0)
    t = det["pos"][2] / cz
    return _image(det, x + t * dx, y + t * dy, E, w)


def _exact_projection(case, seed):
    ins = _instrument(case, seed)
    src, ph, det = ins["components"][0], ins["components"][-2], ins["components"][-1]
    N, G = case["rays"], case["strata"]
    while G > 1 and 16 * G * G > N:
        G -= 1
    ray = np.arange(N, dtype=np.uint64)
    g2 = np.uint64(G * G)
    cell = ray * g2 // np.uint64(N)
    start = lambda c: (c * np.uint64(N) + g2 - np.uint64(1)) // g2  # noqa: E731
    factor = (N / (G * G)) / (start(cell + np.uint64(1)) - start(cell)).astype(np.float64)
    cx, cy = (cell % np.uint64(G)).astype(np.float64), (cell // np.uint64(G)).astype(np.float64)
    u = [_uniforms(seed, ray, i) for i in range(3)]
    a, b = 2.0 * (cx + u[0]) / G - 1.0, 2.0 * (cy + u[1]) / G - 1.0
    wide = np.abs(a) > np.abs(b)
    rad = np.where(wide, a, b)
    phi = np.where(wide, math.pi / 4 * b / np.where(wide, a, 1.0), math.pi / 2 - math.pi / 4 * a / np.where(wide, 1.0, b))
    s = math.sin(0.5 * src["half_angle"])
    sh = np.abs(rad) * s
    k = 2.0 * s * np.sqrt(1.0 - sh * sh)
    d = np.stack([k * rad * np.cos(phi), k * rad * np.sin(phi), 1.0 - 2.0 * sh * sh], 1)
    E = src["emin"] + (src["emax"] - src["emin"]) * u[2]
    t = det["pos"][2] / d[:, 2]
    x, y = t * d[:, 0], t * d[:, 1]
    hit = (x >= det["xmin"]) & (x < det["xmax"]) & (y >= det["ymin"]) & (y < det["ymax"])
    d, E, x, y, factor = d[hit], E[hit], x[hit], y[hit], factor[hit]
    e0 = src["e0"]
    cont = src["f_cont"] / (e0 * math.log(src["emax"] / src["emin"]) - (src["emax"] - src["emin"])) * (e0 - E) / E
    for line, f in (("1", src["f_line1"]), ("2", src["f_line2"])):
        z = (E - src["e_line" + line]) / src["line_sigma"]
        cont = cont + f * np.exp(-0.5 * z * z) / (src["line_sigma"] * math.sqrt(2.0 * math.pi))
    w = (src["emax"] - src["emin"]) * cont * factor
    rot, pos, vol, v = np.asarray(ph["rot"]), np.asarray(ph["pos"]), ph["volume"], ph["voxel"]
    mu = np.asarray(ph["mu_table"])
    e = np.clip(np.floor((E - ph["table_emin"]) * (mu.shape[1] / (ph["table_emax"] - ph["table_emin"]))), 0, mu.shape[1] - 1).astype(int)
    q, dl = -(rot @ pos), d @ rot.T
    n = np.array(vol.shape[::-1])
    corner = -0.5 * n * v
    tau = np.zeros(len(E))
    for i0 in range(0, len(E), 20_000):
        dd = dl[i0:i0 + 20_000]
        cuts = [(corner[i] + v * np.arange(n[i] + 1) - q[i])[None, :] / dd[:, i:i + 1] for i in range(3)]
        near = np.maximum.reduce([np.minimum(c[:, 0], c[:, -1]) for c in cuts] + [np.zeros(len(dd))])
        far = np.minimum.reduce([np.maximum(c[:, 0], c[:, -1]) for c in cuts])
        far = np.maximum(far, near)
        alpha = np.sort(np.clip(np.concatenate(cuts, 1), near[:, None], far[:, None]), 1)
        mid, length = 0.5 * (alpha[:, 1:] + alpha[:, :-1]), np.diff(alpha, axis=1)
        idx = [np.clip(np.floor((q[i] + mid * dd[:, i:i + 1] - corner[i]) / v), 0, n[i] - 1).astype(int) for i in range(3)]
        tau[i0:i0 + 20_000] = np.sum(mu[vol[idx[2], idx[1], idx[0]], e[i0:i0 + 20_000, None]] * length, 1) / 10.0
    return _image(det, x, y, E, w * np.exp(-tau))


def _network(p, ctx):
    """Outputs of the network in 64 bits at its bfloat16 parameters."""
    at, w = 0, []
    for shape in ((6, 128), (128,), (128, 128), (128,), (128, 56), (56,)):
        size = math.prod(shape)
        w.append(p[at:at + size].reshape(shape))
        at += size
    h = torch.nn.functional.silu(ctx @ w[0] + w[1])
    h = torch.nn.functional.silu(h @ w[2] + w[3])
    return h @ w[4] + w[5]


def _head(o, lo, hi):
    lo, hi = (torch.tensor(b, dtype=torch.float64) for b in (lo, hi))
    o = o.reshape(-1, 8, 7)
    mu = 0.5 * (lo + hi) + 0.5 * (hi - lo) * torch.tanh(o[:, :, 1:4])
    sigma = 0.5 * (hi - lo) * (1e-3 + torch.nn.functional.softplus(o[:, :, 4:7], threshold=1e9))
    return torch.softmax(o[:, :, 0], 1), mu, sigma


def exact(case, seed):
    kind = case["kind"]
    if kind == "basic" and case["rays"] <= 4_000_000:
        return _exact_basic(case, seed)
    if kind == "projection" and case["rays"] <= 1_000_000 and case["n"] <= 128 and not case["early_out"]:
        return _exact_projection(case, seed)
    if kind == "mixtures":
        p = torch.tensor(_parameters(seed)).bfloat16().double()
        o = _network(p, torch.tensor(_contexts(case["rows"], np.random.default_rng(seed + 1))).double())
        pi, mu, sigma = _head(o, *_box())
        return dict(out=o, gmm=torch.cat([pi[:, :, None], mu, sigma], 2).reshape(-1, 56))
    if kind == "gradient":
        p, ctx, y, omega = _gradient_inputs(case, seed)
        p = torch.tensor(p).bfloat16().double().requires_grad_()
        lo, hi = _box()
        pi, mu, sigma = _head(_network(p, torch.tensor(ctx).double()), lo, hi)
        z = (torch.tensor(y)[:, None, :] - mu) / sigma
        dens = torch.log(pi) - (0.5 * z * z + torch.log(sigma) + 0.5 * math.log(2.0 * math.pi)).sum(2)
        edge = lambda b: torch.special.ndtr((torch.tensor(b, dtype=torch.float64) - mu) / sigma)  # noqa: E731
        mass = (pi * (edge(hi) - edge(lo)).prod(2)).sum(1)
        w = torch.tensor(omega)
        loss = (w * (torch.log(mass) - torch.logsumexp(dens, 1))).sum() / w.sum()
        loss.backward()
        return dict(loss=loss.detach().reshape(1), grad=p.grad)
    return None
