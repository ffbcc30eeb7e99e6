"""Performance cases of the particle-filter library.

A case is a plain dict; `listed()` gives the fixed ones, `draw()` more of the
same ranges, `prepare()` what a program holds before the call, `run()` one
pass through the public entry points, `work()` what the pass cannot do
without, and `exact()` the same outputs in plain 64-bit torch.

Kinds of case:
  track     one filter over one movie: reset, one step per frame, the
            estimate read after every frame (a live tracker) or the
            log-likelihood alone at the end (offline analysis), and the
            resampled cloud at the end
  batch     one filter per spot of a movie, stepped together, every track's
            statistics read after every frame
  loglik    log p^ of a movie and its gradient through torch autograd
            (parameter fitting): forward and backward
  resample  standalone resampling of log weights, systematic (with caller
            scratch or the library's static scratch) or RNA
  schedule  a dynamic load balancing schedule of group counts

A movie pass starts from a reset, so each pass covers the spread-out first
frames, where the cloud collapses onto the spot, as well as the steady ones.
"""
import math

import numpy as np
import torch

import paper_1310_5045_amd as ppf
from paper_1310_5045_amd import synth

BACKGROUND, NOISE, INTENSITY = 10.0, 3.0, 30.0
# process noise, and the priors of the velocities and the intensity
Q = (0.5, 0.5, 0.1, 0.1, 1.0)
# linear-Gaussian model: prior, and the sds of the three observed components
LG_MEAN, LG_SD, LG_R = (64.0, 64.0, 0.5, -0.3, 30.0), (2.0, 2.0, 0.3, 0.3, 3.0), (0.7, 0.7, 1.5)
SCHEMES = {"systematic": (0, 0), "rna": (1, 0), "arna": (3, 0), "rpa_gs": (2, 0), "rpa_sgs": (2, 1)}
INITS = {"uniform": 0, "gaussian": 1, "stratified": 2, "zorder": 3}
SCHEDULES = {"sgs": 1, "lgs": 2}


def track(name, n, width, height, sigma, frames, **more):
    """A `track` case. box: half width of the initial box around the spot's
    first position (0: the whole frame); half: resample when ESS < N / 2
    instead of at every step; each: read the estimate after every frame."""
    c = dict(name=name, kind="track", n=n, width=width, height=height, sigma=sigma, frames=frames,
             scheme="systematic", group=0, half=False, init="uniform", box=0, model="spot",
             graph=False, each=True, shape=0)
    c.update(more)
    if name is None:
        del c["name"]
    return c


def listed():
    return [
        # the smallest workload of the benchmark's table: a live tracker on a
        # small crop, bound by launches and by reading the estimate
        track("live_4k", 4096, 128, 128, 1.5, 10),
        # the middle workload: a camera frame at 2^20 particles, resampled
        # when the sample degenerates, the step replayed as a HIP graph
        track("live_1m", 1 << 20, 512, 512, 1.5, 20, half=True, init="zorder", graph=True),
        # the headline workload: 38 million particles, 13 x 13 patches
        track("movie_38m", 38_000_000, 1024, 1024, 2.0, 8, init="zorder", shape=1),
        # a wide spot (25 x 25 patches, the largest) on a frame that is not
        # square, from a Gaussian prior around it; a ragged particle count
        track("wide_spot_250k", 250_007, 640, 480, 4.0, 8, init="gaussian", box=4),
        # the linear-Gaussian model over a long record, read only at its end
        track("linear_100k", 100_003, 0, 0, 0.0, 50, half=True, init="gaussian", model="linear",
              each=False),
        # distributed resampling, one group per workgroup: RNA, ARNA, and
        # proportional allocation with sorted greedy routing
        track("rna_1m", 1 << 20, 512, 512, 1.5, 10, scheme="rna", group=256, half=True,
              init="zorder", graph=True),
        track("arna_300k", 300_000, 512, 512, 1.5, 10, scheme="arna", group=1000, half=True,
              init="zorder"),
        track("rpa_sgs_1m", 1 << 20, 512, 512, 1.5, 10, scheme="rpa_sgs", group=256, half=True,
              init="zorder", graph=True),
        # one evaluation of the objective of a parameter fit, with its gradient
        dict(name="loglik_grad_262k", kind="loglik", n=1 << 18, width=512, height=512, sigma=1.7,
             frames=30),
        # every spot of a movie at once
        dict(name="spots_256", kind="batch", tracks=256, n_lo=1024, n_hi=262144, width=1024,
             height=1024, sigma_lo=1.2, sigma_hi=2.5, frames=5, graph=True),
        # the standalone resampler in another program's filter
        dict(name="resample_16m", kind="resample", scheme="systematic", n=16_777_213, spread=4.0,
             group=0),
        # the schedule of Sorted Greedy for the groups of the 38 M workload
        dict(name="schedule_152k", kind="schedule", schedule="sgs", groups=152_000, n=250),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["live", "movie", "movie", "wide", "linear", "group", "group", "loglik",
                       "batch", "resample", "rna", "schedule"])
    if kind == "live":  # small crops, from a box around the spot
        w = rng.randint(48, 256)
        return track(None, _log(rng, 500, 60_000), w, rng.randint(48, 256),
                     round(rng.uniform(0.7, 2.6), 3), rng.randint(5, 15), box=rng.randint(8, 20),
                     graph=rng.random() < 0.5, half=rng.random() < 0.5)
    if kind == "movie":
        n = _log(rng, 60_000, 16_000_000)
        return track(None, n, rng.randint(256, 1024), rng.randint(256, 1024),
                     round(rng.uniform(1.0, 2.3), 3), rng.randint(4, 8),
                     init=rng.choice(["zorder", "stratified"]), half=rng.random() < 0.5,
                     each=rng.random() < 0.7, graph=rng.random() < 0.5, shape=rng.randint(0, 1))
    if kind == "wide":
        return track(None, _log(rng, 20_000, 1_000_000), rng.randint(200, 1024),
                     rng.randint(200, 1024), round(rng.uniform(2.4, 4.3), 3), rng.randint(4, 10),
                     init=rng.choice(["gaussian", "zorder"]), box=rng.randint(3, 8))
    if kind == "linear":
        return track(None, _log(rng, 1000, 2_000_000), 0, 0, 0.0, rng.randint(10, 50),
                     half=rng.random() < 0.7, init="gaussian", model="linear",
                     each=rng.random() < 0.5, graph=rng.random() < 0.5)
    if kind == "group":
        scheme = rng.choice(["rna", "arna", "rpa_gs", "rpa_sgs"])
        group = rng.choice([100, 250, 256, 512, 777, 1000, 1024])
        return track(None, group * _log(rng, 40, 4000), rng.randint(128, 640),
                     rng.randint(128, 640), round(rng.uniform(1.0, 2.0), 3), rng.randint(5, 12),
                     scheme=scheme, group=group, half=rng.random() < 0.6, init="zorder",
                     graph=rng.random() < 0.5)
    if kind == "loglik":
        return dict(kind="loglik", n=_log(rng, 5000, 2_000_000), width=rng.randint(128, 768),
                    height=rng.randint(128, 768), sigma=round(rng.uniform(1.0, 2.3), 3),
                    frames=rng.randint(8, 30))
    if kind == "batch":
        return dict(kind="batch", tracks=rng.randint(5, 256), n_lo=1024,
                    n_hi=_log(rng, 8192, 262144), width=rng.randint(512, 1024),
                    height=rng.randint(512, 1024), sigma_lo=1.2, sigma_hi=2.5,
                    frames=rng.randint(3, 6), graph=rng.random() < 0.5)
    if kind == "resample":
        n = _log(rng, 1000, 16_000_000)
        static = n <= ppf.STATIC_MAX_N and rng.random() < 0.5
        return dict(kind="resample", scheme="static" if static else "systematic", n=n,
                    spread=round(rng.uniform(0.5, 30.0), 2), group=0)
    if kind == "rna":
        group = rng.choice([64, 250, 256, 999, 1024])
        return dict(kind="resample", scheme="rna", n=group * _log(rng, 20, 16_000),
                    spread=round(rng.uniform(0.5, 10.0), 2), group=group)
    return dict(kind="schedule", schedule=rng.choice(["sgs", "lgs"]),
                groups=_log(rng, 50, 152_000), n=rng.randint(32, 1024))


# ---------------------------------------------------------------- inputs
def _movie(c, seed):
    """The movie (or observation record) of a track or loglik case, and the
    parameters of its filter."""
    if c.get("model") == "linear":
        rec = synth.linear_gaussian_track(c["frames"], LG_MEAN, LG_SD, Q, LG_R, seed=seed)
        p = dict(obs_model=ppf.OBS_LINEAR_GAUSSIAN, init_kind=ppf.INIT_GAUSSIAN, init_a=LG_MEAN,
                 init_b=LG_SD, lg_r=LG_R)
        return rec.obs, p
    W, H = c["width"], c["height"]
    mv = synth.render_movie(W, H, c["frames"], intensity=INTENSITY, sigma=c["sigma"],
                            background=BACKGROUND, noise_sd=NOISE, seed=seed)
    x, y = (float(v) for v in mv.truth[0, 0])
    r = c.get("box", 5)
    lo, hi = (-1, -1, INTENSITY / 2), (1, 1, 1.5 * INTENSITY)
    if c.get("init") == "gaussian":
        a, b = (x, y, 0, 0, INTENSITY), (r, r, 0.7, 0.7, INTENSITY / 5)
    elif r:
        a, b = (x - r, y - r) + lo, (x + r, y + r) + hi
    else:
        a, b = (0, 0) + lo, (W, H) + hi
    p = dict(width=W, height=H, psf_sigma=c["sigma"], background=BACKGROUND, noise_sigma=NOISE,
             init_kind=INITS[c.get("init", "uniform")], init_a=a, init_b=b)
    return mv.frames, p


def _params(c, p, seed):
    resample, dlb = SCHEMES[c.get("scheme", "systematic")]
    n = c["n"]
    more = {}
    if c.get("group"):
        more = dict(rna_group=c["group"])
    if c.get("scheme") == "arna":
        more.update(rna_exchange=0.5, arna_min=0.05)
    return ppf.params(n_particles=n, q=Q, resample=resample, dlb=dlb, seed=seed,
                      ess_threshold=n / 2 if c.get("half") else math.inf, **more, **p)


def _spots(c, seed):
    """A movie of many spots and the parameters of one filter per spot."""
    W, H, T = c["width"], c["height"], c["tracks"]
    mv = synth.render_movie(W, H, c["frames"], n_spots=T, intensity=(15.0, 60.0),
                            sigma=(c["sigma_lo"], c["sigma_hi"]), vmax=2.0,
                            start_box=(0, W, 0, H), seed=seed)
    rng = np.random.default_rng(seed)
    ns = np.rint(np.exp(rng.uniform(math.log(c["n_lo"]), math.log(c["n_hi"]), T))).astype(int)
    if c["tracks"] == 256:  # the sizes are the workload's own, whatever the seed
        ns = np.rint(np.exp(np.random.default_rng(1).uniform(math.log(c["n_lo"]),
                                                             math.log(c["n_hi"]), T))).astype(int)
    ps = []
    for t in range(T):
        x, y = (float(v) for v in mv.truth[0, t])
        I = float(mv.intensity[t])
        ps.append(ppf.params(n_particles=int(ns[t]), width=W, height=H,
                             psf_sigma=float(mv.sigma[t]), background=BACKGROUND,
                             noise_sigma=NOISE, q=Q, init_a=(x - 5, y - 5, -2, -2, I / 2),
                             init_b=(x + 5, y + 5, 2, 2, 1.5 * I), ess_threshold=math.inf,
                             seed=seed, track_id=t))
    return mv.frames, ps


def _frames(frames):
    dev = torch.from_numpy(np.ascontiguousarray(frames, dtype=np.float32)).cuda()
    return [dev[k] for k in range(dev.shape[0])]


def _weights(c, seed):
    """Log weights as a likelihood gives them: minus half the square of a
    normal, times the spread (the larger, the fewer particles that matter)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    z = torch.randn(c["n"], generator=g, device="cuda")
    return (-0.5 * c["spread"] * z * z).contiguous()


def _counts(c, seed):
    """Offspring counts of the groups under a posterior that favours some of
    them, summing to groups * n. The seed deals the same counts to other
    groups: the number of schedule entries is then the same for every seed."""
    share = np.random.default_rng(1).gamma(0.5, 1.0, c["groups"])
    edges = np.floor(np.cumsum(share) / share.sum() * c["groups"] * c["n"] + 0.5).astype(np.int64)
    counts = np.diff(edges, prepend=0).astype(np.int32)
    return np.random.default_rng(seed).permutation(counts)


def prepare(case, seed):
    c, kind = case, case["kind"]
    seed = seed & 0x7FFFFFFF
    if kind == "track":
        obs, p = _movie(c, seed)
        f = ppf.Filter(_params(c, p, seed))
        if c["shape"]:
            f.set_shape(c["shape"])
        if c["graph"]:
            f.graph(True)
        out = torch.empty((5, c["n"]), dtype=torch.float32, device="cuda")
        return dict(kind=kind, filter=f, frames=_frames(obs), each=c["each"], out=out)
    if kind == "batch":
        frames, ps = _spots(c, seed)
        b = ppf.Batch(ps)
        if c["graph"]:
            b.graph(True)
        return dict(kind=kind, batch=b, frames=_frames(frames))
    if kind == "loglik":
        obs, p = _movie(c, seed)
        base = _params(c, p, seed)
        theta = torch.tensor(ppf.theta_of(base), dtype=torch.float64)
        return dict(kind=kind, theta=theta, base=base, frames=torch.from_numpy(obs).cuda())
    if kind == "resample":
        lw = _weights(c, seed)
        rng = np.random.default_rng(seed)
        st = dict(kind=kind, scheme=c["scheme"], logw=lw, u=float(rng.random()))
        if c["scheme"] == "rna":
            st.update(group=c["group"], moved=c["group"] // 10,
                      u=torch.from_numpy(rng.random(c["n"] // c["group"])).cuda())
        return st
    return dict(kind=kind, schedule=SCHEDULES[c["schedule"]], n=c["n"],
                counts=torch.from_numpy(_counts(c, seed)).cuda())


# ------------------------------------------------------------------ one pass
def run(state):
    kind = state["kind"]
    if kind == "track":
        f = state["filter"]
        f.reset()
        seen = []
        for z in state["frames"]:
            f.step(z)
            if state["each"]:
                seen.append(f.estimate())
        if not state["each"]:
            seen.append(f.estimate())
        cum, _ = f.loglik()
        return {"mean": np.stack([m for m, _ in seen]), "ess": np.array([e for _, e in seen]),
                "loglik": cum, "cloud": f.gather(state["out"])}
    if kind == "batch":
        b = state["batch"]
        b.reset()
        mean, ess, delta = [], [], []
        for z in state["frames"]:
            b.step(z)
            sts = b.stats()
            mean.append([s["mean"] for s in sts])
            ess.append([s["ess"] for s in sts])
            delta.append([s["delta"] for s in sts])
        return {"mean": np.array(mean), "ess": np.array(ess), "delta": np.array(delta)}
    if kind == "loglik":
        theta = state["theta"].clone().requires_grad_(True)
        value = ppf.loglik(theta, state["frames"], state["base"])
        value.backward()
        return {"loglik": value.detach(), "grad": theta.grad}
    if kind == "resample":
        if state["scheme"] == "rna":
            anc, lwg = ppf.resample_rna(state["logw"], state["group"], state["moved"], state["u"])
            return {"ancestors": anc, "group_logw": lwg}
        if state["scheme"] == "static":
            return {"ancestors": ppf.resample_systematic_static(state["logw"], state["u"])}
        return {"ancestors": ppf.resample_systematic(state["logw"], state["u"])}
    return {"entries": ppf.dlb_schedule(state["schedule"], state["counts"], state["n"])}


def _patch(sigma):
    return 2 * int(math.floor(3.0 * float(np.float32(sigma)))) + 1


def work(case):
    """Per particle and frame: the parent's index and state read, the new
    state and weight written, the weight read and the ancestor written by the
    resampling (56 bytes), and the P x P patch (a multiply-add for the spot's
    profile and one for the residual's square per pixel, in 64 bits)."""
    c, kind = case, case["kind"]
    if kind == "track":
        n, T = c["n"], c["frames"]
        per = 4 * _patch(c["sigma"]) ** 2 if c["model"] == "spot" else 60
        # the initial cloud written; the resampled cloud read and written
        return {"bytes": n * T * 56 + n * 20 + n * 44 + T * 4 * c["width"] * c["height"],
                "flops": n * T * per}
    if kind == "loglik":
        n, T = c["n"], c["frames"]
        # and seven tangents per particle read and written; three operations a pixel
        return {"bytes": n * T * (56 + 56) + n * 48 + T * 4 * c["width"] * c["height"],
                "flops": n * T * 8 * _patch(c["sigma"]) ** 2}
    if kind == "batch":
        # the mean of log-uniform particle counts, and of the squared patch edge
        span = c["n_hi"] - c["n_lo"]
        n = c["tracks"] * span / math.log(c["n_hi"] / c["n_lo"])
        return {"bytes": n * c["frames"] * 56 + n * 20 + c["frames"] * 4 * c["width"] * c["height"],
                "flops": n * c["frames"] * 4 * 11 ** 2}
    if kind == "resample":
        return {"bytes": c["n"] * 8, "flops": c["n"] * 20}
    # the counts read, an entry of three numbers for each group or so written
    return {"bytes": c["groups"] * 16, "flops": c["groups"] * 20}


# ------------------------------------------------------- 64-bit references
M32 = 0xFFFFFFFF


def _mulhilo(a, x):
    """High and low halves of the 64-bit product of the constant a and x < 2^32."""
    lo16, hi16 = a * (x & 0xFFFF), a * (x >> 16)
    return (hi16 + (lo16 >> 16)) >> 16, (lo16 + ((hi16 & 0xFFFF) << 16)) & M32


def _philox(index, k, purpose, block, seed, track):
    """Philox4x32-10 (Salmon et al., SC'11) of the counters (index, k, purpose
    << 24 | block, track) under the key `seed`."""
    x = [index & M32, torch.full_like(index, k), torch.full_like(index, purpose << 24 | block),
         torch.full_like(index, track)]
    k0, k1 = seed & M32, seed >> 32
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2511F53, x[0])
        h1, l1 = _mulhilo(0xCD9E8D57, x[2])
        x = [h1 ^ x[1] ^ k0, l1, h0 ^ x[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return x


def _normals(w):
    """Five normals of one block: radius fields of 24 bits and angle fields of
    18, end to end from bit 0, through Box-Muller."""
    fields = [(w[0] & 0xFFFFFF, (w[0] >> 24 | w[1] << 8) & 0x3FFFF),
              ((w[1] >> 10 | w[2] << 22) & 0xFFFFFF, (w[2] >> 2) & 0x3FFFF),
              ((w[2] >> 20 | w[3] << 12) & 0xFFFFFF, (w[3] >> 12) & 0x3FFFF)]
    out = []
    for r, a in fields:
        rad = torch.sqrt(-2.0 * torch.log((r.double() + 1.0) / 2.0 ** 24))
        ang = a.double() * (2.0 * math.pi / 2.0 ** 18)
        out += [rad * torch.cos(ang), rad * torch.sin(ang)]
    return torch.stack(out[:5])


def _u53(index, k, purpose, seed, track):
    w = _philox(index, k, purpose, 0, seed, track)
    return (w[0].double() * 2097152.0 + (w[1] >> 11).double()) * 2.0 ** -53


def _spread16(v):
    out = torch.zeros_like(v)
    for j in range(16):
        out |= ((v >> j) & 1) << (2 * j)
    return out


def _initial(p, i):
    """The initial cloud, rounded to 32 bits as the filter stores it."""
    n, seed, tr = p.n_particles, p.seed, p.track_id
    a = torch.tensor(list(p.init_a), dtype=torch.float64, device=i.device)[:, None]
    b = torch.tensor(list(p.init_b), dtype=torch.float64, device=i.device)[:, None]
    if p.init_kind == INITS["gaussian"]:
        return (a + b * _normals(_philox(i, 0, 1, 0, seed, tr))).float().double()
    w = _philox(i, 0, 1, 0, seed, tr) + _philox(i, 0, 1, 1, seed, tr)[:1]
    f = torch.stack([(v >> 8).double() / 2.0 ** 24 for v in w])
    if p.init_kind == INITS["stratified"]:
        t = max(0, n.bit_length() - 3)
        cell = (i << t) // n
        cx, cy = torch.zeros_like(i), torch.zeros_like(i)
        for j in range(t):
            bit = (cell >> j) & 1
            if j % 2 == 0:
                cx |= bit << (j // 2)
            else:
                cy |= bit << (j // 2)
        f[0] = (cx.double() + f[0]) / 2.0 ** ((t + 1) // 2)
        f[1] = (cy.double() + f[1]) / 2.0 ** (t // 2)
    if p.init_kind == INITS["zorder"]:
        key = _spread16(w[0] >> 16) | (_spread16(w[1] >> 16) << 1)
        f = f[:, torch.sort(key, stable=True).indices]
    return (a + (b - a) * f).float().double()


def _patch_loglik(x, frame, p):
    """Log likelihood of every particle on its patch (Eq. 4 with the spot of
    Eq. 3)."""
    P = ppf.patch_size(p)
    h, H, W = (P - 1) // 2, p.height, p.width
    s, sig = float(p.psf_sigma), float(p.noise_sigma)
    pad = torch.nn.functional.pad(frame.double() - float(p.background), (2 * P,) * 4)
    off = torch.arange(-h, h + 1, device=x.device)
    n = x.shape[1]
    out = torch.empty(n, dtype=torch.float64, device=x.device)
    chunk = max(1, (1 << 28) // (P * P))
    for j in range(0, n, chunk):
        px, py, I = x[0, j:j + chunk], x[1, j:j + chunk], x[4, j:j + chunk, None, None]
        cx, cy = torch.floor(px + 0.5), torch.floor(py + 0.5)
        ix = (cx.clamp(-P, W + P).long() + 2 * P)[:, None] + off
        iy = (cy.clamp(-P, H + P).long() + 2 * P)[:, None] + off
        ix, iy = ix.clamp(0, W + 4 * P - 1), iy.clamp(0, H + 4 * P - 1)
        ex = ((cx - px)[:, None] + off)[:, None, :]
        ey = ((cy - py)[:, None] + off)[:, :, None]
        g = torch.exp(-ex * ex / (2 * s * s)) * torch.exp(-ey * ey / (2 * s * s))
        at = iy[:, :, None] * pad.shape[1] + ix[:, None, :]
        r = pad.reshape(-1)[at] - I * g
        ssq = (r * r).sum((1, 2))
        out[j:j + chunk] = -ssq / (2 * sig * sig) - P * P * math.log(sig * math.sqrt(2 * math.pi))
    return out


def _systematic(w, u, n):
    """s(i) = min{ j : (i + u) / n < C_j } for the normalised weights w."""
    C = torch.cumsum(w, 0)
    us = (torch.arange(n, device=w.device, dtype=torch.float64) + u) / n
    return torch.searchsorted(C / C[-1], us, right=True).clamp(max=n - 1)


def _rna(w, p, k):
    """RNA (Section 3): the slots' ancestors and log weights."""
    n, m = p.n_particles, p.rna_group
    G, moved = n // m, int(math.floor(float(p.rna_exchange) * m))
    g = torch.arange(G, device=w.device)
    u = _u53(g, k, 4, p.seed, p.track_id)
    wg = w.reshape(G, m)
    Wg = wg.sum(1)
    C = torch.cumsum(wg / Wg.clamp(min=1e-300)[:, None], 1)
    us = (torch.arange(m, device=w.device, dtype=torch.float64) + u[:, None]) / m
    loc = torch.searchsorted(C, us, right=True).clamp(max=m - 1)
    loc = torch.where((Wg > 0)[:, None], loc, torch.arange(m, device=w.device)) + (g * m)[:, None]
    lw = torch.log(Wg / m)[:, None].expand(G, m).clone()
    prev = (g - 1) % G
    loc[:, m - moved:], lw[:, m - moved:] = loc[prev, m - moved:], lw[prev, m - moved:]
    return loc.reshape(-1), lw.reshape(-1)


def _rpa(anc, p):
    """Proportional allocation of the systematic ancestors over the groups,
    the surplus routed by Greedy or Sorted Greedy (Section 4)."""
    n, m = p.n_particles, p.rna_group
    G = n // m
    cnt = torch.bincount(anc // m, minlength=G)
    first = torch.cumsum(cnt, 0) - cnt
    order = torch.arange(G, device=anc.device)
    send, recv = order[cnt > m], order[cnt < m]
    if p.dlb == ppf.DLB_SGS:
        send = send[torch.sort(m - cnt[send], stable=True).indices]
        recv = recv[torch.sort(cnt[recv] - m, stable=True).indices]

    def ranges(start, length):
        ends = torch.cumsum(length, 0)
        r = torch.arange(int(ends[-1]) if len(ends) else 0, device=anc.device)
        return torch.repeat_interleave(start - (ends - length), length) + r

    keep = cnt.clamp(max=m)
    out = torch.empty_like(anc)
    out[ranges(order * m, keep)] = anc[ranges(first, keep)]
    out[ranges(recv * m + cnt[recv], m - cnt[recv])] = anc[ranges(first[send] + m, cnt[send] - m)]
    return out


def _filter(p, frames):
    """The filter of Algorithm 1 in 64 bits: estimates, ESS and log p^ per
    frame, and the resampled cloud."""
    dev = torch.device("cuda")
    n, seed, tr = int(p.n_particles), int(p.seed), int(p.track_id)
    i = torch.arange(n, device=dev)
    x = _initial(p, i)
    lw = torch.full((n,), -math.log(n), dtype=torch.float64, device=dev)
    q = torch.tensor(list(p.q), dtype=torch.float64, device=dev)[:, None]
    means, esses, deltas = [], [], []
    for k, z in enumerate(frames, 1):
        noise = _normals(_philox(i, k, 2, 0, seed, tr))
        x = x + q * noise + torch.stack([x[2], x[3], x[2] * 0, x[2] * 0, x[2] * 0])
        if p.obs_model == ppf.OBS_LINEAR_GAUSSIAN:
            r = torch.tensor(list(p.lg_r), dtype=torch.float64, device=dev)[:, None]
            e = (z.double()[:, None] - x[[0, 1, 4]]) / r
            like = (-0.5 * e * e - torch.log(r * math.sqrt(2 * math.pi))).sum(0)
        else:
            like = _patch_loglik(x, z, p)
        l = lw + like
        m = l.max()
        delta = m + torch.log(torch.exp(l - m).sum())
        lw = l - delta
        w = torch.exp(lw)
        ess = float(1.0 / (w * w).sum())
        means.append((x * w).sum(1).cpu().numpy())
        esses.append(ess)
        deltas.append(float(delta))
        if ess < p.ess_threshold:
            if p.resample == ppf.RESAMPLE_RNA:
                anc, lw = _rna(w, p, k)
            else:
                u = float(_u53(torch.zeros(1, dtype=torch.int64, device=dev), k, 3, seed, tr))
                anc = _systematic(w, u, n)
                if p.resample == ppf.RESAMPLE_RPA:
                    anc = _rpa(anc, p)
                lw = torch.full_like(lw, -math.log(n))
            x = x[:, anc]
    return dict(mean=np.stack(means), ess=np.array(esses), delta=np.array(deltas), cloud=x)


def exact(case, seed):
    c, kind = case, case["kind"]
    seed = seed & 0x7FFFFFFF
    if kind == "track":
        if c["scheme"] == "arna":
            return None  # its redrawn rings have no short form in plain torch
        obs, p = _movie(c, seed)
        r = _filter(_params(c, p, seed), _frames(obs))
        rows = slice(None) if c["each"] else slice(-1, None)
        return {"mean": r["mean"][rows], "ess": r["ess"][rows], "loglik": float(r["delta"].sum()),
                "cloud": r["cloud"]}
    if kind == "loglik":
        obs, p = _movie(c, seed)
        # the gradient has no 64-bit value to compare with: the ancestors that
        # fall the other way under 32-bit weights change the lines of descent
        # that its tangents sum over
        r = _filter(_params(c, p, seed), _frames(obs))
        return {"loglik": torch.tensor(r["delta"].sum()), "grad": None}
    if kind == "batch":
        frames, ps = _spots(c, seed)
        dev = _frames(frames)
        rs = [_filter(p, dev) for p in ps]
        return {key: np.stack([r[key] for r in rs], 1) for key in ("mean", "ess", "delta")}
    if kind == "resample" and c["scheme"] == "rna":
        lw = _weights(c, seed).double()
        lse = torch.logsumexp(lw, 0)
        per = torch.logsumexp(lw.reshape(-1, c["group"]), 1) - lse - math.log(c["group"])
        return {"ancestors": None, "group_logw": per}
    return None
