"""The work that a user of this library has it do, as measurable cases.

Every case is a tracker stepping its filters on video frames that lie in device
memory, and reading the estimates the way its kind of program does:

  realtime    one frame arrives at a time and the estimate is wanted on the
              host before the next one: one step and one read per pass;
  clip        a recorded clip of some frames is stepped through without
              waiting; each frame's estimate goes to a track on the device;
  checkpoint  some steps, then the whole state is exported to the host;
  fleet       one tick of many small streams of equal frames, stepped as one
              batch; the estimates stay on the device;
  serving     one tick of a server's streams: other frame sizes, radii and
              particle counts per stream, a part of them active, estimates
              read back to the host.

The videos are disks on a flat background with Gaussian pixel noise (the
tracking workload of the repository's benchmark), drawn on the device.  The
object moves (1, -2) pixels per frame through the clip and back again, so that
a pass after a pass goes on tracking; the filters do not know the direction
(drift 0) and spread with the transition deviations (5, 2).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2308_00763_amd as pf

FG, BG, KAPPA, SIGMA = 228, 100, 50.0, (5.0, 2.0)
VELOCITY = (1, -2)


def _clip(name, dtype, n, width, height, radius, frames, noise=2.0, resampler="systematic"):
    return dict(name=name, kind="clip", dtype=dtype, n=n, width=width, height=height, radius=radius,
                frames=frames, noise=noise, resampler=resampler)


def listed():
    return [
        # the smallest call: a camera at 128 x 128 tracked with a thousand
        # particles in double, every estimate needed at once
        dict(name="realtime_f64_n1000", kind="realtime", dtype="f64", n=1000, width=128, height=128, radius=5,
             frames=16, noise=2.0, resampler="systematic"),
        # the larger of the two particle counts of the paper's speedup study
        _clip("clip_f16_n64k", "f16", 65536, 512, 512, 5, 16),
        # the precision sweep of the benchmark: one video, 2^20 particles
        _clip("clip_f16_n1m", "f16", 1 << 20, 1024, 1024, 5, 8),
        _clip("clip_f32_n1m", "f32", 1 << 20, 1024, 1024, 5, 8),
        _clip("clip_f64_n1m", "f64", 1 << 20, 1024, 1024, 5, 8),
        # an odd camera format, an odd particle count and a larger object
        _clip("clip_bf16_n3m_ragged", "bf16", 3000001, 641, 481, 12, 4, 4.0),
        # the largest single filters: a noisy video, 2^24 particles in half,
        # 2^23 + 1 in double
        _clip("clip_f16_n16m", "f16", 1 << 24, 512, 512, 8, 4, 8.0),
        _clip("clip_f64_n8m", "f64", (1 << 23) + 1, 512, 512, 8, 4, 8.0),
        # the scan-free alternative whose offspring counts are unbiased
        _clip("clip_f32_rejection", "f32", 1 << 18, 512, 512, 5, 4, 2.0, "rejection"),
        # a long-running tracker saving its state between clips
        dict(name="checkpoint_f64_n70001", kind="checkpoint", dtype="f64", n=70001, width=512, height=512, radius=5,
             frames=4, noise=2.0, resampler="systematic"),
        # thousands of small streams advanced together
        dict(name="fleet_f16_4096", kind="fleet", dtype="f16", streams=4096, n_lo=256, n_hi=65536, side=256, radius=5),
        # a server's tick: streams of every size, two thirds with a new frame
        dict(name="serving_f32_192", kind="serving", dtype="f32", streams=192, n_lo=1000, n_hi=1000000, side=1024,
             radius=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["realtime", "clip", "clip", "clip", "clip", "resampler", "checkpoint", "fleet", "serving"])
    if kind == "fleet":
        return dict(kind="fleet", dtype=rng.choice(["f16", "bf16", "f32"]), streams=_log_int(rng, 48, 4096), n_lo=256,
                    n_hi=65536, side=rng.choice([128, 256]), radius=rng.choice([3, 5, 8]))
    if kind == "serving":
        return dict(kind="serving", dtype=rng.choice(["f16", "f32", "f64"]), streams=_log_int(rng, 16, 192),
                    n_lo=1000, n_hi=rng.choice([100000, 300000]), side=rng.choice([256, 1024]), radius=0)
    c = dict(kind="clip", dtype=rng.choice(["f64", "f32", "f16", "bf16"]), n=0, width=rng.randint(128, 1024),
             height=rng.randint(128, 1024), radius=rng.randint(2, 12), frames=8, noise=rng.choice([2.0, 4.0, 8.0]),
             resampler="systematic")
    if kind == "realtime":
        c.update(kind="realtime", n=_log_int(rng, 128, 65536), frames=16)
    elif kind == "checkpoint":
        c.update(kind="checkpoint", dtype="f64", n=_log_int(rng, 1000, 200000), frames=4)
    elif kind == "resampler":
        c.update(n=_log_int(rng, 1 << 14, 1 << 17), resampler=rng.choice(["rejection", "metropolis"]), radius=5,
                 noise=2.0, frames=4)
    else:
        c["n"] = _log_int(rng, 128, 1 << (22 if c["dtype"] == "f64" else 23))
        c["frames"] = 16 if c["n"] < 1 << 18 else 8 if c["n"] < 1 << 21 else 4
        if c["n"] > 1 << 21:
            c["radius"] = min(c["radius"], 8)
    return c


# ---------------------------------------------------------------------------
# Inputs.

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) & (2**63 - 1))
    return g


def _render(centres, width, height, radius, noise, g):
    """(len(centres), height, width) uint8 frames with the disk at the given centres."""
    c = torch.as_tensor(np.asarray(centres, dtype=np.float32), device="cuda")
    dx2 = (torch.arange(width, device="cuda", dtype=torch.float32) - c[:, 0, None]) ** 2
    dy2 = (torch.arange(height, device="cuda", dtype=torch.float32) - c[:, 1, None]) ** 2
    out = torch.empty((len(centres), height, width), dtype=torch.uint8, device="cuda")
    for t in range(len(centres)):
        img = torch.where(dy2[t, :, None] + dx2[t, None, :] < float(radius * radius), float(FG), float(BG))
        img += torch.randn((height, width), generator=g, device="cuda") * noise
        out[t] = torch.clamp(torch.floor(img + 0.5), 0, 255).to(torch.uint8)
    return out


def _centres(case, rng):
    """Centres of frames 0 .. T, every disk inside the frame."""
    T, r = case["frames"], case["radius"]
    x0 = int(rng.integers(r, case["width"] - r - T * VELOCITY[0]))
    y0 = int(rng.integers(r - T * VELOCITY[1], case["height"] - r))
    return [(x0 + VELOCITY[0] * t, y0 + VELOCITY[1] * t) for t in range(T + 1)]


def _params(case, seed, x0, y0, n=None, width=None, height=None, radius=None, stream_id=0):
    res = case.get("resampler", "systematic")
    return pf.make_params(n or case["n"], width or case["width"], height or case["height"], case["dtype"],
                          radius=radius or case["radius"], x0=x0, y0=y0, drift=(0.0, 0.0), sigma=SIGMA,
                          seed=seed, stream_id=stream_id, fg=FG, bg=BG, kappa=KAPPA,
                          rejection_trials=4096 if res == "rejection" else 0,
                          metropolis_steps=32 if res == "metropolis" else 0)


def _single_inputs(case, seed):
    rng = np.random.default_rng(seed)
    centres = _centres(case, rng)
    return centres, _render(centres, case["width"], case["height"], case["radius"], case["noise"], _gen(seed))


def _sizes(case):
    """Particle counts of the streams: evenly spread over the logarithm of their range."""
    s, lo, hi = case["streams"], math.log(case["n_lo"]), math.log(case["n_hi"])
    return [int(round(math.exp(lo + (hi - lo) * (i + 0.5) / s))) for i in range(s)]


def _batch_inputs(case, seed):
    """Per stream: (n, side, radius, start), its filter's seed, and frames 0 and 1."""
    rng = np.random.default_rng(seed)
    sizes = np.asarray(_sizes(case))[rng.permutation(case["streams"])]
    streams = []
    for i, n in enumerate(sizes):
        side = case["side"]
        radius = case["radius"]
        if case["kind"] == "serving":
            side = int(2 ** rng.integers(6, int(math.log2(case["side"])) + 1))
            radius = int(rng.choice([3, 5, 5, 5, 8]))
        start = (int(rng.integers(radius, side - radius - 1)), int(rng.integers(radius + 2, side - radius)))
        streams.append((int(n), side, radius, start))
    g = _gen(seed)
    if case["kind"] == "fleet":  # frames of one size: a few draws
        side, r = case["side"], case["radius"]
        ax = torch.arange(side, device="cuda", dtype=torch.float32)
        start = torch.as_tensor([s[3] for s in streams], device="cuda", dtype=torch.float32)
        frames = []
        for t in range(2):
            f = torch.empty((len(streams), side, side), dtype=torch.uint8, device="cuda")
            for k in range(0, len(streams), 512):
                c = start[k:k + 512] + torch.tensor(VELOCITY, device="cuda", dtype=torch.float32) * t
                d2 = ((ax - c[:, 1, None]) ** 2)[:, :, None] + ((ax - c[:, 0, None]) ** 2)[:, None, :]
                img = torch.where(d2 < float(r * r), float(FG), float(BG))
                img += torch.randn(img.shape, generator=g, device="cuda") * 4.0
                f[k:k + 512] = torch.clamp(torch.floor(img + 0.5), 0, 255).to(torch.uint8)
            frames.append(list(f))
        return streams, frames
    pairs = [_render([s[3], (s[3][0] + VELOCITY[0], s[3][1] + VELOCITY[1])], s[1], s[1], s[2], 4.0, g)
             for s in streams]
    return streams, [[p[t] for p in pairs] for t in range(2)]


def prepare(case, seed):
    if case["kind"] in ("fleet", "serving"):
        streams, frames = _batch_inputs(case, seed)
        params = [_params(case, seed, s[3][0], s[3][1], n=s[0], width=s[1], height=s[1], radius=s[2], stream_id=i)
                  for i, s in enumerate(streams)]
        state = dict(case=case, batch=pf.Batch(params), pos=0, frames=frames, active=None,
                     est=torch.zeros((len(streams), 2), dtype=torch.float64, device="cuda"))
        state["ptrs"] = [np.array([f.data_ptr() for f in fr], dtype=np.uint64) for fr in frames]
        state["pitches"] = np.array([s[1] for s in streams], dtype=np.int64)
        if case["kind"] == "serving":  # every third stream waits for its next frame
            state["active"] = [np.array([i % 3 != k for i in range(len(streams))], dtype=np.uint8) for k in range(3)]
        return state
    centres, frames = _single_inputs(case, seed)
    T = case["frames"]
    track = torch.zeros((T, 2), dtype=torch.float64, device="cuda")
    return dict(case=case, filter=pf.Filter(_params(case, seed, *centres[0])), pos=0,
                # the clip forward, then backward
                frames=[frames[t] for t in list(range(1, T + 1)) + list(range(T - 1, -1, -1))],
                track=track, track_ptrs=[track[i].data_ptr() for i in range(T)])


# ---------------------------------------------------------------------------
# One pass.  Outside the double mode an estimate is a float value (the library
# widens it to double on its way out), and is kept as one.

def run(state):
    case = state["case"]
    kind, wide = case["kind"], case["dtype"] == "f64"
    if kind in ("fleet", "serving"):
        b, i = state["batch"], state["pos"]
        state["pos"] = i + 1
        # the object moves one frame on, then one back
        active = None if state["active"] is None else state["active"][i % 3]
        b.step_ptrs(state["ptrs"][(i + 1) % 2], state["pitches"], active)
        if kind == "serving":
            est = b.estimates()
            return est if wide else est.astype(np.float32)
        pf.pf_batch_estimates_async(b.handle, state["est"].data_ptr())
        return state["est"] if wide else state["est"].float()
    f, frames, i = state["filter"], state["frames"], state["pos"]
    if kind == "realtime":
        f.step(frames[i])
        state["pos"] = (i + 1) % len(frames)
        est = f.estimate()
        return np.array(est, dtype=np.float64 if wide else np.float32)
    T = case["frames"]
    state["pos"] = (i + T) % len(frames)
    if kind == "checkpoint":
        for k in range(T):
            f.step(frames[i + k])
        got = f.export()
        return {"x": got["x"], "y": got["y"], "t": got["t"]}
    for k in range(T):
        f.step(frames[i + k])
        pf.pf_estimate_async(f.handle, state["track_ptrs"][k])
    return state["track"].clone() if wide else state["track"].float()


# ---------------------------------------------------------------------------
# What a pass cannot do without: the state read and written once per step, the
# pixels its particles look at read once; about 130 operations per particle
# (random numbers, the move, the pixel cell, the disk's row sums, the weight,
# the scan and the resampling), more of them in the trials of a chain.

ELT = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}


def _disk(radius):
    return sum(1 for i in range(-radius, radius + 1) for j in range(-radius, radius + 1)
               if i * i + j * j < radius * radius)


def work(case):
    if case["kind"] in ("fleet", "serving"):
        sizes = _sizes(case)
        share = 1.0 if case["kind"] == "fleet" else 2.0 / 3.0
        n, steps, windows, radius = sum(sizes) * share, 1, len(sizes) * share, case["radius"] or 5
    else:
        n, windows, radius = case["n"], 1, case["radius"]
        steps = 1 if case["kind"] == "realtime" else case["frames"]
    window = (6 * SIGMA[0] + 2 * radius) * (6 * SIGMA[1] + 2 * radius)
    ops = 112 + 4 * radius + {"metropolis": 32 * 30, "rejection": 32 * 30}.get(case.get("resampler"), 0)
    return {"bytes": steps * (4.0 * ELT[case["dtype"]] * n + window * windows + 16 * windows),
            "flops": steps * float(ops) * n}


# ---------------------------------------------------------------------------
# The same passes in plain torch, in 64 bits: Philox4x32-10 streams (the top
# 24 bits of their words outside the double mode), Box-Muller, the disk sums
# pixel by pixel, and the resampler's definition.

def _philox(c0, c1, c2, c3, seed):
    m = 0xFFFFFFFF
    k0, k1 = seed & m, (seed >> 32) & m
    c = [torch.as_tensor(v, dtype=torch.int64, device="cuda") for v in (c0, c1, c2, c3)]
    for _ in range(10):
        p0, p1 = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((p1 >> 32) & m) ^ c[1] ^ k0, p1 & m, ((p0 >> 32) & m) ^ c[3] ^ k1, p0 & m]
        k0, k1 = (k0 + 0x9E3779B9) & m, (k1 + 0xBB67AE85) & m
    return c


def _u53(hi, lo):
    return ((hi << 21) | (lo >> 11)).double() * 2.0 ** -53


class _Exact:
    """One filter in 64 bits."""

    def __init__(self, case, seed, n, radius, x0, y0, stream_id):
        self.case, self.seed, self.n, self.sid, self.t = case, seed, n, stream_id, 0
        self.wide = case["dtype"] == "f64"
        self.x = torch.full((n,), float(x0), dtype=torch.float64, device="cuda")
        self.y = torch.full((n,), float(y0), dtype=torch.float64, device="cuda")
        self.k = torch.arange(n, device="cuda")
        self.r = radius
        off = [(i, j) for i in range(-radius, radius + 1) for j in range(-radius, radius + 1)
               if i * i + j * j < radius * radius]
        self.dy, self.dx = torch.tensor(off, device="cuda").T

    def step(self, frame, resample=True):
        self.t += 1
        w = _philox(self.k, self.t, self.sid, 0, self.seed)
        if self.wide:
            ua, ub = _u53(w[0], w[1]), _u53(w[2], w[3])
        else:
            ua, ub = (w[0] >> 8).double() * 2.0 ** -24, (w[2] >> 8).double() * 2.0 ** -24
        rho = torch.sqrt(-2.0 * torch.log(1.0 - ua))
        x = self.x + SIGMA[0] * (rho * torch.cos(2.0 * math.pi * ub))
        y = self.y + SIGMA[1] * (rho * torch.sin(2.0 * math.pi * ub))
        H, W = frame.shape
        # the likelihood of every pixel cell that a particle lies in
        cx, cy = torch.floor(x + 0.5).long(), torch.floor(y + 0.5).long()
        r = self.r
        cx, cy = cx.clamp(-r, W - 1 + r), cy.clamp(-r, H - 1 + r)
        bx, by = int(cx.min()), int(cy.min())
        gy = torch.arange(by, int(cy.max()) + 1, device="cuda")
        gx = torch.arange(bx, int(cx.max()) + 1, device="cuda")
        pix = (frame.double() - BG) ** 2 - (frame.double() - FG) ** 2
        S = pix[(gy[:, None, None] + self.dy).clamp(0, H - 1), (gx[:, None] + self.dx).clamp(0, W - 1)].sum(-1)
        L = S[cy - by, cx - bx] / (KAPPA * len(self.dy))
        wt = torch.exp(L - L.max())
        Z = wt.sum()
        self.est = torch.stack([(wt * x).sum() / Z, (wt * y).sum() / Z])
        if resample:
            a = self._ancestors(L, wt, Z)
            self.x, self.y = x[a], y[a]

    def _words(self, j, q):
        """The proposal and acceptance words of both trials of pair q of the slots j."""
        return _philox(j, self.t, self.sid, 2 + q, self.seed)

    def _unit(self, word):
        return (word.double() + 0.5) * 2.0 ** -32 if self.wide else ((word >> 8).double() + 0.5) * 2.0 ** -24

    def _ancestors(self, L, wt, Z):
        n, res = self.n, self.case.get("resampler", "systematic")
        if res == "systematic":
            u = _philox(0, self.t, self.sid, 1, self.seed)
            c = torch.cumsum(wt, 0) / Z
            c[-1] = 1.0
            return torch.searchsorted(c, (self.k.double() + _u53(u[0], u[1])) / n).clamp(max=n - 1)
        if res == "metropolis":
            a = self.k.clone()
            for b in range(32):
                w = self._words(self.k, b >> 1)
                i = (w[2 * (b & 1)] * n) >> 32
                a = torch.where(self._unit(w[2 * (b & 1) + 1]) <= torch.exp(L[i] - L[a]), i, a)
            return a
        a, left = self.k.clone(), self.k
        for m in range(4096):
            if not len(left):
                break
            w = self._words(left, m >> 1)
            no = self._unit(w[2 * (m & 1)]) > wt[a[left]]
            if m + 1 < 4096:
                a[left[no]] = (w[2 * (m & 1) + 1][no] * n) >> 32
            left = left[no]
        return a


def exact(case, seed):
    if case["kind"] in ("fleet", "serving"):
        streams, frames = _batch_inputs(case, seed)
        out = np.array([s[3] for s in streams], dtype=np.float64)
        for i, (n, _, radius, start) in enumerate(streams):
            if case["kind"] == "serving" and i % 3 == 0:
                continue
            f = _Exact(case, seed, n, radius, start[0], start[1], i)
            f.step(frames[1][i], resample=False)
            out[i] = f.est.cpu().numpy()
        return out
    centres, frames = _single_inputs(case, seed)
    f = _Exact(case, seed, case["n"], case["radius"], centres[0][0], centres[0][1], 0)
    T = 1 if case["kind"] == "realtime" else case["frames"]
    track = []
    for t in range(1, T + 1):
        f.step(frames[t], resample=case["kind"] == "checkpoint" or t < T)
        track.append(f.est.cpu().numpy())
    if case["kind"] == "checkpoint":
        return {"x": f.x.cpu().numpy(), "y": f.y.cpu().numpy(), "t": None}
    return track[0] if case["kind"] == "realtime" else np.stack(track)
