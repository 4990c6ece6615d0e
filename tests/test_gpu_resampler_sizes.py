"""Metropolis and rejection resampling on both sides of the sizes and the
likelihoods at which their kernels change: Metropolis in groups of eight or a
pair of steps at a time, rejection with its marks in LDS (two workgroup sizes)
or in memory, with trials ahead or one at a time by the chance of a trial, and
both behind the streaming pass A.

The oracle runs on the GPU's own integer disk terms, so every step is checked
whatever the pixel ties.  A slot may differ only where one of its tests lies
within the arithmetic's resolution of its threshold: FP64 1e-12; reduced modes
2^-24 + 2.5e-6 (the uniform is the top 24 bits of the word, and the exponent
carries at most 24 * 2^-23 of error where the threshold is above 2^-24, plus one
ulp of the exponential)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2308_00763_amd as pf
import pfsynth
from test_gpu_stream import _frames, _run

pytestmark = pytest.mark.gpu

MARGIN = {"f64": 1e-12, "f32": 2.0 ** -24 + 2.5e-6, "f16": 2.0 ** -24 + 2.5e-6, "bf16": 2.0 ** -24 + 2.5e-6}
ND = oracle.disk(5)[0].size


def _steps(dtype, n, kappa=50.0, steps=2, **kw):
    w = pfsynth.WORKLOADS["disk128_n1000"]
    vid = pfsynth.workload_video(w, frames=steps + 1)
    fr = torch.from_numpy(vid.frames).to("cuda:0")
    x0, y0 = vid.centres[0]
    f = pf.Filter(pf.make_params(n, w.width, w.height, dtype, radius=5, x0=x0, y0=y0, seed=11, stream_id=3,
                                 kappa=kappa, diagnostics=True, **kw))
    for t in range(1, steps + 1):
        print(f"[sizes] {dtype} n={n} kappa={kappa} {kw} step={t}", flush=True)
        f.step(fr[t])
        got, gs = f.export(), f.export_step()
        yield t, got, gs, gs["disk_sum"].astype(np.float64) / (kappa * ND)
    f.close()


def _check(dtype, got, gs, anc, margin):
    mism = got["anc"] != anc
    assert np.all(margin[mism] <= MARGIN[dtype]), np.flatnonzero(mism & (margin > MARGIN[dtype]))[:10]
    assert np.array_equal(got["x"], gs["x_prop"][got["anc"]]) and np.array_equal(got["y"], gs["y_prop"][got["anc"]])


@pytest.mark.parametrize("dtype, n, B", [
    ("f16", 65536, 1), ("f16", 65536, 2), ("f32", 65536, 4), ("f32", 65536, 5), ("f64", 65536, 8), ("f16", 65536, 13),
    ("f32", 65536, 15), ("f64", 1000, 23), ("f16", 65537, 1), ("f32", 65537, 2), ("f64", 65537, 3), ("bf16", 65537, 8),
    ("f16", 65537, 17), ("f32", 300001, 33)])
def test_metropolis(dtype, n, B):
    for t, got, gs, L in _steps(dtype, n, metropolis_steps=B):
        anc, margin = oracle.metropolis(L, B, 11, 3, t)
        _check(dtype, got, gs, anc, margin)


@pytest.mark.parametrize("dtype, n, cap, kappa", [
    # chance of a trial about 0.01 (kappa 50), 0.025 (3000), 0.06 (6000), 0.3 (20000), nearly 1 (1e6)
    ("f32", 700, 64, 20000.0), ("f64", 65536, 64, 6000.0), ("f16", 65537, 64, 20000.0), ("f32", 65537, 64, 50.0),
    ("f32", 262145, 128, 50.0), ("f16", 262145, 64, 6000.0), ("f64", 262145, 64, 6000.0), ("bf16", 262145, 64, 1e6),
    ("f32", 524288, 64, 20000.0), ("f16", 524289, 128, 50.0), ("f32", 524289, 64, 3000.0), ("f64", 524289, 64, 6000.0),
    ("f16", 524289, 64, 1e6), ("f16", 1048577, 64, 3000.0)])
def test_rejection(dtype, n, cap, kappa):
    for t, got, gs, L in _steps(dtype, n, kappa, rejection_trials=cap):
        anc, margin, trials = oracle.rejection(L, cap, 11, 3, t)
        print(f"[sizes] trials {trials.min()}..{trials.max()} mean {trials.mean():.2f}", flush=True)
        _check(dtype, got, gs, anc, margin)


@pytest.mark.parametrize("dtype, kw", [("f16", dict(rejection_trials=64)), ("f32", dict(rejection_trials=64)),
                                       ("bf16", dict(metropolis_steps=3)), ("f32", dict(metropolis_steps=9))])
def test_behind_the_streaming_pass(dtype, kw):
    """Against the one-tile pass A (which a filter with the per-pixel likelihood
    takes), bit for bit."""
    n, start = 6 * (1 << 20) + 777, (128, 128)
    fr = _frames(256, 5, start, 5)
    a = _run(n, dtype, 5, 256, fr, start, (5.0, 2.0), None, **kw)
    b = _run(n, dtype, 5, 256, fr, start, (5.0, 2.0), None, naive_likelihood=True, **kw)
    for u, v in zip(a, b):
        assert np.array_equal(u, v)
