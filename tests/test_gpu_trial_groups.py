"""Rejection and Metropolis resampling at the edges of their trial groups: two
trials, then eight at a time, then 128 for one slot; steps in groups of eight.
FP64 against the oracle: the same ancestor except where one of the slot's tests
lies within 1e-12 of its threshold."""
import numpy as np
import pytest
import torch

import oracle
import paper_2308_00763_amd as pf
import pfsynth
from gpu_common import make_filter, near_half, oracle_params, oracle_step_parts

pytestmark = pytest.mark.gpu


def _steps(n, kappa_sigma, **kw):
    """Two teacher-forced steps; a wide cloud of few particles makes most
    proposals fail (slots run out of trials), a still one accepts at once."""
    w = pfsynth.WORKLOADS["disk128_n1000"]
    vid = pfsynth.workload_video(w, frames=3)
    fr = torch.from_numpy(vid.frames).to("cuda:0")
    x0, y0 = vid.centres[0]
    f = make_filter("f64", n, w.width, w.height, 5, x0, y0, seed=3, stream_id=2, sigma=kappa_sigma, **kw)
    op = oracle_params(n, w.width, w.height, 5, seed=3, stream_id=2, sigma=kappa_sigma)
    x, y = np.full(n, x0), np.full(n, y0)
    for t in (1, 2):
        f.load(x, y, t - 1)
        f.step(fr[t])
        got, gs = f.export(), f.export_step()
        ref = oracle_step_parts(op, t, vid.frames[t], x, y)
        bad = gs["disk_sum"].astype(np.int64) != ref["S"]
        assert np.all((near_half(ref["x_prop"]) | near_half(ref["y_prop"]))[bad])
        if not bad.any():
            yield t, got, gs, ref, op
        x, y = ref["x_prop"][got["anc"]], ref["y_prop"][got["anc"]]
    f.close()


def _check(got, gs, anc, margin):
    mism = got["anc"] != anc
    assert np.all(margin[mism] <= 1e-12), np.flatnonzero(mism & (margin > 1e-12))[:10]
    assert np.array_equal(got["x"], gs["x_prop"][got["anc"]])


@pytest.mark.parametrize("n, cap, sigma", [(1, 64, (5.0, 2.0)), (63, 64, (9.0, 9.0)), (65, 128, (9.0, 9.0)),
                                           (300, 192, (9.0, 9.0)), (2049, 16320, (9.0, 9.0)), (4096, 64, (0.0, 0.0)),
                                           # marks in LDS: the larger workgroups, their largest size; read from memory
                                           (262145, 256, (5.0, 2.0)), (524288, 128, (5.0, 2.0)),
                                           (524289, 128, (5.0, 2.0))])
def test_rejection_groups(n, cap, sigma):
    for t, got, gs, ref, op in _steps(n, sigma, rejection_trials=cap):
        anc, margin, trials = oracle.rejection(ref["L"], cap, op.seed, op.stream_id, t)
        print(f"[groups] n={n} cap={cap} trials {trials.min()}..{trials.max()}", flush=True)
        _check(got, gs, anc, margin)


@pytest.mark.parametrize("n, steps", [(1, 1), (257, 7), (257, 8), (1000, 9), (1000, 255)])
def test_metropolis_groups(n, steps):
    for t, got, gs, ref, op in _steps(n, (5.0, 2.0), metropolis_steps=steps):
        anc, margin = oracle.metropolis(ref["L"], steps, op.seed, op.stream_id, t)[:2]
        _check(got, gs, anc, margin)
