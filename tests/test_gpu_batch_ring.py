"""A host that runs ahead of the device by more steps than the batch has staging
buffers: each step's plan (stepped set and frames) is the one it was given."""
import numpy as np
import pytest
import torch

import paper_2308_00763_amd as pf
import pfsynth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("own_stream", [False, True])
def test_plans_survive_a_busy_stream(own_stream):
    sizes = [1000, 1024, 5000, 30000, 70001] * 8
    v = torch.from_numpy(pfsynth.moving_disk(96, 96, 12, 5, (40, 60), (1, -2), 4.0, 3).frames).to("cuda:0")
    ps = [pf.make_params(n, 96, 96, "f32", x0=40, y0=60, seed=2, stream_id=i) for i, n in enumerate(sizes)]
    stream = torch.cuda.Stream() if own_stream else torch.cuda.current_stream()
    a = torch.randn((4096, 4096), device="cuda:0")
    torch.cuda.synchronize()
    rng = np.random.default_rng(1)
    plans = [((rng.random(len(sizes)) < 0.6).astype(np.uint8), rng.integers(0, 12, len(sizes))) for _ in range(10)]
    b = pf.Batch(ps, stream=stream)
    frames = [[v[j] for j in fr] for _, fr in plans]
    with torch.cuda.stream(stream):
        for _ in range(40):  # tens of milliseconds of work before the first step
            a = a @ a * 1e-4
        ahead = torch.cuda.Event()
        ahead.record(stream)
    for (active, _), fr in zip(plans[:3], frames[:3]):
        b.step(fr, active)
    assert not ahead.query()  # the staging buffers are all waiting to be read
    for (active, _), fr in zip(plans[3:], frames[3:]):
        b.step(fr, active)
    est = b.estimates()
    for i in range(len(sizes)):
        f = pf.Filter(ps[i])
        for active, fr in plans:
            if active[i]:
                f.step(v[int(fr[i])])
        assert f.estimate() == tuple(est[i])
        u, w = f.export(), b.export(i)
        assert np.array_equal(u["x"], w["x"]) and np.array_equal(u["y"], w["y"])
        f.close()
    b.close()
