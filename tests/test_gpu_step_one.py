"""The one-launch step of a filter of one tile against the separate kernels,
which a filter being profiled takes: bit for bit, with exports between steps,
diagnostics, an import, and as a captured graph."""
import numpy as np
import pytest
import torch

import paper_2308_00763_amd as pf
import pfsynth

pytestmark = pytest.mark.gpu


def _filter(dtype, n, r, diag, vid):
    x0, y0 = vid.centres[0]
    return pf.Filter(pf.make_params(n, 128, 128, dtype, radius=r, x0=x0, y0=y0, seed=5, stream_id=3, diagnostics=diag))


@pytest.mark.parametrize("dtype", ["f64", "f32", "f16", "bf16"])
@pytest.mark.parametrize("n, r, diag", [(1, 5, False), (63, 3, True), (257, 8, False), (1000, 5, True), (1024, 5, False),
                                        (1024, 12, False)])
def test_one_launch_equals_the_separate_kernels(dtype, n, r, diag):
    vid = pfsynth.moving_disk(128, 128, 7, r, (64, 64), (1, -2), 3.0, 11)
    fr = torch.from_numpy(vid.frames).to("cuda:0")
    a, b = _filter(dtype, n, r, diag, vid), _filter(dtype, n, r, diag, vid)
    pf.pf_profile_start(b.handle, 16)
    for t in range(1, 7):
        a.step(fr[t])
        b.step(fr[t])
        assert a.estimate() == b.estimate()
        if t in (2, 5, 6):
            u, v, us, vs = a.export(), b.export(), a.export_step(), b.export_step()
            for k in ("x", "y") + (("w", "anc") if diag else ()):
                assert np.array_equal(u[k], v[k]), (t, k)
            assert np.array_equal(us["x_prop"], vs["x_prop"]) and u["t"] == v["t"] == t
        if t == 3:
            x = 64.0 + np.arange(n) % 7
            a.load(x, x, t)
            b.load(x, x, t)
    a.close()
    b.close()


@pytest.mark.parametrize("dtype", ["f64", "f16"])
def test_one_launch_in_a_graph(dtype):
    vid = pfsynth.moving_disk(128, 128, 7, 5, (64, 64), (1, -2), 3.0, 11)
    fr = torch.from_numpy(vid.frames).to("cuda:0")
    s = torch.cuda.Stream()
    x0, y0 = vid.centres[0]
    f = pf.Filter(pf.make_params(1000, 128, 128, dtype, x0=x0, y0=y0, seed=5, stream_id=3), stream=s)
    buf = fr[1].clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        f.step(buf)
    e = pf.Filter(pf.make_params(1000, 128, 128, dtype, x0=x0, y0=y0, seed=5, stream_id=3))
    for t in range(1, 7):
        buf.copy_(fr[t])
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        e.step(fr[t])
        assert f.estimate() == e.estimate()
    u, v = f.export(), e.export()
    assert np.array_equal(u["x"], v["x"]) and np.array_equal(u["y"], v["y"])
    e.close()
    f.close()


@pytest.mark.parametrize("dtype", ["f64", "bf16"])
def test_one_launch_on_the_static_scratch(dtype):
    vid = pfsynth.moving_disk(128, 128, 5, 5, (64, 64), (1, -2), 3.0, 11)
    fr = torch.from_numpy(vid.frames).to("cuda:0")
    x0, y0 = vid.centres[0]
    a = _filter(dtype, 1000, 5, False, vid)
    b = pf.Filter(pf.make_params(1000, 128, 128, dtype, x0=x0, y0=y0, seed=5, stream_id=3, state_only=True))
    for t in range(1, 5):
        a.step(fr[t])
        b.step(fr[t])
        assert a.estimate() == b.estimate()
    u, v = a.export(), b.export()
    assert np.array_equal(u["x"], v["x"]) and np.array_equal(u["y"], v["y"])
    a.close()
    b.close()
