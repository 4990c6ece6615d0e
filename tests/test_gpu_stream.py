"""The streaming pass A (a table of pixel cells kept over a run of tiles)
against the one-tile pass A, bit for bit: both form the same integer disk sums
and the same sums of weights in the same order.  A filter with the per-pixel
likelihood always takes the one-tile kernel."""
import numpy as np
import pytest
import torch

import paper_2308_00763_amd as pf
import pfsynth

pytestmark = pytest.mark.gpu

N = 4096 * 1024 + 777  # the fewest tiles that stream, and a ragged one


def _frames(side, r, start, seed, pitch=None):
    v = pfsynth.moving_disk(side, side, 4, r, start, (1, -2), 4.0, seed)
    pitch = pitch or side
    buf = torch.zeros((4, side, pitch), dtype=torch.uint8, device="cuda:0")
    buf[:, :, :side] = torch.from_numpy(v.frames)
    return buf[:, :, :side]


def _run(n, dtype, r, side, fr, start, sigma, state, **kw):
    f = pf.Filter(pf.make_params(n, side, side, dtype, radius=r, x0=start[0], y0=start[1], drift=(1.0, -2.0),
                                 sigma=sigma, seed=9, **kw))
    if state is not None:
        f.load(state[0], state[1], 0)
    est = []
    for t in range(1, 4):
        f.step(fr[t])
        est.append(f.estimate())
    got = f.export()
    f.close()
    return np.array(est), got["x"], got["y"]


def _state(kind, n, start):
    x = np.full(n, float(start[0]))
    y = np.full(n, float(start[1]))
    k = np.arange(n)
    if kind == "outliers":      # now and then a particle far off: the table is rebuilt, then given up
        far = k % 3001 == 17
        x[far] += 60.0 * ((k[far] // 3001) % 5 - 2)
    elif kind == "two_places":  # tiles with different maxima, in blocks
        away = (k // 5000) % 2 == 1
        x[away] += 25.0
    elif kind == "spread":      # wider than the row-prefix window
        x += (k % 211) - 105.0
        y += (k % 97) - 48.0
    else:
        return None
    return x, y


@pytest.mark.parametrize("dtype, r, side, start, sigma, kind, pitch, n", [
    ("f16", 5, 256, (128, 128), (5.0, 2.0), None, None, N),
    ("bf16", 12, 255, (128, 128), (5.0, 2.0), None, 257, N),        # rows not 4-byte aligned
    ("f32", 1, 64, (3, 61), (5.0, 2.0), None, None, N),             # cells clamped at the frame's edges
    ("f16", 8, 128, (8, 119), (9.0, 7.0), None, None, N),           # an edge, a larger table
    ("f32", 3, 256, (128, 128), (0.0, 0.0), None, None, N),         # one cell
    ("f16", 5, 256, (128, 128), (20.0, 9.0), None, None, N),        # box within the window, too many cells
    ("bf16", 5, 256, (128, 128), (60.0, 60.0), None, None, N),      # sums straight from the frame
    ("f16", 5, 256, (128, 128), (5.0, 2.0), "outliers", None, N),
    ("f32", 8, 256, (128, 128), (3.0, 3.0), "two_places", None, N),
    ("bf16", 5, 256, (128, 128), (5.0, 2.0), "spread", None, N),
    ("f16", 8, 256, (128, 128), (5.0, 2.0), None, None, 8193 * 1024 - 5),  # past the write-through sizes
])
def test_stream_equals_one_tile_pass(dtype, r, side, start, sigma, kind, pitch, n):
    fr = _frames(side, r, start, 5, pitch)
    st = _state(kind, n, start)
    a = _run(n, dtype, r, side, fr, start, sigma, st)
    b = _run(n, dtype, r, side, fr, start, sigma, st, naive_likelihood=True)
    for u, v in zip(a, b):
        assert np.array_equal(u, v)


@pytest.mark.parametrize("dtype, radii", [("f16", (5,)), ("bf16", (8,)), ("f32", (3, 12, 5))])
def test_streamed_batch_equals_alone(dtype, radii):
    """Members of 1 to 200 tiles in one grid (runs that end inside a
    workgroup's share), two pass-A sizes among them, some inactive."""
    sizes = [1, 1024, 1025, 70001, 204800] * 20
    side = 128
    ps, frs = [], []
    for i, n in enumerate(sizes):
        r = radii[i % len(radii)]
        frs.append(_frames(side, r, (60 + i % 9, 64), 100 + i))
        ps.append(pf.make_params(n, side, side, dtype, radius=r, x0=60 + i % 9, y0=64, seed=4, stream_id=i,
                                 threads_a=512 if i % 7 == 3 else None))
    b = pf.Batch(ps)
    active = np.array([i % 11 != 5 for i in range(len(sizes))], dtype=np.uint8)
    for t in range(1, 4):
        b.step([f[t] for f in frs], active if t == 2 else None)
    est = b.estimates()
    for i in range(0, len(sizes), 3):
        f = pf.Filter(ps[i])
        for t in range(1, 4):
            if t != 2 or active[i]:
                f.step(frs[i][t])
        assert f.estimate() == tuple(est[i])
        u, v = f.export(), b.export(i)
        assert np.array_equal(u["x"], v["x"]) and np.array_equal(u["y"], v["y"])
        f.close()
    b.close()
