"""The streaming pass A at sizes that stream by the rule of radius and
deviations, bit for bit against the one-tile pass (which a filter with the
per-pixel likelihood always takes), and batches on both sides of the rule
against their members alone."""
import numpy as np
import pytest
import torch

import paper_2308_00763_amd as pf
from test_gpu_stream import _frames, _run, _state

pytestmark = pytest.mark.gpu

M = 1 << 20


@pytest.mark.parametrize("dtype, r, side, start, sigma, kind, pitch, n", [
    ("f16", 5, 256, (128, 128), (5.0, 2.0), None, None, 6 * M + 777),
    ("bf16", 12, 255, (128, 128), (5.0, 2.0), None, 257, 5 * M - 1),     # rows not 4-byte aligned
    ("f32", 1, 64, (3, 61), (3.0, 3.0), None, None, 6 * M + 777),        # cells clamped at the frame's edges
    ("f16", 8, 128, (8, 119), (5.0, 4.0), None, None, 6 * M + 1),        # an edge, a larger table
    ("f16", 16, 256, (128, 128), (2.0, 6.0), None, None, 4 * M + 5),     # sums straight from the frame
    ("f16", 5, 256, (128, 128), (5.0, 2.0), "outliers", None, 6 * M + 777),
    ("f32", 8, 256, (128, 128), (3.0, 3.0), "two_places", None, 5 * M + 777),
    ("bf16", 5, 256, (128, 128), (5.0, 2.0), "spread", None, 6 * M + 777),
    ("f32", 8, 256, (128, 128), (5.0, 2.0), "outliers", None, 8193 * 1024 - 5),  # FP32 past the write-through sizes
    ("f16", 5, 256, (128, 128), (5.0, 2.0), None, None, 8193 * 1024 - 5),
])
def test_stream_equals_one_tile_pass(dtype, r, side, start, sigma, kind, pitch, n):
    fr = _frames(side, r, start, 5, pitch)
    st = _state(kind, n, start)
    a = _run(n, dtype, r, side, fr, start, sigma, st)
    b = _run(n, dtype, r, side, fr, start, sigma, st, naive_likelihood=True)
    for u, v in zip(a, b):
        assert np.array_equal(u, v)


@pytest.mark.parametrize("dtype, radii, sizes", [
    ("f16", (5,), [1, 1024, 1025, 70001, 204800] * 45),    # streams: a run's last tile, runs of one tile
    ("bf16", (8,), [1, 1024, 1025, 70001, 204800] * 45),
    ("f32", (8,), [1, 1024, 1025, 70001, 204800] * 45),
    ("f32", (3, 12, 5), [1, 1024, 1025, 70001, 204800] * 45),
    ("f16", (5, 12), [1000] * 4100),                       # enough tiles, one each: does not stream
])
def test_batch_equals_alone(dtype, radii, sizes):
    """Some members of another pass-A size, some whose table does not fit, some
    inactive."""
    side = 128
    ps, frs = [], []
    scenes = [[_frames(side, r, (60 + i, 64), 100 + i) for i in range(9)] for r in radii]
    for i, n in enumerate(sizes):
        frs.append(scenes[i % len(radii)][i % 9])
        ps.append(pf.make_params(n, side, side, dtype, radius=radii[i % len(radii)], x0=60 + i % 9, y0=64, seed=4,
                                 stream_id=i, threads_a=512 if i % 9 == 3 else None,
                                 sigma=(9.0, 9.0) if i % 31 == 7 else (5.0, 2.0)))
    b = pf.Batch(ps)
    active = np.array([i % 11 != 5 for i in range(len(sizes))], dtype=np.uint8)
    for t in range(1, 4):
        b.step([f[t] for f in frs], active if t == 2 else None)
    est = b.estimates()
    for i in range(0, len(sizes), max(7, len(sizes) // 40)):
        f = pf.Filter(ps[i])
        for t in range(1, 4):
            if t != 2 or active[i]:
                f.step(frs[i][t])
        assert f.estimate() == tuple(est[i])
        u, v = f.export(), b.export(i)
        assert np.array_equal(u["x"], v["x"]) and np.array_equal(u["y"], v["y"])
        f.close()
    b.close()
