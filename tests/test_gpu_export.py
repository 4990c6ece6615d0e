"""Exports of one coordinate and of both agree, at the sizes up to which both
are copied at once and past them, and on a filter with a pending resampling."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2308_00763_amd as pf

pytestmark = pytest.mark.gpu


def _get(h, n, x, y, step):
    out = [np.full(n, np.nan) if want else None for want in (x, y)]
    p = [None if o is None else ctypes.c_void_p(o.ctypes.data) for o in out]
    if step:
        assert pf.lib().pf_export_step(h, p[0], p[1], None) == 0
    else:
        assert pf.lib().pf_export(h, p[0], p[1], None, None, None) == 0
    return out


@pytest.mark.parametrize("dtype, n", [("f64", 1), ("f64", 70001), ("f32", 32768), ("f32", 32769), ("f16", 65536),
                                      ("f16", 65537), ("bf16", 1023), ("bf16", 70001)])
def test_one_coordinate_or_both(dtype, n):
    f = pf.Filter(pf.make_params(n, 128, 96, dtype, x0=60.25, y0=40.5, seed=5))
    frame = torch.randint(0, 255, (96, 128), dtype=torch.uint8, device="cuda:0")
    for step in (True, False):  # the propagated positions; the state, resampled for the export
        f.step(frame)
        x, y = _get(f.handle, n, True, True, step)
        assert np.all(np.isfinite(x)) and np.all(np.isfinite(y))
        assert np.abs(x - 60).max() < 80 and np.abs(y - 40).max() < 60
        assert np.array_equal(_get(f.handle, n, True, False, step)[0], x)
        assert np.array_equal(_get(f.handle, n, False, True, step)[1], y)
        assert _get(f.handle, n, False, False, step) == [None, None]
    f.close()
