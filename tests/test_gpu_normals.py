"""The double mode's normals against 80-bit arithmetic on the same random words.

A filter at the origin with no drift and unit deviations moves each particle
by exactly its normals, so the propagated positions are the normals.  Bound:
-2 ln(1 - u) to 1 ulp (its square root then to 2^-53), the square root's own
rounding, cosine and sine to 3.5 2^-53 of one (the reduced angle's rounding,
the polynomial and its last sum), the product: under 8 2^-53 of the radius."""
import numpy as np
import pytest
import torch

import oracle
import paper_2308_00763_amd as pf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seed, sid, t", [(0, 0, 1), (2**63 + 12345, 7, 3)])
def test_f64_normals_against_long_double(seed, sid, t):
    n = 6000
    f = pf.Filter(pf.make_params(n, 64, 64, "f64", x0=0.0, y0=0.0, drift=(0.0, 0.0), sigma=(1.0, 1.0), seed=seed,
                                 stream_id=sid))
    f.load(np.zeros(n), np.zeros(n), t - 1)
    f.step(torch.zeros((64, 64), dtype=torch.uint8, device="cuda:0"))
    got = f.export_step()
    f.close()
    w = np.array([oracle.philox_words(seed, k, t, sid, 0) for k in range(n)], dtype=np.uint64)
    u = ((w[:, 0::2] << np.uint64(21)) | (w[:, 1::2] >> np.uint64(11))).astype(np.longdouble) / np.longdouble(2) ** 53
    rho = np.sqrt(-2 * np.log1p(-u[:, 0]))
    turn = 8 * np.arctan(np.longdouble(1)) * u[:, 1]
    tol = 8 * 2.0 ** -53 * rho
    assert np.all(np.abs(got["x_prop"] - rho * np.cos(turn)) <= tol)
    assert np.all(np.abs(got["y_prop"] - rho * np.sin(turn)) <= tol)
