"""The numeric primitives at the edges of their ranges: the double mode's normals
on random words near the ends and the splits of its logarithm and cosine, its
weights over likelihoods down to the smallest doubles, and the reduced modes'
pixel cells at ties, at the floats beside them and far outside the frame."""
import numpy as np
import pytest
import torch

import oracle
import paper_2308_00763_amd as pf

pytestmark = pytest.mark.gpu

ND = oracle.disk(5)[0].size
SEED, SID = 12345, 7


@pytest.mark.parametrize("t, k, what", [
    (7752, 679, "1 - u near 1"), (40349, 236, "1 - u near 1"), (61315, 376, "1 - u small"), (39962, 887, "1 - u small"),
    (28623, 629, "mantissa beside sqrt(1/2)"), (64288, 82, "mantissa beside sqrt(1/2)"),
    (64943, 808, "mantissa beside sqrt(1/2)"), (44728, 798, "angle beside a quarter turn"),
    (1926, 670, "angle beside a quarter turn"), (865, 142, "angle beside an eighth"), (5898, 22, "angle beside an eighth")])
def test_f64_normals_at_edge_words(t, k, what):
    """As in test_gpu_normals (same bound: 8 2^-53 of the radius), at words
    found by a search over 2^26 counters; every other particle of the step too."""
    n = 1024
    f = pf.Filter(pf.make_params(n, 64, 64, "f64", x0=0.0, y0=0.0, drift=(0.0, 0.0), sigma=(1.0, 1.0), seed=SEED,
                                 stream_id=SID))
    f.load(np.zeros(n), np.zeros(n), t - 1)
    f.step(torch.zeros((64, 64), dtype=torch.uint8, device="cuda:0"))
    got = f.export_step()
    f.close()
    w = np.array([oracle.philox_words(SEED, j, t, SID, 0) for j in range(n)], dtype=np.uint64)
    u = ((w[:, 0::2] << np.uint64(21)) | (w[:, 1::2] >> np.uint64(11))).astype(np.longdouble) / np.longdouble(2) ** 53
    a, q = float(1 - u[k, 0]), float(4 * u[k, 1])
    edge = {"1 - u near 1": 1 - a, "1 - u small": a, "mantissa beside sqrt(1/2)": abs(np.frexp(a)[0] - 0.5 ** 0.5),
            "angle beside a quarter turn": abs(q - round(q)), "angle beside an eighth": abs(abs(q - round(q)) - 0.5)}[what]
    assert edge < 1e-7
    rho = np.sqrt(-2 * np.log1p(-u[:, 0]))
    turn = 8 * np.arctan(np.longdouble(1)) * u[:, 1]
    tol = 8 * 2.0 ** -53 * rho
    assert np.all(np.abs(got["x_prop"] - rho * np.cos(turn)) <= tol)
    assert np.all(np.abs(got["y_prop"] - rho * np.sin(turn)) <= tol)


@pytest.mark.parametrize("kappa", [0.5, 5.0, 50.0, 5000.0])
def test_f64_weights_relative_to_the_largest(kappa):
    """w_k / w_max against exp of the difference of the disk terms' likelihoods
    (the GPU's own integers, divided and subtracted as it does).  Bound: the
    exponential 0.861 ulp (1.72 2^-53), a rounding each of the two divisions by the
    normaliser, and of the quotient here: under 5 2^-53 where the weights are
    normal numbers; as many units of the last place below."""
    n, side = 1000, 64
    rng = np.random.default_rng(5)
    fr = torch.from_numpy(rng.integers(0, 256, (side, side)).astype(np.uint8)).to("cuda:0")
    f = pf.Filter(pf.make_params(n, side, side, "f64", x0=32.0, y0=32.0, sigma=(9.0, 9.0), seed=3, kappa=kappa,
                                 diagnostics=True))
    f.step(fr)
    got, S = f.export(), f.export_step()["disk_sum"]
    f.close()
    L = S.astype(np.float64) / (kappa * ND)
    d = L - L.max()
    want = np.exp(d.astype(np.longdouble))
    ratio = got["w"].astype(np.longdouble) / got["w"].max()
    z = float(got["w"].max())
    normal = (want > 2.3e-308) & (got["w"] > 2.3e-308)
    print(f"[edges] kappa {kappa}: least exponent {d.min():.1f}, {normal.sum()} normal weights", flush=True)
    assert np.all(np.abs(ratio - want)[normal] <= 5 * 2.0 ** -53 * want[normal])
    assert np.all(np.abs(ratio - want)[~normal] <= 5 * 5e-324 / z)


def _offsets(dtype):
    """Offsets from the origin cell: ties, the representable numbers beside them,
    zeros, and positions far off."""
    v = [0.0, -0.0, 0.25, -0.25, 0.49999997, -0.49999997]
    for h in np.arange(-12.5, 13.0, 0.5):
        h = np.float32(h)
        v += [h, np.nextafter(h, np.float32(99)), np.nextafter(h, np.float32(-99))]
    for h in (-12.5, -3.5, -0.5, 0.5, 1.5, 7.5):
        for ulp in (2.0 ** -10, 2.0 ** -7, 2.0 ** -11, 2.0 ** -8):  # beside the ties in 16 bits
            v += [h * (1 + ulp), h * (1 - ulp)]
    far = [300.5, -300.5, 4095.5, -4096.5, 30000.0, -30000.0]
    if dtype != "f16":
        far += [8388607.5 / 16, -8388607.5 / 16, 9e5, -9e5]
    return np.array(v), np.array(far)


@pytest.mark.parametrize("axis", ["x", "y"])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16", "f64"])
def test_pixel_cells(dtype, axis):
    """A frame whose grey value is the coordinate: the disk sum gives the cell."""
    side, origin = 256, 128
    near, far = _offsets(dtype)
    off = np.concatenate([near, far])
    off = np.concatenate([off, -off])  # mean 0: the origin cell is 128
    n = off.size
    ramp = np.arange(side, dtype=np.uint8)
    frame = np.broadcast_to(ramp[None, :] if axis == "x" else ramp[:, None], (side, side)).copy()
    p = pf.make_params(n, side, side, dtype, x0=origin, y0=origin, drift=(0.0, 0.0), sigma=(0.0, 0.0),
                       diagnostics=True)
    f = pf.Filter(p)
    pos, mid = origin + off, np.full(n, float(origin))
    f.load(*((pos, mid) if axis == "x" else (mid, pos)), 0)
    f.step(torch.from_numpy(frame).to("cuda:0"))
    got = f.export_step()
    f.close()
    x = got["x_prop"] if axis == "x" else got["y_prop"]
    cell = origin + np.floor((x - origin) + 0.5)  # exact: few bits beside the origin
    dy, dx = np.mgrid[-5:6, -5:6]
    d = dx[dx * dx + dy * dy < 25]
    want = np.clip(cell[:, None] + d[None, :], 0, side - 1).sum(1)
    S = 2 * (228 - 100) * want - ND * (228 ** 2 - 100 ** 2)
    assert np.array_equal(got["disk_sum"].astype(np.int64), S.astype(np.int64))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_pixel_cells_of_the_streaming_pass(dtype):
    side, origin, n = 256, 128, 6 * (1 << 20) + 777
    near, far = _offsets(dtype)
    off = np.concatenate([near, -near])
    off = np.tile(off, n // off.size + 1)[:n]
    off[-2 * (off.size % 2) - 1] = 0.0
    far_at = np.arange(50000, n, 700001)
    off[far_at] = far[np.arange(far_at.size) % far.size]
    frame = np.broadcast_to(np.arange(side, dtype=np.uint8)[None, :], (side, side)).copy()
    f = pf.Filter(pf.make_params(n, side, side, dtype, x0=origin, y0=origin, drift=(0.0, 0.0), sigma=(0.0, 0.0),
                                 diagnostics=True))
    f.load(origin + off, np.full(n, float(origin)), 0)
    f.step(torch.from_numpy(frame).to("cuda:0"))
    got = f.export_step()
    f.close()
    o = got["x_prop"] - origin
    cell = origin + np.floor(o + 0.5)
    dy, dx = np.mgrid[-5:6, -5:6]
    d = dx[dx * dx + dy * dy < 25]
    table = np.array([np.clip(c + d, 0, side - 1).sum() for c in range(-10, side + 10)])
    want = table[np.clip(cell, -10, side + 9).astype(np.int64) + 10]
    S = 2 * (228 - 100) * want - ND * (228 ** 2 - 100 ** 2)
    assert np.array_equal(got["disk_sum"].astype(np.int64), S)
