"""GPU parity of the bilateral depth filter against the float64 oracle.
Bar: the set of valid outputs is exact (an output is 0 exactly where the
input is invalid) and values agree within 5e-6 m.  Derivation: the kernel's
float32 weights carry a relative error of a few 1e-6 (exp of an argument up
to ~20 that matters), which moves the mean by at most that times the depth
spread of the weighted window (~3 sigma_range = 0.075 m): < 1e-6 m; the
float32 accumulation of at most 225 terms of w (d_q - d_p) adds < 2e-6 m;
the final rounding of a depth below 4 m adds 2.4e-7 m."""
import numpy as np
import pytest

from gpu_helpers import to_device
from synth import Intrinsics, configs, render_depth

pytestmark = pytest.mark.gpu

TOL = 5e-6


def _run(depth, radius, ss, sr):
    import torch
    import paper_1708_00783_amd as T
    d = to_device(depth)
    out = torch.full(depth.shape, -1.0, dtype=torch.float32, device="cuda")
    T.tf_bilateral(d, out, radius, ss, sr)
    return out.cpu().numpy()


def _check(depth_m, got, radius, ss, sr, tag):
    from oracle.bilateral import bilateral
    want = bilateral(depth_m, radius, ss, sr)
    assert np.array_equal(got > 0, want > 0), tag
    assert np.array_equal(got == 0, depth_m == 0), tag
    err = np.abs(got.astype(np.float64) - want).max()
    assert err <= TOL, f"{tag}: max error {err:.3g} m"
    return err


def test_full_frame_u16_matches_oracle():
    mm = configs.c2_frame(7)
    dm = (mm.astype(np.float32) / np.float32(1000.0)).astype(np.float32)
    for radius, ss, sr in ((2, 2.5, 0.025), (1, 1.0, 0.01), (7, 4.0, 0.05)):
        got = _run(mm, radius, ss, sr)
        err = _check(dm, got, radius, ss, sr, f"640x480 r{radius}")
        print(f"r={radius} ss={ss} sr={sr}: max error {err:.2e} m", flush=True)
    # the same depth as float32 metres gives the same output
    assert np.array_equal(_run(dm, 2, 2.5, 0.025), _run(mm, 2, 2.5, 0.025))


def test_ragged_image_with_holes_and_tiny_images():
    K = Intrinsics(270.0, 268.0, 166.3, 124.8, 333, 251)
    d = render_depth(configs.c2_scene(3), configs.c2_poses(300, 3)[40], K).astype(np.float32)
    rng = np.random.default_rng(5)
    d[rng.random(d.shape) < 0.1] = 0.0
    d[:, :5] = 0.0
    _check(d, _run(d, 3, 2.0, 0.03), 3, 2.0, 0.03, "333x251")
    for shape in ((1, 1), (1, 37), (23, 1), (17, 16)):
        t = rng.uniform(0.5, 3.0, shape).astype(np.float32)
        t[rng.random(shape) < 0.2] = 0.0
        _check(t, _run(t, 2, 1.5, 0.5), 2, 1.5, 0.5, f"{shape}")


def test_rejects_bad_arguments():
    import torch
    import paper_1708_00783_amd as T
    d = torch.zeros((8, 8), dtype=torch.float32, device="cuda")
    with pytest.raises(T.TsdfError):
        T.tf_bilateral(d, d, 2, 2.0, 0.02)          # output overlaps the input
    out = torch.empty_like(d)
    with pytest.raises(T.TsdfError):
        T.tf_bilateral(d, out, 8, 2.0, 0.02)        # radius beyond 7
    with pytest.raises(T.TsdfError):
        T.tf_bilateral(d, out, 2, 0.0, 0.02)


@pytest.mark.parametrize("radius", [1, 2, 3, 4, 5, 6, 7])
def test_every_radius_and_a_range_that_overflows(radius):
    """the window of each radius has its own kernel: on an image of ragged tiles; and with a range so narrow that the exponent of a far neighbour
    overflows, where only equal depths count"""
    rng = np.random.default_rng(radius)
    d = rng.choice([0.0, 0.5, 0.5625, 12.0], size=(35, 50), p=[0.1, 0.4, 0.3, 0.2]).astype(np.float32)
    _check(d, _run(d, radius, 2.0, 0.05), radius, 2.0, 0.05, f"r{radius}")
    assert np.array_equal(_run(d, radius, 2.0, 3e-19), d)


@pytest.mark.parametrize("lo,hi", [(-87.0, -18.0), (-103.0, -87.5)])
def test_range_weights_are_as_exact_as_expf(lo, hi):
    """The exponential of the range weight, read off the output: beside a pixel
    of 2^-126 m one of 2^60 m with weight w < 2^-25 makes it 2^-126 +
    2^60 w / (1 + w), which is 2^60 w in float32, subnormal w too.  Its error against 64 bits is within expf's over all
    floats of the interval (mean 0.257, at most 0.852 ulp; among the subnormals
    0.273 and 1.0), the mean with room for a sample of 4096."""
    import torch
    import paper_1708_00783_amd as T
    n = 4096
    sr = (2.0 ** 60 * np.sqrt(-0.5 / np.linspace(lo, hi, n))).astype(np.float32)
    d = torch.tensor([[2.0 ** -126, 2.0 ** 60]], dtype=torch.float32, device="cuda")
    out = torch.zeros((n, 1, 2), dtype=torch.float32, device="cuda")
    for k in range(n):
        T.tf_bilateral(d, out[k], 1, 1e6, float(sr[k]))
    w = out[:, 0, 0].cpu().numpy().astype(np.float64) * 2.0 ** -60
    t = -(1.0 / (2.0 * sr.astype(np.float64) ** 2)).astype(np.float32).astype(np.float64) * 2.0 ** 120
    x = np.exp(t)
    ulp = np.ldexp(1.0, np.maximum(np.frexp(x)[1], -125) - 24)
    err = np.abs(w - x) / ulp
    mean, most = (0.27, 0.86) if lo == -87.0 else (0.285, 1.0)
    print(f"exp over [{lo}, {hi}]: mean {err.mean():.4f} max {err.max():.4f} ulp", flush=True)
    assert err.mean() <= mean and err.max() <= most
