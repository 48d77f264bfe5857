"""FDK on every path of the back-projection against the FP64 oracle: volumes of
few tiles (the views summed in parts), windows of either size, boxes inside the
detector and past its edges, and voxels too coarse for a window, without and
with motion.  Bar as in test_gpu_fdk.py (FP32 positions)."""
import math

import numpy as np
import pytest

from oracle import fdk as ofdk
from oracle.geometry import moved_projection
from paper_1806_02637_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eng():
    import torch

    from paper_1806_02637_amd import engine

    assert torch.cuda.is_available()
    e = engine.Engine(0)
    yield e
    e.close()


@pytest.mark.parametrize("n_views,W,H,pitch,vol", [
    (40, 96, 80, 2.4, (48, 40, 24, 2.4)),   # parts of the views, 44-row windows, boxes inside the detector
    (15, 96, 80, 2.4, (16, 16, 16, 3.0)),   # one tile, one part
    (41, 130, 65, 2.4, (18, 17, 33, 4.6)),  # 56-row windows, boxes past the detector
    (33, 64, 50, 4.0, (24, 24, 9, 9.0)),    # no window fits
    (25, 3, 2, 60.0, (7, 5, 3, 8.0)),       # a detector of a few pixels
])
@pytest.mark.parametrize("moved", [False, True])
def test_fdk_paths(eng, n_views, W, H, pitch, vol, moved):
    import torch

    print(f"case: fdk {n_views} views {W}x{H}, volume {vol}, moved {moved}", flush=True)
    g = inputs.ScanGeometry(n_views, W, H, pitch)
    P, intr, betas, arc = g.projection_matrices(), g.intrinsics(), g.orbit_angles(), math.radians(g.arc_deg)
    imgs = inputs.project(g, inputs.random_phantom(5, 6, contained_radius=0.9 * g.fov_radius(), semi_range=(5.0, 30.0),
                                                   centre_radius=20.0))
    theta = inputs.smooth_motion(3, n_views, peak=3.0, params=(0, 1, 2, 3, 4, 5)) if moved else None
    Pm = None if theta is None else np.array(
        [moved_projection([list(r) for r in P[i]], list(theta[i])) for i in range(n_views)])
    scan = eng.load_scan(P, intr, imgs)
    got = scan.fdk(torch.tensor(imgs, device="cuda"), vol, theta=theta).cpu().numpy()
    ref = ofdk.fdk(imgs, P, intr, betas, arc, g.sid_mm, ofdk.Volume(*vol), moved_P=Pm)
    scan.free()
    peak = np.abs(ref).max()
    err = np.abs(got - ref)
    assert err.max() <= 1e-4 * peak and np.sqrt(np.mean(err ** 2)) <= 1e-5 * peak


@pytest.mark.parametrize("n_views,W,H", [
    (20, 255, 7),   # 2 blocks of outputs per wave, odd width, rows past the last tile
    (20, 514, 5),   # 3
    (20, 801, 4),   # 4
    (20, 1278, 4),  # 5
    (20, 1283, 3),  # two column tiles
    (16, 4096, 2),  # the widest detector (the largest table of taps)
])
def test_fdk_filter_widths(eng, n_views, W, H):
    """The ramp filter over its column tilings.  Q = x / 4 + off-diagonal sum
    nearly cancels on wide smooth rows, so its FP32 error is a rounding of the
    two terms, up to 2^-23 x_max / 4 each, scaled by f / D; the back-projection
    adds it over the arc with weights near 1.  Bar: that, twice, plus the
    position bar of 1e-4 of the peak."""
    import torch

    print(f"case: fdk filter {n_views} views {W}x{H}", flush=True)
    g = inputs.ScanGeometry(n_views, W, H, 380.0 / W)
    P, intr, betas, arc = g.projection_matrices(), g.intrinsics(), g.orbit_angles(), math.radians(g.arc_deg)
    imgs = inputs.project(g, inputs.random_phantom(6, 6))
    vol = (20, 18, 2, 0.6 * g.pitch_mm)
    scan = eng.load_scan(P, intr, imgs)
    got = scan.fdk(torch.tensor(imgs, device="cuda"), vol).cpu().numpy()
    ref = ofdk.fdk(imgs, P, intr, betas, arc, g.sid_mm, ofdk.Volume(*vol))
    scan.free()
    bar = 1e-4 * np.abs(ref).max() + 2.0 * arc * (2.0 ** -23 * imgs.max() / 2.0) * g.f_px / g.sid_mm
    err = np.abs(got - ref).max()
    print(f"  max err {err:.2e} of peak {np.abs(ref).max():.3g}, bar {bar:.2e}", flush=True)
    assert err <= bar
