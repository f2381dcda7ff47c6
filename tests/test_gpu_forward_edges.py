"""Forward trace at the edges of its steps: list lengths around the groups of
four, the chunks of 64 positions and the window of 128, copies of one Gaussian
(equal depths; more of them than a lane's pool holds), and hits that stay
pending longer than the pool and the window hold.

Against the fp64 oracle, at the bars of test_gpu_parity: pixels 1e-5 (fp32
colours of order 1), hits per pixel exact, gradients 1e-4 relative L2.  Pixels
within rounding of a decision are left out of all three: their upstream
gradient is zero on both sides.
"""
import numpy as np
import pytest

import oracle
from helpers import random_tiny_scene, rel_l2, run_gpu
from paper_2608_17298_amd.scenes import pinhole_camera

pytestmark = pytest.mark.gpu


def _check(sc, tiny=0.0, **kw):
    o = oracle.OracleScene(sc)
    ren = o.render()
    # (a margin of exactly 0 is a tie of equal depths, which the index decides on both sides)
    ok = (ren["margin"] >= 1e-9) | (ren["margin"] == 0)
    assert ok.mean() > 0.9
    sc.dl_dimage.reshape(-1, 3)[~ok] = 0.0
    gpu = run_gpu(sc, **kw)
    assert np.array_equal(gpu["n_hits"][ok], ren["n_included"][ok])
    assert np.abs(gpu["image"].reshape(-1, 3) - ren["color"])[ok].max() <= 1e-5
    assert np.abs(gpu["t_final"].astype(np.float64) - ren["T_final"])[ok].max() <= 1e-6
    ref = o.backward(sc.dl_dimage)
    for k, v in gpu["grads"].items():
        if np.linalg.norm(ref[k]) < tiny:  # fp32 sums cannot hold it
            assert np.linalg.norm(v) < 2 * tiny, k
        else:
            assert rel_l2(v, ref[k]) <= 1e-4, k
    return gpu


@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 63, 64, 65, 127, 128, 129, 260])
def test_list_lengths(n, tile):
    # every Gaussian covers the whole image, one tile and a ragged edge
    sc, _, _ = random_tiny_scene(np.random.default_rng(100 + n), n, tile + 3, tile + 1, 3, tile=tile, spread=0.2,
                                 ls_mu=-0.6, ls_sd=0.2, logit_mu=-3.5, logit_sd=0.3, high_sd=0.1)
    gpu = _check(sc)
    assert np.diff(gpu["tile_range"]).max() == n


@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("copies", [2, 12, 16, 40])
def test_copies_of_one_gaussian(copies, tile):
    """Equal depths are composited in index order, also where a lane's pool
    cannot hold all of them."""
    sc, _, _ = random_tiny_scene(np.random.default_rng(copies), 60, 21, 18, 1, tile=tile, spread=0.4, ls_mu=-1.5,
                                 ls_sd=0.3, logit_mu=-2.5, logit_sd=0.3)
    src = 7
    at = np.random.default_rng(3).choice(60, copies, replace=False)
    for name in ("means", "log_scales", "quats", "opacity_logits"):
        getattr(sc, name)[at] = getattr(sc, name)[src]
    _check(sc)


@pytest.mark.parametrize("tile", [8, 16])
def test_long_pending_hits(tile):
    """Flat Gaussians tilted against the rays: their depth varies over a tile
    by more than the spacing of the list, so that hits stay pending past the
    pool (rescans) and past the window of list positions."""
    n = 400
    sc, _, _ = random_tiny_scene(np.random.default_rng(11), n, 40, 33, 2, tile=tile, spread=0.3, ls_mu=-0.7, ls_sd=0.2,
                                 logit_mu=-3.5, logit_sd=0.3)
    sc.log_scales[:, 2] = -4.0
    from paper_2608_17298_amd import gart
    gpu = _check(sc)
    assert gpu["counters"][gart.CNT_FWD_RESCANS] > 0 and gpu["counters"][gart.CNT_FWD_DROPS] > 0


POOL = 11  # entries of the smallest pool a lane has


@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("n,step", [(40, 0.0), (130, 0.0), (130, 2e-8), (60, 4e-7)])
def test_equal_depths_take_few_passes(n, step, tile):
    """Gaussians at the same depth, and closer together than the pool's keys
    tell apart: every pass over the list composites a pool of hits a lane."""
    sc, _, _ = random_tiny_scene(np.random.default_rng(n), n, tile + 5, tile - 1, 1, tile=tile, logit_mu=-4.0, logit_sd=0.2)
    sc.means[:] = 0.0
    sc.means[:, 2] = np.random.default_rng(5).permutation(n) * np.float32(step)
    sc.log_scales[:] = [-0.2, -0.6, -0.4]
    sc.quats[:] = sc.quats[0]
    gpu = _check(sc)
    from paper_2608_17298_amd import gart
    waves = -(-(tile + 5) // 8) * -(-(tile - 1) // 8)
    assert gpu["n_hits"].max() == n
    assert gpu["counters"][gart.CNT_FWD_RESCANS] <= waves * (-(-n // POOL) - 1)


@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("n,steps", [(40, 1), (40, 400), (130, 3)])
def test_depths_below_the_float_range(n, steps, tile):
    """Depths that are subnormal floats, some of them with the smallest keys."""
    cam = pinhole_camera(tile + 5, tile - 1, 60.0, 0.0)
    rng = np.random.default_rng(n + steps)
    sc, _, _ = random_tiny_scene(rng, n, tile + 5, tile - 1, 1, tile=tile, logit_mu=-4.0, logit_sd=0.2, cam=cam)
    sc.means[:] = 0.0
    sc.means[:, 2] = np.float32(2.0 ** -149) * rng.integers(1, steps * n, n)
    sc.log_scales[:] = [-0.2, -0.6, -0.4]
    sc.quats[:] = sc.quats[0]
    # the offsets of the rays from the means, and with them three groups' gradients, are subnormal as well
    gpu = _check(sc, tiny=np.finfo(np.float32).tiny)
    assert gpu["n_hits"].max() == n


@pytest.mark.parametrize("tile", [8, 16])
def test_scales_beyond_the_square_root_of_the_range(tile):
    """Gaussians whose squared inverse scales are subnormal, and which are still
    visible (axis-aligned, opacity within rounding of alpha_min, so that their
    rectangle is the image): hit by every ray, in the order of their depths."""
    n, huge = 40, 12
    cam = pinhole_camera(13, 11)
    cam.cx = cam.cy = 0.0
    rng = np.random.default_rng(1)
    sc, _, _ = random_tiny_scene(rng, n, 13, 11, 1, tile=tile, ls_mu=-0.6, ls_sd=0.3, logit_mu=-2.0, logit_sd=0.3, cam=cam)
    alpha_min = float(np.float32(1 / 255))
    threshold = np.log(alpha_min / (1 - alpha_min))
    sc.means[:huge, :2] = 0.0
    sc.log_scales[:huge] = rng.uniform(354.0, 358.0, (huge, 3))
    sc.quats[:huge] = [1, 0, 0, 0]
    sc.opacity_logits[:huge] = np.float32(threshold) + np.float32(4.8e-7) * rng.integers(2, 20, huge)
    o = oracle.OracleScene(sc)
    assert (np.exp(-2.0 * sc.log_scales[:huge].astype(np.float64).min(1)) < np.finfo(np.float64).tiny).sum() > 6
    assert (o.prim_info().area[:huge] == 13 * 11).sum() > 6
    assert o.ray_prim(np.arange(13 * 11), np.zeros(13 * 11, int))["hit"].all()
    gpu = _check(sc)
    assert gpu["n_hits"].min() > 6
