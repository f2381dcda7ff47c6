"""Hybrid pixel walk where neighbouring pixels' terms are added up before they
reach LDS: every pixel on the same Gaussian, ragged edges, single pixels that
share with no neighbour, unequal hit counts, and lists beyond one window of the
walk's accumulators (384 positions on 8x8 tiles, 128 on 16x16).

Against the fp64 oracle at the bar of test_gpu_parity: gradients 1e-4 relative
L2 (fp32 sums of at most a few hundred hits).
"""
import numpy as np
import pytest

import oracle
from helpers import random_tiny_scene, rel_l2, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [8, 16])
@pytest.mark.parametrize("n,width,height,size", [
    (1, 8, 8, "wide"), (1, 17, 3, "wide"), (5, 1, 1, "wide"), (12, 9, 16, "wide"), (40, 33, 18, "mixed"),
    (200, 31, 17, "small"), (130, 17, 9, "wide"), (420, 9, 9, "wide"),
])
def test_hybrid_walk(n, width, height, size, tile):
    ls_mu, ls_sd, spread = {"wide": (-0.6, 0.2, 0.2), "mixed": (-1.8, 0.9, 0.5), "small": (-3.2, 0.3, 0.8)}[size]
    sc, _, _ = random_tiny_scene(np.random.default_rng(7 * n + width), n, width, height, 2, tile=tile, spread=spread,
                                 ls_mu=ls_mu, ls_sd=ls_sd, logit_mu=-3.5, logit_sd=0.3, high_sd=0.1)
    o = oracle.OracleScene(sc)
    ren = o.render()
    assert (ren["margin"] >= 1e-9).all()
    gpu = run_gpu(sc, mode="hybrid")
    ref = o.backward(sc.dl_dimage)
    for k, v in gpu["grads"].items():
        assert rel_l2(v, ref[k]) <= 1e-4, k
