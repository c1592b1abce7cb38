"""Spreading workgroups of every grid length: 2 to 16 interleaved grid copies,
256 and 512 threads, short and long partitions.

Tolerance: relative L2 <= 1e-5 per (pair, chirp) block against the FP64 oracle
(the kernel's aliasing of about 1e-7 and 2^-29 fixed point: about 1e-6).
"""
import numpy as np
import pytest

from oracle import raymeta as R
from paper_2305_14176_amd import rayscene as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rays, n_tx, n_rx, n_chirps", [
    (70, 1, 1, 1),              # one ragged workgroup, fewer rays than threads
    (5000, 3, 4, 16),           # more than a workgroup a CU: 256 threads
    (177000, 3, 4, 16),         # partitions of 4352 rays: long from 512 cells up
    (353000, 3, 4, 16),         # of 8448: long for every grid
])
@pytest.mark.parametrize("n_samples", [32, 33, 128, 256, 257, 513])      # grids of 64 to 2048 cells
def test_spread_grid_copies(n_samples, n_rays, n_tx, n_rx, n_chirps):
    from paper_2305_14176_amd import raymeta as RM
    sc = S.small_scene(n_rays=n_rays, n_chirps=n_chirps, n_samples=n_samples, n_tx=n_tx, n_rx=n_rx)
    sc.amp = S.random_amplitudes(sc, 6)
    sel = sorted({0, 1, n_samples // 2, n_samples - 1})
    pairs = sorted({0, n_tx * n_rx - 1})
    print(f"[gpu] spread grids: {n_rays} rays, {n_tx * n_rx} pairs, {n_chirps} chirps, {n_samples} samples", flush=True)
    ref = R.if_cube(sc, chirps=[n_chirps - 1], samples=sel)[pairs]
    got = RM.if_cube(RM.DeviceScene(sc)).cpu().numpy()[pairs, n_chirps - 1:, :][:, :, sel]
    err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert err.max() <= 1e-5, err.max()
