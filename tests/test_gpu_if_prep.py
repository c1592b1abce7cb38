"""IF cubes at the edges of the call's preparation: hits resolved and tables
computed by the geometry launch (one batch, at most 2^18 rays x chirps) or by a
launch of their own, and one to 64 partial maxima of the weights.

Tolerance: relative L2 <= 1e-5 per (pair, chirp) block against the FP64 oracle
(FP64 phases, FP32 phasors or 2^-29 fixed point: about 1e-6).  The largest
weight sits at the last ray, the smallest partial maximum's share: a maximum
that missed it would overflow the fixed-point grid.
"""
import numpy as np
import pytest

from oracle import raymeta as R
from paper_2305_14176_amd import rayscene as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("method", ["spread", "direct"])
@pytest.mark.parametrize("n_rays, n_chirps, n_samples", [
    (255, 1, 5),            # part of one workgroup's rays; a ragged last table block
    (257, 16, 33),          # the largest batch of one launch
    (257, 17, 33),          # a second batch: a launch of their own
    (2049, 2, 100),         # two partial maxima
    (131072, 2, 64),        # 2^18 rays x chirps: the last inline call; 64 partial maxima
    (131073, 2, 64),        # the first beyond it, more rays than 64 shares of 2048
])
def test_preparation_routes(n_rays, n_chirps, n_samples, method):
    import torch
    from paper_2305_14176_amd import raymeta as RM
    sc = S.small_scene(n_rays=n_rays, n_chirps=n_chirps, n_samples=n_samples, n_tx=1, n_rx=2)
    sc.amp = S.random_amplitudes(sc, 3)
    sc.amp[-1] = 50.0
    # three rays whose meta data are out of range add nothing: for the oracle their weight is zero
    bad = [3, n_rays // 2, n_rays - 2]
    ok = sc.amp.copy()
    ok[bad] = 0.0
    sel = sorted({0, 1, n_samples // 2, n_samples - 1})
    chirps = sorted({0, n_chirps - 1})
    w, sc.amp = sc.amp, ok
    ref = R.if_cube(sc, chirps=chirps, samples=sel)
    sc.amp = w
    sc.hit_mesh, sc.hit_tri = sc.hit_mesh.copy(), sc.hit_tri.copy()
    sc.hit_mesh[sc.ray_off[bad[0]]] = sc.n_meshes
    sc.hit_mesh[sc.ray_off[bad[1]]] = -1
    sc.hit_tri[sc.ray_off[bad[2]]] = 1 << 30
    ds = RM.DeviceScene(sc)
    got = RM.if_cube(ds, weights=torch.from_numpy(w).to(ds.device), method=method).cpu().numpy()
    got = got[:, chirps][:, :, sel]
    err = np.linalg.norm(got - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert err.max() <= 1e-5, err.max()
