"""Which IF calls resolve their hits inside the geometry launch: few rays x chirps
and few hits a ray.  Counted as the kernel nodes of a captured call; rays of many
hits would resolve each of them again for every chirp.

Results against the FP64 oracle: relative L2 <= 1e-5 per (pair, chirp) block, as
for every IF cube (FP64 phases, FP32 phasors or 2^-29 fixed point: about 1e-6).
"""
import ctypes as C

import numpy as np
import pytest

from oracle import raymeta as R
from paper_2305_14176_amd import rayscene as S

pytestmark = pytest.mark.gpu


def _hip():
    """The HIP runtime this process has loaded."""
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    return C.CDLL(sorted(paths)[0])


def _kernels(call):
    """Kernel nodes of one captured call."""
    import torch
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    n = C.c_size_t(0)
    assert _hip().hipGraphGetNodes(C.c_void_p(g.raw_cuda_graph()), None, C.byref(n)) == 0
    return n.value


def _scene(n_rays, n_chirps, hits):
    sc = S.small_scene(n_rays=n_rays, n_chirps=n_chirps, n_samples=40, n_tx=1, n_rx=1)
    rng = np.random.default_rng(hits)
    n = n_rays * hits
    sc.ray_off = (np.arange(n_rays + 1) * hits).astype(np.int32)
    sc.hit_mesh = rng.integers(0, sc.n_meshes, n).astype(np.int32)
    sc.hit_tri = (rng.random(n) * np.diff(sc.mesh_tri_off)[sc.hit_mesh]).astype(np.int32)
    u = rng.random(n)
    sc.hit_u, sc.hit_v = u.astype(np.float32), (rng.random(n) * (1 - u)).astype(np.float32)
    sc.amp = S.random_amplitudes(sc, 3)
    return sc


@pytest.mark.parametrize("n_rays, n_chirps, hits, inline", [
    (300, 2, 1, True),
    (300, 2, 6, True),          # the most hits a ray
    (300, 2, 7, False),
    (300, 16, 64, False),
    (65536, 4, 2, True),        # the most rays x chirps
    (65537, 4, 2, False),
    (65536, 4, 12, False),
])
@pytest.mark.parametrize("method", ["spread", "direct"])
def test_hits_are_resolved_where_it_is_cheaper(method, n_rays, n_chirps, hits, inline):
    from paper_2305_14176_amd import raymeta as RM
    sc = _scene(n_rays, n_chirps, hits)
    ds = RM.DeviceScene(sc)
    syn = RM.Synthesizer(ds, method=method)
    got = syn.run(0, ds.amp).cpu().numpy()
    # geometry, sum over rays, finish or reduce; and a launch of its own to resolve the hits
    assert _kernels(lambda: syn.run(0, ds.amp)) == (3 if inline else 4)
    sel = [0, 17, 39]
    ref = R.if_cube(sc, chirps=[n_chirps - 1], samples=sel)
    err = np.linalg.norm(got[:, n_chirps - 1:, sel] - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert err.max() <= 1e-5, err.max()
