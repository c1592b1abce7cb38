"""Which launch an IF call takes, read from the kernel nodes of a captured call:
four workgroups of synth_kernel a compute unit where the grid has more than three
for each, and fewer copies of the spreading grid for few rays.

Results against the FP64 oracle: relative L2 <= 1e-5 per (pair, chirp) block, as
for every IF cube (FP64 phases, FP32 phasors or 2^-29 fixed point: about 1e-6).
"""
import ctypes as C

import numpy as np
import pytest

from oracle import raymeta as R
from paper_2305_14176_amd import rayscene as S

pytestmark = pytest.mark.gpu


class _Dim3(C.Structure):
    _fields_ = [("x", C.c_uint), ("y", C.c_uint), ("z", C.c_uint)]


class _Node(C.Structure):
    """hipKernelNodeParams."""
    _fields_ = [("block", _Dim3), ("extra", C.c_void_p), ("func", C.c_void_p), ("grid", _Dim3),
                ("params", C.c_void_p), ("lds", C.c_uint)]


def _hip():
    """The HIP runtime this process has loaded."""
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    return C.CDLL(sorted(paths)[0])


def _launches(call):
    """Launch parameters of the kernels of one captured call, in order."""
    import torch
    hip = _hip()
    g = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(g):
        call()
    graph, n = C.c_void_p(g.raw_cuda_graph()), C.c_size_t(0)
    assert hip.hipGraphGetNodes(graph, None, C.byref(n)) == 0
    nodes = (C.c_void_p * n.value)()
    assert hip.hipGraphGetNodes(graph, nodes, C.byref(n)) == 0
    out = [_Node() for _ in nodes]
    for node, p in zip(nodes, out):
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)) == 0
    return out


def _run(method, n_rays, n_pairs, n_chirps, n_samples):
    """The sum over rays' launch (after the geometry) of a call checked against the oracle."""
    from paper_2305_14176_amd import raymeta as RM
    sc = S.small_scene(n_rays=n_rays, n_chirps=n_chirps, n_samples=n_samples, n_tx=1, n_rx=n_pairs)
    sc.amp = S.random_amplitudes(sc, 3)
    ds = RM.DeviceScene(sc)
    syn = RM.Synthesizer(ds, method=method)
    got = syn.run(0, ds.amp).cpu().numpy()
    sel = [0, n_samples // 2, n_samples - 1]
    ref = R.if_cube(sc, chirps=[n_chirps - 1], samples=sel)
    err = np.linalg.norm(got[:, n_chirps - 1:, sel] - ref, axis=-1) / np.linalg.norm(ref, axis=-1)
    assert err.max() <= 1e-5, err.max()
    return _launches(lambda: syn.run(0, ds.amp))[1]


@pytest.mark.parametrize("n_rays, n_pairs, n_chirps, n_samples", [
    (100, 48, 16, 40),          # three workgroups a compute unit
    (100, 49, 16, 40),          # more
    (100, 64, 16, 300),
    (100, 32, 16, 520),         # two passes over the samples
    (3000, 48, 16, 40),         # partitions
])
def test_direct_launch_fills_its_compute_units(n_rays, n_pairs, n_chirps, n_samples):
    k = _run("direct", n_rays, n_pairs, n_chirps, n_samples)
    assert k.grid.x >= n_pairs * n_chirps and k.block.x == 256
    per_cu = C.c_int(0)
    assert _hip().hipOccupancyMaxActiveBlocksPerMultiprocessor(C.byref(per_cu), C.c_void_p(k.func), 256,
                                                               C.c_size_t(k.lds)) == 0
    assert per_cu.value == (4 if k.grid.x > 3 * 256 else 3)


@pytest.mark.parametrize("n_rays, n_samples, copies", [
    (1, 30, 8), (95, 30, 8), (96, 30, 8), (1023, 30, 8), (1024, 30, 16),            # 64 cells
    (95, 60, 4), (96, 60, 8), (1023, 60, 8), (1024, 60, 16),                        # 128
    (95, 120, 2), (96, 120, 4), (1023, 120, 4), (1024, 120, 8),                     # 256
    (95, 250, 2), (1023, 250, 2), (1024, 250, 4),                                   # 512
    (95, 500, 2), (1024, 500, 2),                                                   # 1024
])
@pytest.mark.parametrize("n_pairs", [1, 20])                                        # 16 and 320 workgroups
def test_spread_copies_follow_the_rays(n_pairs, n_rays, n_samples, copies):
    k = _run("spread", n_rays, n_pairs, 16, n_samples)
    cells = 1 << (2 * n_samples - 1).bit_length()
    assert (k.grid.x, k.block.x) == (16 * n_pairs, 256 if n_pairs > 16 else 512)
    assert k.lds == copies * 2 * (cells + 8) * 8
