"""The rows per tile that the automatic launch takes for FP64 rows of three to
five waves: as many as 16 waves hold where that saves the fullest compute unit
work, rounds of workgroups counted; and the same bits as a fixed shape.
"""
import numpy as np
import pytest

from paper_2305_14176_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims, rows, planes", [
    ((150, 130, 110), 4, 16),       # three waves: 15 in a workgroup, not 12
    ((192, 96, 160), 3, 20),        # the smaller tile fills the chip as it is
    ((224, 64, 40), 2, 5),          # four waves: the larger tile saves less than a twentieth
    ((193, 130, 64), 3, 13),        # 16 waves
    ((256, 192, 256), 3, 64),       # both march 64 planes: two rounds of the smaller tile, one of the larger
    ((256, 256, 256), 2, 64),       # two rounds of either
    ((257, 34, 110), 2, 8),         # five waves: 15, not 10
])
def test_automatic_f64_tile(dims, rows, planes):
    from paper_2305_14176_amd.solver import YeeSolver
    nx, ny, nz = dims
    wl = W.cpml_block_lattice(nx, steps=3, seed=sum(dims), precision="f64", cpml=5, nprobes=6, nfreq=2, block=16,
                              ny=ny, nz=nz)
    init = W.random_initial_fields(wl, seed=7)
    got = []
    for shape in ({}, {"tile_rows": 1, "chunk_planes": 32}):
        s = YeeSolver(wl, **shape)
        for c, f in init.items():
            s.set_field(c, f)
        s.step(wl.steps)
        got.append((s.launch_info(), s.series(), [s.field(c) for c in W.COMP_INDEX]))
        s.close()
    (info, y0, f0), (_, y1, f1) = got
    assert (info["tile_rows"], info["chunk_planes"], info["samples_per_lane"]) == (rows, planes, 1)
    assert np.array_equal(y0, y1)
    for a, b in zip(f0, f1):
        assert np.array_equal(a, b) and np.abs(a).max() > 0
