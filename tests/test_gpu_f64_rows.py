"""FP64 rows of three and four waves: the automatic tile (up to 16 waves a
workgroup) against a fixed shape, bit for bit.

Every launch shape runs the same per-sample arithmetic, so the fields, CPML
auxiliaries and probe samples have to be equal.
"""
import numpy as np
import pytest

from paper_2305_14176_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims, cpml", [
    ((130, 65, 300), (5, 4, 6)),     # three waves a row; ragged tiles and chunks
    ((192, 41, 230), (8, 1, 9)),     # three full waves
    ((193, 63, 170), (7, 3, 2)),     # four waves, one sample into the last
    ((256, 34, 251), (0, 5, 4)),     # four full waves
])
def test_automatic_f64_tile_equals_a_fixed_shape(dims, cpml):
    import torch
    from paper_2305_14176_amd.solver import YeeSolver
    nx, ny, nz = dims
    wl = W.cpml_block_lattice(nx, steps=5, seed=sum(dims), precision="f64", cpml=0, nprobes=12, nfreq=2, block=7,
                              ny=ny, nz=nz)
    wl.cpml_cells = cpml
    init = W.random_initial_fields(wl, seed=4)
    got = []
    for shape in ({}, {"tile_rows": 2, "chunk_planes": 16}):
        s = YeeSolver(wl, **shape)
        for c, f in init.items():
            s.set_field(c, f)
        s.step(wl.steps)
        state = s.save_state(torch.zeros(s.state_bytes(), dtype=torch.uint8, device="cuda:0"))
        got.append((s.launch_info(), s.series(), s.dft(), state.cpu().numpy().view(np.uint64)))
        s.close()
    (i0, y0, d0, a), (i1, y1, d1, b) = got
    assert i1["chunk_planes"] == 16 and i0["chunk_planes"] > 1      # both march
    assert np.array_equal(y0, y1) and np.array_equal(d0, d1)
    zero = np.uint64(1) << np.uint64(63)                            # a zero may carry either sign
    assert np.array_equal(np.where(a == zero, 0, a), np.where(b == zero, 0, b))
