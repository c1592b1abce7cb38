"""Which small grids the no-march step takes, and their bits on both sides of the line.

The line was drawn from measured times; wide rows and thin plates whose march
is faster by more than a run's spread have to march, the small ones must not.
"""
import numpy as np
import pytest

from paper_2305_14176_amd import workloads as W

pytestmark = pytest.mark.gpu


def _solver(dims, precision, cpml, **shape):
    from paper_2305_14176_amd.solver import YeeSolver
    nx, ny, nz = dims
    wl = W.cpml_block_lattice(nx, ny=ny, nz=nz, steps=5, precision=precision, cpml=0, nprobes=4, nfreq=2, block=7,
                              seed=sum(dims))
    wl.cpml_cells = tuple(min(cpml, n // 3) for n in dims)
    if precision == "f16":
        wl.fp16_exp = (12, 12, 12, 21, 21, 21)
    s = YeeSolver(wl, **shape)
    for c, f in W.random_initial_fields(wl, seed=5).items():
        s.set_field(c, f)
    s.step(wl.steps)
    return s


@pytest.mark.parametrize("dims, precision, cpml, marches", [
    # us a step without a march / with it
    ((64, 64, 64), "f32", 10, False),        # 8.1 / 12.6
    ((100, 72, 72), "f32", 10, False),       # 15.2 / 19.2
    ((64, 126, 127), "f16", 10, False),      # rows of one wave, 4 MiB: 20.6 / 21.5
    ((150, 43, 44), "f64", 10, False),       # 17.3 / 21.8
    ((320, 40, 40), "f32", 6, False),        # 16.4 / 23.3
    ((150, 10, 95), "f64", 0, True),         # a second round of few workgroups: 12.6 / 10.9
    ((128, 8, 501), "f64", 6, True),         # 23.6 / 21.9
    ((256, 63, 63), "f32", 6, True),         # 25.2 / 20.4
    ((150, 73, 73), "f32", 0, True),         # 23.2 / 20.1
    ((256, 40, 40), "f16", 0, True),         # 14.0 / 13.1
    ((384, 51, 52), "f32", 6, True),         # 32.2 / 24.3
    ((321, 8, 334), "f16", 6, True),         # 35.7 / 20.7
    ((384, 36, 37), "f64", 6, True),         # 29.8 / 24.8
])
def test_the_faster_step_is_taken(dims, precision, cpml, marches):
    s = _solver(dims, precision, cpml)
    info = s.launch_info()
    assert (info["chunk_planes"] > 1) == marches, info
    other = _solver(dims, precision, cpml, tile_rows=1, chunk_planes=4)
    assert other.launch_info()["chunk_planes"] == 4
    for c in W.COMP_INDEX:
        assert np.array_equal(s.field(c), other.field(c)), c
    assert np.array_equal(s.series(), other.series()) and np.array_equal(s.dft(), other.dft())
    s.close()
    other.close()
