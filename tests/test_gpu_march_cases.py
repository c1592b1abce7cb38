"""The march of the step kernel on small grids, where the automatic launch takes
the step without a march: tile ownership, guard bands and the FP64 oracle.

Every case states the launch it means and checks it, so that another automatic
choice cannot move the case to another kernel.

* Write counts: every stored sample counts exactly one store (it belongs to one
  tile of one chunk), padding columns at most one, the zero plane none.
* Guard bands around the workspace stay intact over single steps.
* Oracle, relative L2 per final field: FP64 1e-12 (rounding order and FMA
  contraction), FP32 1e-5, FP16 storage 1e-3 (few steps from a common state:
  both take the same rounding decisions almost everywhere).
"""
import numpy as np
import pytest

from paper_2305_14176_amd import workloads as W
from _helpers import oracle_from_workload, rel_l2, stored

pytestmark = pytest.mark.gpu

COMPS = ("Ex", "Ey", "Ez", "Hx", "Hy", "Hz")


def _wl(dims, precision, cpml, steps=4):
    nx, ny, nz = dims
    if precision == "f16":
        return W.fp16_substrate(nx, ny, nz, steps=steps, cpml=cpml)
    wl = W.cpml_block_lattice(nx, ny=ny, nz=nz, steps=steps, precision=precision, cpml=0, nprobes=0, nfreq=0, block=4)
    wl.cpml_cells = (cpml, max(cpml - 1, 0), max(cpml - 2, 0))
    wl.cpml_kappa_max, wl.cpml_alpha_max = 2.0, 0.05
    if min(dims) < 4:
        wl.sources = []
    return wl


def _solver(wl, launch, expect, **kw):
    from paper_2305_14176_amd.solver import YeeSolver
    s = YeeSolver(wl, tile_rows=launch[0], chunk_planes=launch[1], samples_per_lane=launch[2], **kw)
    info = s.launch_info()
    print(f"[gpu] {wl.nx}x{wl.ny}x{wl.nz} {wl.precision} {info}", flush=True)
    assert (info["tile_rows"], info["chunk_planes"], info["samples_per_lane"]) == expect
    return s


@pytest.mark.parametrize("dims, precision, cpml, launch, expect", [
    ((2, 2, 2), "f32", 0, (1, 2, 0), (1, 2, 1)),
    ((37, 29, 23), "f64", 4, (3, 5, 0), (3, 5, 1)),             # ragged tiles and chunks
    ((33, 17, 9), "f64", 3, (2, 4, 0), (2, 4, 1)),
    ((150, 130, 110), "f64", 6, (0, 0, 0), (4, 16, 1)),         # three waves a row, 15 in a workgroup
    ((193, 130, 64), "f64", 5, (0, 0, 0), (3, 13, 1)),          # four waves a row, 16 in a workgroup
    ((257, 34, 110), "f64", 4, (0, 0, 0), (2, 8, 1)),           # five waves a row
    ((256, 20, 33), "f32", 4, (2, 8, 0), (2, 8, 1)),
    ((70, 40, 36), "f16", 4, (2, 6, 1), (2, 6, 1)),             # FP16 storage, one sample a lane
    ((300, 40, 40), "f16", 4, (3, 8, 2), (3, 8, 2)),            # two samples a lane
    ((301, 21, 18), "f16", 4, (2, 7, 2), (2, 7, 2)),            # ragged rows of two samples a lane
    ((301, 64, 80), "f16", 4, (0, 0, 0), (3, 8, 2)),            # the same, too large for the other step
])
def test_march_owns_every_sample_once(dims, precision, cpml, launch, expect):
    nx, ny, nz = dims
    s = _solver(_wl(dims, precision, cpml), launch, expect, series_len=4)
    for _ in range(2):                      # two calls: counts start at zero each time
        counts = s.write_counts(1)
        inner = counts[:, :nz, :ny, :nx]
        assert inner.min() == 1 and inner.max() == 1, (inner.min(), inner.max())
        assert counts[:, :nz, :ny, nx:].max(initial=0) <= 1
        assert counts[:, nz].max() == 0
    s.close()


@pytest.mark.parametrize("dims, precision, launch, expect", [
    ((90, 33, 40), "f32", (4, 8, 0), (4, 8, 1)),
    ((90, 33, 40), "f16", (4, 8, 0), (4, 8, 1)),
    ((90, 33, 40), "f64", (4, 8, 0), (4, 8, 1)),
    ((301, 33, 20), "f16", (3, 6, 2), (3, 6, 2)),
    ((150, 130, 110), "f64", (0, 0, 0), (4, 16, 1)),
])
def test_march_stays_between_guard_bands(dims, precision, launch, expect):
    wl = _wl(dims, precision, 6)
    s = _solver(wl, launch, expect, series_len=16, guard_bytes=1 << 16)
    assert s.check_guards()
    for c, a in W.random_initial_fields(wl, 12).items():
        s.set_field(c, a)
    s.step(13)
    s.status()
    state = s.save_state()
    s.step(3)
    s.load_state(state)
    s.step(2)
    assert s.check_guards()
    s.close()


@pytest.mark.parametrize("dims, precision, cpml, launch, expect, tol", [
    ((37, 29, 23), "f64", 4, (3, 5, 0), (3, 5, 1), 1e-12),
    ((200, 12, 30), "f64", 5, (3, 8, 0), (3, 8, 1), 1e-12),     # four waves a row, 16 in a workgroup
    ((300, 9, 11), "f64", 4, (2, 4, 0), (2, 4, 1), 1e-12),      # five waves a row, 15 in a workgroup
    ((300, 17, 26), "f32", 6, (3, 4, 2), (3, 4, 2), 1e-5),      # two samples a lane, three waves a row
    ((300, 40, 40), "f16", 4, (3, 8, 2), (3, 8, 2), 1e-3),
    ((301, 40, 40), "f16", 4, (3, 8, 2), (3, 8, 2), 1e-3),      # ragged rows of two samples a lane
    ((300, 40, 40), "f16", 4, (2, 8, 1), (2, 8, 1), 1e-3),      # one sample a lane, five waves a row
])
def test_march_against_the_oracle(dims, precision, cpml, launch, expect, tol):
    wl = _wl(dims, precision, cpml)
    s = _solver(wl, launch, expect)
    init = W.random_initial_fields(wl, 51)
    for c, a in init.items():
        s.set_field(c, a)
    s.step(wl.steps)
    sim = oracle_from_workload(wl, initial=init)
    assert sim.dt == s.dt
    sim.run(wl.steps)
    for c in COMPS:
        err = rel_l2(s.field(c), stored(sim, c))
        assert err <= tol, (c, err)
    s.close()


@pytest.mark.parametrize("shape", [{"samples_per_lane": 1}, {"tile_rows": 3}, {"chunk_planes": 5}])
def test_any_launch_value_selects_the_march(shape):
    """A grid that takes the step without a march by itself marches once any
    value of the launch shape is set."""
    from paper_2305_14176_amd.solver import YeeSolver
    wl = W.cpml_block_lattice(48, steps=2, cpml=8, nprobes=4, nfreq=2)
    own = YeeSolver(wl)
    assert own.launch_info()["chunk_planes"] == 1
    s = YeeSolver(wl, **shape)
    assert s.launch_info()["chunk_planes"] > 1
    for q in (own, s):
        q.step(wl.steps)
    assert np.array_equal(own.series(), s.series())
    own.close()
    s.close()
