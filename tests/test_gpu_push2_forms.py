"""The 2D push where a tile's current box changes form: tiles that fit the LDS
as a whole, tiles that only fit a work-group's particles at a time, groups
that do not fit either, patches across the period's seam, a partial last
group.  Cells, offsets and integer currents of a field-free push must equal
the contract's."""
import numpy as np
import pytest

from test_gpu_pic2d import _contract_currents, _gpu_particles, _oracle, _zero_fields
from workloads import preset2d, random_particles2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("tile,capacity", [(256, 0), (512, 1 << 18), (1024, 1 << 20)])
@pytest.mark.parametrize("rows,group,patch,n", [
    (64, 256, (10, 10), 2348),   # patches of 256 particles: their tile's box does not fit
    (64, 256, (16, 48), 1024),   # patches near the largest box
    (64, 256, (30, 62), 1300),   # patches over the whole period that do not fit
    (64, 1024, (12, 12), 2048),  # whole tiles that fit
    (5, 256, (4, 5), 1500),      # a period of 5 rows
])
def test_push_boxes_bit_exact(precision, tile, capacity, rows, group, patch, n):
    from paper_1008_1685_amd.run2d import Run2D

    print(f"\n[gpu] push2 {precision} tile {tile}, {rows} rows, {group} per {patch}", flush=True)
    cfg = preset2d("d1", precision=precision, box_y=rows / 32, x_foil=1.0)
    sim = _oracle(cfg)
    nx, ny = sim.nx, sim.ny
    parts = []
    for s in (0, 1):
        p = random_particles2d(7 + s, n, 0, 1, 1, sim.w_ref, 1e-2, 1e3, False)
        rng = np.random.default_rng(n + s)
        g = np.arange(n) // group
        x0 = rng.integers(2, nx - 2 - patch[0], g[-1] + 1)
        y0 = rng.integers(0, ny, g[-1] + 1)
        p["ix"] = x0[g] + rng.integers(0, patch[0], n)
        p["iy"] = (y0[g] + rng.integers(0, patch[1], n)) % ny
        parts.append(p)
    run = Run2D(cfg, capacity=max(n, capacity))
    assert run.info["tile"] == tile
    run.set_state({s: _gpu_particles(run, parts[s]) for s in (0, 1)}, fields=_zero_fields(nx, ny), step=0)
    run.push_deposit()
    st = run.get_state()
    J, moved = _contract_currents(cfg, sim, {0: parts[0], 1: parts[1]}, st, run)
    for s in range(2):
        g = st[f"sp{s}"]
        ix1, iy1, ox1, oy1 = moved[s]
        assert np.array_equal(g["cell"], run.encode(ix1, iy1))
        if precision == "fp32":  # (the contract's offsets are float32)
            assert np.array_equal(g["ox"], ox1) and np.array_equal(g["oy"], oy1)
    if precision == "fp32":
        for k, name in enumerate(("Jx_int", "Jy_int", "Jz_int")):
            assert np.array_equal(st[name], J[k]), name
    # exact continuity at any precision: the carried charge follows the particles
    run.field_advance()
    assert run.diag()["gauss_int"] == 0
    run.close()
