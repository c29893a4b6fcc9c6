"""The 2D sort's and push's forms in FP64: every particle once and in key
order through the sort's window, key table and global claims; cells, offsets
and all three integer currents of a field-free push equal to the contract's
evaluated in double precision, whichever box a tile's current goes through."""
import numpy as np
import pytest

import test_gpu_sort_forms as sorts
from oracle import contract2d
from test_gpu_pic2d import _contract_currents, _gpu_particles, _oracle, _zero_fields
from workloads import preset2d, random_particles2d

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 2048, 2049, 7000])
@pytest.mark.parametrize("cols,rows", [(1, 1), (8, 64), (64, 64), (65, 64), (300, 500), (2560, 512)])
def test_sort_2d_fp64(n, cols, rows, monkeypatch):
    monkeypatch.setattr(sorts, "preset2d", lambda name, **kw: preset2d(name, precision="fp64", **kw))
    sorts.test_sort_2d(n, cols, rows)


@pytest.mark.parametrize("tile,capacity", [(256, 0), (512, 1 << 18), (1024, 1 << 20)])
@pytest.mark.parametrize("rows,group,patch,n,mixed_w", [
    (64, 256, (10, 10), 2348, False),   # patches of 256 particles: their tile's box does not fit
    (64, 256, (16, 48), 1024, False),   # patches near the largest box
    (64, 256, (30, 62), 1300, False),   # patches over the whole period that do not fit
    (64, 1024, (12, 12), 2048, False),  # whole tiles that fit
    (5, 256, (4, 5), 1500, False),      # a period of 5 rows
    (64, 256, (10, 10), 2348, True),    # particles of other weights than the reference
])
def test_push_currents_fp64(tile, capacity, rows, group, patch, n, mixed_w, monkeypatch):
    from paper_1008_1685_amd.run2d import Run2D

    print(f"\n[gpu] push2 fp64 tile {tile}, {rows} rows, {group} per {patch} {mixed_w}", flush=True)
    monkeypatch.setattr(contract2d, "F32", np.float64)  # the contract's one rounding per operation, in double
    cfg = preset2d("d1", precision="fp64", box_y=rows / 32, x_foil=1.0)
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
        p["ox"], p["oy"] = rng.random(n), rng.random(n)  # (all 53 bits)
        for k in ("ux", "uy", "uz"):
            p[k] = p[k] * (1.0 + 1e-9 * rng.random(n))
        if mixed_w:
            p["w"] = p["w"] * np.array([1.0, 0.37, 1.0, 1.6, 1.0, 2.9])[np.arange(n) % 6]
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
        assert np.array_equal(g["ox"], ox1) and np.array_equal(g["oy"], oy1)
    for k, name in enumerate(("Jx_int", "Jy_int", "Jz_int")):
        assert np.array_equal(st[name], J[k]), name
    run.field_advance()
    assert run.diag()["gauss_int"] == 0
    run.close()
