"""The column-strip field kernel against the tile kernel, bit for bit, where
the strips' rows and columns change form (one, two and more waves over the
period, a partial last one, strips narrower than their halos, a box of one
strip) and where the columns that hold a current change: a foil in a wide
vacuum, currents and step counters set by the host between steps."""
import numpy as np
import pytest

from workloads import preset2d

pytestmark = pytest.mark.gpu

GRIDS = ("Ex", "Ey", "Ez", "Bx", "By", "Bz", "Jx_int", "Jy_int", "Jz_int", "charge_int")


def _same(runs, what):
    a, b = (r.get_state(particles=False) for r in runs)
    for k in GRIDS:
        assert np.array_equal(a[k], b[k]), (what, k)
    for k in ("E_in", "E_out_left", "E_out_right"):
        # row sums of the same terms; the tiles' products may be fused differently
        assert a["budget"][k] == pytest.approx(b["budget"][k], rel=1e-13, abs=1e-300), (what, k)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("cols,rows", [(320, 64), (9, 2), (40, 3), (75, 61), (64, 62), (130, 122), (100, 123),
                                       (700, 337), (60, 512)])
def test_strips_match_tiles(precision, cols, rows):
    from paper_1008_1685_amd.run2d import Run2D

    print(f"\n[gpu] field2 {precision} {cols} x {rows}", flush=True)
    cfg = preset2d("d1", precision=precision, box_x=cols / 32, box_y=rows / 32, pol="CP", waist=0.3,
                   x_foil=min(2.0, cols / 64), thickness=min(1.0, cols / 128), t_rise=0.5, t_flat=20.0,
                   sort_interval=7)  # (in the pulse's fall the kernels' incident waves differ by an ulp in FP64)
    runs = [Run2D(dict(cfg, field_kernel=k)) for k in ("strips", "tiles")]
    assert [r.get_info()["field_kernel"] for r in runs] == ["strips", "tiles"]
    rng = np.random.default_rng(cols * rows)
    nx, ny = runs[0].info["nx"], runs[0].info["ny"]
    f = {k: rng.uniform(-50, 50, (nx + (2 if k in ("Ex", "By", "Bz") else 1), ny)) for k in GRIDS[:6]}
    for r in runs:
        r.set_state(fields=f)
    for n in (1, 1, 5, 20):
        for r in runs:
            r.step(n)
        _same(runs, n)
    # currents of the host's in columns no push touches
    j = {k: rng.integers(-(1 << 30), 1 << 30, (nx + (2 if k == "Jx_int" else 3), ny)) for k in GRIDS[6:9]}
    for r in runs:
        r.set_state(fields=j)
        r.field_advance()
    _same(runs, "host currents")
    for r in runs:
        r.step(3)
    _same(runs, "after host currents")
    # the step counter set by the host, to the same and to the other parity
    for step in (101, 260):
        st = runs[0].get_state()
        for r in runs:
            r.set_state(particles={0: st["sp0"], 1: st["sp1"]}, step=step)
            r.step(4)
        _same(runs, ("step", step))
    for r in runs:
        r.close()


def test_automatic_choice_is_strips_at_any_period():
    from paper_1008_1685_amd.run2d import Run2D

    for prec, rows in (("fp32", 1100), ("fp64", 601)):
        print(f"\n[gpu] field2 auto {prec} {rows}", flush=True)
        cfg = preset2d("d1", precision=prec, box_x=2.0, box_y=rows / 32, x_foil=0.5, thickness=0.25, ppc_x=1, ppc_y=1)
        runs = [Run2D(dict(cfg, field_kernel=k)) for k in ("auto", "tiles")]
        assert runs[0].get_info()["field_kernel"] == "strips"
        for r in runs:
            r.step(40)
        _same(runs, rows)
        for r in runs:
            r.close()
