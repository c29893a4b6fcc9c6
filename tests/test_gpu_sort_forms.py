"""The cell sort at the sizes where its position claims change form: tiles
whose keys fit the LDS window, fill an LDS table of keys, or span more than
the table's 2^20 keys; particle counts at the edges of a tile; all particles
of a wave in one cell, or each in its own.  Every particle must come out
once, in key order; the order within a cell is open."""
import numpy as np
import pytest

from workloads import preset, preset2d

pytestmark = pytest.mark.gpu


def _check(before, after, keys, order_of):
    for s in ("sp0", "sp1"):
        a, b = before[s], after[s]
        oa, ob = (np.lexsort([p[k] for k in keys]) for p in (a, b))
        for k in a:
            assert np.array_equal(a[k][oa], b[k][ob]), (s, k)
        assert np.array_equal(order_of(b), np.sort(order_of(b), kind="stable")), s


def _particles(rng, n, cell, rdt, extra):
    d = dict(cell=cell.astype(np.int32), w=np.full(n, 0.5))
    for k in ("ux", "uy", "uz"):
        d[k] = rng.normal(size=n)
    for k in extra:
        d[k] = rng.integers(0, 1 << 24, n) / float(1 << 24)
    return {k: v if k == "cell" else v.astype(rdt) for k, v in d.items()}


@pytest.mark.parametrize("n", [1, 2048, 2049, 7000])
@pytest.mark.parametrize("cols,rows", [(1, 1), (8, 64), (64, 64), (65, 64), (300, 500), (2560, 512)])
def test_sort_2d(n, cols, rows):
    from paper_1008_1685_amd.run2d import Run2D

    print(f"\n[gpu] sort 2d {n} over {cols} x {rows}", flush=True)
    run = Run2D(preset2d("d1", cells_per_lambda=64, box_x=40.0, box_y=8.0, ppc_x=1, ppc_y=1,
                         thickness=1 / 64, x_foil=1.0), capacity=max(n, 512))
    rng = np.random.default_rng(n + cols)
    part = {}
    for s in (0, 1):
        ix, iy = rng.integers(0, cols, n), rng.integers(0, rows, n)
        ix[: n // 4], iy[: n // 4] = ix[0], iy[0]  # a dense cell among the others
        part[s] = _particles(rng, n, run.encode(ix, iy), run.rdt, ("ox", "oy"))
    run.set_state(particles=part)
    before = run.get_state()
    run.sort()
    sx, sy = run.get_info()["sort_block_shift"]

    def order_of(p):
        ix, iy = run.decode(p["cell"])
        return (((ix >> sx) << 20 | (iy >> sy)) << 20) | (ix & ((1 << sx) - 1)) << 10 | (iy & ((1 << sy) - 1))

    _check(before, run.get_state(), ("uz", "uy", "ux", "ox", "oy"), order_of)
    run.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,span", [(1, 1), (2048, 3), (2049, 4096), (7000, 4097), (7000, 5900)])
def test_sort_1d(precision, n, span):
    from paper_1008_1685_amd import Run

    print(f"\n[gpu] sort 1d {precision} {n} over {span}", flush=True)
    run = Run(preset("c1", precision=precision, ppc=1, thickness=0.01, box_lambda=60.0), capacity=n)
    rng = np.random.default_rng(n + span)
    run.set_state(particles={s: _particles(rng, n, rng.integers(50, 50 + span, n), run.rdt, ("off",))
                             for s in (0, 1)})
    before = run.get_state()
    run.sort()
    _check(before, run.get_state(), ("uz", "uy", "ux", "off"), lambda p: p["cell"])
    run.close()
