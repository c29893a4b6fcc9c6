"""Steps whose field pass shares a launch with the next push (runs in small
tiles), against the same steps taken stage by stage: the same bits, in the
cases where the tiles' own field update changes form: tiles at either end of
the box (boundary guards), tiles wider than their LDS (each particle's fields
computed alone), one-particle and remainder tiles, removed particles."""
import numpy as np
import pytest

from workloads import preset

pytestmark = pytest.mark.gpu


def _state(rng, n, lo, hi, nx, rdt, order):
    u = lambda s: (rng.normal(size=n) * s).astype(rdt)  # noqa: E731
    cell = rng.integers(lo, hi, n).astype(np.int32)
    if order:
        cell.sort()
    off = (rng.integers(0, 1 << 24, n) / float(1 << 24)).astype(rdt)
    return lambda s, w: dict(cell=cell, off=off, ux=u(s), uy=u(s), uz=u(s), w=np.full(n, w, rdt))


def _fields(rng, nx, rdt):
    f = lambda m: rng.uniform(-200, 200, m).astype(rdt)  # noqa: E731
    return dict(Ey=f(nx + 1), Ez=f(nx + 1), By=f(nx + 2), Bz=f(nx + 2),
                Ex_int=rng.integers(-(1 << 40), 1 << 40, nx + 2))


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("tile", [256, 512, 1024])
@pytest.mark.parametrize("n,lo,hi,order", [
    (1, 5, 6, True), (1023, 0, 3, True), (1025, 1997, 2000, True), (5000, 0, 2000, True),
    (3000, 0, 2000, False),     # unsorted: every tile spans the box
    (2100, 700, 1040, False),   # about the widest tile that fits in FP64
    (2100, 700, 1210, False),   # and in FP32
    (9000, 0, 1, True)])
def test_fused_steps_match_stages(precision, tile, n, lo, hi, order):
    from paper_1008_1685_amd import Run

    print(f"\n[gpu] fused {precision} tile {tile} {n} [{lo}, {hi}) {order}", flush=True)
    # (the quiet start only chooses the tile: the state replaces it)
    cfg = preset("c1", precision=precision, ppc={256: 1, 512: 100000, 1024: 200000}[tile], thickness=0.01,
                 sort_interval=4, pol="CP")
    runs, out = [], []
    for _ in range(2):
        rng = np.random.default_rng(n + lo)
        r = Run(cfg, capacity=n)
        assert r.info["tile"] == tile
        nx = r.info["n_cells"]
        part = _state(rng, n, lo, hi, nx, r.rdt, order)
        r.set_state(particles={0: part(5.0, r.info["w_ref"]), 1: part(0.1, 0.7 * r.info["w_ref"])},
                    fields=_fields(rng, nx, r.rdt), step=161)
        runs.append(r)
    for chunk in (3, 1, 2, 5, 13):  # odd and even numbers of steps, with and without a sort between
        runs[0].step(chunk)
        for _ in range(chunk):
            r = runs[1]
            if r.get_info()["step"] % 4 == 0:
                r.sort()
            r.push_deposit()
            r.field_advance()
        out = [r.get_state() for r in runs]
        assert out[0]["step"] == out[1]["step"]
        for k in ("Ex", "Ey", "Ez", "By", "Bz", "Ex_int", "Jx_int", "Jy_int", "Jz_int"):
            assert np.array_equal(out[0][k], out[1][k]), (chunk, k)
        for s in ("sp0", "sp1"):
            a, b = out[0][s], out[1][s]
            keys = ("uz", "uy", "ux", "off", "cell")  # (the order within a cell is open after a sort)
            oa, ob = (np.lexsort([p[k] for k in keys]) for p in (a, b))
            for k in a:
                assert np.array_equal(a[k][oa], b[k][ob]), (chunk, s, k)
        for k in ("E_in", "E_out_left", "E_out_right"):
            assert out[0]["budget"][k] == out[1]["budget"][k]
    for r in runs:
        r.close()
