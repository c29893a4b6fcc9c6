"""The diagnostics' integer charge at the sizes where its kernels change form:
tiles whose charge fits LDS in sixteen to one copies and tiles that do not,
particle counts at the edges of a tile, periods of a few rows.  The charge is
an exact integer and is computed again with numpy; kinetic energies are FP64
sums of n terms."""
import numpy as np
import pytest

from workloads import preset, preset2d

pytestmark = pytest.mark.gpu


def _u(rng, n):
    return np.exp(rng.uniform(np.log(1e-2), np.log(300.0), n)).astype(np.float32).astype(np.float64)


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("n,span", [(1, 1), (63, 2), (2047, 3), (2048, 239), (2049, 240), (5000, 1300),
                                    (6001, 4096), (6001, 4500)])
def test_charge_1d(precision, n, span):
    from paper_1008_1685_amd import Run

    print(f"\n[gpu] charge 1d {precision} {n} {span}", flush=True)
    run = Run(preset("c1", precision=precision, ppc=1, thickness=0.01, box_lambda=60.0), capacity=n)
    nx, w_ref = run.info["n_cells"], run.info["w_ref"]
    rng = np.random.default_rng(n)
    parts, rho, kin = {}, np.zeros(nx + 1, np.int64), []
    for s, Z, M in ((0, -1, 1.0), (1, 1, 1836.0)):
        cell = rng.integers(700, 700 + span, n).astype(np.int32)
        off = rng.integers(0, 1 << 24, n) / float(1 << 24)
        qw = rng.choice([256, 200], n)
        # (not sorted: every tile spans the whole range)
        u = _u(rng, n)
        z = np.zeros(n)
        parts[s] = dict(cell=cell, off=off, ux=u, uy=z, uz=z, w=qw * w_ref / 256.0)
        q = (off * (1 << 24)).astype(np.int64)
        np.add.at(rho, cell, Z * qw * ((1 << 24) - q))
        np.add.at(rho, cell + 1, Z * qw * q)
        w = (qw * w_ref / 256.0).astype(run.rdt).astype(np.float64)
        kin.append((w * M * (np.sqrt(1.0 + u * u) - 1.0)).sum())
    run.set_state(particles=parts, fields=dict(Ex_int=np.zeros(nx + 2, np.int64)))
    for _ in range(2):  # (the second read finds the charge cleared)
        d = run.diag()
        assert d["gauss_int"] == np.abs(rho[1:nx]).max()
        assert d["n_alive"] == (n, n)
        # sqrt(1 + u^2) - 1 loses up to eps / u^2 of a term of u = 1e-2: 1e-11 of the sum at most
        assert d["K_e"] == pytest.approx(kin[0], rel=1e-11)
        assert d["K_i"] == pytest.approx(kin[1], rel=1e-11)
    run.close()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("rows,cols,n", [(2, 1, 1), (3, 4, 2047), (8, 40, 2049), (64, 30, 5000),
                                         (64, 62, 5000), (64, 200, 6001), (37, 3, 4097)])
def test_charge_2d(precision, rows, cols, n):
    from paper_1008_1685_amd.run2d import Run2D

    print(f"\n[gpu] charge 2d {precision} {rows} x {cols}, {n}", flush=True)
    run = Run2D(preset2d("d1", precision=precision, box_y=rows / 32, ppc_x=1, ppc_y=1, thickness=1 / 32),
                capacity=max(n, rows))
    ny, w_ref = run.info["ny"], run.info["w_ref"]
    assert ny == rows
    rng = np.random.default_rng(n + rows)
    rho, parts = np.zeros((run.info["nx"] + 1, ny), np.int64), {}
    for s, Z in ((0, -1), (1, 1)):
        ix, iy = rng.integers(20, 20 + cols, n), rng.integers(0, ny, n)
        o = rng.integers(0, 1 << 24, (2, n)) / float(1 << 24)
        qw = rng.choice([256, 200], n)
        z = np.zeros(n)
        parts[s] = dict(cell=run.encode(ix, iy), ox=o[0], oy=o[1], ux=_u(rng, n), uy=z, uz=z,
                        w=qw * w_ref / 256.0)
        qx, qy = (np.floor(v * 4096).astype(np.int64) for v in o)
        for a, sx in ((0, 4096 - qx), (1, qx)):
            for b, sy in ((0, 4096 - qy), (1, qy)):
                np.add.at(rho, (ix + a, (iy + b) % ny), 2 * Z * qw * sx * sy)
    run.set_state(particles=parts)  # (the running charge restarts from the particles')
    st = run.get_state(particles=False)
    assert np.array_equal(st["charge_int"], rho)
    for _ in range(2):
        d = run.diag()
        assert d["gauss_int"] == 0
        assert d["n_alive"] == (n, n)
    st["charge_int"][25, 0] += 12345  # a planted difference shows
    run.set_state(fields=dict(charge_int=st["charge_int"]))
    assert run.diag()["gauss_int"] == 12345
    run.close()
