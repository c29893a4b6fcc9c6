"""Runs whose step counter is set back or forward without new particles: no
current of an earlier step may enter a later one.  What follows must equal,
bit for bit, the steps of a run that never held those currents."""
import numpy as np
import pytest

from workloads import preset, preset2d

pytestmark = pytest.mark.gpu

GRIDS = ("Ex", "Ey", "Ez", "By", "Bz", "Ex_int")


def _moving(run, rng):
    """Random fields and momenta, so that every step carries a current."""
    n = run.info["n_cells"]
    st = run.get_state()
    for s, u in ((0, 3.0), (1, 0.05)):
        for k in ("ux", "uy", "uz"):
            st[f"sp{s}"][k] = (rng.normal(size=st[f"sp{s}"]["cell"].size) * u).astype(run.rdt)
    run.set_state(particles={0: st["sp0"], 1: st["sp1"]},
                  fields={k: rng.uniform(-5, 5, n + (1 if k in ("Ey", "Ez") else 2)) for k in GRIDS[:5]})


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("size,before", [("large", 1), ("large", 2), ("large", 4), ("small", 1), ("small", 2),
                                         ("small", 3), ("small", 4)])
def test_rewound_run_joins_a_batch(size, before, precision):
    from paper_1008_1685_amd import Run
    from paper_1008_1685_amd.serve import Batch

    print(f"\n[gpu] rewind {size} {before} {precision}", flush=True)
    cfg = preset("c1", precision=precision, ppc=16 if size == "small" else 14000, pol="CP", sort_interval=8)
    batch = Batch(precision=precision, max_slots=1, quantum=8, max_particles=10 ** 7, max_cells=10 ** 5)
    out = []
    for in_batch in (False, True):
        run = Run(cfg, stream=batch.stream)
        assert (run.info["tile"] == 5120) == (size == "large")
        _moving(run, np.random.default_rng(before))
        run.step(before)
        run.set_state(step=0)
        if in_batch:
            slot = batch.admit(run, 12)
            batch.step(2)
            batch.release(slot)
        else:
            run.step(12)
        assert run.get_info()["step"] == 12
        out.append((run.get_state(), run.diag()))
        run.close()
    (a, da), (b, db) = out
    for k in GRIDS:
        assert np.array_equal(a[k], b[k]), k
    for s in ("sp0", "sp1"):  # (the order within a cell is open)
        for k in ("cell", "off", "ux", "uy", "uz"):
            assert np.array_equal(np.sort(a[s][k]), np.sort(b[s][k])), (s, k)
    for k in ("E_in", "E_out_left", "E_out_right"):
        assert da[k] == db[k]
    batch.close()


GRIDS_2D = ("Ex", "Ey", "Ez", "Bx", "By", "Bz", "Jx_int", "Jy_int", "Jz_int", "charge_int")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("kernel", ["strips", "tiles"])
@pytest.mark.parametrize("before,step", [(1, 0), (1, 2), (2, 1), (2, 7), (2, 0), (5, 100), (6, 101)])
def test_step_set_alone_2d(before, step, kernel, precision):
    from paper_1008_1685_amd.run2d import Run2D

    print(f"\n[gpu] step 2d {before} -> {step} {kernel} {precision}", flush=True)
    cfg = preset2d("d1", precision=precision, box_x=3.0, box_y=1.91, x_foil=1.0, thickness=0.5, pol="CP",
                   field_kernel=kernel, sort_interval=1000)
    a, b = Run2D(dict(cfg)), Run2D(dict(cfg))
    rng = np.random.default_rng(before)
    st = a.get_state()
    for s, u in ((0, 3.0), (1, 0.05)):
        for k in ("ux", "uy", "uz"):
            st[f"sp{s}"][k] = (rng.normal(size=st[f"sp{s}"]["cell"].size) * u).astype(a.rdt)
    a.set_state(particles={0: st["sp0"], 1: st["sp1"]},
                fields={k: rng.uniform(-5, 5, st[k].shape) for k in GRIDS_2D[:6]})
    a.step(before)
    st = a.get_state()
    a.set_state(step=step)
    # a run that never held a current, given the same particles and fields
    b.set_state(particles={0: st["sp0"], 1: st["sp1"]}, step=step,
                fields={k: st[k] for k in GRIDS_2D if k[0] != "J"})
    for n in (1, 1, 3):
        a.step(n)
        b.step(n)
        sa, sb = a.get_state(), b.get_state()
        for k in GRIDS_2D:
            assert np.array_equal(sa[k], sb[k]), (n, k)
        for s in ("sp0", "sp1"):
            for k in sa[s]:
                assert np.array_equal(sa[s][k], sb[s][k]), (n, s, k)
        assert a.diag()["gauss_int"] == 0
    # the current of a push whose fields are still due stays with the run
    a.push_deposit()
    before = a.get_state(particles=False)
    a.set_state(step=before["step"] + 1)
    after = a.get_state(particles=False)
    for k in GRIDS_2D:
        assert np.array_equal(before[k], after[k]), k
    assert np.any(after["Jx_int"])
