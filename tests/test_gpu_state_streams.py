"""State reads and writes beside work on streams: what a call clears is clear
before the caller's next launch, on a stream that does not wait for the null
stream too, and a read changes nothing that a step in flight could touch."""
import numpy as np
import pytest

from workloads import preset, preset2d

pytestmark = pytest.mark.gpu

GRIDS_2D = ("Ex", "Ey", "Ez", "Bx", "By", "Bz", "Jx_int", "Jy_int", "Jz_int", "charge_int")


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("what", ["particles", "particles and fields", "particles and step"])
def test_push_follows_the_cleared_currents_2d(what, precision):
    import torch

    from paper_1008_1685_amd.run2d import Run2D

    print(f"\n[gpu] cleared currents {what} {precision}", flush=True)
    # a grid whose clearing takes a while against a push of few particles
    cfg = preset2d("d1", precision=precision, box_x=60.0, box_y=15.9, x_foil=1.0, thickness=0.1)
    with torch.cuda.stream(torch.cuda.Stream()):
        a, b = Run2D(dict(cfg)), Run2D(dict(cfg))
        rng = np.random.default_rng(3)
        st = a.get_state()
        for s, u in ((0, 3.0), (1, 0.05)):
            for k in ("ux", "uy", "uz"):
                st[f"sp{s}"][k] = (rng.normal(size=st[f"sp{s}"]["cell"].size) * u).astype(a.rdt)
        kw = dict(particles={0: st["sp0"], 1: st["sp1"]})
        if "fields" in what:
            kw["fields"] = {k: rng.uniform(-5, 5, st[k].shape) for k in GRIDS_2D[:6]}
        if "step" in what:
            kw["step"] = 1
        # (the current of a push in progress is what has to go)
        a.set_state(particles=kw["particles"])
        a.push_deposit()
        for r in (a, b):
            r.set_state(**kw)
            r.push_deposit()
        sa, sb = a.get_state(), b.get_state()
    for k in GRIDS_2D:
        if "fields" in what or k[0] in "Jc":
            assert np.array_equal(sa[k], sb[k]), k
    assert np.any(sa["Jx_int"])


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("before", [0, 1])
@pytest.mark.parametrize("dims", [1, 2])
def test_reads_write_scratch_only(dims, before, precision):
    import torch

    from paper_1008_1685_amd import Run
    from paper_1008_1685_amd.run2d import Run2D

    print(f"\n[gpu] reads {dims}D {before} {precision}", flush=True)
    if dims == 1:
        run = Run(preset("c1", precision=precision))
        scratch = (run.info["n_cells"] + 2) * np.dtype(run.rdt).itemsize
    else:
        run = Run2D(preset2d("d1", precision=precision, box_x=3.0, box_y=1.91, x_foil=1.0, thickness=0.5))
        scratch = (run.info["nx"] + 2) * run.info["ny"] * np.dtype(run.rdt).itemsize
    rng = np.random.default_rng(before)
    run.step(before)
    st = run.get_state(particles=False)
    run.set_state(fields={k: rng.uniform(-5, 5, v.shape) for k, v in st.items()
                          if isinstance(v, np.ndarray) and k[0] in "EB" and not k.endswith("_int")})
    run.step(3)  # (both parities of the fields hold values of their own)
    torch.cuda.synchronize()
    old = run.ws.clone()
    run.get_state()
    run.get_state(particles=False)
    at = torch.nonzero(run.ws[: run.ws_bytes] != old[: run.ws_bytes]).flatten()
    # nothing but one component's worth of scratch, outside every array of the run
    assert at.numel() == 0 or int(at[-1] - at[0]) < scratch, (int(at[0]), int(at[-1]), scratch)
    run.step(1)
    torch.cuda.synchronize()
    new = run.ws.clone()
    if at.numel():
        lo, hi = int(at[0]), int(at[-1]) + 1
        run.step(4)
        torch.cuda.synchronize()
        assert torch.equal(run.ws[lo:hi], new[lo:hi])
