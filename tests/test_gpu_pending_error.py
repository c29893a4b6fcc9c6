"""A HIP error that some other library left pending on the thread: state reads
and writes go through, as they check only their own calls, and a diagnostics
call that reports it leaves nothing behind for the next."""
import ctypes as C

import numpy as np
import pytest

from workloads import preset, preset2d

pytestmark = pytest.mark.gpu


def _run(dims, precision):
    """A few steps of electrons with momenta of their own, so that the charge
    and the currents are not zero."""
    from paper_1008_1685_amd import Run
    from paper_1008_1685_amd.run2d import Run2D

    if dims == 1:
        run = Run(preset("c1", precision=precision))
    else:
        run = Run2D(preset2d("d1", precision=precision, box_x=3.0, box_y=1.91, x_foil=1.0, thickness=0.5))
    st = run.get_state()
    rng = np.random.default_rng(dims)
    for k in ("ux", "uy", "uz"):
        st["sp0"][k] = rng.normal(size=st["sp0"]["cell"].size).astype(run.rdt)
    run.set_state(particles={0: st["sp0"], 1: st["sp1"]})
    run.step(3)
    return run


class _Pending:
    """An invalid device number leaves hipErrorInvalidDevice behind."""

    def __init__(self):
        from paper_1008_1685_amd import _native as N

        self.hip = N.load()

    def __enter__(self):
        self.hip.hipSetDevice.argtypes = [C.c_int]
        assert self.hip.hipSetDevice(1 << 20) != 0

    def __exit__(self, *_):
        self.hip.hipGetLastError()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dims", [1, 2])
def test_state_calls_go_through(dims, precision):
    print(f"\n[gpu] pending error, state {dims}D {precision}", flush=True)
    run = _run(dims, precision)
    want = run.get_state()
    with _Pending():
        got = run.get_state()
    for k, v in want.items():
        if isinstance(v, np.ndarray):
            assert np.array_equal(v, got[k]), k
    fields = {k: v for k, v in want.items() if isinstance(v, np.ndarray)}
    with _Pending():
        run.set_state(fields=fields, step=100)
    got = run.get_state()
    assert got["step"] == 100
    for k in fields:
        assert np.array_equal(fields[k], got[k]), k


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dims", [1, 2])
def test_diagnostics_after_a_failed_call(dims, precision):
    from paper_1008_1685_amd import PicError

    print(f"\n[gpu] pending error, diag {dims}D {precision}", flush=True)
    run = _run(dims, precision)
    run.step(3)
    want = run.diag()
    assert want["gauss_int"] == 0
    with _Pending():
        try:
            run.diag()
        except PicError:
            pass
    for _ in range(2):
        assert run.diag() == want
