"""Tracked electrons whose momentum squared overflows the format: 1 / gamma
is zero, so without radiation reaction the electron stays where it is and
gains the field's kick only, and its neighbours are tracked as they are
alone."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scheme", ["leapfrog", "rk4"])
@pytest.mark.parametrize("u", [1e160, -3e200, 1e300])
def test_overflowing_momentum(u, scheme):
    from paper_1008_1685_amd.track import track

    print(f"\n[gpu] track {scheme} {u}", flush=True)
    n = 5
    x, v = np.linspace(0, 1, n), np.tile([0.5, -2.0, 3.0], (n, 1))
    kw = dict(a_y=5.0, a_z=2.0, psi=0.3, scheme=scheme, rr="off", precision="fp64", dt=0.01, steps=10)
    want = track(x, v, **kw)
    for c in range(3):
        w = v.copy()
        w[2, c] = u
        got = track(x, w, **kw)
        for g, r in zip(got, want):
            assert np.array_equal(np.delete(g, 2, 0), np.delete(r, 2, 0)), c
        assert got[0][2] == x[2] and got[1][2, c] == u
        assert np.all(np.isfinite(got[1][2]))


def test_overflow_by_the_radiation_force():
    # an explicit RR step far past its stability squares a momentum: in the
    # step that takes its square past the largest number the electron stays
    # in place, and keeps its finite momentum if that was the last step
    from paper_1008_1685_amd.track import track

    print("\n[gpu] track, RR overflow", flush=True)
    n = 200
    x, u = np.linspace(0, 1, n), np.zeros((n, 3))
    u[:, 0] = -np.logspace(60, 110, n)
    kw = dict(a_y=350.0, scheme="leapfrog", rr="reduced", precision="fp64", dt=0.01)
    seen = 0
    for steps in range(1, 4):
        x0, _ = track(x, u, steps=steps - 1, **kw)
        x1, u1 = track(x, u, steps=steps, **kw)
        hit = np.all(np.isfinite(u1), 1) & (np.max(np.abs(u1), 1) > 1.4e154)
        assert np.array_equal(x1[hit], x0[hit]), steps
        seen += int(hit.sum())
    assert seen > 0
