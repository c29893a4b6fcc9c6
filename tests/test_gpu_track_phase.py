"""The wave phases of tracked electrons: sine and cosine over the reduced
range, at the seams of the reduction (multiples of pi / 4), and past the phases
the short reduction takes."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("span", [1.0, 30.0, 1e3, 0.99e5, 1e7, 1e12])
def test_one_small_kick_reads_the_wave(span):
    from paper_1008_1685_amd.track import track

    print(f"\n[gpu] track phases up to {span}", flush=True)
    rng = np.random.default_rng(int(span))
    k = np.floor(rng.uniform(-span, span, 4000) / (np.pi / 4))
    seams = k * (np.pi / 4) + rng.choice([0.0, 1e-16, -1e-12, 1e-9], k.size) * np.maximum(1.0, abs(k))
    ph = np.concatenate([rng.uniform(-span, span, 20000), seams, [0.0, -0.0, 1e-300, 1e-17]])
    # an electron at rest, one step without RR at an amplitude so small that
    # the magnetic rotation (1e-9 squared) does not enter: u = -dt E, E = (-a cos, a sin)
    a, dt = 1e-7, 0.01
    _, u = track(-ph, np.zeros((ph.size, 3)), a, a, dt=dt, steps=1, rr="off")
    # up to 1 ulp of the sine or cosine and half a unit each of four products: 3 x 2.2e-16
    assert np.max(np.abs(u[:, 1] / (dt * a) - np.cos(ph))) < 6.7e-16
    assert np.max(np.abs(-u[:, 2] / (dt * a) - np.sin(ph))) < 6.7e-16
