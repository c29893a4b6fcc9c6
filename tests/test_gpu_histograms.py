"""The ion spectrum and the friction histogram at the sizes where their
kernels change form: bins that fill the LDS counters with one to eight copies
each, the first size past them (global atomics), and particle counts at the
edges of a wave and of a work-group.  Expected values come from numpy."""
import numpy as np
import pytest

from workloads import preset

pytestmark = pytest.mark.gpu

MC2 = 1836.0 * 0.51099895


def _run(precision, n, u, w):
    from paper_1008_1685_amd import Run

    cfg = preset("c1", precision=precision, ppc=1, thickness=0.01, x_foil=1.0)
    run = Run(cfg, capacity=n)
    rng = np.random.default_rng(3)
    cell = np.sort(rng.integers(100, 400, n)).astype(np.int32)
    z = np.zeros(n)
    part = dict(cell=cell, off=rng.integers(0, 1 << 24, n) / float(1 << 24), ux=u, uy=z, uz=z, w=w)
    run.set_state(particles={0: part, 1: part})
    return run


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("bins", [1, 512, 513, 4096, 4097, 65536])
def test_spectrum_counts(precision, bins):
    """Energies at bin centres: every bin's weight is exact (the counts are integers)."""
    import torch

    print(f"\n[gpu] spectrum {precision} {bins}", flush=True)
    top = 800.0
    rng = np.random.default_rng(bins)
    for n in (1, 63, 1025, 60001):
        b = rng.integers(0, bins, n)
        b[: n // 2] = b[0]  # bunched: half the particles in one bin
        E = (b + 0.5) * top / bins
        E[n // 3: n // 3 + 5] = 1.5 * top  # past the range: not counted
        u = np.sqrt((1.0 + E / MC2) ** 2 - 1.0)
        run = _run(precision, n, u, np.ones(n))
        w_ref = run.info["w_ref"]
        run.close()
        units = rng.choice([256, 300], n)
        run = _run(precision, n, u, units * w_ref / 256.0)
        ok = E < top
        expect = np.bincount(b[ok], weights=units[ok], minlength=bins) * (w_ref / 256.0) / (top / bins)
        for got in (run.spectrum(bins, top), run.spectrum_static(bins, top)):
            # one multiplication and one division by the host, in FP64
            assert np.allclose(got, expect, rtol=4e-16, atol=0.0)
        run.close()
    torch.cuda.synchronize()


@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_friction_forms_agree(precision):
    """Twice the bins past the LDS form, added pairwise, against the LDS form
    (bin edges are the same numbers: the bin index only doubles)."""
    print(f"\n[gpu] friction {precision}", flush=True)
    n = 30011
    rng = np.random.default_rng(5)
    u = np.exp(rng.uniform(np.log(1e-3), np.log(500.0), n))
    run = _run(precision, n, u, np.full(n, 0.5))
    nx = run.info["n_cells"]
    run.set_state(fields=dict(Ey=rng.uniform(-300, 300, nx + 1), Ez=rng.uniform(-300, 300, nx + 1),
                              Ex=rng.uniform(-50, 50, nx + 2), By=rng.uniform(-300, 300, nx + 2),
                              Bz=rng.uniform(-300, 300, nx + 2)))
    lo, hi = -3.0, 3.0
    small, s0 = run.friction(4094, lo, hi)
    large, s1 = run.friction(8188, lo, hi)
    one, s2 = run.friction(1, lo, hi)
    total = 0.5 * n
    for h, st in ((small, s0), (large, s1), (one, s2)):
        # sums of n equal weights, exact in FP64 (multiples of 1/2 below 2^52)
        assert h.sum() + st["below"] + st["above"] == total
    assert np.array_equal(large.reshape(-1, 2).sum(1), small)
    assert (s0["below"], s0["above"], s0["max"]) == (s1["below"], s1["above"], s1["max"])
    # FP64 sums of n terms in different orders: n eps of the sum of the (positive) terms
    assert s0["mean"] == pytest.approx(s1["mean"], rel=n * 2.3e-16)
    assert s2["mean"] == pytest.approx(s1["mean"], rel=n * 2.3e-16)
    run.close()
