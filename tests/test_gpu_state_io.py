"""Field arrays in and out of a run one component at a time: each lands in
its own place and nowhere else, reads leave the run as it was (the next step
equals, bit for bit, that of a twin that was never read), at either step
parity, and two threads may read one run."""
from concurrent.futures import ThreadPoolExecutor

import numpy as np
import pytest

from workloads import preset, preset2d

pytestmark = pytest.mark.gpu


def _pair(dims, precision, rng):
    from paper_1008_1685_amd import Run
    from paper_1008_1685_amd.run2d import Run2D

    if dims == 1:
        cfg = preset("c1", precision=precision)
        runs = [Run(dict(cfg)) for _ in range(2)]
        n = runs[0].info["n_cells"]
        shape = dict(Ex=n + 2, Ey=n + 1, Ez=n + 1, By=n + 2, Bz=n + 2)
    else:
        cfg = preset2d("d1", precision=precision, box_x=3.0, box_y=1.91, x_foil=1.0, thickness=0.5)
        runs = [Run2D(dict(cfg)) for _ in range(2)]
        nx, ny = runs[0].info["nx"], runs[0].info["ny"]
        shape = {k: (nx + (2 if k in ("Ex", "By", "Bz") else 1), ny) for k in ("Ex", "Ey", "Ez", "Bx", "By", "Bz")}
    return runs, {k: rng.uniform(-1, 1, v).astype(runs[0].rdt) for k, v in shape.items()}


@pytest.mark.parametrize("before", [0, 1])
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
@pytest.mark.parametrize("dims", [1, 2])
def test_components_land_alone_and_reads_leave_no_trace(dims, precision, before):
    (a, b), f = _pair(dims, precision, np.random.default_rng(dims))
    for r in (a, b):
        r.step(before)
    want = {k: a.get_state(particles=False)[k] for k in f}
    for k in f:
        a.set_state(fields={k: f[k]})
        want[k] = f[k]
        got = a.get_state(particles=False)
        for m in f:
            assert np.array_equal(got[m], want[m]), (k, m)
    b.set_state(fields=f)
    with ThreadPoolExecutor(2) as pool:
        for st in pool.map(lambda _: a.get_state(), range(8)):
            assert all(np.array_equal(st[m], f[m]) for m in f)
    for n in (1, 2):
        for r in (a, b):
            r.step(n)
        sa, sb = (r.get_state(particles=False) for r in (a, b))
        for k in sa:
            if isinstance(sa[k], np.ndarray):
                assert np.array_equal(sa[k], sb[k]), (n, k)
