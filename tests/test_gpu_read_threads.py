"""Several threads read one context at once: each gets what the call gives alone, to the bit.

Two uneven lattices of a batch, one whose fields go in several chunks and one whose fields are one chunk; fields of both
in a loop, observables and droplets beside them."""
import threading

import numpy as np
import pytest

from paper_1711_10984_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_threads_read_one_batch():
    from paper_1711_10984_amd import lbm
    params, phi, c, f, drops = [], [], [], [], []
    for nx, ny, nd in ((257, 250, 5), (61, 40, 1)):
        g, p, q = W.random_state(nx, ny, nx)
        params.append(dict(W.ACTIVE, nx=nx, ny=ny))
        phi.append(p), c.append(q), f.append(g)
        drops.append([dict(x=nx * (k + 0.5) / nd, y=0.5 * ny, R=9.0, Rs=3.0, active=1) for k in range(nd)])
    sim = lbm.Sim(params, phi, c, drops, f_pre=f)
    sim.step(7)
    same = lambda a, b: all(np.array_equal(a[k], b[k]) for k in b)
    calls = [(name, i) for name in ("fields", "observables", "droplets") for i in range(2)]
    want = {(name, i): getattr(sim, name)(i) for name, i in calls}
    wrong = []

    def read(name, i):
        for _ in range(30):
            got = getattr(sim, name)(i)
            ok = got == want[name, i] if name == "droplets" else same(got, want[name, i])
            if not ok:
                wrong.append((name, i))

    threads = [threading.Thread(target=read, args=call) for call in calls]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    sim.close()
    assert not wrong, wrong
