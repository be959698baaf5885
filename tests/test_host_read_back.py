"""Read-backs on the host side, without a GPU: calls on one context from several threads do not meet, and contexts share
the page-locked memory that they go through."""
import threading

import numpy as np

from hoststub import Context, stubbed


def test_threads_that_read_one_context_get_their_own_data(monkeypatch):
    """Two threads read the droplets of two lattices of a batch: each gets its lattice's table in every call."""
    lbm, lib = stubbed(monkeypatch)
    tables = [[dict(x=float(100 * i + k), y=float(k), R=5.0) for k in range(3 + i)] for i in range(2)]
    ctx = Context(lbm, [(32, 32), (48, 40)], tables)
    want = [[(d["x"], d["y"]) for d in t] for t in tables]
    wrong = []

    def read(i):
        for _ in range(300):
            got = ctx.centres(i)
            if got != want[i]:
                wrong.append((i, got))

    threads = [threading.Thread(target=read, args=(i,)) for i in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    ctx.close()
    assert not wrong, (len(wrong), wrong[0])


def test_new_contexts_lock_no_memory_of_their_own(monkeypatch):
    """Contexts that are read once each, all of them alive: two blocks serve them all (one of each size), and they are
    not freed and locked again with the contexts."""
    lbm, lib = stubbed(monkeypatch)
    before = lib.stub_host_allocs()
    contexts = [Context(lbm, [(64, 64)], [[dict(x=9.0, y=8.0, R=5.0)]]) for _ in range(12)]
    out = {k: np.empty((64, 64)) for k in ("phi", "c", "n", "ux", "uy")}
    for c in contexts:
        assert c.centres() == [(9.0, 8.0)]
        assert lbm.lbm_fields(c.h, 0, np.empty((9, 64, 64)), **out) == lbm.LBM_OK
    for c in contexts:
        c.close()
    again = Context(lbm, [(64, 64)], [[dict(x=9.0, y=8.0, R=5.0)]])
    assert again.centres() == [(9.0, 8.0)]
    again.close()
    assert lib.stub_host_allocs() - before <= 2


def test_the_shared_memory_is_bounded_and_given_back(monkeypatch):
    """As many blocks as calls at once; of those four of a size are kept, and one once no context is left."""
    lbm, lib = stubbed(monkeypatch)
    ctx = Context(lbm, [(32, 32)], [[dict(x=9.0, y=8.0, R=5.0)]])
    threads = [threading.Thread(target=lambda: [ctx.centres() for _ in range(20)]) for _ in range(12)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert lib.stub_host_live() <= 8
    ctx.close()
    assert lib.stub_host_live() <= 2
