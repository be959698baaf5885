"""Read-backs on the host side, without a GPU: calls on one context from several threads do not meet."""
import threading

import pytest

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
