"""State transfers between host FP64 arrays and the device: one piece on the
calling thread, many pieces on several (with a ragged last one), both buffers
of the ping-pong pair, invalid values anywhere in a large array, and transfers
of several handles at once.  What is read back is what was set, rounded to the
stencil type, with dry cells at rest."""
import ctypes
import sys
import threading

import numpy as np
import pytest

from paper_1705_00614_amd import scenarios as S

pytestmark = pytest.mark.gpu

swe = pytest.importorskip("paper_1705_00614_amd.swe")


@pytest.fixture(autouse=True)
def _announce(request):
    print("\n[gpu] %s" % request.node.nodeid, flush=True)
    sys.stdout.flush()
    yield


def _layer(nx, ny, seed):
    rng = np.random.default_rng(seed)
    H = np.maximum(rng.normal(0.5, 1.0, (ny, nx)), 0.0)
    H[rng.uniform(size=H.shape) < 0.05] = 5e-5          # films: inert, kept
    return H, rng.normal(size=H.shape), rng.normal(size=H.shape)


def _stored(layer, prec):
    t = np.float32 if prec == 32 else np.float64
    H, Qx, Qy = layer
    wet = H > 1e-4
    return tuple(a.astype(t).astype(np.float64) for a in (H, np.where(wet, Qx, 0.0), np.where(wet, Qy, 0.0)))


# 1 cell; odd sides in one piece; just below and above the threaded size
# (2 MB in all); several pieces a thread with a ragged last one
@pytest.mark.parametrize("nx,ny,prec", [(1, 1, 32), (33, 7, 64), (417, 419, 32), (419, 419, 32), (1100, 701, 64),
                                        (2051, 2049, 32)])
def test_state_round_trip(nx, ny, prec):
    sc = S.dam_break(nx, ny, x_dam=nx / 2.0, precision=prec)
    sc["H0"], sc["Qx0"], sc["Qy0"] = _layer(nx, ny, 1)
    g = swe.Solver(sc)
    for a, b in zip(g.state(), _stored((sc["H0"], sc["Qx0"], sc["Qy0"]), prec)):
        assert np.array_equal(a, b)
    g.run(1)                                            # the other buffer is current now
    after = g.state()
    layer = _layer(nx, ny, 2)
    g.set_state(*layer)
    for a, b in zip(g.state(), _stored(layer, prec)):
        assert np.array_equal(a, b)
    g.set_state(sc["H0"], sc["Qx0"], sc["Qy0"])
    g.set_time(0.0)
    g.run(1)
    assert all(np.array_equal(a, b) for a, b in zip(g.state(), after))
    only = np.empty((ny, nx))                           # one field wanted
    assert swe.load().swe_get_state(g._h, None, only.ctypes.data_as(ctypes.POINTER(ctypes.c_double)), None) == 0
    assert np.array_equal(only, after[1])


@pytest.mark.parametrize("nx,ny", [(40, 30), (1500, 900)])
def test_invalid_state_is_refused_and_changes_nothing(nx, ny):
    sc = S.dam_break(nx, ny, x_dam=nx / 2.0, precision=32)
    g = swe.Solver(sc)
    before = g.state()
    for field, bad in ((0, -1e-3), (0, np.nan), (1, np.inf), (2, np.nan)):
        layer = [np.array(a) for a in _layer(nx, ny, 3)]
        layer[field][-1, -1] = bad
        with pytest.raises(swe.SweError):
            g.set_state(*layer)
    assert all(np.array_equal(a, b) for a, b in zip(g.state(), before))


def test_transfers_of_several_threads():
    """Handles used by different host threads share the pinned pool."""
    sizes = [(900, 800, 32), (64, 64, 64), (700, 650, 64), (300, 200, 32)]
    failed = []

    def work(k):
        nx, ny, prec = sizes[k]
        try:
            g = swe.Solver(S.dam_break(nx, ny, x_dam=nx / 2.0, precision=prec), stream=None)
            for it in range(4):
                layer = _layer(nx, ny, 10 * k + it)
                g.set_state(*layer)
                if not all(np.array_equal(a, b) for a, b in zip(g.state(), _stored(layer, prec))):
                    failed.append((k, it))
            g.close()
        except Exception as e:   # a thread's exception would be lost
            failed.append((k, repr(e)))

    th = [threading.Thread(target=work, args=(k,)) for k in range(len(sizes))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not failed, failed


def test_per_thread_stream_orders_transfers_after_queued_steps():
    """On hipStreamPerThread a state read after queued steps is theirs, though
    several host threads move it (the handle names another stream in each)."""
    per_thread = 2   # hipStreamPerThread
    sc = S.dam_break(900, 700, x_dam=450.0, precision=32)
    g, ref = swe.Solver(sc, stream=per_thread), swe.Solver(sc, stream=None)
    for steps in (1, 7):
        g.enqueue(steps)
        ref.run(steps)
        assert all(np.array_equal(a, b) for a, b in zip(g.state(), ref.state()))
    g.close()
