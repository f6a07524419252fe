"""Tensors read back through the pinned staging buffers: sizes below, at and
above one staged chunk and a ragged last chunk, against the same elements read
in pieces small enough for the plain copy; concurrent reads from two contexts
share the buffers.  Bytes have to be equal."""

import sys
import threading

import numpy as np
import pytest

import cct_inputs as ci
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu

PIECE = 100_000  # elements: 0.8 MB, below the staged path


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _pieces(eng):
    n = eng.ntri * eng.v ** 3
    return np.concatenate([eng.copy_r3(i, min(PIECE, n - i)) for i in range(0, n, PIECE)])


def _engine(o, v, seed):
    s = ci.make_system(o, v, 2 * (o + v), seed, sigma=0.02)
    eng = binding.Engine(o, v, s["naux"])
    eng.set_fock(s["f"])
    eng.set_eri_df(s["B"])
    eng.init_mp2()
    eng.update()
    return eng


# packed R3 of 1.0, 2.0, 2.1, 6.2 and 41 MB
@pytest.mark.parametrize("o,v", [(3, 23), (4, 23), (2, 41), (5, 28), (7, 39)])
def test_staged_copies_equal_small_copies(o, v):
    say(f"[host copy] o={o} v={v}")
    with _engine(o, v, o + v) as eng:
        _, r2, r3, _ = eng.residual()
        assert np.array_equal(r3.ravel(), _pieces(eng))
        n = eng.ntri * v ** 3
        whole = eng.copy_r3(1, n - 1)  # odd offset
        assert np.array_equal(whole, r3.ravel()[1:])
        t = eng.get_amplitudes()
        eng.set_amplitudes(*t)
        for a, b in zip(t, eng.get_amplitudes()):
            assert np.array_equal(a, b)


def test_concurrent_reads_share_the_buffers():
    say("[host copy] two contexts, a thread each")
    with _engine(6, 36, 1) as a, _engine(6, 37, 2) as b:
        want = {}
        for eng in (a, b):
            _, _, r3, _ = eng.residual()
            want[eng] = r3.ravel()
        bad = []

        def read(eng):
            for _ in range(5):
                if not np.array_equal(eng.copy_r3(0, len(want[eng])), want[eng]):
                    bad.append(eng)

        # a context serves one thread at a time: one thread per context
        th = [threading.Thread(target=read, args=(e,)) for e in (a, b)]
        for t in th:
            t.start()
        for t in th:
            t.join()
        assert not bad
