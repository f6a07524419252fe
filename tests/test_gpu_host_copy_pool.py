"""The pinned staging buffers are allocated when enough is read back to be worth
it (16 MB in all), not for one small tensor: until then the driver's mappings of
the process do not grow by the 32 MB of the pool.  (They need not grow later
either: the runtime may hand out what it pinned before.)  Bytes are equal on
both paths."""

import numpy as np
import pytest

import cct_inputs as ci
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu


def _mapped():
    n = 0
    with open("/proc/self/maps") as f:
        for line in f:
            if "/dev/dri/" in line:
                a, b = line.split()[0].split("-")
                n += int(b, 16) - int(a, 16)
    return n


def test_small_reads_pin_nothing():
    o, v = 4, 27  # T3 of 3.1 MB
    print(f"[host copy pool] o={o} v={v}", flush=True)
    s = ci.make_system(o, v, 2 * (o + v), 3, sigma=0.02)
    with binding.Engine(o, v, s["naux"]) as eng:
        eng.set_fock(s["f"])
        eng.set_eri_df(s["B"])
        eng.init_mp2()
        eng.update()
        n = eng.ntri * v ** 3
        want = np.concatenate([eng.copy_r3(i, min(100_000, n - i)) for i in range(0, n, 100_000)])
        before = _mapped()
        for k in range(1, 9):
            assert np.array_equal(eng.copy_r3(0, n), want)
            if 8 * n * k < 16 << 20:
                assert _mapped() - before < 32 << 20, k
