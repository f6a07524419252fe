"""E_(Q) in the occupied-tuple order at the sizes where its products and block
orbits change path: fewer virtuals than one 4-block, an exact and a ragged last
block, rows of 16 and 17, odd occupied counts with even virtuals (element
loads), the three widths of the skinny tiles, more than 16 occupied, and task
batches that do not hold every task.  Against the full-tensor oracle (small) or
the virtual-tuple order on the same amplitudes; tolerance as in the other (Q)
tests (1e-11 of the sum of the tasks' magnitudes: sums of at most 1e7 terms
that round at 1e-16 each)."""

import sys

import numpy as np
import pytest

import cct_inputs as ci
from oracle import rccsdt as R
from oracle import rccsdt_q as Q
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _engine(o, v, seed):
    s = ci.make_system(o, v, 2 * (o + v), seed, sigma=0.1)
    t2 = ci.random_amplitudes(o, v, seed, 0.0, 0.05, 0.0, triples=False)[1]
    t3p = ci.random_t3_packed(o, v, seed + 1, 0.03)
    eng = binding.Engine(o, v, s["naux"])
    eng.set_fock(s["f"])
    eng.set_eri_df(s["B"])
    eng.set_amplitudes(np.zeros((o, v)), t2, t3p)
    return s, t2, t3p, eng


@pytest.mark.parametrize("o,v", [(2, 1), (3, 2), (2, 3), (4, 4), (3, 8), (5, 6), (2, 12), (4, 7)])
def test_tasks_match_the_oracle(o, v):
    say(f"[q shapes] o={o} v={v}")
    s, t2, t3p, eng = _engine(o, v, 60 + o + v)
    with eng:
        e, tasks = eng.energy_q(tasks=True)
    V = R.eri_phys_from_B(s["B"])
    t3 = R.unpack_t3(t3p, o)
    want = [Q.task_energy(s["f"], V, t2, t3, o, (i, j, k, l)) if len({i, j, k}) > 1 and len({j, k, l}) > 1 else 0.0
            for i in range(o) for j in range(i, o) for k in range(j, o) for l in range(k, o)]
    scale = max(float(np.abs(want).sum()), 1e-300)
    assert np.abs(tasks - np.array(want)).max() <= 1e-11 * scale
    assert abs(e - Q.energy_q(s["f"], V, t2, t3, o)) <= 1e-11 * scale


@pytest.mark.parametrize("o,v,block", [(3, 32, 8), (2, 33, 8), (2, 48, 12), (2, 49, 10), (3, 40, 10), (17, 5, 5), (9, 10, 5)])
def test_equals_virtual_tuple_order(o, v, block):
    say(f"[q shapes] vs virtual tuples o={o} v={v}")
    _, _, _, eng = _engine(o, v, 70 + o + v)
    with eng:
        e, tasks = eng.energy_q(tasks=True)
        ref = eng.energy_q_abc(block)["e_q"]
    assert abs(e - ref) <= 1e-11 * max(float(np.abs(tasks).sum()), abs(ref))
    assert abs(e - tasks.sum()) <= 1e-12 * float(np.abs(tasks).sum())
