"""The T3 feedback into R1 and R2 (and, through W^{ab}_{dj} and W^{al}_{ij}, into
the drivers D1 and D2) at the sizes where its two products change shape: o + v
at, below and above whole 16-column fragments and past one 128-column tile,
padded and unpadded slot runs, fewer rows than a tile, one slot per batch.
Against the oracle; FP64 tolerance 1e-11 of the largest element (sums of at most
1e5 terms that round at 1e-16 each)."""

import sys

import numpy as np
import pytest

import cct_inputs as ci
from oracle import rccsdt as R
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("o,v,ws", [(1, 1, 0), (3, 13, 0), (3, 14, 0), (2, 16, 0), (4, 28, 0), (3, 30, 0), (2, 46, 0),
                                    (2, 47, 0), (5, 20, 1e-9), (2, 63, 0), (1, 130, 0)])
def test_feedback_matches_the_oracle(o, v, ws):
    say(f"[feedback] o={o} v={v} workspace={'least' if ws else 'default'}")
    seed = 300 + o + v
    s = ci.make_system(o, v, o + v, seed, sigma=0.05)
    f = ci.random_fock(o, v, seed)
    t1, t2, _ = ci.random_amplitudes(o, v, seed, 0.02, 0.03, 0.0, triples=False)
    t3p = ci.random_t3_packed(o, v, seed + 1, 0.02)
    terms = ("D1", "D2")
    with binding.Engine(o, v, s["naux"], opts={"workspace_gb": ws} if ws else None) as eng:
        eng.set_fock(f)
        eng.set_eri_df(s["B"])
        eng.set_amplitudes(t1, t2, t3p)
        g1, g2, g3, _ = eng.residual(terms)
    r1, r2, r3 = R.residuals(f, R.eri_phys_from_B(s["B"]), t1, t2, R.unpack_t3(t3p, o), o, terms=terms)
    r3p = R.pack_t3(R.postprocess_r3(r3))
    for name, a, b in (("R1", g1, r1), ("R2", g2, r2), ("R3", g3, r3p)):
        scale = max(1.0, float(np.abs(b).max()))
        assert np.abs(a - b).max() <= 1e-11 * scale, name
