"""The T3 unpack and the R3 fold at the edges of their 16^3 tiles and of the
order in which tiles are dealt out (1, 8, 27 and 64 tiles per block; 729 in
the feedback test):
the whole residual against the oracle.  FP64: 1e-11 of the largest element
(sums of at most 1e5 terms that round at 1e-16 each).  Split BF16: 1e-3; a
product keeps 2^-16 of its factors, and a misplaced element is of the order of
the largest one."""

import numpy as np
import pytest

import cct_inputs as ci
from oracle import rccsdt as R
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("o,v,prec", [
    (2, 1, "fp64"), (3, 15, "fp64"), (3, 16, "bf16x3"), (4, 17, "bf16x3"), (3, 33, "fp64"), (2, 33, "bf16x3"),
    (2, 48, "bf16x3"), (2, 49, "fp64"),
])
def test_residual_matches_the_oracle(o, v, prec):
    print(f"[unpack] o={o} v={v} {prec}", flush=True)
    seed = 500 + o + v
    s = ci.make_system(o, v, o + v, seed, sigma=0.05)
    f = ci.random_fock(o, v, seed)
    t1, t2, _ = ci.random_amplitudes(o, v, seed, 0.02, 0.03, 0.0, triples=False)
    t3p = ci.random_t3_packed(o, v, seed + 1, 0.02)
    with binding.Engine(o, v, s["naux"], precision=prec) as eng:
        eng.set_fock(f)
        eng.set_eri_df(s["B"])
        eng.set_amplitudes(t1, t2, t3p)
        g1, g2, g3, _ = eng.residual()
    r1, r2, r3 = R.residuals(f, R.eri_phys_from_B(s["B"]), t1, t2, R.unpack_t3(t3p, o), o)
    r3p = R.pack_t3(R.postprocess_r3(r3))
    tol = 1e-11 if prec == "fp64" else 1e-3
    for name, a, b in (("R1", g1, r1), ("R2", g2, r2), ("R3", g3, r3p)):
        assert np.abs(a - b).max() <= tol * max(1.0, float(np.abs(b).max())), name

