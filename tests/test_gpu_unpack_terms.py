"""The unpack and the fold at the edges of their 16^3 tiles, one R3 term at a
time against the oracle, each judged by its own largest element: the terms they
feed are a hundredth of the whole residual, where the Fock term would hide a
misplaced element.  FP64 terms 1e-11 (sums of at most 1e5 terms that round at
1e-16 each).  Rings: FP32 2e-6 (operands round at 6e-8, sums of 128 products in
FP32), split BF16 5e-5 (a split factor keeps 2^-16, a dropped lo lo product is no larger)."""

import numpy as np
import pytest

import cct_inputs as ci
from oracle import rccsdt as R
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu

RINGS = {"fp64": 1e-11, "fp32": 2e-6, "bf16x3": 5e-5}


@pytest.mark.parametrize("o,v,prec", [
    (3, 15, "fp64"), (3, 16, "bf16x3"), (4, 17, "bf16x3"), (3, 17, "fp32"), (2, 33, "bf16x3"), (3, 33, "fp64"),
    (2, 48, "bf16x3"), (2, 49, "fp64"), (2, 49, "fp32"),
])
def test_each_term_matches_the_oracle(o, v, prec):
    print(f"[unpack terms] o={o} v={v} {prec}", flush=True)
    seed = 500 + o + v
    s = ci.make_system(o, v, o + v, seed, sigma=0.05)
    f = ci.random_fock(o, v, seed)
    t1, t2, _ = ci.random_amplitudes(o, v, seed, 0.02, 0.03, 0.0, triples=False)
    t3p = ci.random_t3_packed(o, v, seed + 1, 0.02)
    V, t3 = R.eri_phys_from_B(s["B"]), R.unpack_t3(t3p, o)
    with binding.Engine(o, v, s["naux"], precision=prec) as eng:
        eng.set_fock(f)
        eng.set_eri_df(s["B"])
        eng.set_amplitudes(t1, t2, t3p)
        for term in ("RA", "RB", "RC", "HH", "F1", "F2", "D1", "D2"):
            got = eng.residual((term,))[2]
            want = R.pack_t3(R.postprocess_r3(R.residuals(f, V, t1, t2, t3, o, terms=(term,))[2]))
            tol = RINGS[prec] if term in ("RA", "RB", "RC") else 1e-11
            err = float(np.abs(got - want).max() / np.abs(want).max())
            print(f"  {term} largest {np.abs(want).max():.1e}, error {err:.1e} of it", flush=True)
            assert err <= tol, term
