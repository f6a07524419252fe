"""Large products of the generally strided kernel with few rows (odd v, so that
the hole ladder takes that kernel): 64 x 64 tiles where 128 x 128 ones would be
mostly padding.  36 and 28 rows (o = 8, 7), ragged columns.  FP64 residual
against the oracle, 1e-11 of the largest element (sums of at most 1e5 terms that
round at 1e-16 each)."""

import numpy as np
import pytest

import cct_inputs as ci
from oracle import rccsdt as R
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("o,v", [(8, 33), (7, 37)])
def test_residual_matches_the_oracle(o, v):
    print(f"[strided tiles] o={o} v={v}", flush=True)
    seed = 800 + o + v
    s = ci.make_system(o, v, o + v, seed, sigma=0.05)
    f = ci.random_fock(o, v, seed)
    t1, t2, _ = ci.random_amplitudes(o, v, seed, 0.02, 0.03, 0.0, triples=False)
    t3p = ci.random_t3_packed(o, v, seed + 1, 0.02)
    with binding.Engine(o, v, s["naux"]) as eng:
        eng.set_fock(f)
        eng.set_eri_df(s["B"])
        eng.set_amplitudes(t1, t2, t3p)
        g1, g2, g3, _ = eng.residual()
    r1, r2, r3 = R.residuals(f, R.eri_phys_from_B(s["B"]), t1, t2, R.unpack_t3(t3p, o), o)
    r3p = R.pack_t3(R.postprocess_r3(r3))
    for name, a, b in (("R1", g1, r1), ("R2", g2, r2), ("R3", g3, r3p)):
        assert np.abs(a - b).max() <= 1e-11 * max(1.0, float(np.abs(b).max())), name
