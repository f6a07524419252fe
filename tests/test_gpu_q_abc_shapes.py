"""E_(Q) in the virtual-tuple order where its launches change: the Z products
in one launch (contractions up to 64 labels) and one by one (65), the label
triples of a ragged last tile beside full ones in one launch, o at and past the
column counts that the Wbar builds hold (8, 16, 32).  Against the occupied-tuple
order on the same amplitudes, which shares none of these kernels: 1e-11 of the
energy's scale (both sum FP64 terms of it)."""

import numpy as np
import pytest

import cct_inputs as ci
from oracle import rccsdt as R
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("o,v,nb", [(2, 64, 16), (2, 65, 16), (3, 11, 4), (8, 13, 5), (9, 8, 3), (16, 4, 3), (17, 4, 2)])
def test_q_abc_equals_occupied_order_at_edges(o, v, nb):
    print(f"[q_abc] o={o} v={v} block={nb}", flush=True)
    s = ci.make_system(o, v, o + v, 700 + o + v, sigma=0.1)
    _, t2, t3 = ci.random_amplitudes(o, v, 701 + v, 0.02, 0.05, 0.05)
    t3p = R.pack_t3(R.orthogonalize_r3(R.purify_r3(t3)))
    with binding.Engine(o, v, s["naux"]) as eng:
        eng.set_fock(s["f"])
        eng.set_eri_df(s["B"])
        eng.set_amplitudes(np.zeros((o, v)), t2, t3p)
        e_occ = eng.energy_q()
        e_abc = eng.energy_q_abc(nb)["e_q"]
    assert e_occ != 0.0
    assert abs(e_abc - e_occ) <= 1e-11 * max(1.0, abs(e_occ))
