"""DIIS on the device at the edges of its chunks (256 x 16 elements of T1/T2
or of one T3 block), for histories of one vector, around the eight sums that
are reduced together, and beyond; T3 whole, a sub-cube, or left out."""
import numpy as np
import pytest

import cct_inputs as ci
from oracle import rccsdt as R
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("o,v,space,t3,niter", [
    (2, 16, 8, "full", 11),         # a T3 block is one chunk; the ring wraps
    (2, 17, 3, "full", 8),          # one chunk and 817 elements
    (3, 21, 9, "full", 12),         # two chunks and a part; nine sums: 8 + 1
    (2, 17, 2, "subspace:16", 6),
    (2, 17, 7, "subspace:3", 10),
    (3, 13, 10, "none", 12),
    (1, 2, 1, "full", 4),           # one vector: the Jacobi step stands
])
def test_diis_follows_the_oracle(o, v, space, t3, niter):
    s = ci.make_system(o, v, 2 * (o + v), 100 + v)
    f, B = s["f"], s["B"]
    V = R.eri_phys_from_B(B)
    mode = int(t3.split(":")[1]) if ":" in t3 else t3
    t1, t2, t3o = R.mp2_guess(f, V, o)
    d = R.DIIS(space)
    ref = []
    for _ in range(niter):
        t1, t2, t3o, e, _ = R.iterate(f, V, t1, t2, t3o, o, diis=d, diis_t3=mode)
        ref.append(e)
    with binding.Engine(o, v, B.shape[0], opts={"diis_t3": t3, "diis_space": space}) as eng:
        eng.set_fock(f)
        eng.set_eri_df(B)
        eng.init_mp2()
        got = [eng.update()[0] for _ in range(niter)]
        g1, g2, g3 = eng.get_amplitudes()
    print(f"[diis] o={o} v={v} space={space} {t3}: max |dE| {np.max(np.abs(np.array(got) - np.array(ref))):.2e}",
          flush=True)
    assert np.max(np.abs(np.array(got) - np.array(ref))) < 1e-10
    assert np.abs(g1 - t1).max() < 1e-9
    assert np.abs(g2 - t2).max() < 1e-9
    assert np.abs(g3 - R.pack_t3(t3o)).max() < 1e-9
