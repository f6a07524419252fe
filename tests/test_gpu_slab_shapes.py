"""Slab terms at the sizes where their launches change path: v^2 with and
without padding to whole K tiles, odd and even o and v (element and 16-byte
loads of the driver items), one block, blocks with repeated labels, the default
panel (all of W) and panels of one row.  Against the block oracle; tolerances of
the slab tests (1e-11 FP64, 2e-6 FP32, 5e-5 split-BF16 of the largest element)."""

import sys

import numpy as np
import pytest

import cct_inputs as ci
from oracle import blocks
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-11, "fp32": 2e-6, "bf16x3": 5e-5}


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


@pytest.mark.parametrize("prec,o,v,first,count,panel", [
    ("fp64", 1, 1, 0, 1, None), ("fp64", 2, 3, 0, 4, None), ("fp64", 3, 8, 2, 6, None), ("fp64", 4, 9, 5, 15, 1),
    ("fp64", 5, 16, 0, 35, None), ("fp64", 3, 17, 0, 10, 16), ("fp64", 2, 33, 1, 3, None), ("fp64", 4, 32, 7, 1, None),
    ("fp32", 3, 13, 0, 10, None), ("fp32", 4, 24, 3, 9, None), ("bf16x3", 3, 15, 0, 10, None),
    ("bf16x3", 4, 32, 0, 20, None)])
def test_slab_shapes(prec, o, v, first, count, panel):
    say(f"[slab shapes] {prec} o={o} v={v} [{first},{first + count}) panel={panel}")
    seed = 500 + o + v
    rng = np.random.default_rng(seed)
    naux = o + 2 * v + 1
    s = ci.make_system(o, v, naux, seed, sigma=0.1)
    t1, t2, _ = ci.random_amplitudes(o, v, seed, 0.03, 0.03, 0.0, triples=False)
    Bt = blocks.dressed_factors(s["B"], t1)
    Fvv, Wvvvo, Wvooo = rng.normal(0, 0.1, (v, v)), rng.normal(0, 0.1, (v, v, v, o)), rng.normal(0, 0.1, (v, o, o, o))
    t3p = ci.hashed_t3_packed(o, v, seed + 1, 0.02, threads=4)
    tri = ci.packed_triples(o)
    W = blocks.w_vvvv(Bt, t2, o)
    with binding.Slab(o, v, naux, first, count, precision=prec, opts=None if panel is None else {"panel": panel}) as sl:
        sl.set_intermediates(Bt, t2, Fvv, np.ascontiguousarray(Wvvvo.transpose(3, 0, 1, 2)), Wvooo)
        sl.set_t3(t3p[first:first + count])
        for terms in (("PP", "F1", "D1", "D2"), ("PP",), ("D1",), ("D2",), ("D1", "D2", "F1")):
            got, _ = sl.residual(terms)
            ref = np.array([blocks.local_terms_block(W, Fvv, Wvvvo, Wvooo, t2, t3p[n], tri[n], terms=terms)
                            for n in range(first, first + count)])
            assert np.abs(got - ref).max() <= TOL[prec] * max(float(np.abs(ref).max()), 1e-300), terms
