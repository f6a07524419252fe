"""The work that users of this framework have it do, as measurable cases.

Kinds (each through the public classes of ``paper_2607_00981_amd.binding``):

``iterate``   a CCSDT run: MP2 guess, a few iterations (residuals, Jacobi
              update, DIIS, energy), amplitudes read back
``residual``  one residual evaluation at given amplitudes, R1, R2, R3 read back
``batch``     one iteration of a batch of independent small systems
``q``         the perturbative quadruples correction, occupied-tuple order
``qabc``      the same in the virtual-tuple order, a share of its tasks
``slab``      the block-local R3 terms of a share of the packed triples
``quad``      the quadruples ladder on compact T4

Shapes are named by o occupied and v virtual orbitals; naux = 2 (o + v).
Integrals are random with the (pq|rs) variance of the o=4, v=20 system at
every size, so that the iterations stay bounded, and amplitudes come from
iterations on them or are Gaussian of the size such iterations give.
"""

import itertools
import math

import numpy as np
import torch

from paper_2607_00981_amd import binding


def listed():
    return [
        # The smallest single molecule: a whole run is bound by launches and read-backs.
        {"name": "iterate-o4v20-fp64", "kind": "iterate", "o": 4, "v": 20, "prec": "fp64", "iters": 8},
        # A small molecule of odd sizes in the FP32 mode.
        {"name": "iterate-o6v37-fp32", "kind": "iterate", "o": 6, "v": 37, "prec": "fp32", "iters": 4},
        # The ordinary single molecule, all in FP64 ...
        {"name": "iterate-o10v90-fp64", "kind": "iterate", "o": 10, "v": 90, "prec": "fp64", "iters": 3},
        # ... and with split-BF16 ladder and ring products.
        {"name": "iterate-o10v90-bf16x3", "kind": "iterate", "o": 10, "v": 90, "prec": "bf16x3", "iters": 3},
        # A residual for a solver of the caller's own, at an odd number of virtuals.
        {"name": "residual-o8v61-fp64", "kind": "residual", "o": 8, "v": 61, "prec": "fp64"},
        # Many small molecules iterated together (sizes o 3..8, v 20..60).
        {"name": "batch-48-fp64", "kind": "batch", "nsys": 48, "omax": 8, "vmax": 60, "prec": "fp64"},
        # (Q) after a run of the smallest molecule: launch-bound.
        {"name": "q-o4v20", "kind": "q", "o": 4, "v": 20},
        # (Q) of an ordinary molecule.
        {"name": "q-o6v48", "kind": "q", "o": 6, "v": 48},
        # The virtual-tuple order on a spread-out share of its tasks, as one process of several takes them.
        {"name": "qabc-o8v60-b6", "kind": "qabc", "o": 8, "v": 60, "block": 6, "ntasks": 24},
        # One process's share of a sharded run, mixed precision.
        {"name": "slab-o12v96-bf16x3", "kind": "slab", "o": 12, "v": 96, "first": 100, "count": 24, "prec": "bf16x3"},
        # The same in FP64 at odd sizes.
        {"name": "slab-o9v75-fp64", "kind": "slab", "o": 9, "v": 75, "first": 3, "count": 20, "prec": "fp64"},
        # The leading RCCSDTQ term of a small molecule.
        {"name": "quad-o4v24-fp64", "kind": "quad", "o": 4, "v": 24, "prec": "fp64"},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: any kind, any precision it takes, sizes over the whole range, odd ones included."""
    kind = rng.choice(["iterate", "iterate", "iterate", "residual", "batch", "q", "qabc", "slab", "quad"])
    prec = rng.choice(["fp64", "fp64", "fp32", "bf16x3"])
    if kind == "iterate":
        o, v = rng.randint(3, 9), _log_int(rng, 14, 80)
        return {"kind": kind, "o": o, "v": v, "prec": prec, "iters": rng.randint(2, 3)}
    if kind == "residual":
        return {"kind": kind, "o": rng.randint(2, 8), "v": _log_int(rng, 12, 64), "prec": prec}
    if kind == "batch":
        return {"kind": kind, "nsys": rng.randint(6, 40), "omax": rng.randint(4, 8), "vmax": rng.randint(24, 60),
                "prec": prec}
    if kind == "q":
        return {"kind": kind, "o": rng.randint(2, 6), "v": _log_int(rng, 12, 48)}
    if kind == "qabc":
        return {"kind": kind, "o": rng.randint(3, 8), "v": _log_int(rng, 18, 60), "block": rng.randint(3, 7),
                "ntasks": rng.randint(6, 24)}
    if kind == "slab":
        o = rng.randint(4, 12)
        n = o * (o + 1) * (o + 2) // 6
        count = rng.randint(6, 20)
        return {"kind": kind, "o": o, "v": _log_int(rng, 30, 96), "first": rng.randint(0, n - count), "count": count,
                "prec": prec}
    return {"kind": kind, "o": rng.randint(2, 4), "v": _log_int(rng, 12, 26), "prec": prec}


# --- inputs ------------------------------------------------------------------


def _system(o, v, seed):
    """Diagonal Fock matrix and fitting factors B[P][p][q], symmetric in (p, q)."""
    n, naux = o + v, 2 * (o + v)
    rng = np.random.default_rng(seed)
    f = np.diag(np.concatenate([np.sort(rng.uniform(-1.5, -0.5, o)), np.sort(rng.uniform(0.3, 3.0, v))]))
    # the weak-coupling variant of the named workloads: (pq|rs) small enough for every size to converge
    B = rng.normal(0.0, 0.05 * math.sqrt(48.0 / naux) / 3.0, (naux, n, n))
    return f, np.ascontiguousarray(np.triu(B) + np.swapaxes(np.triu(B, 1), 1, 2))


def _pair_t2(rng, o, v, scale):
    x = rng.normal(0.0, scale, (o, o, v, v))
    return np.ascontiguousarray(0.5 * (x + x.transpose(1, 0, 3, 2)))


def _triples(o):
    return [(i, j, k) for i in range(o) for j in range(i, o) for k in range(j, o)]


def _packed_t3(rng, blocks, v, scale):
    """Packed T3 blocks with the symmetry that equal occupied indices force."""
    t = rng.random((len(blocks), v, v, v))
    t -= 0.5
    t *= scale
    for m, (i, j, k) in enumerate(blocks):
        if i == j == k:
            t[m] = sum(t[m].transpose(p) for p in itertools.permutations(range(3))) / 6.0
        elif i == j:
            t[m] = 0.5 * (t[m] + t[m].transpose(1, 0, 2))
        elif j == k:
            t[m] = 0.5 * (t[m] + t[m].transpose(0, 2, 1))
    return t


def _amplitudes(c, seed):
    o, v = c["o"], c["v"]
    rng = np.random.default_rng([seed, 1])
    return (rng.normal(0.0, 0.02, (o, v)), _pair_t2(rng, o, v, 0.02), _packed_t3(rng, _triples(o), v, 0.02))


def _batch_sizes(c):
    """The sizes belong to the case, not to the seed: the same batch with other integrals."""
    rng = np.random.default_rng(4)
    return [(int(rng.integers(3, c["omax"] + 1)), int(rng.integers(20, c["vmax"] + 1))) for _ in range(c["nsys"])]


def _qabc_tasks(c):
    total = binding.q_abc_task_count(c["v"], c["block"])
    n = min(c["ntasks"], total)
    return [int((m + 0.5) * total / n) for m in range(n)]


def _slab_inputs(c, seed):
    o, v, n = c["o"], c["v"], c["o"] + c["v"]
    rng = np.random.default_rng([seed, 2])
    uniform = lambda shape, scale: (rng.random(shape) - 0.5) * scale  # noqa: E731
    B = _system(o, v, seed)[1]
    blocks = _triples(o)[c["first"]:c["first"] + c["count"]]
    return (B, _pair_t2(rng, o, v, 0.02), uniform((v, v), 0.2), uniform((o, v, v, v), 0.2), uniform((v, o, o, o), 0.2),
            _packed_t3(rng, blocks, v, 0.02))


def _quad_inputs(c, seed):
    o, v = c["o"], c["v"]
    rng = np.random.default_rng([seed, 3])
    W = rng.random((v, v, v, v))
    W -= 0.5
    W = np.ascontiguousarray(W + W.transpose(1, 0, 3, 2))  # W^{ab}_{ef} = W^{ba}_{fe}
    quads = list(itertools.combinations_with_replacement(range(o), 4))
    t4 = rng.random((len(quads), v, v, v, v))
    t4 -= 0.5
    t4 *= 0.01
    for m, q in enumerate(quads):  # equal occupied indices: symmetric in their virtual axes
        sym = [p for p in itertools.permutations(range(4)) if tuple(q[x] for x in p) == q]
        if len(sym) > 1:
            t4[m] = sum(t4[m].transpose(p) for p in sym) / len(sym)
    return W, t4


def prepare(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind in ("iterate", "residual", "q", "qabc"):
        o, v = c["o"], c["v"]
        f, B = _system(o, v, seed)
        eng = binding.Engine(o, v, B.shape[0], precision=c.get("prec", "fp64"))
        eng.set_fock(f)
        eng.set_eri_df(B)
        state = {"c": c, "eng": eng}
        if kind == "residual":
            eng.set_amplitudes(*_amplitudes(c, seed))
        elif kind in ("q", "qabc"):
            eng.init_mp2()
            for _ in range(2):
                eng.update()
            if kind == "qabc":
                state["tasks"] = _qabc_tasks(c)
        return state
    if kind == "batch":
        sizes = _batch_sizes(c)
        batch = binding.Batch([(o, v, 2 * (o + v)) for o, v in sizes], precision=c["prec"])
        for s, (o, v) in enumerate(sizes):
            batch.set_system(s, *_system(o, v, [seed, s]))
        batch.iterate(1)  # records the graph; triples are non-zero from here on
        return {"c": c, "batch": batch}
    if kind == "slab":
        Bt, t2, Fvv, Wt, Wvooo, t3 = _slab_inputs(c, seed)
        slab = binding.Slab(c["o"], c["v"], Bt.shape[0], c["first"], c["count"], precision=c["prec"])
        slab.set_intermediates(Bt, t2, Fvv, Wt, Wvooo)
        slab.set_t3(t3)
        return {"c": c, "slab": slab}
    quad = binding.Quad(c["o"], c["v"], precision=c["prec"])
    quad.set(*_quad_inputs(c, seed))
    return {"c": c, "quad": quad}


def run(state):
    c = state["c"]
    kind = c["kind"]
    if kind == "iterate":
        eng = state["eng"]
        eng.init_mp2()
        history = [eng.update() for _ in range(c["iters"])]
        t1, t2, t3 = eng.get_amplitudes()
        return {"e": np.array([e for e, _ in history]), "norms": np.array([n for _, n in history]),
                "t1": t1, "t2": t2, "t3": t3}
    if kind == "residual":
        r1, r2, r3, norms = state["eng"].residual()
        return {"r1": r1, "r2": r2, "r3": r3, "norms": norms}
    if kind == "batch":
        batch = state["batch"]
        e, norms = batch.iterate(1)
        amps = [batch.system(s).get_amplitudes(with_t3=False) for s in range(c["nsys"])]
        return {"e": e, "norms": norms, "t1": np.concatenate([a[0].ravel() for a in amps]),
                "t2": np.concatenate([a[1].ravel() for a in amps])}
    if kind == "q":
        e, tasks = state["eng"].energy_q(tasks=True)
        return {"e": e, "tasks": tasks}
    if kind == "qabc":
        got = state["eng"].energy_q_abc(c["block"], state["tasks"], tuples=True)
        return {"e": got["e_q"], "tasks": got["e_tasks"], "tuples": got["e_tuples"]}
    if kind == "slab":
        r3, norm2 = state["slab"].residual()
        return {"r3": r3, "norm2": norm2}
    r4, norm2 = state["quad"].ladder()
    return {"r4": r4, "norm2": norm2}


# --- work ----------------------------------------------------------------------


def _residual_work(o, v):
    """(multiply-adds, doubles) of one residual with the compact storage: the
    ladder in its symmetric / antisymmetric form, rings, hole ladder, T3
    feedback, drivers, Fock term, the T2 ladder and the integrals."""
    n, naux, ntri = o + v, 2 * (o + v), o * (o + 1) * (o + 2) // 6
    npair = o * (o + 1) // 2
    macs = 1.5 * ntri * v ** 5 + (2 * npair + o * o) * (o * v) ** 2 * v ** 2 + o ** 3 * npair * v ** 3
    macs += 3 * o ** 3 * v ** 4 + o ** 4 * v ** 3 + 3 * ntri * v ** 4 + 0.5 * o * o * v ** 4 + 0.5 * naux * n ** 4
    return macs, 2 * ntri * v ** 3 + 2 * (o * v) ** 2 + naux * n * n


def _q_task_macs(o, v):
    """Per ordered occupied tuple: two v^5 and two o v^4 contractions."""
    return 2 * v ** 5 + 2 * o * v ** 4


def work(case):
    c = dict(case)
    kind, o, v = c["kind"], c.get("o", 0), c.get("v", 0)
    if kind in ("iterate", "residual"):
        macs, doubles = _residual_work(o, v)
        it = c.get("iters", 1)
        return {"bytes": 8.0 * doubles * it, "flops": 2.0 * macs * it}
    if kind == "batch":
        each = [_residual_work(*s) for s in _batch_sizes(c)]
        return {"bytes": 8.0 * sum(d for _, d in each), "flops": 2.0 * sum(m for m, _ in each)}
    n, ntri = o + v, o * (o + 1) * (o + 2) // 6
    if kind == "q":
        ordered = o ** 4 - 4 * o * (o - 1) - o  # no three equal indices
        return {"bytes": 8.0 * (ntri * v ** 3 + (o * v) ** 2 + 2 * n ** 3 + o ** 4),
                "flops": 2.0 * (ordered * _q_task_macs(o, v) + o * o * v ** 5 + n ** 5)}
    if kind == "qabc":
        nb, nt = c["block"], c["ntasks"]
        per = nb ** 4 * (12 * (o ** 4 * v + o ** 5) * 2)
        return {"bytes": 8.0 * (2 * ntri * v ** 3 + (o * v) ** 2 + 2 * n ** 3 + nt * nb ** 4),
                "flops": 2.0 * (nt * per + n ** 5)}
    if kind == "slab":
        count, naux = c["count"], 2 * n
        macs = 1.5 * count * v ** 5 + 0.5 * (naux + o * o) * v ** 4 + 9 * count * v ** 4 + 6 * count * o * v ** 3
        return {"bytes": 8.0 * (2 * count * v ** 3 + o * v ** 3 + naux * n * n + (o * v) ** 2), "flops": 2.0 * macs}
    nq = o * (o + 1) * (o + 2) * (o + 3) // 24
    return {"bytes": 8.0 * (2 * nq + 1) * v ** 4, "flops": 2.0 * 3 * nq * v ** 6}


# --- 64-bit values ---------------------------------------------------------------
# The paper's equations on full tensors (Appendix A; the (Q) appendix), written
# out with torch.einsum in float64: no packed storage, no splitting.

_es = torch.einsum
_PERM3 = list(itertools.permutations(range(3)))
_PERM4 = list(itertools.permutations(range(4)))


def _dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda" if torch.cuda.is_available() else "cpu")


def _swap_virt(t, p):
    """t[i,j,k,a,b,c] with its virtual axes permuted."""
    return t.permute(0, 1, 2, 3 + p[0], 3 + p[1], 3 + p[2])


def _unpack3(t3p, o):
    """Full T3 from packed blocks i <= j <= k by the column symmetry."""
    v = t3p.shape[1]
    full = torch.empty((o, o, o, v, v, v), dtype=torch.float64, device=t3p.device)
    for m, ijk in enumerate(_triples(o)):
        for p in _PERM3:
            full[ijk[p[0]], ijk[p[1]], ijk[p[2]]] = t3p[m].permute(p)
    return full


def _pack3(t):
    return torch.stack([t[i, j, k] for i, j, k in _triples(t.shape[0])])


def _coulomb(B):
    """v^{pq}_{rs} = sum_P B_pr B_qs."""
    return _es("Ppr,Pqs->pqrs", B, B)


def _dress(f, B, t1):
    o, v = t1.shape
    n = o + v
    x, y = torch.eye(n, dtype=f.dtype, device=f.device), torch.eye(n, dtype=f.dtype, device=f.device)
    x[o:, :o] -= t1.T
    y[:o, o:] += t1
    G = 2.0 * _es("Prs,P->rs", B, _es("Pia,ia->P", B[:, :o, o:], t1)) - _es("Pri,Pis->rs", B[:, :, o:] @ t1.T, B[:, :o])
    return x @ (f + G) @ y.T, _es("pt,Ptu,ru->Ppr", x, B, y)


def _residuals64(f, B, t1, t2, t3):
    """R1, R2 and the post-processed R3 on full tensors."""
    o, v = t1.shape
    O, U = slice(0, o), slice(o, o + v)
    ft, Bt = _dress(f, B, t1)
    V = _coulomb(Bt)
    chk = lambda x: 2.0 * x - x.transpose(2, 3)  # noqa: E731
    oovv, C = V[O, O, U, U], chk(V[O, O, U, U])
    tau = chk(t2)
    s1 = 2.0 * t3 - _swap_virt(t3, (1, 0, 2)) - _swap_virt(t3, (2, 1, 0))
    s12 = 2.0 * s1 - _swap_virt(s1, (0, 2, 1))
    Covvo = 2.0 * V[O, U, U, O] - V[O, U, O, U].transpose(2, 3)
    Coovo = 2.0 * V[O, O, U, O] - V[O, O, O, U].transpose(2, 3)
    Fvv = ft[U, U] - _es("kldc,kldb->bc", C, t2)
    Foo = ft[O, O] + _es("lkcd,ljcd->kj", C, t2)
    Woooo = V[O, O, O, O] + _es("klcd,ijcd->klij", oovv, t2)
    Wovvo = Covvo + 0.5 * _es("lkdc,lida->kaci", C, tau)
    Wovov = V[O, U, O, U] - 0.5 * _es("lkcd,ilda->kaic", oovv, t2)
    r1 = ft[U, O].T + _es("kc,ikac->ia", ft[O, U], tau) + _es("akcd,ikcd->ia", V[U, O, U, U], tau)
    r1 = r1 - _es("klic,klac->ia", V[O, O, O, U], tau) + 0.5 * _es("jkbc,jkibca->ia", oovv, s12)
    X2 = 0.5 * V[U, U, O, O].permute(2, 3, 0, 1) + _es("bc,ijac->ijab", Fvv, t2) - _es("kj,ikab->ijab", Foo, t2)
    X2 = X2 + 0.5 * _es("abcd,ijcd->ijab", V[U, U, U, U], t2) + 0.5 * _es("klij,klab->ijab", Woooo, t2)
    X2 = X2 + 0.5 * _es("kaci,kjcb->ijab", Wovvo, tau) - 0.5 * _es("kaic,jkcb->ijab", Wovov, t2)
    X2 = X2 - _es("kbic,jkca->ijab", Wovov, t2) + 0.5 * _es("kc,kijcab->ijab", ft[O, U], s1)
    X2 = X2 + _es("bkcd,kijdac->ijab", V[U, O, U, U], s1) - _es("kljc,likcab->ijab", V[O, O, O, U], s1)
    r2 = X2 + X2.permute(1, 0, 3, 2)
    Wvvvo = V[U, U, U, O] + 0.5 * _es("laed,ljeb->abdj", chk(V[O, U, U, U]), tau)
    Wvvvo = Wvvvo - 0.5 * _es("lade,jleb->abdj", V[O, U, U, U], t2) - _es("lbde,jlea->abdj", V[O, U, U, U], t2)
    Wvvvo = Wvvvo + _es("lmdj,lmab->abdj", V[O, O, U, O], t2) - _es("lmde,mjleba->abdj", oovv, s1)
    Wvooo = V[U, O, O, O] + _es("ld,ijad->alij", ft[O, U], t2) + 0.5 * _es("mldj,mida->alij", Coovo, tau)
    Wvooo = Wvooo - 0.5 * _es("mljd,imda->alij", V[O, O, O, U], t2) - _es("mlid,jmda->alij", V[O, O, O, U], t2)
    Wvooo = Wvooo + _es("alde,ijde->alij", V[U, O, U, U], t2) + _es("lmde,mijead->alij", oovv, s1)
    Wb1 = Wovvo + 0.5 * _es("mled,miea->ladi", C, tau)
    Wb2 = Wovov - 0.5 * _es("mlde,imea->laid", oovv, t2)
    Wvvvv = V[U, U, U, U] + _es("lmde,lmab->abde", oovv, t2)
    X3 = _es("abdj,ikdc->ijkabc", Wvvvo, t2) - _es("alij,lkbc->ijkabc", Wvooo, t2)
    X3 += 0.5 * _es("ad,ijkdbc->ijkabc", Fvv, t3)
    X3 -= 0.5 * _es("li,ljkabc->ijkabc", Foo, t3)
    X3 += 0.25 * _es("ladi,ljkdbc->ijkabc", Wb1, s1)
    X3 -= 0.5 * _es("laid,jlkdbc->ijkabc", Wb2, t3)
    X3 -= _es("lbid,jlkdac->ijkabc", Wb2, t3)
    X3 += 0.5 * _es("lmij,lmkabc->ijkabc", Woooo, t3)
    X3 += 0.5 * _es("abde,ijkdec->ijkabc", Wvvvv, t3)
    r3 = torch.zeros_like(X3)
    for p in _PERM3:
        r3 += X3.permute(*p, *(3 + q for q in p))
    for i in range(o):
        r3[i, i, i] = 0.0
    return r1, r2, r3 - sum(_swap_virt(r3, p) for p in _PERM3) / 6.0


def _denominators(f, o):
    e = torch.diagonal(f)
    d1 = e[:o, None] - e[None, o:]
    d2 = d1[:, None, :, None] + d1[None, :, None, :]
    return d1, d2, d2[:, :, None, :, :, None] + d1[None, None, :, None, None, :]


def _norms(r1, r2, r3):
    return [float((r * r).sum()) for r in (r1, r2, r3)]


def _run64(f, B, o, iters):
    """MP2 guess and `iters` iterations with DIIS over (T1, T2, T3): 8 vectors,
    from the second on, error = Jacobi step."""
    v = f.shape[0] - o
    d = _denominators(f, o)
    V = _es("Pia,Pjb->ijab", B[:, :o, o:], B[:, :o, o:])
    t = [torch.zeros_like(d[0]), V / d[1], torch.zeros((o, o, o, v, v, v), dtype=f.dtype, device=f.device)]
    vecs, errs, energies, norms = [], [], [], []
    for _ in range(iters):
        r = _residuals64(f, B, *t)
        norms.append(_norms(*r))
        step = [x / y for x, y in zip(r, d)]
        t = [x + y for x, y in zip(t, step)]
        vecs, errs = (vecs + [t])[-8:], (errs + [step])[-8:]
        m = len(vecs)
        if m >= 2:
            A = np.zeros((m + 1, m + 1))
            A[m, :m] = A[:m, m] = -1.0
            for a in range(m):
                for b in range(m):
                    A[a, b] = sum(float((x * y).sum()) for x, y in zip(errs[a], errs[b]))
            rhs = np.zeros(m + 1)
            rhs[m] = -1.0
            w = np.linalg.solve(A, rhs)[:m]
            t = [sum(w[a] * vecs[a][k] for a in range(m)) for k in range(3)]
        tau = t[1] + _es("ia,jb->ijab", t[0], t[0])
        energies.append(float((_es("ijab,ijab->", 2.0 * V - V.transpose(2, 3), tau)
                               + 2.0 * (f[:o, o:] * t[0]).sum())))
    return t, energies, norms


def _quadruples64(V, t2, t3, eo, ev, occ, vir):
    """z and t4 on the box of the label sets occ[4], vir[4] (lists), as
    [i,j,k,l,a,b,c,d]: the 24-permutation sums of X + V and X + Y over column
    orders, each order evaluated on the permuted label sets."""
    o = t2.shape[0]
    O, U = slice(0, o), slice(o, None)
    take = lambda t, *ix: t[torch.meshgrid(*(  # noqa: E731
        torch.arange(t.shape[k], device=t.device)[x] if isinstance(x, slice) else torch.tensor(x, device=t.device)
        for k, x in enumerate(ix)), indexing="ij")]
    A = slice(None)
    z = t4 = 0.0
    for p in _PERM4:
        # the term whose first column is column p[0] of the box, and so on
        i, j, k, l = (occ[x] for x in p)
        a, b, c, d = (vir[x] for x in p)
        g = lambda x: [o + y for y in x]  # noqa: E731
        X = 0.5 * _es("abej,iklecd->ijklabcd", take(V, g(a), g(b), U, j), take(t3, i, k, l, A, c, d))
        X = X - 0.5 * _es("amij,mklbcd->ijklabcd", take(V, g(a), O, i, j), take(t3, A, k, l, b, c, d))
        Wv = 0.5 * (_es("abef,jkfc->ejkabc", take(V, g(a), g(b), U, U), take(t2, j, k, A, c))
                    + _es("acef,kjfb->ejkabc", take(V, g(a), g(c), U, U), take(t2, k, j, A, b)))
        Y = 0.5 * _es("ejkabc,iled->ijklabcd", Wv, take(t2, i, l, A, d))

        def half(i_, j_, a_, b_, spec):
            w = (_es("maei,jkbe->ijkabm", take(V, O, g(a_), U, i_), take(t2, j_, k, b_, A))
                 + _es("make,jibe->ijkabm", take(V, O, g(a_), k, U), take(t2, j_, i_, b_, A))
                 - 0.5 * _es("mnki,njab->ijkabm", take(V, O, O, k, i_), take(t2, A, j_, a_, b_)))
            return w.permute(spec)

        Wo = half(i, j, a, b, (0, 1, 2, 3, 4, 5)) + half(j, i, b, a, (1, 0, 2, 4, 3, 5))
        Y = Y - 0.5 * _es("ijkabm,mlcd->ijklabcd", Wo, take(t2, A, l, c, d))
        W = 0.25 * _es("abij,klcd->ijklabcd", take(V, g(a), g(b), i, j), take(t2, k, l, c, d))
        inv = [p.index(x) for x in range(4)]
        order = (*inv, *(4 + x for x in inv))
        z = z + (X + W).permute(order)
        t4 = t4 + (X + Y).permute(order)
    den = 0.0
    for s in range(4):
        den = den + eo[occ[s]].reshape([-1 if x == s else 1 for x in range(8)])
        den = den - ev[vir[s]].reshape([-1 if x == 4 + s else 1 for x in range(8)])
    return z, t4 / den


def _spin_sum4(t, first):
    """The fully spin-summed amplitude: label exchanges on the four axes from `first` on."""
    def x(u, p, q):
        return u.transpose(first + p, first + q)
    u = 2.0 * t - x(t, 0, 1) - x(t, 0, 2) - x(t, 0, 3)
    u = 2.0 * u - x(u, 1, 2) - x(u, 1, 3)
    return 2.0 * (2.0 * u - x(u, 2, 3))


def _orders(q):
    return len(set(itertools.permutations(q)))


def _q64(c, seed):
    o, v = c["o"], c["v"]
    f, B = (_dev(x) for x in _system(o, v, seed))
    t, _, _ = _run64(f, B, o, 2)
    V, e = _coulomb(B), torch.diagonal(f)
    everything = list(range(v))
    out = []
    for q in itertools.combinations_with_replacement(range(o), 4):
        if max(q.count(x) for x in q) >= 3:
            out.append(0.0)
            continue
        z, t4 = _quadruples64(V, t[1], t[2], e[:o], e[o:], [[x] for x in q], [everything] * 4)
        out.append(float((z * _spin_sum4(t4, 4)).sum()) * _orders(q) / 24.0)
    return {"e": float(sum(out)), "tasks": np.array(out)}


def _qabc64(c, seed):
    o, v, nb = c["o"], c["v"], c["block"]
    f, B = (_dev(x) for x in _system(o, v, seed))
    t, _, _ = _run64(f, B, o, 2)
    V, e = _coulomb(B), torch.diagonal(f)
    tiles = [list(range(x, min(x + nb, v))) for x in range(0, v, nb)]
    boxes = list(itertools.combinations_with_replacement(range(len(tiles)), 4))
    tasks = _qabc_tasks(c)
    tuples = np.zeros((len(tasks), nb ** 4))
    for m, task in enumerate(tasks):
        vir = [tiles[x] for x in boxes[task]]
        z, t4 = _quadruples64(V, t[1], t[2], e[:o], e[o:], [list(range(o))] * 4, vir)
        # exchanging virtual labels at fixed occupied ones = exchanging the occupied labels (column symmetry)
        share = (z * _spin_sum4(t4, 0)).sum(dim=(0, 1, 2, 3)).reshape(-1).cpu().numpy() / 24.0
        for at, q in enumerate(itertools.product(*vir)):
            if list(q) == sorted(q) and max(q.count(x) for x in q) < 3:
                tuples[m, at] = share[at] * _orders(q)
    return {"e": float(tuples.sum()), "tasks": tuples.sum(axis=1), "tuples": tuples}


def _slab64(c, seed):
    o, v = c["o"], c["v"]
    Bt, t2, Fvv, Wt, Wvooo, t3 = (_dev(x) for x in _slab_inputs(c, seed))
    V = _es("Pad,Pbe->abde", Bt[:, o:, o:], Bt[:, o:, o:])
    V += _es("lmde,lmab->abde", _es("Pld,Pme->lmde", Bt[:, :o, o:], Bt[:, :o, o:]), t2)
    out, norm2 = torch.zeros_like(t3), 0.0
    for m, occ in enumerate(_triples(o)[c["first"]:c["first"] + c["count"]]):
        if occ[0] == occ[2]:
            continue
        r = torch.zeros_like(t3[m])
        for p in _PERM3:
            i, j, k = (occ[x] for x in p)
            t = t3[m].permute(p)  # t_ijk^{xyz}
            y = 0.5 * _es("xyde,dez->xyz", V, t) + 0.5 * _es("xd,dyz->xyz", Fvv, t)
            y = y + _es("xyd,dz->xyz", Wt[j], t2[i, k]) - _es("xl,lyz->xyz", Wvooo[:, :, i, j], t2[:, k])
            r += y.permute([p.index(x) for x in range(3)])
        out[m] = r - sum(r.permute(p) for p in _PERM3) / 6.0
        norm2 += _orders(occ) * float((out[m] * out[m]).sum())
    return {"r3": out, "norm2": norm2}


def _quad64(c, seed):
    o = c["o"]
    W, t4 = (_dev(x) for x in _quad_inputs(c, seed))
    out = torch.zeros_like(t4)
    out += _es("xyef,nefcd->nxycd", W, t4) + _es("xyef,nebfd->nxbyd", W, t4) + _es("xyef,nebcf->nxbcy", W, t4)
    out += _es("xyef,naefd->naxyd", W, t4) + _es("xyef,naecf->naxcy", W, t4) + _es("xyef,nabef->nabxy", W, t4)
    weight = torch.tensor([float(_orders(q)) for q in itertools.combinations_with_replacement(range(o), 4)],
                          dtype=out.dtype, device=out.device)
    return {"r4": out, "norm2": float((weight * (out * out).sum(dim=(1, 2, 3, 4))).sum())}


def exact(case, seed):
    c = dict(case)
    kind = c["kind"]
    if kind == "q":
        return _q64(c, seed)
    if kind == "qabc":
        return _qabc64(c, seed)
    if kind == "slab":
        return _slab64(c, seed)
    if kind == "quad":
        return _quad64(c, seed)
    if kind == "batch":
        e, norms, t1, t2 = [], [], [], []
        for s, (o, v) in enumerate(_batch_sizes(c)):
            f, B = (_dev(x) for x in _system(o, v, [seed, s]))
            t, energies, n = _run64(f, B, o, 2)
            e.append(energies[-1])
            norms.append(n[-1])
            t1.append(t[0].reshape(-1))
            t2.append(t[1].reshape(-1))
        return {"e": np.array(e), "norms": np.array(norms), "t1": torch.cat(t1), "t2": torch.cat(t2)}
    o = c["o"]
    f, B = (_dev(x) for x in _system(o, c["v"], seed))
    if kind == "residual":
        t1, t2, t3 = (_dev(x) for x in _amplitudes(c, seed))
        r1, r2, r3 = _residuals64(f, B, t1, t2, _unpack3(t3, o))
        return {"r1": r1, "r2": r2, "r3": _pack3(r3), "norms": np.array(_norms(r1, r2, r3))}
    t, energies, norms = _run64(f, B, o, c["iters"])
    return {"e": np.array(energies), "norms": np.array(norms), "t1": t[0], "t2": t[1], "t3": _pack3(t[2])}
