"""GPU: objects and calls where device memory is short.  The card is filled but
for a stated rest (hipMalloc, freed at the end), or the caller's allocator
refuses above a limit; what ran before on that rest has to run, and a refusal
has to be CCT_ENOMEM with nothing left behind.  Results are compared with those
of the same object where memory is plentiful (equal bits where the same launches
run, else the tolerance of the object's own tests)."""

import contextlib
import ctypes as C
import sys
import threading
import time

import numpy as np
import pytest

import cct_inputs as ci
from paper_2607_00981_amd import binding

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def _hip():
    """The libamdhip64 already mapped into this process by libcct."""
    binding.load()
    with open("/proc/self/maps") as f:
        paths = {line.split()[-1] for line in f if "libamdhip64" in line}
    assert paths, "libamdhip64 is not loaded"
    hip = C.CDLL(sorted(paths)[0])
    hip.hipMemGetInfo.argtypes = [C.POINTER(C.c_size_t), C.POINTER(C.c_size_t)]
    hip.hipMalloc.argtypes = [C.POINTER(C.c_void_p), C.c_size_t]
    hip.hipFree.argtypes = [C.c_void_p]
    return hip


def free_bytes():
    fr, tot = C.c_size_t(), C.c_size_t()
    assert _hip().hipMemGetInfo(C.byref(fr), C.byref(tot)) == 0
    return fr.value


@contextlib.contextmanager
def rest_of_card(rest):
    """All but `rest` bytes of the free device memory taken."""
    hip = _hip()
    held = []
    try:
        for _ in range(50):  # memory freed shortly before turns up a little later
            more = free_bytes() - rest
            if more > 8 << 20:
                p = C.c_void_p()
                assert hip.hipMalloc(C.byref(p), more) == 0
                held.append(p)
            time.sleep(0.01)
        say(f"  {free_bytes() / 1e6:.0f} MB left of {rest / 1e6:.0f} asked for")
        yield
    finally:
        for p in held:
            assert hip.hipFree(p) == 0


def _engine(o, v, seed, **kw):
    s = ci.make_system(o, v, 2 * (o + v), seed, sigma=0.1)
    t2 = ci.random_amplitudes(o, v, seed, 0.0, 0.05, 0.0, triples=False)[1]
    eng = binding.Engine(o, v, s["naux"], **kw)
    eng.set_fock(s["f"])
    eng.set_eri_df(s["B"])
    eng.set_amplitudes(np.zeros((o, v)), t2, ci.random_t3_packed(o, v, seed + 1, 0.03))
    return eng


def test_a_refused_object_leaves_no_error_pending():
    say("[memory limits] slab of 8 TB refused, then an iteration")
    with _engine(3, 8, 1) as eng:
        with pytest.raises(binding.CCTError) as err:
            binding.Slab(1, 1000, 1_000_000, 0, 1)
        assert err.value.code == binding.CCT_ENOMEM
        eng.update()


def _slab_inputs(o, v, naux, count, seed):
    rng = np.random.default_rng(seed)
    s = ci.make_system(o, v, naux, seed, sigma=0.1)
    t2 = ci.random_amplitudes(o, v, seed, 0.03, 0.03, 0.0, triples=False)[1]
    return (s["B"], t2, rng.normal(0, 0.1, (v, v)), rng.normal(0, 0.1, (o, v, v, v)),
            rng.normal(0, 0.1, (v, o, o, o)), ci.random_t3_packed(o, v, seed + 1, 0.02)[:count])


def _slab_residual(inputs, o, v, naux, count, **kw):
    with binding.Slab(o, v, naux, 0, count, **kw) as sl:
        sl.set_intermediates(*inputs[:-1])
        sl.set_t3(inputs[-1])
        return sl.residual()[0]


def test_slab_panel_narrows_when_memory_is_short():
    """The whole of W is 680 MB here, eight rows of it 57 MB."""
    o, v, naux, count = 2, 96, 20, 1
    say(f"[memory limits] slab panel o={o} v={v}")
    inputs = _slab_inputs(o, v, naux, count, 5)
    want = _slab_residual(inputs, o, v, naux, count, opts={"panel": 8})
    with rest_of_card(400 << 20):
        got = _slab_residual(inputs, o, v, naux, count)
    assert np.array_equal(got, want)


def _q_bound(o, v):
    """Bytes that cct_energy_q may take, as include/cct.h has it."""
    per = 28 * v ** 4 + 48 * 4096 * ((v + 7) // 8) ** 4 if v % 2 == 0 and o <= 16 else 52 * v ** 4
    return max(8 * ((o + v) ** 4 + o ** 2 * v ** 4 + o ** 3 * v ** 3 + 2 * o ** 4 * v ** 2 + per), 128 << 20)


@pytest.mark.parametrize("o,v", [(10, 24), (8, 32), (5, 33), (17, 6)])
def test_q_takes_no_more_than_documented(o, v):
    say(f"[memory limits] (Q) o={o} v={v}, bound {_q_bound(o, v) / 1e6:.0f} MB")
    with _engine(o, v, 7) as eng:
        before = free_bytes()
        e = eng.energy_q()
        kept = before - free_bytes()
        say(f"  {kept / 1e6:.0f} MB kept")
        assert kept <= _q_bound(o, v) + (16 << 20)
        assert eng.energy_q() == e


def test_q_runs_where_little_more_than_its_need_is_free():
    o, v = 10, 24
    say(f"[memory limits] (Q) o={o} v={v} on a nearly full card")
    with _engine(o, v, 7) as eng:
        with rest_of_card(_q_bound(o, v) + (600 << 20)):
            e, tasks = eng.energy_q(tasks=True)
    with _engine(o, v, 7) as eng:
        e2, tasks2 = eng.energy_q(tasks=True)
    assert e == e2 and np.array_equal(tasks, tasks2)


class LimitedAllocator:
    """The caller's allocator over hipMalloc: refuses above `limit` bytes in all."""

    def __init__(self):
        self.hip, self.live, self.limit, self.most = _hip(), {}, None, 0

    def alloc(self, nbytes):
        if self.limit is not None and sum(self.live.values()) + nbytes > self.limit:
            return None
        p = C.c_void_p()
        if self.hip.hipMalloc(C.byref(p), nbytes) != 0:
            return None
        self.live[p.value] = nbytes
        self.most = max(self.most, sum(self.live.values()))
        return p.value

    def free(self, ptr):
        del self.live[ptr]
        self.hip.hipFree(C.c_void_p(ptr))

    def pair(self):
        return self.alloc, self.free


@pytest.mark.parametrize("o,v", [(6, 20), (5, 13)])
def test_q_takes_fewer_tasks_at_a_time_where_memory_is_refused(o, v):
    say(f"[memory limits] (Q) o={o} v={v} under an allocator's limit")
    al = LimitedAllocator()
    with _engine(o, v, 9, allocator=al.pair()) as eng:
        own = sum(al.live.values())
        want = eng.energy_q(tasks=True)
        full = al.most - own
        least = None
        for part in (0.9, 0.7, 0.5, 0.3, 0.1, 0.02):
            al.limit = own + int(part * full)
            try:
                e, tasks = eng.energy_q(tasks=True)
            except binding.CCTError as err:
                assert err.code == binding.CCT_ENOMEM
                assert sum(al.live.values()) == own
                continue
            assert e == want[0] and np.array_equal(tasks, want[1])
            least = part
        say(f"  {full / 1e6:.1f} MB by itself, down to {least} of it")
        assert least is not None and least <= 0.7
        al.limit = None
        assert eng.energy_q(tasks=True)[0] == want[0]
    assert not al.live


def _alone(o, v, seed, f):
    with _engine(o, v, seed) as eng:
        return f(eng)


def test_q_memory_is_one_block_and_goes_with_its_last_user():
    o, v = 8, 32
    say(f"[memory limits] (Q) o={o} v={v} on three contexts")
    engines = [_engine(o, v, 20 + k) for k in range(3)]
    try:
        before = free_bytes()
        energies = [e.energy_q() for e in engines]
        assert before - free_bytes() <= _q_bound(o, v) + (16 << 20)
        engines.pop(0).close()
        assert [e.energy_q() for e in engines] == energies[1:]
    finally:
        for e in engines:
            e.close()
    for k in range(3):
        assert _alone(o, v, 20 + k, lambda e: e.energy_q()) == energies[k]


def test_q_memory_is_given_back_on_destroy():
    say("[memory limits] (Q) memory after destroy")
    _engine(8, 32, 20).close()
    time.sleep(0.5)
    before = free_bytes()
    with _engine(8, 32, 20) as eng:
        eng.energy_q()
    for _ in range(100):
        if before - free_bytes() <= 16 << 20:
            break
        time.sleep(0.05)
    assert before - free_bytes() <= 16 << 20


def test_virtual_tuple_order_takes_the_kept_memory():
    """o = 10, v = 24, block 8: 1.5 GB with its margin; (Q) keeps 0.68 of what is free."""
    o, v, block = 10, 24, 8
    say(f"[memory limits] both orders o={o} v={v} on a nearly full card")
    tasks = [0, 3, 14]
    want = _alone(o, v, 7, lambda e: e.energy_q_abc(block, tasks)["e_tasks"])
    with _engine(o, v, 7) as eng:
        eng.energy_q()
        with rest_of_card(1100 << 20):
            got = eng.energy_q_abc(block, tasks)["e_tasks"]
    assert np.array_equal(got, want)


def test_new_objects_take_the_kept_memory():
    say("[memory limits] a quadruples object beside kept (Q) memory")
    with _engine(8, 32, 20) as eng:
        eng.energy_q()
        with rest_of_card(300 << 20):
            with binding.Quad(4, 30):  # 35 blocks of 6.5 MB, three times: 0.7 GB
                pass


def test_q_after_new_amplitudes_equals_a_fresh_context():
    o, v = 4, 20
    say("[memory limits] (Q) twice on a context, other amplitudes")
    rng = np.random.default_rng(3)
    t2 = rng.normal(0, 0.05, (o, o, v, v))
    t2 = 0.5 * (t2 + t2.transpose(1, 0, 3, 2))
    t3p = ci.random_t3_packed(o, v, 77, 0.03)

    def second(eng, first):
        if first:
            eng.energy_q()
        eng.set_amplitudes(np.zeros((o, v)), t2, t3p)
        return eng.energy_q(tasks=True)

    e1, x1 = _alone(o, v, 30, lambda e: second(e, True))
    e2, x2 = _alone(o, v, 30, lambda e: second(e, False))
    assert e1 == e2 and np.array_equal(x1, x2)


def test_q_on_two_threads():
    say("[memory limits] (Q) on two contexts, a thread each")
    sizes = [(5, 20, 40), (4, 25, 41)]
    want = [_alone(*s, lambda e: e.energy_q(tasks=True)[1]) for s in sizes]
    got = [[], []]

    def work(k):
        with _engine(*sizes[k]) as eng:
            for _ in range(20):
                got[k].append(eng.energy_q(tasks=True)[1])

    ts = [threading.Thread(target=work, args=(k,)) for k in range(2)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    for k in range(2):
        assert len(got[k]) == 20
        for x in got[k]:
            assert np.array_equal(x, want[k])


def _slab_bytes_unrelabelled(o, v, naux, count):
    """An FP64 slab's buffers with T3 read in place and eight rows of W, exactly
    (rows of W padded to 16, o to even), and 256 kB for the small ones."""
    v2, op = v * v, (o + 1) // 2 * 2
    rows = min(v, 8) * v * ((v2 + 15) // 16 * 16)
    n = v2 * naux + 3 * v2 * o * o + v2 + o * v ** 3 + v * o * o * op + 2 * count * v ** 3 + rows
    return 8 * (n + 64 * count) + 6 * count * 208 + (256 << 10)


# v^2 odd, even without whole K tiles, and of whole K tiles
@pytest.mark.parametrize("o,v,count", [(5, 33, 35), (5, 30, 30), (4, 32, 20), (1, 1, 1), (3, 47, 9)])
def test_slab_relabels_in_parts_where_memory_is_short(o, v, count):
    say(f"[memory limits] FP64 slab o={o} v={v} count={count} under an allocator's limit")
    naux = 2 * v
    inputs = _slab_inputs(o, v, naux, count, 11)
    want = _slab_residual(inputs, o, v, naux, count)
    least = _slab_bytes_unrelabelled(o, v, naux, count)
    block = 3 * v * ((v * v + 15) // 16 * 16) * 8
    full = LimitedAllocator()
    _slab_residual(inputs, o, v, naux, count, allocator=full.pair())
    for limit in (full.most, full.most - 1, least + count // 2 * block, least + 2 * block, least + block, least):
        al = LimitedAllocator()
        al.limit = limit
        got = _slab_residual(inputs, o, v, naux, count, allocator=al.pair())
        assert np.abs(got - want).max() <= 1e-11 * max(float(np.abs(want).max()), 1e-300)
        assert not al.live
        say(f"  {limit / 1e6:.2f} MB allowed, {al.most / 1e6:.2f} taken")


def test_slab_copies_of_t3_are_bounded():
    o, v, count = 9, 111, 165
    say(f"[memory limits] FP64 slab o={o} v={v} count={count}: 5.3 GB of padded copies")
    al = LimitedAllocator()
    with binding.Slab(o, v, 20, 0, count, allocator=al.pair()):
        assert al.most <= _slab_bytes_unrelabelled(o, v, 20, count) + (5 << 30)


@pytest.mark.parametrize("o,v", [(50, 25), (1, 9)])
def test_the_smallest_workspace_holds_the_feedback(o, v):
    say(f"[memory limits] feedback in the smallest workspace o={o} v={v}")
    s = ci.make_system(o, v, 12, 5, sigma=0.02)
    got = []
    for gb in (1e-6, 2.0):
        with binding.Engine(o, v, 12, opts={"diis": False, "workspace_gb": gb}) as eng:
            eng.set_fock(s["f"])
            eng.set_eri_df(s["B"])
            eng.init_mp2()
            eng.update()
            got.append(eng.residual(want_r3=False))
    for a, b in zip(got[0], got[1]):
        if a is not None:
            assert np.abs(a - b).max() <= 1e-11 * np.abs(b).max()
