"""The LDS layouts that the planner falls back to, against the oracle:
records halved or cut to one per thread, a winner table of 256 entries beside
more records, no learned-occurrence bits, the program that no layout holds;
tables and probe windows that a round overflows; and the least layout, which a
large batch takes.

Atoms that head no rule cost a variable each and nothing in the search, so a
small program reaches every size.  LDS bytes of a workgroup: 56 per record, 16
per table entry, 4 per thread, 512, and bits for V + 1 variables (two each), A + 1
atoms and A + Rh + 1 learned occurrences, in words.
"""
import numpy as np
import pytest

import aspgen
import oracle
from parity import STATUS, assert_same_stats

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1909_01786_amd as P
    P.lib()
    return P


def _rules_of(p):
    return [(int(h), [int(x) for x in p.body_lits[p.body_off[r]:p.body_off[r + 1]]])
            for r, h in enumerate(p.head)]


def _padded(atoms, seed=0):
    """A 200-atom program that learns, a choice that implies 300 atoms at once,
    and atoms without rules up to `atoms`."""
    p = aspgen.single_random(1000 + seed)
    n = p.n_atoms
    rules = _rules_of(p) + [(n + 1, [-(n + 2)]), (n + 2, [-(n + 1)])]
    rules += [(n + 3 + i, [n + 1]) for i in range(300)] + [(n + 303 + i, [n + 2]) for i in range(300)]
    return aspgen.from_rules(atoms, rules, f"padded{atoms}")


def _same(P, prog, threads, limit=-1, **kw):
    rc, m, st = oracle.solve(prog, limits=oracle.make_limits(limit), **kw)
    g = P.Program(prog, **kw)
    layout = P.Batch([g], threads=threads).launch_lds()[0]
    g.bind("cuda", threads=threads)
    grc, gm, gst = g.solve(P.limits(limit, 60000))
    assert grc == STATUS[rc], prog.name
    assert_same_stats(st, gst, (prog.name, threads))
    if rc == oracle.SAT:
        assert np.array_equal(gm, m)
    words = lambda bits: 4 * ((bits + 31) // 32)
    V, A = g.n_vars, prog.n_atoms
    base = words(2 * (V + 1)) + words(A + 1) + 512 + 4 * threads + 56 * layout[2] + 16 * layout[3]
    if kw.get("learning"):
        base += 8 * threads
    return layout[2], layout[3], layout[1] - base >= words(A + 1)


@pytest.mark.parametrize("threads,atoms,learning,layout", [
    (128, 20000, 0, (512, 1024, True)),
    (128, 60000, 0, (1024, 2048, True)),
    (128, 200000, 0, (512, 1024, True)),      # halved
    (128, 240000, 0, (256, 512, True)),       # halved twice
    (256, 240000, 0, (256, 512, True)),
    (128, 290000, 0, (128, 256, True)),       # one per thread
    (128, 350000, 0, (128, 256, False)),      # and no learned-occurrence bits
    (1024, 160000, 0, (1024, 256, True)),     # 256 entries beside all records
    (1024, 220000, 0, (1024, 256, False)),
    (128, 350000, 1, (256, 512, False)),
    (1024, 220000, 1, (1024, 256, False)),
])
def test_fallback_layouts(P, threads, atoms, learning, layout):
    prog = _padded(atoms, seed=5 if atoms >= 200000 else 0)     # SAT, UNSAT
    assert _same(P, prog, threads, learning=learning) == layout


@pytest.mark.parametrize("threads,atoms", [(1024, 270000), (128, 420000)])
def test_beyond_every_layout(P, threads, atoms):
    from paper_1909_01786_amd.binding import AspError
    with pytest.raises(AspError, match="LDS"):
        P.Program(_padded(atoms)).bind("cuda", threads=threads)


def _fanout(n, atoms):
    """x :- not y.  y :- not x.  h_i :- x (i = 1..n).  :- h_1, h_n."""
    rules = [(1, [-2]), (2, [-1])] + [(2 + i, [1]) for i in range(1, n + 1)] + [(0, [3, 2 + n])]
    return aspgen.from_rules(max(atoms, n + 2), rules, f"fanout{n}")


@pytest.mark.parametrize("learning", [0, 1])
@pytest.mark.parametrize("threads", [64, 256])
@pytest.mark.parametrize("n,atoms,table", [(600, 0, 512), (1300, 0, 1024), (2600, 30000, 2048)])
def test_more_variables_than_table_entries(P, n, atoms, table, threads, learning):
    """A round that implies more variables than its winner table has entries:
    the rest go through the global keys and the pending map."""
    assert _same(P, _fanout(n, atoms), threads, learning=learning)[1] == table < n


@pytest.mark.parametrize("copies", [1, 33, 34, 36])
@pytest.mark.parametrize("threads", [64, 256])
def test_full_probe_window(P, copies, threads):
    """One-wave rounds that imply `copies` atoms of one hash bucket, one of
    them twice: from the 33rd on, the probe window is full and the round is left
    to the general one."""
    atoms, bits = 90000, 11                       # 2048 entries above 32767 variables
    x = np.arange(3, atoms + 1, dtype=np.uint64)
    h = ((x * np.uint64(0x9E3779B1)) & np.uint64(0xffffffff)) >> np.uint64(32 - bits)
    bucket = x[h == np.argmax(np.bincount(h.astype(np.int64)))][:copies]
    assert bucket.size == copies
    rules = [(1, [-2]), (2, [-1])] + [(int(a), [1]) for a in bucket] + [(int(bucket[0]), [1])]
    prog = aspgen.from_rules(atoms, rules, f"bucket{copies}")
    assert _same(P, prog, threads)[:2] == (1024, 2048)


@pytest.mark.parametrize("learning", [0, 1])
def test_least_layout_of_a_large_batch(P, learning):
    """3000 programs at once take the least records and table: the same
    results as each alone."""
    progs = [aspgen.single_random(1000 + s) for s in range(3)] + [_fanout(300, 0), _fanout(60, 0)]
    opt = {"learning": learning, "learned_cap_ng": 2048, "learned_cap_lits": 1 << 16}
    gs = [P.Program(p, **opt) for p in progs]
    b = P.Batch([gs[i % 5] for i in range(3000)]).bind("cuda")
    assert all(r[2:] in ((128, 256), (256, 256), (256, 512)) for r in b.launch_lds())
    b.solve(P.limits(300, 60000))
    verd, models, stats = b.results()
    lim = oracle.make_limits(300, 2048, 1 << 16)
    want = [oracle.solve(p, limits=lim, learning=learning) for p in progs]
    for i in range(3000):
        rc, m, st = want[i % 5]
        assert verd[i] == STATUS[rc], i
        assert_same_stats(st, stats[i], i)
        if rc == oracle.SAT:
            assert np.array_equal(models[i], m), i
