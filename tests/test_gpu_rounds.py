"""Runs of one-wave rounds at their edges, against the oracle.

A run takes the rounds whose visits fit one wave (two per lane) and leaves
the others to the general round; single steps never start one (the frontier
records are in LDS only between the steps of one launch), so each program is
run from the start for n steps at once and the whole state is compared.
"""
import numpy as np
import pytest
import torch  # noqa: F401  (loads the HIP runtime the library uses)

import aspgen
import oracle
from parity import STATUS, assert_same_state, assert_same_stats, to_lib_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1909_01786_amd as P
    P.lib()
    return P


def fan(width, per_atom):
    """`width` atoms that all follow from one choice, each with `per_atom`
    rules (support nogoods of per_atom + 1 literals), and a second layer
    needing two of them, so that one round implies many variables, some of
    them twice."""
    rules = [(1, [-2]), (2, [-1])]
    for i in range(width):
        a = 3 + i
        rules += [(a, [1])] + [(a, [2, -(3 + (i + 1 + j) % width)]) for j in range(per_atom - 1)]
        rules.append((3 + width + i // 2, [a, 3 + (i + 1) % width]))
    return aspgen.from_rules(3 + width + width // 2, rules, f"fan{width}_{per_atom}")


def _compare(P, prog, n, threads, **kw):
    o = oracle.Solver(prog, learning=kw.get("learning", 0))
    for _ in range(n):
        if o.next_step() == oracle.ST_DONE:
            return False
        o.step()
    g = P.Program(prog, **kw).bind("cuda", threads=threads)
    rc, st = g.run_steps(n, P.limits(-1, 30000))
    s = o.state()
    assert rc == STATUS[s.status], (prog.name, n)
    if s.status == oracle.RUNNING:
        assert_same_state(s, g.export_state(), (prog.name, n))
    assert_same_stats(o.stats(), st, (prog.name, n))
    return True


@pytest.mark.parametrize("threads", [64, 128, 256])
@pytest.mark.parametrize("width,per_atom", [(1, 1), (20, 3), (21, 4), (22, 7), (31, 2), (32, 8),
                                            (43, 1), (63, 1), (64, 1), (65, 3), (127, 1), (129, 2),
                                            (16, 9), (9, 17)])
def test_round_edges(P, width, per_atom, threads):
    """Frontiers and visit counts around one and two per lane, and nogoods of
    2 to 18 literals, after every number of steps up to 40."""
    prog = fan(width, per_atom)
    for n in range(1, 41):
        if not _compare(P, prog, n, threads):
            break


@pytest.mark.parametrize("threads", [64, 256])
@pytest.mark.parametrize("width,per_atom", [(255, 1), (256, 1), (257, 1), (511, 2), (512, 2),
                                            (513, 2), (1023, 10), (1024, 10), (1025, 10)])
def test_record_edges(P, width, per_atom, threads):
    """Rounds that imply as many variables as LDS holds records for (256 below
    4096 variables, 512 below 32768, then 1024), one fewer, and one more."""
    prog = fan(width, per_atom)
    for n in (3, 4, 5, 6, 7, 8, 12, 40):
        if not _compare(P, prog, n, threads):
            break


@pytest.mark.parametrize("learning", [0, 1])
@pytest.mark.parametrize("seed", range(6))
def test_learned_visits(P, seed, learning):
    """Searches with learned nogoods: the state after 50, 200, 400 steps."""
    for prog in (aspgen.single_random(1000 + seed), aspgen.batch_hamiltonian(seed, n_lo=20, n_hi=30)):
        for n in (50, 200, 400):
            _compare(P, prog, n, 128, learning=learning)


@pytest.mark.parametrize("threads", [64, 128, 256])
@pytest.mark.parametrize("decision", [0, 2, 3])
@pytest.mark.parametrize("lookahead", [2, 8])
def test_ordered_candidates(P, lookahead, decision, threads):
    """The lookahead's candidates, taken one after another from the rules'
    order: neighbours in one 64-position chunk (a colouring's first
    decisions), spread over many chunks, and fewer than asked for."""
    for prog in (aspgen.gnp_coloring(1, 40, 3.0), fan(5, 2), aspgen.batch_random(3, a_lo=200, a_hi=400)):
        g = P.Program(prog, lookahead=lookahead, decision=decision).bind("cuda", threads=threads)
        rc, m, st = g.solve(P.limits(60, 30000))
        orc, om, ost = oracle.solve(prog, lookahead=lookahead, decision=decision,
                                    limits=oracle.make_limits(60))
        assert rc == STATUS[orc], prog.name
        assert_same_stats(ost, st, prog.name)


@pytest.mark.parametrize("steps", [2, 40, 300])
@pytest.mark.parametrize("seed", range(4))
def test_import_ignores_variable_0(P, seed, steps):
    """The arrays of an imported state have an entry 0 that belongs to no
    variable: whatever a caller leaves there, the search goes on the same."""
    prog = aspgen.single_random(1000 + seed)
    o = oracle.Solver(prog)
    while o.stats()["decisions"] < 3:
        o.step()
    st = to_lib_state(o.state(), o.stats())
    st.val[0], st.deps[0] = 1, np.uint64(2 ** 64 - 1)
    g = P.Program(prog).bind("cuda", threads=128)
    g.import_state(st)
    for _ in range(steps):
        if o.next_step() == oracle.ST_DONE:
            break
        o.step()
    rc, gst = g.run_steps(steps, P.limits(-1, 30000))
    s = o.state()
    assert rc == STATUS[s.status]
    if s.status == oracle.RUNNING:
        assert_same_state(s, g.export_state(), (seed, steps))
    assert_same_stats(o.stats(), gst, (seed, steps))
