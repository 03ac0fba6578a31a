"""How many searches of a batch a CU holds at once: the LDS records of a
launch class trade a round's latency for residency, so a batch of many
searches must not get fewer per CU than the least records allow, and a batch
of few gets every record it can use.  The plan needs no GPU.
"""
import numpy as np
import pytest

import aspgen

CUS, CU_LDS, STATIC = 256, 160 * 1024, 512


@pytest.fixture(scope="module")
def P():
    import paper_1909_01786_amd as P
    P.lib()
    return P


def _facts(n_vars):
    """A program of n_vars variables: one fact per atom (four variables each)."""
    n = n_vars // 4
    return aspgen.from_rules(n, [(a, []) for a in range(1, n + 1)], f"facts{n}")


def _check(batch, sizes, waves):
    """Every class against the least records (one per thread, 128 at least)
    and table (256 entries); sizes: the programs' variables.  Fewer searches a
    CU than with the least are sound only where all run at once, or where all
    of them, by their variables, take 0.7 of the time of the largest sixteenth."""
    info, order = batch.launch_info()
    rows = batch.launch_lds()
    need = weighted = 0.0
    fewer = []
    for (first, count, threads, _), (held, lds, rec, tab) in zip(info, rows):
        least = max(threads, 128)
        assert rec in (128, 256, 512, 1024) and rec >= least
        assert 256 <= tab <= 2 * rec and lds <= CU_LDS - 1024
        slots = max(1, waves * 64 // threads)
        assert held == max(1, min(slots, CU_LDS // (lds + STATIC)))
        low = lds - 56 * (rec - least) - 16 * (tab - 256)
        fewer.append(held < max(1, min(slots, CU_LDS // (low + STATIC))))
        need += count / held
        weighted += sum(sizes[i] for i in order[first:first + count]) / held
    largest = np.sort(sizes)[-(-(-len(sizes) // 16)):].mean()
    assert need <= CUS or weighted <= 0.7 * CUS * largest or not any(fewer), (need, weighted, rows)
    return rows


@pytest.mark.parametrize("n,threads,held", [(200, 256, 1), (256, 128, 1), (300, 128, 2), (452, 256, 2), (600, 128, 4),
                                            (4000, 256, 4), (4000, 128, 4)])
def test_equal_large_programs(P, n, threads, held):
    """n programs of 44 thousand variables: at least `held` a CU, and one
    (every record) where each gets a CU of its own."""
    g = P.Program(_facts(44000))
    b = P.Batch([g] * n, threads=threads)
    (per_cu, _, rec, tab), = _check(b, [g.n_vars] * n, 16)
    assert per_cu >= held
    if n <= CUS:
        assert (rec, tab) == (1024, 2048)


@pytest.mark.parametrize("classes,cth", [(4, (256, 128, 128, 128)), (4, (128,) * 4), (3, (256, 128, 128)),
                                         (2, (256, 128)), (1, (128,))])
@pytest.mark.parametrize("scale,full", [(1, False), (16, True)])
def test_uneven_batch(P, classes, cth, scale, full):
    """4096 programs in the proportions of a log-uniform batch of 100..5000
    atoms hold as many searches a CU as with the least records; 256 of them
    get every record."""
    gs = [P.Program(_facts(v)) for v in (63700, 46000, 32700, 24000, 16300, 9000, 4090, 1500)]
    progs = [g for g, n in zip(gs, (52, 400, 119, 600, 507, 1000, 418, 1000)) for _ in range(n // scale)]
    b = P.Batch(progs, threads=cth[-1], classes=classes, class_threads=list(cth))
    rows = _check(b, [g.n_vars for g in progs], 16)
    if full:
        assert rows[0][2] == 1024
    else:
        assert rows[0][0] >= 3 and all(r[0] >= 6 for r in rows[1:])


@pytest.mark.parametrize("seed", range(12))
def test_residency_rule(P, seed):
    """Random mixes over every width, Learning step and search mode."""
    rng = np.random.default_rng(seed)
    mode = [{}, {"learning": 1}, {"max_models": 4}, {"learn_conflicts": 4}, {"lookahead": 4}][seed % 5]
    gs = [P.Program(_facts(int(v)), **mode) for v in np.exp(rng.uniform(np.log(40), np.log(120000), 5))]
    for _ in range(20):
        progs = [gs[i] for i in rng.integers(0, 5, int(np.exp(rng.uniform(0, np.log(5000)))))]
        cth = [int(t) for t in rng.choice([64, 128, 256, 512, 1024], 4)]
        classes = int(rng.integers(1, 5))
        b = P.Batch(progs, threads=cth[-1], classes=classes, class_threads=cth)
        _check(b, [g.n_vars for g in progs], 12 if mode else 16)


@pytest.mark.parametrize("threads", [64, 128, 256, 1024])
@pytest.mark.parametrize("n", [1, 3000])
def test_wide_deps_take_the_least(P, n, threads):
    """Searches with Deps of several words have one layout."""
    g = P.Program(_facts(44000), W=2)
    (held, lds, rec, tab), = _check(P.Batch([g] * n, threads=threads), [g.n_vars] * n, 16)
    assert (rec, tab) == (max(threads, 128), 256)
