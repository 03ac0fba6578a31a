"""The learned Decision's training kernels against the float reference.

asp_scorer_train runs the float scorer's forward and backward passes on the
matrix cores with bfloat16 operands and float32 accumulation; the reference
(oracle/mpnn_train.py) is the same model in float64 with autograd.  Bfloat16
keeps 8 significant bits, so each product carries a relative error up to
2^-8 and the passes through three layers compound it; clamp masks may flip
for the few pre-activations within that error of 0 or 1.  The comparison is
therefore norm-wise per parameter group: relative L2 error at most 0.05 and
cosine at least 0.995, loss within 1%.  Adam moves every parameter with a
non-zero gradient by about lr whatever the gradient's size, so parameters
whose gradient is within bf16 noise of 0 move either way and two runs'
parameters part after the first step; the Adam arithmetic is therefore
checked on the device's own gradient (to float32 rounding), and the
trajectory on the loss curve.
"""
import os

import numpy as np
import pytest
import torch

import aspgen
import oracle
from oracle import mpnn_train as T
from parity import STATUS

pytestmark = pytest.mark.gpu

torch.set_num_threads(8)


@pytest.fixture(scope="module")
def P():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    import paper_1909_01786_amd as P
    P.lib()
    return P


def _setup(seed):
    progs = [aspgen.tiny_program(20 + seed, 10, 16), aspgen.single_random(1001 + seed),
             aspgen.batch_hamiltonian(seed + 3)]
    rng = np.random.default_rng(seed)
    labels = [np.where(rng.random(p.n_atoms) < 0.7, rng.integers(0, 2, p.n_atoms), -1).astype(np.float32)
              for p in progs]
    w = aspgen.mpnn_weights(seed, spread=90)
    for k in ("ev", "ec", "bc", "bv"):
        w[k] = w[k] // 4
    return progs, labels, w


@pytest.mark.parametrize("seed", [0, 1])
def test_gradient_pass_matches_reference(P, seed):
    from paper_1909_01786_amd import binding as B
    progs, labels, w = _setup(seed)
    vec = B.dequantize(w)
    gp = [P.Program(p) for p in progs]
    _, loss, grad = B.train_scorer(gp, labels, vec, steps=0)
    ref_loss, ref_grad = T.loss_and_grad(vec.astype(np.float64), progs, labels)
    assert abs(loss[0] - ref_loss) <= 0.01 * abs(ref_loss), (loss[0], ref_loss)
    gd, rd = T.split(grad.astype(np.float64)), T.split(ref_grad)
    for name, _ in T.layout():
        a, b = gd[name].reshape(-1), rd[name].reshape(-1)
        nb = np.linalg.norm(b)
        if nb < 1e-9:
            assert np.linalg.norm(a) < 1e-6, name
            continue
        rel = np.linalg.norm(a - b) / nb
        cos = float(a @ b) / (np.linalg.norm(a) * nb + 1e-30)
        assert rel <= 0.05 and cos >= 0.995, (name, rel, cos)


def test_adam_steps_match_reference(P):
    """One step from the device's own gradient is Adam to float32 rounding;
    ten steps follow the reference's loss curve within 2%."""
    from paper_1909_01786_amd import binding as B
    progs, labels, w = _setup(2)
    vec = B.dequantize(w)
    gp = [P.Program(p) for p in progs]
    lr, steps = 2e-3, 10
    one, _, g1 = B.train_scorer(gp, labels, vec, steps=1, lr=lr)
    want, _ = T.adam(vec.astype(np.float64), lambda v: (0.0, g1.astype(np.float64)), 1, lr)
    assert np.abs(one - want).max() <= 1e-6, float(np.abs(one - want).max())
    _, losses, _ = B.train_scorer(gp, labels, vec, steps=steps, lr=lr)
    _, ref_losses = T.adam(vec.astype(np.float64),
                           lambda v: T.loss_and_grad(v, progs, labels), steps, lr)
    assert np.allclose(losses, ref_losses, rtol=0.02), (losses, ref_losses)


def test_training_lowers_the_loss_and_quantizes(P):
    """Labels the network can represent -- an atom is 1 when its occurrence
    count is at least the program's median, which the degree features carry
    -- fall from about ln 2 within 40 steps; the quantized result is a valid
    weight set the integer scorer and the search accept."""
    from paper_1909_01786_amd import binding as B
    progs, _, w = _setup(3)
    labels = []
    for p in progs:
        occ = oracle.Solver(p).occ()[1:].astype(np.float64)
        labels.append((occ >= np.median(occ)).astype(np.float32))
    gp = [P.Program(p) for p in progs]
    vec, losses, _ = B.train_scorer(gp, labels, B.dequantize(w), steps=40, lr=5e-3)
    assert losses[-1] < 0.85 * losses[0] and losses[-1] < 0.6, (losses[0], losses[-1])
    codes = B.quantize(vec)
    g = P.Program(progs[1], decision=P.DECISION_SCORE).bind("cuda")
    sc = g.score(codes)
    from oracle import mpnn
    assert np.array_equal(sc[1:], mpnn.scores(codes, progs[1])[1:])
    rc, m, st = g.solve(P.limits(2000, 60000))
    orc, om, ost = oracle.solve(progs[1], scores=sc, fallback_after=10,
                                limits=oracle.make_limits(2000))
    assert rc == STATUS[orc] and st["trace_hash"] == ost["trace_hash"]


def test_batch_learned_nogoods_are_the_oracles(P):
    """The conflict traces read back from a batch (asp_batch_learned) are
    the oracle's learned nogoods, nogood for nogood."""
    progs = [aspgen.batch_random(i, a_lo=100, a_hi=400) for i in range(12)]
    gp = [P.Program(p, learned_cap_ng=4096, learned_cap_lits=1 << 18) for p in progs]
    b = P.Batch(gp).bind("cuda")
    b.solve(P.limits(300, 60000))
    torch.cuda.synchronize()
    for i, prog in enumerate(progs):
        s = oracle.Solver(prog)
        s.run(oracle.make_limits(300, 4096, 1 << 18))
        st = s.state()
        n0 = st.n_static
        base = int(st.ng_off[n0])
        o_off = (st.ng_off[n0:] - base).astype(np.int32)
        o_lits = st.ng_lits[base:].astype(np.int32)
        off, lits = b.learned(i)
        assert np.array_equal(off, o_off) and np.array_equal(lits, o_lits), i


@pytest.mark.parametrize("atoms,rules,copies", [(4, 4, 1), (16, 16, 2), (13, 17, 2), (16, 16, 4),
                                                (60, 200, 8), (700, 2100, 4)])
def test_gradient_over_row_tiles(P, atoms, rules, copies):
    """The mean loss of a program's copies, and its gradient, are the
    program's own: the copies' rows fall at other places of the 64-row tiles
    (64 variable rows exactly, one more, one less, many tiles).  A copy count
    that is a power of two scales every term exactly, so what differs is the
    order of the float32 sums over rows: for n rows, about sqrt(n) 2^-24 of
    the terms' size, below 1e-4 here even after some cancellation.  Two runs
    give the same bits."""
    from paper_1909_01786_amd import binding as B
    rng = np.random.default_rng(atoms)
    prog = aspgen.random_program(np.random.default_rng(rules), atoms, rules, 0, 3)
    lab = rng.integers(0, 2, atoms).astype(np.float32)
    w = aspgen.mpnn_weights(atoms, spread=40)
    for k in ("ev", "ec", "bc", "bv"):
        w[k] = w[k] // 8
    vec = B.dequantize(w)
    gp = [P.Program(prog) for _ in range(copies)]
    _, l1, g1 = B.train_scorer(gp[:1], [lab], vec, steps=0)
    _, ln, gn = B.train_scorer(gp, [lab] * copies, vec, steps=0)
    _, lm, gm = B.train_scorer(gp, [lab] * copies, vec, steps=0)
    assert np.array_equal(gn, gm) and np.array_equal(ln, lm)
    assert abs(l1[0] - ln[0]) <= 1e-5 * abs(l1[0])
    a, b = T.split(gn.astype(np.float64)), T.split(g1.astype(np.float64))
    for name, _ in T.layout():
        d, n = np.linalg.norm(a[name] - b[name]), np.linalg.norm(b[name])
        assert d <= 1e-4 * n + 1e-9, (name, d, n)
    # against float64 arithmetic with the same bfloat16 operands; float32
    # sums move a product by about 2^-20 and now and then an operand across
    # a rounding boundary (2^-9 of it), a few 1e-5 of each term
    rl, rg = _rounded_gradient(vec, prog, lab)
    assert abs(l1[0] - rl) <= 1e-4 * abs(rl)
    assert np.linalg.norm(g1 - rg) <= 1e-2 * np.linalg.norm(rg)


def _rounded_gradient(vec, prog, lab):
    """Loss and gradient in float64 with the operands of every 64-wide
    product -- activations, matrices, backward derivatives -- rounded to
    bfloat16, the derivatives written out by hand."""
    W = {k: v for k, v in T.split(torch.tensor(vec.astype(np.float64))).items()}
    g, xv, xc, deg = T.graph_tensors(prog)
    xv, xc = torch.tensor(xv), torch.tensor(xc)
    v, c, pos = torch.tensor(g.var - 1), torch.tensor(g.ng_of_lit), torch.tensor(g.pos)
    cs = torch.tensor(2.0 ** -T.log2ceil(g.lens).astype(np.float64))[:, None]
    vs = torch.tensor(2.0 ** -T.log2ceil(deg).astype(np.float64))[:, None]

    def R(x):
        return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)

    def edges(n, dst, src, x, m):
        return torch.zeros((n, 64), dtype=torch.float64).index_add(0, dst[m], x[src[m]])

    def mask(d, a):
        return torch.where((a > 0) & (a < 1), d, torch.zeros_like(d))
    L = 3
    av, ac = [torch.clamp(xv @ W["Ev"] / 4 + W["ev"], 0, 1)], [torch.clamp(xc @ W["Ec"] / 4 + W["ec"], 0, 1)]
    for l in range(L):
        e = edges(g.n, c, v, R(av[l]) @ R(W["P"][l]), pos) + edges(g.n, c, v, R(av[l]) @ R(W["N"][l]), ~pos)
        ac.append(torch.clamp((R(ac[l]) @ R(W["S"][l]) + cs * e) / 4 + W["bc"][l], 0, 1))
        e = edges(g.V, v, c, R(ac[l + 1]) @ R(W["Q"][l]), pos) + \
            edges(g.V, v, c, R(ac[l + 1]) @ R(W["R"][l]), ~pos)
        av.append(torch.clamp((R(av[l]) @ R(W["T"][l]) + vs * e) / 4 + W["bv"][l], 0, 1))
    y = torch.tensor(lab.astype(np.float64))
    A = y.shape[0]
    z = av[L][:A] @ W["wo"] + W["bo"]
    loss = torch.nn.functional.binary_cross_entropy_with_logits(z, y)
    dz = (torch.sigmoid(z) - y) / A
    G = {k: torch.zeros_like(x) for k, x in W.items()}
    G["wo"], G["bo"] = dz @ av[L][:A], dz.sum()
    dv, dc = torch.zeros_like(av[L]), torch.zeros_like(ac[L])
    dv[:A] = dz[:, None] * W["wo"]
    for l in reversed(range(L)):
        m = mask(dv, av[l + 1])
        G["bv"][l], gv = m.sum(0), m / 4
        gq, gr = edges(g.n, c, v, vs * gv, pos), edges(g.n, c, v, vs * gv, ~pos)
        G["T"][l] = R(av[l]).T @ R(gv)
        G["Q"][l], G["R"][l] = R(ac[l + 1]).T @ R(gq), R(ac[l + 1]).T @ R(gr)
        m = mask(dc + R(gq) @ R(W["Q"][l]).T + R(gr) @ R(W["R"][l]).T, ac[l + 1])
        G["bc"][l], gc = m.sum(0), m / 4
        gp, gn = edges(g.V, v, c, cs * gc, pos), edges(g.V, v, c, cs * gc, ~pos)
        G["S"][l] = R(ac[l]).T @ R(gc)
        G["P"][l], G["N"][l] = R(av[l]).T @ R(gp), R(av[l]).T @ R(gn)
        dv = R(gv) @ R(W["T"][l]).T + R(gp) @ R(W["P"][l]).T + R(gn) @ R(W["N"][l]).T
        dc = R(gc) @ R(W["S"][l]).T
    for name, x, d, a in (("v", xv, dv, av[0]), ("c", xc, dc, ac[0])):
        m = mask(d, a)
        G["e" + name], G["E" + name] = m.sum(0), x.T @ (m / 4)
    return float(loss), np.concatenate([G[k].numpy().reshape(-1) for k, _ in T.layout()])
