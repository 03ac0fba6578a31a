"""The work a user has this library do, as a list of timed cases.

Every case is one pass through the Python binding of libasp on seeded
synthetic programs of the families the library's own benchmark, tests and
training script use: uniform random normal programs, 3-colourings of G(n, p),
and Hamiltonian-cycle programs.  A case's "kind" is the entry point:

* ``solve``  -- ``Program.solve``: one ground program to a verdict, or to a
  conflict budget (a user's single query);
* ``batch``  -- ``Batch.solve`` as a HIP-graph replay and ``Batch.results``: many
  programs at once, in one of the search modes;
* ``learned`` -- ``Batch.score`` and the score-driven search after it;
* ``score``  -- ``Batch.score`` alone, with the atom scores read back;
* ``train``  -- ``train_scorer``: gradient pass (``steps`` 0) or Adam steps.

The searches return whole numbers and bytes (verdicts, answer sets, counters,
trace hashes) and the scorer integer codes; only training computes floating
point results, so only it has an ``exact`` form.
"""
from concurrent.futures import ThreadPoolExecutor
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_1909_01786_amd as P
from paper_1909_01786_amd import binding as B

COUNTERS = ("rounds", "visits", "literal_checks", "propagations", "decisions", "conflicts",
            "learned", "learned_len", "gate_failures", "completes", "trace_hash", "models",
            "restarts", "exhausted")

# Options of each search mode of a batch (the benchmark's legs).
MODES = {
    "plain": {},
    "jw": {"decision": P.DECISION_JW},
    "activity": {"decision": P.DECISION_ACTIVITY},
    "res": {"learning": P.LEARN_RES},
    "multi": {"learn_conflicts": 4},
    "enum": {"max_models": 16},
    "restart": {"restart_every": 64},
    "lookahead": {"lookahead": 4},
}

# Learned store of a budgeted search: the training script's.
STORE = {"learned_cap_ng": 4096, "learned_cap_lits": 1 << 18}


def listed():
    return [
        # the smallest query there is: a handful of rules, where launch,
        # set-up and read-back are everything
        {"name": "solve_tiny", "kind": "solve", "family": "random", "atoms": 20, "ratio": 2.5,
         "kmin": 0, "kmax": 4, "budget": -1, "W": 1},
        # an ordinary single query: the 200-atom, 600-rule program, to its verdict
        {"name": "solve_200", "kind": "solve", "family": "random", "atoms": 200, "ratio": 3.0,
         "kmin": 1, "kmax": 3, "budget": -1, "W": 1},
        # a large single query: the 2000-vertex 3-colouring under a budget
        {"name": "solve_coloring_2000", "kind": "solve", "family": "coloring", "vertices": 2000,
         "degree": 4.2, "budget": 400, "W": 1},
        # the main workload: a batch of very uneven random programs
        {"name": "batch_random", "kind": "batch", "mode": "plain", "family": "random", "n": 1024,
         "a_lo": 100, "a_hi": 5000, "budget": 400},
        # many small programs at once, all to their verdicts or 1000 conflicts
        {"name": "batch_small", "kind": "batch", "mode": "plain", "family": "random", "n": 2000,
         "a_lo": 100, "a_hi": 400, "budget": 1000},
        # recursive programs (stability checks and constraints at work)
        {"name": "batch_hamiltonian", "kind": "batch", "mode": "plain", "family": "hamiltonian",
         "n": 256, "v_lo": 60, "v_hi": 200, "budget": 400},
        # resolution-based learning, the method's other Learning step
        {"name": "batch_res", "kind": "batch", "mode": "res", "family": "random", "n": 256,
         "a_lo": 100, "a_hi": 5000, "budget": 250},
        # up to 16 answer sets of each program
        {"name": "batch_enum", "kind": "batch", "mode": "enum", "family": "random", "n": 512,
         "a_lo": 100, "a_hi": 2000, "budget": 400},
        # lookahead over four candidate decisions
        {"name": "batch_lookahead", "kind": "batch", "mode": "lookahead", "family": "random",
         "n": 512, "a_lo": 100, "a_hi": 2000, "budget": 200},
        # the learned Decision: scoring, sorting, and the search it drives
        {"name": "learned_random", "kind": "learned", "family": "random", "n": 512, "a_lo": 100,
         "a_hi": 5000, "budget": 200},
        # the scorer alone, its scores read back
        {"name": "score_random", "kind": "score", "family": "random", "n": 512, "a_lo": 100,
         "a_hi": 5000},
        # training the scorer: ten full-batch Adam steps on a small training set
        {"name": "train_steps", "kind": "train", "n": 64, "a_lo": 100, "a_hi": 5000, "steps": 10},
    ]


def _logu(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above (sizes spread over their logarithm)."""
    kind = rng.choice(("solve", "solve", "batch", "batch", "batch", "learned", "score", "train"))
    if kind == "solve":
        if rng.random() < 0.5:
            return {"kind": kind, "family": "coloring", "vertices": _logu(rng, 60, 2000),
                    "degree": rng.uniform(3.6, 4.6), "budget": rng.randrange(50, 400),
                    "W": rng.choice((1, 1, 2))}
        return {"kind": kind, "family": "random", "atoms": _logu(rng, 12, 1500),
                "ratio": rng.uniform(2.0, 4.0), "kmin": rng.choice((0, 1)),
                "kmax": rng.choice((3, 4)), "budget": rng.randrange(200, 800),
                "W": rng.choice((1, 1, 2))}
    if kind == "train":
        a_hi = _logu(rng, 150, 5000)
        return {"kind": kind, "n": _logu(rng, 2, 48), "a_lo": 100, "a_hi": a_hi,
                "steps": rng.choice((0, 0, 1, 3, 6))}
    case = {"kind": kind, "family": rng.choice(("random", "random", "hamiltonian"))}
    if case["family"] == "random":
        case.update(n=_logu(rng, 16, 500), a_lo=rng.choice((50, 100, 300)),
                    a_hi=_logu(rng, 400, 4000))
    else:
        v_lo = rng.randrange(20, 100)
        case.update(n=_logu(rng, 16, 250), v_lo=v_lo, v_hi=v_lo + rng.randrange(1, 100))
    if kind == "batch":
        case["mode"] = rng.choice(tuple(MODES))
    if kind != "score":
        slow = case.get("mode") in ("res", "lookahead", "multi")
        case["budget"] = rng.randrange(20, 120 if slow else 250)
    return case


# ------------------------------------------------------------------ programs
def _rng(*seed):
    return np.random.Generator(np.random.PCG64(np.random.SeedSequence([17, *seed])))


def _program(n_atoms, head, off, lits):
    return SimpleNamespace(n_atoms=int(n_atoms), head=np.ascontiguousarray(head, np.int32),
                           body_off=np.ascontiguousarray(off, np.int64),
                           body_lits=np.ascontiguousarray(lits, np.int32))


def _random_programs(rng, atoms, rules, kmin, kmax):
    """Uniform random normal programs (bodies of kmin..kmax distinct atoms,
    each negated with probability one half), all drawn together."""
    atoms, rules = np.asarray(atoms, np.int64), np.asarray(rules, np.int64)
    of = np.repeat(atoms, rules)                       # atoms of each rule's program
    head = rng.integers(1, of + 1)
    k = np.minimum(rng.integers(kmin, kmax + 1, size=of.shape[0]), of)
    m = rng.integers(1, of[:, None] + 1, size=(of.shape[0], kmax))
    valid = np.arange(kmax)[None, :] < k[:, None]
    while True:                                        # redraw the later of two equal atoms
        dup = np.zeros_like(valid)
        for j in range(1, kmax):
            for i in range(j):
                dup[:, j] |= m[:, i] == m[:, j]
        dup &= valid
        if not dup.any():
            break
        m[dup] = rng.integers(1, np.broadcast_to(of[:, None], m.shape)[dup] + 1)
    lits = m[valid]
    lits = np.where(rng.random(lits.shape[0]) < 0.5, -lits, lits)
    off = np.zeros(of.shape[0] + 1, np.int64)
    np.cumsum(k, out=off[1:])
    out, r = [], 0
    for a, n in zip(atoms.tolist(), rules.tolist()):
        o = off[r:r + n + 1]
        out.append(_program(a, head[r:r + n], o - o[0], lits[o[0]:o[-1]]))
        r += n
    return out


def _coloring(rng, n, degree):
    """3-colouring of G(n, p): one choice per vertex through even negative
    cycles, one constraint per edge and colour."""
    iu, ju = np.triu_indices(n, k=1)
    keep = rng.random(iu.shape[0]) < degree / (n - 1)
    u, w = iu[keep], ju[keep]
    v, c = np.repeat(np.arange(n), 3), np.tile(np.arange(3), n)
    head = np.concatenate([3 * v + c + 1, np.zeros(3 * u.shape[0], np.int64)])
    body = np.stack([-(3 * v + (c + 1) % 3 + 1), -(3 * v + (c + 2) % 3 + 1)], 1)
    cu = (3 * u[:, None] + np.arange(3) + 1).reshape(-1)
    cw = (3 * w[:, None] + np.arange(3) + 1).reshape(-1)
    lits = np.concatenate([body.reshape(-1), np.stack([cu, cw], 1).reshape(-1)])
    return _program(3 * n, head, 2 * np.arange(head.shape[0] + 1), lits)


def _hamiltonian(rng, deg):
    """Hamiltonian cycle of a random digraph with the given out-degrees:
    in(e), out(e) and reach(v) atoms, recursive reachability from vertex 0."""
    n = deg.shape[0]
    t = np.argsort(rng.random((n, n - 1)), axis=1)[:, :6]
    t = t + (t >= np.arange(n)[:, None])
    pick = np.arange(t.shape[1])[None, :] < deg[:, None]
    u = np.broadcast_to(np.arange(n)[:, None], t.shape)[pick]
    w = t[pick]
    E = u.shape[0]
    e = np.arange(E)
    inn, out, reach = e + 1, E + e + 1, 2 * E + 1
    heads, lens, lits = [], [], []

    def put(head, body):
        heads.append(np.broadcast_to(head, body.shape[:1]))
        lens.append(np.full(body.shape[0], body.shape[1]))
        lits.append(body.reshape(-1))
    put(inn, -out[:, None])
    put(out, -inn[:, None])
    s = u == 0
    put(reach + w[s], inn[s][:, None])
    put(reach + w[~s], np.stack([reach + u[~s], inn[~s]], 1))
    for end in (u, w):                                 # at most one edge out of / into a vertex
        same = np.triu(end[:, None] == end[None, :], 1)
        a, b = np.nonzero(same)
        put(np.int64(0), np.stack([inn[a], inn[b]], 1))
    put(np.int64(0), -(reach + np.arange(n))[:, None])
    off = np.zeros(sum(x.shape[0] for x in lens) + 1, np.int64)
    np.cumsum(np.concatenate(lens), out=off[1:])
    return _program(2 * E + n, np.concatenate(heads), off, np.concatenate(lits))


def _sizes(case):
    """Atoms and rules of each random program of a batch, or the out-degrees
    (3..6) of each Hamiltonian-cycle graph: the case's own, whatever the seed."""
    rng = np.random.Generator(np.random.PCG64(case["n"]))
    if case.get("family") == "hamiltonian":
        return [np.minimum(rng.integers(3, 7, size=int(v)), int(v) - 1)
                for v in rng.integers(case["v_lo"], case["v_hi"] + 1, case["n"])]
    a = np.rint(np.exp(rng.uniform(math.log(case["a_lo"]), math.log(case["a_hi"]),
                                   case["n"]))).astype(np.int64)
    return a, np.rint(a * rng.uniform(2.0, 4.0, case["n"])).astype(np.int64)


def _programs(case, seed):
    rng = _rng(seed)
    if case["kind"] == "solve":
        if case["family"] == "coloring":
            return [_coloring(rng, case["vertices"], case["degree"])]
        return _random_programs(rng, [case["atoms"]], [int(round(case["atoms"] * case["ratio"]))],
                                case["kmin"], case["kmax"])
    if case.get("family") == "hamiltonian":
        return [_hamiltonian(rng, deg) for deg in _sizes(case)]
    return _random_programs(rng, *_sizes(case), 1, 4)


def _encode(progs, **options):
    with ThreadPoolExecutor(16) as ex:
        return list(ex.map(lambda p: P.Program(p, **options), progs))


# ------------------------------------------------------------------- prepare
def prepare(case, seed):
    """Programs encoded and bound to the device (and weights, labels and
    starting parameters), as a user's program holds them between calls."""
    kind = case["kind"]
    progs = _programs(case, seed)
    st = SimpleNamespace(kind=kind)
    if kind == "solve":
        st.prog = P.Program(progs[0], W=case["W"]).bind("cuda")
        st.lim = P.limits(case["budget"], 120000)
        return st
    if kind == "train":
        st.progs = _encode(progs, **STORE)
        st.labels, st.params, st.steps = *_training_inputs(progs, seed), case["steps"]
        return st
    if kind == "batch":
        st.handles = _encode(progs, **STORE, **MODES[case["mode"]])
        st.all_models = case["mode"] == "enum"
    else:
        st.handles = _encode(progs, **STORE, decision=P.DECISION_SCORE)
        st.weights = B.load_weights()
        st.all_models = False
    stream = torch.cuda.Stream()       # graph launches need a stream of their own
    with torch.cuda.stream(stream):
        st.batch = P.Batch(st.handles).bind("cuda", stream=stream)
        if kind != "batch":
            st.ws = st.batch.scorer_workspace("cuda")
    if kind != "score":
        st.lim = P.limits(case["budget"], 120000)
    return st


def _training_inputs(progs, seed):
    """Labels as the training script draws them from traces (only atoms that
    head a rule carry one, about a twentieth of them 1) and seeded starting
    parameters (matrices within 24/128, biases within 1/8)."""
    rng = _rng(seed, 1)
    labels = []
    for p in progs:
        y = np.full(p.n_atoms, -1.0, np.float32)
        h = np.unique(p.head[p.head > 0]) - 1
        y[h] = rng.random(h.shape[0]) < 0.05
        labels.append(y)
    H, L, FH = B.SCORER_H, B.SCORER_L, B.SCORER_F * B.SCORER_H
    mat = rng.integers(-24, 25, 2 * FH + 6 * L * H * H) / 128.0
    bias = rng.integers(-(1 << 14), (1 << 14) + 1, 2 * H + 2 * L * H) / 131072.0
    wo = rng.integers(-127, 128, H) / 128.0
    params = np.concatenate([mat[:2 * FH], bias[:2 * H], mat[2 * FH:], bias[2 * H:], wo, [0.0]])
    return labels, params.astype(np.float32)


# ----------------------------------------------------------------------- run
def _counters(stats):
    return np.array([[s[k] & 0x7fffffffffffffff for k in COUNTERS] for s in stats], np.int64)


def run(state):
    if state.kind == "solve":
        verdict, model, stats = state.prog.solve(state.lim)
        if model is None:
            model = np.zeros(state.prog.n_atoms, np.uint8)
        return [verdict, model, _counters([stats])]
    if state.kind == "train":
        params, losses, grad = B.train_scorer(state.progs, state.labels, state.params,
                                              steps=state.steps, lr=3e-3)
        return [params, losses, grad]
    b = state.batch
    if state.kind in ("learned", "score"):
        b.score(state.weights, state.ws)
        if state.kind == "score":
            return np.concatenate([b.get_scores(i) for i in range(len(state.handles))])
    b.solve(state.lim, graph=True)
    verdicts, models, stats = b.results(all_models=state.all_models)
    # the answer sets, each at its place (an instance leaves the places it
    # found none for unspecified: 0 here)
    out = np.zeros(b.model_bytes, np.uint8)
    at = 0
    for i, h in enumerate(state.handles):
        kept = models[i] if state.all_models else [models[i]] if verdicts[i] == P.SAT else []
        for j, m in enumerate(kept):
            out[at + j * h.n_atoms:at + (j + 1) * h.n_atoms] = m
        at += h.n_atoms * max(1, int(h.opt.max_models))
    return [verdicts, out, _counters(stats)]


# ---------------------------------------------------------------------- work
def _expected(case):
    """Expected variables, static nogoods and literals of all programs (the
    completion of a rule with k body literals has 5 + k nogoods and 9 + 3k
    literals, and its atom's support nogoods add two literals and one nogood
    per rule; three auxiliary variables per rule)."""
    if case.get("family") == "coloring":
        a, edges = 3 * case["vertices"], case["vertices"] * case["degree"] / 2
        r, k, con, clits = a, 2.0, 3 * edges, 6 * edges
    elif case.get("family") == "hamiltonian":
        v = case["n"] * (case["v_lo"] + case["v_hi"]) / 2
        a, r, k = v * 10.0, v * 13.5, 1.3
        con, clits = v * 19.0, v * 37.0
    else:
        if case["kind"] == "solve":
            a, ratio, k = case["atoms"], case["ratio"], (case["kmin"] + case["kmax"]) / 2
        else:
            lo, hi = case["a_lo"], case["a_hi"]
            a = case["n"] * ((hi - lo) / math.log(hi / lo) if hi > lo else lo)
            ratio, k = 3.0, 2.5
        r, con, clits = a * ratio, 0.0, 0.0
    return a, r, a + 3 * r, r * (6 + k) + a + con, r * (12 + 3 * k) + a + clits


def work(case):
    """Bytes and operations of one pass that no implementation can avoid:
    the programs read once, the results written once; how many rounds a
    search takes is the input's business.  The scorer and its training do
    two products per node and sign (64 x 64) and an addition per literal and
    column in each layer and direction; training reads the programs once per
    step (its activations count as kept on the chip)."""
    a, r, v, ng, lits = _expected(case)
    n, H, L = case.get("n", 1), B.SCORER_H, B.SCORER_L
    read = 4 * (lits + ng + v)
    fwd = 2.0 * H * H * 3 * L * (v + ng) + 2.0 * H * L * 2 * lits
    if case["kind"] == "train":
        passes = max(1, case["steps"])
        return {"bytes": passes * (read + 8 * B.SCORER_NPARAM), "flops": passes * 3 * fwd}
    flops = fwd if case["kind"] in ("learned", "score") else 0
    if case["kind"] == "score":
        return {"bytes": read + 4 * a, "flops": flops}
    return {"bytes": read + a * MODES[case.get("mode", "plain")].get("max_models", 1) + 112 * n,
            "flops": flops}


# --------------------------------------------------------------------- exact
def _graph(progs):
    """Edges (nogood, variable row, negative) of all programs' completions and
    the nodes' input features, as float64 tensors."""
    cs, vs, sg, kinds, atoms = [], [], [], [], []
    nc = nv = 0
    for p in progs:
        A, R = p.n_atoms, p.head.shape[0]
        j = np.arange(R)
        b, t, q = A + 3 * j + 1, A + 3 * j + 2, A + 3 * j + 3
        k = np.diff(p.body_off)
        rule, lit = np.repeat(j, k), p.body_lits.astype(np.int64)
        pos = lit > 0
        o = nc + np.arange(R)                         # the fixed nogoods of each rule
        groups = [(o, -b), (o, t), (o, q)]            # {F b, T t, T n}
        o = o + R
        groups += [(o, b), (o, -t)]                   # {T b, F t}
        o = o + R
        groups += [(o, b), (o, -q)]                   # {T b, F n}
        o = o + R
        groups += [(o, -t), (o[rule[pos]], lit[pos])]     # {F t} u body+
        o = o + R
        groups += [(o, -q), (o[rule[~pos]], lit[~pos])]   # {F n} u F body-
        o = nc + 5 * R + np.arange(lit.shape[0])      # {T t, F p}, {T n, T q} per body literal
        groups += [(o, np.where(pos, t[rule], q[rule])), (o, np.where(pos, -lit, -lit))]
        o = nc + 5 * R + lit.shape[0] + j             # {F p, T b} per rule
        groups += [(o, -p.head.astype(np.int64)), (o, b)]
        o = nc + 6 * R + lit.shape[0] + np.arange(A)  # {T p} u {F b of its rules}
        groups += [(o, np.arange(1, A + 1)), (o[p.head - 1], -b)]
        c = np.concatenate([g[0] for g in groups])
        l = np.concatenate([g[1] for g in groups])
        cs.append(c)
        vs.append(nv + np.abs(l) - 1)
        sg.append(l < 0)
        kind = np.zeros(A + 3 * R, np.int64)
        kind[A:] = 1 + np.tile(np.arange(3), R)
        kinds.append(kind)
        atoms.append(np.arange(A + 3 * R) < A)
        nc += 6 * R + lit.shape[0] + A
        nv += A + 3 * R
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    c, v, s = (torch.from_numpy(np.concatenate(x)).to(dev) for x in (cs, vs, sg))
    kind = torch.from_numpy(np.concatenate(kinds)).to(dev)
    f64 = {"dtype": torch.float64, "device": dev}

    def count(idx, n):
        return torch.zeros(n, **f64).index_add_(0, idx, torch.ones(idx.shape[0], **f64))

    def bits(x):                                       # bit length of a non-negative integer
        return torch.where(x > 0, torch.floor(torch.log2(torch.clamp(x, min=1))) + 1, 0 * x)
    ln, npos = count(c, nc), count(c[~s], nc)
    dp, dn = count(v[~s], nv), count(v[s], nv)
    z = torch.zeros(nc, **f64)
    xc = torch.stack([z + 32, torch.floor((32 + torch.floor(ln / 2)) / ln), 32. * (ln == 1),
                      32. * (ln == 2), 32. * (ln == 3), 32. * (ln >= 4),
                      torch.floor((32 * npos + torch.floor(ln / 2)) / ln), z], 1) / 256
    xv = torch.stack([torch.full((nv,), 32., **f64)] + [32. * (kind == i) for i in range(4)] +
                     [torch.clamp(16 * bits(d), max=255) for d in (dp, dn, dp + dn)], 1) / 256
    scale = [torch.exp2(-torch.ceil(torch.log2(torch.clamp(d, min=1)))) for d in (ln, dp + dn)]
    return c, v, s, xc, xv, scale[0][:, None], scale[1][:, None], \
        torch.from_numpy(np.concatenate(atoms)).to(dev)


def _loss(p, graph, y):
    """Mean binary cross-entropy of the scorer's float form."""
    c, v, s, xc, xv, sc, sv, _ = graph
    H, L, F = B.SCORER_H, B.SCORER_L, B.SCORER_F
    shapes = [(F, H)] * 2 + [(H,)] * 2 + [(L, H, H)] * 6 + [(L, H)] * 2 + [(H,), (1,)]
    parts = torch.split(p, [math.prod(x) for x in shapes])
    Ev, Ec, ev, ec, Pp, Nn, S, Q, R, T, bc, bv, wo, bo = (q.view(x) for q, x in zip(parts, shapes))

    def gather(dst, src, n, x_pos, x_neg):
        out = torch.zeros(n, H, dtype=p.dtype, device=p.device)
        out = out.index_add(0, dst[~s], x_pos[src[~s]])
        return out.index_add(0, dst[s], x_neg[src[s]])
    av, ac = (torch.clamp(x @ E / 4 + e, 0, 1) for x, E, e in ((xv, Ev, ev), (xc, Ec, ec)))
    for l in range(L):
        ac = torch.clamp((ac @ S[l] + sc * gather(c, v, xc.shape[0], av @ Pp[l], av @ Nn[l])) / 4
                         + bc[l], 0, 1)
        av = torch.clamp((av @ T[l] + sv * gather(v, c, xv.shape[0], ac @ Q[l], ac @ R[l])) / 4
                         + bv[l], 0, 1)
    keep = y >= 0
    z = av[keep] @ wo + bo
    return torch.nn.functional.binary_cross_entropy_with_logits(z, y[keep])


def exact(case, seed):
    """Training in 64-bit floating point: parameters, losses and gradient."""
    if case["kind"] != "train":
        return None
    progs = _programs(case, seed)
    labels, params = _training_inputs(progs, seed)
    graph = _graph(progs)
    c, _, _, xc, xv, _, _, atom = graph
    y = torch.full((xv.shape[0],), -1.0, dtype=torch.float64, device=c.device)
    y[atom] = torch.from_numpy(np.concatenate(labels)).to(y)
    p = torch.from_numpy(params).to(y)
    H, L, F = B.SCORER_H, B.SCORER_L, B.SCORER_F
    lim = torch.full_like(p, 127 / 128)
    lim[2 * F * H:2 * F * H + 2 * H] = 128
    lim[-1 - H - 2 * L * H:-1 - H] = 128
    lim[-1] = 512
    m, w, losses, steps = torch.zeros_like(p), torch.zeros_like(p), [], case["steps"]
    for t in range(1, max(steps, 1) + 1):
        q = p.clone().requires_grad_(True)
        loss = _loss(q, graph, y)
        g, = torch.autograd.grad(loss, q)
        losses.append(loss.item())
        if steps:
            m = 0.9 * m + 0.1 * g
            w = 0.999 * w + 0.001 * g * g
            p = p - 3e-3 * (m / (1 - 0.9 ** t)) / (torch.sqrt(w / (1 - 0.999 ** t)) + 1e-8)
            p = torch.minimum(torch.maximum(p, -lim), lim)
    return [p.cpu().numpy(), np.array(losses), g.cpu().numpy()]
