"""The work that programs have this framework do, as cases that can be timed: integer recursions and
while-loops, and recursive tree networks forward and with their gradients, each one call of tdf.eval
or tdf.eval_grad on inputs that are resident on the GPU.

A case is a dict of plain values; `kind` names the program:

  fib, tak   recursive integer functions (one and three parameters), a batch of argument tuples
  gcd        the subtractive gcd while-loop, a batch of pairs
  tree       TreeRNN / TreeLSTM over a batch of binary trees; `mode` is
               states   forward, the root states h (and c)
               losses   forward with the 5-class head, one loss per tree
               train    the same with the gradients of W, b and E
               nodes    fully labelled trees: a loss term at every node, with the gradients
"""
import functools

import numpy as np
import torch

from paper_2410_20225_amd import programs, tdf

DEV = "cuda"
CLASSES = 5


def _tree(name, cell, dtype, mode, trees, lo, hi, hidden, vocab, zipf=False, chains=0.0, complete=0.0):
    c = dict(kind="tree", cell=cell, dtype=dtype, mode=mode, trees=trees, lo=lo, hi=hi, hidden=hidden, vocab=vocab,
             zipf=zipf, chains=chains, complete=complete)
    return dict(c, name=name) if name else c


def listed():
    return [
        # a handful of small calls, as a service gets them: launches and round trips are all there is
        dict(name="fib_few", kind="fib", calls=8, lo=3, hi=10),
        # the batch fib(0) .. fib(20), 57 thousand tags
        dict(name="fib_batch", kind="fib", calls=21, lo=0, hi=20),
        # three large recursions side by side, 14 million tags
        dict(name="fib_large", kind="fib", calls=3, lo=30, hi=32),
        # a recursion with three parameters whose arguments are themselves calls
        dict(name="tak_batch", kind="tak", calls=256, hi=12),
        # while-loops with data-dependent trip counts, many at once
        dict(name="gcd_loops", kind="gcd", calls=65536, hi=1024),
        # one sentence encoded by a TreeLSTM, as a server answers a single request
        _tree("lstm_one", "lstm", "bf16", "states", 1, 20, 50, 256, 20000, zipf=True),
        # a batch of sentences encoded by a TreeRNN in fp32
        _tree("rnn_states_fp32", "rnn", "f32", "states", 256, 2, 50, 128, 10000),
        # a batch of sentences encoded by a TreeLSTM, a fifth of them left chains
        _tree("lstm_states", "lstm", "bf16", "states", 4096, 2, 128, 256, 20000, zipf=True, chains=0.2),
        # a training step on a minibatch of fully labelled sentences, odd width
        _tree("lstm_nodes_minibatch", "lstm", "bf16", "nodes", 50, 2, 50, 150, 10000, zipf=True),
        # training steps: TreeRNN with a head, ragged width; TreeLSTM on a large batch
        _tree("rnn_train", "rnn", "bf16", "train", 1024, 2, 60, 300, 10000),
        _tree("lstm_train", "lstm", "bf16", "train", 4096, 2, 128, 256, 20000, zipf=True, chains=0.2),
        # a training step on deep recursions: chains of 4096 leaves beside complete trees of as many
        _tree("rnn_train_deep", "rnn", "bf16", "train", 128, 4096, 4096, 512, 10000, chains=0.5, complete=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    what = rng.choice(["fib", "tak", "gcd"] + ["tree"] * 5)
    if what == "fib":
        hi = rng.randint(9, 31)
        return dict(kind="fib", calls=_log_int(rng, 2, max(2, min(4096, 8_000_000 // int(1.7 ** hi)))), lo=rng.randint(0, hi - 6), hi=hi)
    if what == "tak":
        return dict(kind="tak", calls=_log_int(rng, 4, 1024), hi=rng.randint(7, 13))
    if what == "gcd":
        return dict(kind="gcd", calls=_log_int(rng, 16, 65536), hi=_log_int(rng, 20, 1024))
    cell, mode = rng.choice(["rnn", "lstm"]), rng.choice(["states", "losses", "train", "train", "nodes"])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    if rng.random() < 0.15:   # deep recursions
        trees, lo = _log_int(rng, 2, 128), 1 << rng.randint(7, 11)
        hidden = rng.choice([64, 100, 128, 200, 256, 300])
        return _tree(None, cell, dtype, mode, trees, lo, lo, hidden, 10000, chains=0.5, complete=0.5)
    hidden = rng.choice([32, 50, 64, 100, 128, 150, 168, 200, 256, 300, 384, 512])
    hi = _log_int(rng, 8, 128)
    most = 4096 if dtype == "bf16" and hidden <= 256 else 1024
    return _tree(None, cell, dtype, mode, _log_int(rng, 1, most), rng.randint(2, 8), hi, hidden,
                 rng.choice([1000, 10000, 20000]), zipf=rng.random() < 0.5, chains=rng.choice([0.0, 0.0, 0.2]))


# ---- inputs ------------------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _graph(program, *args):
    """A program is compiled once and serves every batch."""
    *prog, grad = args
    g = tdf.graph_build(*getattr(programs, program)(*prog), want_grad=grad)
    tdf.graph_prepare(g)
    return g


def _fib_tags(n):
    a, b = 0, 1
    for _ in range(n + 1):
        a, b = b, a + b
    return 2 * a - 1          # invocations of fib(n)


@functools.lru_cache(maxsize=None)
def _tak(x, y, z):
    """(value, invocations)"""
    if y >= x:
        return z, 1
    a, b, c = _tak(x - 1, y, z), _tak(y - 1, z, x), _tak(z - 1, x, y)
    d = _tak(a[0], b[0], c[0])
    return d[0], 1 + a[1] + b[1] + c[1] + d[1]


def _gcd_trips(a, b):
    """Iterations of the loop over all pairs: the sum of Euclid's quotients, one per subtraction, plus
    the test that leaves (the last subtraction, which would reach zero, is that test)."""
    a, b = a.copy(), b.copy()
    n = 0
    while True:
        on = b > 0
        if not on.any():
            return n
        a, b = a[on], b[on]
        n += int((a // b).sum())
        a, b = b, a % b


def _calls(case, rng, seed):
    """Argument tuples of an integer program and the number of tags they take."""
    n = case["calls"]
    if case["kind"] == "fib":
        v = np.linspace(case["lo"], case["hi"], n).round().astype(np.int64)
        v = np.roll(v, seed) if n < 8 else rng.permutation(v)
        return v[:, None], sum(_fib_tags(int(x)) for x in v)
    if case["kind"] == "tak":
        hi = case["hi"]
        v = np.stack([rng.integers(hi // 2, hi + 1, n), rng.integers(0, hi // 2 + 1, n), rng.integers(0, hi + 1, n)], 1)
        return v, sum(_tak(*map(int, r))[1] for r in v)
    v = rng.integers(1, case["hi"] + 1, (n, 2))
    return v, _gcd_trips(v[:, 0], v[:, 1])


def _forest(case, rng):
    """left, right, is-leaf and roots of the batch's trees, each laid out in pre-order: a node over L
    leaves has its left child, over k leaves, behind it and its right child 2k - 1 places further.  The
    sizes lo .. hi are spread evenly over the batch, in random order."""
    B = case["trees"]
    leaves = rng.permutation(case["lo"] + ((np.arange(B) + 0.5) * (case["hi"] - case["lo"] + 1) / B).astype(np.int64))
    at = np.concatenate([[0], np.cumsum(2 * leaves - 1)])
    left, right = np.full(at[-1], -1, np.int32), np.full(at[-1], -1, np.int32)
    kind = np.zeros(B, np.int64)                   # 0 random split, 1 left chain, 2 complete
    kind[:int(round(B * case["chains"]))] = 1
    kind[int(round(B * case["chains"])):int(round(B * (case["chains"] + case["complete"])))] = 2
    kind = rng.permutation(kind)
    chain = kind == 1
    if chain.any():                                # every right child is a leaf
        n = leaves[chain] - 1
        i = np.arange(n.sum()) - np.repeat(np.cumsum(n) - n, n)
        p, last = np.repeat(at[:-1][chain], n), np.repeat(2 * n, n)
        left[p + i], right[p + i] = p + i + 1, p + last - i
    p, L, k3 = at[:-1][~chain], leaves[~chain], kind[~chain]
    while p.size:
        on = L > 1
        p, L, k3 = p[on], L[on], k3[on]
        k = np.where(k3 == 2, L // 2, 1 + (rng.random(L.size) * (L - 1)).astype(np.int64))
        left[p], right[p] = p + 1, p + 2 * k
        p, L, k3 = np.concatenate([p + 1, p + 2 * k]), np.concatenate([k, L - k]), np.concatenate([k3, k3])
    return left, right, at[:-1]


def prepare(case, seed):
    rng = np.random.default_rng([seed, 20225])
    on_gpu = lambda a, d: torch.from_numpy(np.ascontiguousarray(a)).to(DEV, d)  # noqa: E731
    if case["kind"] != "tree":
        args, n_tags = _calls(case, rng, seed)
        g = _graph("gcd_loop" if case["kind"] == "gcd" else case["kind"], False)
        t_args = on_gpu(args, torch.int64).reshape(-1)
        inputs = tdf.make_inputs(len(args), args=t_args, n_args=args.shape[1], max_tags=n_tags, stats_level=0)
        return dict(graph=g, inputs=inputs, keep=t_args, ws=torch.empty(tdf.workspace_size(g, inputs), dtype=torch.uint8, device=DEV),
                    grad=False, out=dict(out_i64=torch.zeros(len(args), dtype=torch.int64, device=DEV)))

    mode, B, H, V = case["mode"], case["trees"], case["hidden"], case["vocab"]
    head, grad, nodes = mode in ("losses", "train"), mode in ("train", "nodes"), mode == "nodes"
    left, right, roots = _forest(case, rng)
    n = left.size
    leaf = left < 0
    n_leaf = int(leaf.sum())
    if case["zipf"]:
        cdf = np.cumsum(np.arange(1, V + 1, dtype=np.float64) ** -1.1)
        tok = np.minimum(np.searchsorted(cdf, rng.random(n_leaf) * cdf[-1]), V - 1)
    else:
        tok = rng.integers(0, V, n_leaf)
    token = np.full(n, -1, np.int32)
    token[leaf] = tok
    rows = (5 if case["cell"] == "lstm" else 1) * H
    bf16 = case["dtype"] == "bf16"
    gen = torch.Generator(device=DEV).manual_seed(seed)
    el = torch.bfloat16 if bf16 else torch.float32
    f32 = dict(dtype=torch.float32, device=DEV)
    xavier = lambda r, c: (torch.rand(r, c, generator=gen, **f32) * 2 - 1) * (6.0 / (r + c)) ** 0.5  # noqa: E731
    keep = dict(args=on_gpu(np.stack([roots, rng.integers(0, CLASSES, B)], 1) if head else roots[:, None], torch.int64),
                left=on_gpu(left, torch.int32), right=on_gpu(right, torch.int32), token=on_gpu(token, torch.int32),
                E=torch.randn(V, H, generator=gen, **f32).to(el), W=xavier(rows, 2 * H).to(el), b=torch.zeros(rows, **f32),
                U=xavier(CLASSES, H), u0=torch.zeros(CLASSES, **f32))
    if nodes:
        keep["node_label"] = on_gpu(rng.integers(0, CLASSES, n), torch.int32)
    g = _graph("tree", case["cell"], head, nodes, grad)
    inputs = tdf.make_inputs(B, n_args=2 if head else 1, dtype=tdf.BF16 if bf16 else tdf.F32, hidden=H, vocab=V, n_classes=CLASSES,
                             max_tags=n, stats_level=0, **keep)
    out = {}
    if head:
        out["out_f32"] = torch.zeros(B, **f32)
    else:
        out["out_h"] = torch.zeros(B, H, **f32)
        if case["cell"] == "lstm":
            out["out_c"] = torch.zeros(B, H, **f32)
    if nodes:
        out["out_node_loss"] = torch.zeros(n, **f32)
    state = dict(graph=g, inputs=inputs, keep=keep, grad=grad, out=out,
                 ws=torch.empty(tdf.workspace_size(g, inputs, grad), dtype=torch.uint8, device=DEV))
    if grad:
        state["dy"] = torch.full((B,), 1.0 / B, **f32) if head else None
        state["dnode"] = torch.full((n,), 1.0 / n, **f32) if nodes else None
        state["grads"] = dict(dW=torch.empty(rows, 2 * H, **f32), db=torch.empty(rows, **f32), dE=torch.empty(V, H, **f32))
    return state


def run(s):
    if s["grad"]:
        _, stats = tdf.eval_grad(s["graph"], s["inputs"], s["dy"], s["ws"], dnode=s["dnode"], **s["grads"], **s["out"])
        return dict(s["out"], **s["grads"], n_tags=stats.n_tags)
    _, stats = tdf.eval(s["graph"], s["inputs"], s["ws"], **s["out"])
    return dict(s["out"], n_tags=stats.n_tags)


# ---- what a pass cannot do without ------------------------------------------------------------

def work(case):
    """Integer programs: the arguments and results, and the body's arithmetic once per tag.  Trees: the
    forest, the embedding rows the leaves name, the parameters and the results (with the gradients, and
    every row of dE), each moved once, and the products of the cells: forward, input and weight gradient."""
    if case["kind"] != "tree":
        args, n_tags = _calls(case, np.random.default_rng([1, 20225]), 1)
        return {"bytes": 8.0 * args.size + 8.0 * len(args), "flops": {"fib": 4.0, "tak": 4.0, "gcd": 3.0}[case["kind"]] * n_tags}
    B, H, V = case["trees"], case["hidden"], case["vocab"]
    leaves = B * (case["lo"] + case["hi"]) / 2
    nodes, cells = 2 * leaves - B, leaves - B
    rows, el = (5 if case["cell"] == "lstm" else 1) * H, 2 if case["dtype"] == "bf16" else 4
    seen = V * (1 - (1 - 1.0 / V) ** leaves) if not case["zipf"] else min(leaves, V) * 0.5   # distinct tokens, about
    by = 12.0 * nodes + 16 * B + seen * H * el + rows * 2 * H * el + 4 * rows + 4 * CLASSES * H
    flops = 2.0 * cells * rows * 2 * H
    by += 4.0 * B if case["mode"] in ("losses", "train") else 4.0 * B * H * (2 if case["cell"] == "lstm" else 1)
    if case["mode"] == "nodes":
        by += 12.0 * nodes
        flops += 2.0 * nodes * CLASSES * H * 2
    if case["mode"] in ("train", "nodes"):
        by += 4.0 * (rows * 2 * H + rows + V * H)
        flops *= 3
    return {"bytes": by, "flops": flops}


def tolerance(case):
    if case["kind"] != "tree":
        return "exact"
    # bf16: the states are rounded to 8 bits at every level of the recursion; fp32: sums in another order
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-5}
