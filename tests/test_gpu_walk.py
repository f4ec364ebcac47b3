"""The walk over the forest (forest_walk.hip) against the lanes, which run every program: same results, same counts, same
refusals, on forests of every shape: shuffled, with nodes nobody asks for, shared nodes, bad entries, and trees that
leave the walk's stack; and which of the two ran (tdf_stats.tag_phase).  Gradients on both, and where a walk was left to the
lanes, against the oracle."""
import dataclasses
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2410_20225_amd import tdf, programs  # noqa: E402
from paper_2410_20225_amd.programs import _Fn  # noqa: E402
from tdf_workloads import make_config  # noqa: E402
from gpu_util import TreeRun, run_oracle_tree, rel_fro  # noqa: E402

DEV, H, V, C = "cuda:0", 64, 50, 5
KEYS = ("n_tags", "n_tokens", "n_leaf_rows", "n_cell_rows", "n_waves", "max_tag_depth")


def _trees(shapes, rng, shuffle=True):
    """shapes: nested pairs, None a leaf -> left, right, token, roots; nodes numbered at random."""
    left, right, roots = [], [], []

    def add(s):
        todo, top = [(s, None, 0)], len(left)
        while todo:
            s, parent, side = todo.pop()
            v = len(left)
            left.append(-1)
            right.append(-1)
            if parent is not None:
                (left, right)[side][parent] = v
            if s is not None:
                todo += [(s[1], v, 1), (s[0], v, 0)]
        return top

    roots = [add(s) for s in shapes]
    left, right, roots = np.array(left), np.array(right), np.array(roots)
    if shuffle:
        name = rng.permutation(left.size)
        new = lambda a: np.where(a >= 0, name[np.maximum(a, 0)], -1)  # noqa: E731
        l2, r2 = np.empty_like(left), np.empty_like(right)
        l2[name], r2[name] = new(left), new(right)
        left, right, roots = l2, r2, name[roots]
    return left, right, rng.integers(0, V, left.size), roots


def _chain(n, right=None):
    s = None
    for _ in range(n):
        s = (s, right)
    return s


def _random(n, rng):
    if n == 1:
        return None
    k = int(rng.integers(1, n))
    return (_random(k, rng), _random(n - k, rng))


def _swapped():   # cell(f(right), f(left)), with identities in between
    T = tdf
    r = _Fn("result", 2)
    y = r.add(T.OP_CALLFN, [r.add(T.OP_IN, imm=1)], imm=1)
    r.add(T.OP_OUT, [r.add(T.OP_CE_HEAD, [y, r.add(T.OP_IN, imm=0)])])
    f = _Fn("f", 1)
    v = f.add(T.OP_ID, [f.add(T.OP_IN, imm=0)])
    sw = f.add(T.OP_SWITCH, [f.add(T.OP_TREE_ISLEAF, [v]), v])
    leaf, inner = (sw[0], 0), (sw[0], 1)
    e = f.add(T.OP_EMBED, [f.add(T.OP_TREE_TOKEN, [leaf])])
    hl = f.add(T.OP_CALLFN, [f.add(T.OP_TREE_LEFT, [f.add(T.OP_ID, [inner])])], imm=1)
    hr = f.add(T.OP_CALLFN, [f.add(T.OP_TREE_RIGHT, [inner])], imm=1)
    f.add(T.OP_OUT, [f.add(T.OP_ID, [f.add(T.OP_MERGE, [f.add(T.OP_LSTM_CELL, [hr, hl]), e])])])
    return [r.desc(), f.desc()], 0


def _leaf_label():   # not the walk's form: the head's label is a node's token
    T = tdf
    r = _Fn("result", 2)
    v = r.add(T.OP_IN, imm=0)
    y = r.add(T.OP_CALLFN, [v], imm=1)
    r.add(T.OP_OUT, [r.add(T.OP_CE_HEAD, [y, r.add(T.OP_SUB, [r.add(T.OP_IN, imm=1), r.add(T.OP_CONST, imm=0)])])])
    fns, _ = programs.tree("lstm", True)
    return [r.desc(), fns[1]], 0


def _run(prog, forest, walk, max_tags=None, label_first=False, nodes=False, vocab=V):
    left, right, token, roots = forest
    os.environ.pop("TDF_NO_WALK", None)
    if not walk:
        os.environ["TDF_NO_WALK"] = "1"
    try:
        g = tdf.graph_build(*prog)
        B, n = len(roots), len(left)
        lab = np.arange(B) % C
        args = roots[:, None] if nodes else np.stack([lab, roots] if label_first else [roots, lab], 1)
        t = lambda a, d: torch.tensor(np.ascontiguousarray(a), dtype=d, device=DEV)  # noqa: E731
        gen = torch.Generator(device=DEV).manual_seed(3)
        rn = lambda *s: torch.randn(*s, generator=gen, device=DEV) * 0.3  # noqa: E731
        keep = dict(args=t(args, torch.int64), left=t(left, torch.int32), right=t(right, torch.int32), token=t(token, torch.int32),
                    E=rn(vocab, H).bfloat16(), W=rn(5 * H, 2 * H).bfloat16(), b=rn(5 * H), U=rn(C, H), u0=rn(C))
        if nodes:
            keep["node_label"] = t(np.arange(n) % (C + 1) - 1, torch.int32)
        inp = tdf.make_inputs(B, n_args=args.shape[1], dtype=tdf.BF16, hidden=H, vocab=vocab, n_classes=C,
                              max_tags=max(n, B) if max_tags is None else max_tags, stats_level=0, **keep)
        ws = torch.full((tdf.workspace_size(g, inp),), 0x5A, dtype=torch.uint8, device=DEV)
        out = dict(out_h=torch.zeros(B, H, device=DEV), out_c=torch.zeros(B, H, device=DEV), out_node_loss=torch.zeros(n, device=DEV)) if nodes \
            else dict(out_f32=torch.zeros(B, device=DEV))
        res = []
        for _ in range(2):
            st, stats = tdf.eval(g, inp, ws, check=False, **out)
            res.append((st, [getattr(stats, k) for k in KEYS] if st == tdf.OK else None,
                        [o.cpu().numpy().copy() for o in out.values()] if st == tdf.OK else None, stats))
        return res
    finally:
        os.environ.pop("TDF_NO_WALK", None)


def _same(prog, forest, left=False, form=True, **kw):
    """left: the forest is one that the walk leaves to the lanes; form: the program is one that is walked."""
    a, b = _run(prog, forest, True, **kw), _run(prog, forest, False, **kw)
    for k, (x, y) in enumerate(zip(a, b)):
        assert x[0] == y[0] and x[1] == y[1], (x[:2], y[:2])
        if x[0] == tdf.OK:   # (a row's arithmetic does not depend on where the row lies)
            for o, p in zip(x[2], y[2]):
                assert np.array_equal(o, p)
            assert x[3].tag_phase == (tdf.TAGS_WALK if form and not left else tdf.TAGS_LANES) and y[3].tag_phase == tdf.TAGS_LANES
            assert x[3].repeats == (1 if form and left and k == 0 else 0) and y[3].repeats == 0   # (a graph remembers it for a while)
    return a[0]


def _forests():
    rng = np.random.default_rng(5)
    some = [_random(int(n), rng) for n in rng.integers(1, 40, 30)]
    yield "one_leaf", _trees([None], rng)
    yield "one_pair", _trees([(None, None)], rng)
    yield "random", _trees(some, rng)
    yield "in_order", _trees(some, rng, shuffle=False)
    yield "chains", _trees([_chain(70), _chain(3), None], rng)
    yield "right_chain", _trees([tuple_chain(90)], rng)
    # spines of spines of spines: more right children at once than the stack holds (leaves would be taken as they come)
    yield "combs", _trees([_chain(100, _chain(20, _chain(4))), _chain(5)], rng)
    l, r, t, roots = _trees(some, rng)
    yield "nodes_nobody_asks_for", (l, r, t, roots[::3])
    yield "the_same_root_twice", (l, r, t, np.concatenate([roots[:5], roots[3:9]]))
    inner = roots[np.nonzero(l[roots] >= 0)[0][:6]]
    yield "a_root_inside_another_tree", (l, r, t, np.concatenate([inner, l[inner]]))
    l2, r2 = l.copy(), r.copy()
    r2[inner[0]] = l2[inner[0]]
    yield "both_children_the_same", (l2, r2, t, roots)
    l3, r3 = l.copy(), r.copy()
    r3[inner[0]] = l3[inner[1]]
    yield "a_child_of_two_trees", (l3, r3, t, roots)
    for k, bad in (("right_missing", -1), ("right_out_of_range", l.size), ("left_out_of_range", l.size + 7)):
        a, b = l.copy(), r.copy()
        (a if k[0] == "l" else b)[inner[2]] = bad
        yield k, (a, b, t, roots)
    t2 = t.copy()
    t2[np.nonzero(l < 0)[0][3]] = V
    yield "token_out_of_range", (l, r, t2, roots)
    yield "root_out_of_range", (l, r, t, np.concatenate([roots, [l.size]]))
    a, b = l.copy(), r.copy()
    leaf = l[inner[3]]
    while a[leaf] >= 0:
        leaf = a[leaf]
    a[leaf], b[leaf] = inner[3], inner[3]
    yield "a_cycle", (a, b, t, roots)


def tuple_chain(n):
    s = None
    for _ in range(n):
        s = (None, s)
    return s


FORESTS = list(_forests())


SHARED = {"the_same_root_twice", "a_root_inside_another_tree", "both_children_the_same", "a_child_of_two_trees"}


@pytest.mark.parametrize("name,forest", FORESTS, ids=[n for n, _ in FORESTS])
def test_forests(name, forest):
    wrong = {"right_missing", "right_out_of_range", "left_out_of_range", "token_out_of_range", "root_out_of_range", "a_cycle"}
    st, _, _, stats = _same(programs.tree("lstm", True), forest, left=name in SHARED, max_tags=4 * max(len(forest[0]), len(forest[3])))
    assert (st != tdf.OK) == (name in wrong)
    if name == "combs":   # a wave's stack was full (512 nodes, and 64 lanes), so its lanes kept lists
        assert stats.peak_frames >= 512 + 64 + 64


@pytest.mark.parametrize("max_tags", [1, 2])
def test_fewer_tags_than_nodes(max_tags):
    forest = dict(FORESTS)["random"]
    n = len(forest[0])
    assert _same(programs.tree("lstm", True), forest, max_tags=max(n // max_tags, 30))[0] == (tdf.OK if max_tags == 1 else tdf.ERR_TABLE_FULL)


def test_other_programs():
    for name in ("random", "combs", "nodes_nobody_asks_for"):
        forest = dict(FORESTS)[name]
        assert _same(_swapped(), forest, label_first=True)[0] == tdf.OK
        assert _same(_leaf_label(), forest, form=False)[0] == tdf.OK
        assert _same(programs.tree("lstm", False, True), forest, nodes=True)[0] == tdf.OK


@pytest.mark.parametrize("walk", [True, False], ids=["walk", "lanes"])
@pytest.mark.parametrize("shared", [False, True], ids=["trees", "roots_twice"])
@pytest.mark.parametrize("cfg,bf16", [(2, False), (4, True)])
def test_gradients(cfg, bf16, shared, walk, monkeypatch):
    # shared: some instances ask for the same trees, so the first evaluation's walk is left to the lanes half way
    if not walk:
        monkeypatch.setenv("TDF_NO_WALK", "1")
    c = make_config(cfg, n_trees=30, max_leaves=20, hidden=48, vocab=100)
    F = c["forest"]
    n_tags = F.n_nodes
    if shared:
        again = np.arange(0, 30, 4)
        c["forest"] = dataclasses.replace(F, roots=np.concatenate([F.roots, F.roots[again]]), n_leaves=np.concatenate([F.n_leaves, F.n_leaves[again]]))
        c["labels"] = np.concatenate([c["labels"], c["labels"][again]])
        n_tags += int((2 * F.n_leaves[again] - 1).sum())
    B = c["forest"].n_trees
    dy = np.linspace(0.5, 1.5, B) / B
    ref = run_oracle_tree(c, head=True, grad=True, dy=dy)
    run = TreeRun(c, head=True, grad=True, stats_level=0, max_tags=n_tags)
    tol = 2e-2 if bf16 else 2e-5   # (the bars of the other gradient tests)
    for k in range(2):
        st, stats = run.run(dy)
        assert stats.tag_phase == (tdf.TAGS_WALK if walk and not shared else tdf.TAGS_LANES)
        assert stats.repeats == (1 if walk and shared and k == 0 else 0)
        assert stats.n_tags == stats.n_grad_firings == n_tags and stats.n_grad_not_once == 0
        assert rel_fro(run.out_f32.cpu().numpy(), np.array(ref["out"])) < tol
        for name, t in (("dW", run.dW), ("db", run.db), ("dE", run.dE)):
            assert rel_fro(t.cpu().numpy(), ref["grads"][name]) < tol, name


def _complete(levels):
    s = None
    for _ in range(levels):
        s = (s, s)
    return s


@pytest.mark.parametrize("shapes,left", [([_complete(11)], False), ([_complete(14)], True), ([_complete(14)] + [_chain(9)] * 20, True),
                                         ([_complete(12)] * 16, False), ([_chain(9000)], False), ([_chain(3000), _complete(11)], False)],
                         ids=["complete_2k", "complete_16k", "complete_16k_and_small_ones", "16_of_4k", "chain_9k", "chain_and_complete"])
def test_wide_trees_are_left_to_the_lanes(shapes, left):
    assert _same(programs.tree("lstm", True), _trees(shapes, np.random.default_rng(3)), left=left)[0] == tdf.OK


def test_a_refused_evaluation_does_not_keep_the_next_one_from_the_walk():
    # a token out of range; then the same graph on a forest that is in order, and on one with shared nodes
    c = make_config(4, n_trees=12, max_leaves=9, hidden=32, vocab=40)
    run = TreeRun(c, head=True, grad=False, stats_level=0, max_tags=2 * c["forest"].n_nodes)
    run.run()
    want = run.out_f32.clone()
    leaf = int(np.nonzero(c["forest"].left < 0)[0][4])
    good = int(run.t_token[leaf])
    for _ in range(3):
        run.t_token[leaf] = 40
        assert run.run(check=False)[0] == tdf.ERR_BAD_ARG
        run.t_token[leaf] = good
        st, stats = run.run()
        assert stats.tag_phase == tdf.TAGS_WALK and stats.repeats == 0 and torch.equal(run.out_f32, want)
    args = run.t_args.clone()
    run.t_args[1] = run.t_args[0]
    got = [run.run()[1] for _ in range(10)]   # left once, eight at once on the lanes, and the walk has its turn again
    assert [st.repeats for st in got] == [1] + [0] * 8 + [1] and all(st.tag_phase == tdf.TAGS_LANES for st in got)
    run.t_args.copy_(args)
    assert run.run()[1].tag_phase == tdf.TAGS_LANES and torch.equal(run.out_f32, want)


# ---- trees in one piece of memory, which are not walked: the schedule's steps are rounds of doubling (14 at most)

def _in_pieces(shapes, order, rng):
    """Tree after tree, depth first or level by level, the roots in front or (back) behind their trees."""
    left, right, token, roots = _trees(shapes, rng, shuffle=False)
    name = np.arange(left.size)
    if "level" in order:
        for top, end in zip(roots, np.append(roots[1:], left.size)):
            todo = [top]
            for v in todo:
                if left[v] >= 0:
                    todo += [left[v], right[v]]
            name[todo] = np.arange(top, end)
    if "back" in order:
        name = left.size - 1 - name
    new = lambda a: np.where(a >= 0, name[np.maximum(a, 0)], -1)  # noqa: E731
    l2, r2 = np.empty_like(left), np.empty_like(right)
    l2[name], r2[name] = new(left), new(right)
    return l2, r2, token, name[roots]


# (one wave and 512 nodes, four and 4,096, sixteen and 16,384: a workgroup's window by the trees' number and average size)
PIECES = {
    "waves1": lambda rng: [_random(int(n), rng) for n in rng.integers(1, 70, 270)] + [_chain(255), _complete(8), _random(256, rng)],
    "waves4": lambda rng: [_chain(2047), _complete(11), _random(900, rng), None, (None, None)] + [_random(9, rng)] * 20,
    "waves16": lambda rng: [_chain(8191), _random(3000, rng), _complete(13)],
}


@pytest.mark.parametrize("order", ["depth", "depth back", "level", "level back"])
@pytest.mark.parametrize("size", PIECES)
def test_trees_in_one_piece(size, order):
    rng = np.random.default_rng(8)
    stats = _same(programs.tree("lstm", True), _in_pieces(PIECES[size](rng), order, rng))[3]
    assert 0 < stats.n_steps <= 14


@pytest.mark.parametrize("leaves,small", [(257, 300), (2049, 4), (8193, 0)], ids=["waves1", "waves4", "waves16"])
def test_a_tree_too_large_for_the_window_is_walked(leaves, small):
    rng = np.random.default_rng(9)
    stats = _same(programs.tree("lstm", True), _in_pieces([_chain(leaves - 1)] + [_random(20, rng)] * small, "depth", rng))[3]
    assert stats.n_steps > leaves


@pytest.mark.parametrize("order", ["depth", "level back"])
@pytest.mark.parametrize("what", ["a_stranger_inside", "a_child_before_its_parent", "right_is_left", "a_child_of_two_trees", "a_cycle",
                                  "right_missing", "right_out_of_range", "token_out_of_range", "roots_in_another_order", "every_other_tree"])
def test_pieces_that_are_none(what, order):
    rng = np.random.default_rng(10)
    l, r, t, roots = _in_pieces([_chain(40), _random(30, rng), _complete(4), _random(25, rng)], order, rng)
    inner = [next(v for v in (l[x], r[x]) if l[v] >= 0) for x in roots]   # an inner node below each root
    left, st = False, tdf.OK
    if what in ("a_stranger_inside", "a_child_before_its_parent"):   # (another numbering of the same trees)
        n = l.size
        if what == "a_stranger_inside":   # a leaf that belongs to nobody, between two nodes of the first tree
            a = min(roots[0], inner[0]) + 1
            name = np.arange(n) + (np.arange(n) >= a)
            size = n + 1
        else:   # an inner node and the last of its subtree change places
            name, size = np.arange(n), n
            v = inner[1]
            low = r[v] if l[r[v]] < 0 else l[v]
            name[[v, low]] = name[[low, v]]
        new = lambda x: np.where(x >= 0, name[np.maximum(x, 0)], -1)  # noqa: E731
        l2, r2, t2 = np.full(size, -1), np.full(size, -1), np.zeros(size, np.int64)
        l2[name], r2[name], t2[name] = new(l), new(r), t
        l, r, t, roots = l2, r2, t2, name[roots]
    elif what == "right_is_left":
        r[inner[1]], left = l[inner[1]], True
    elif what == "a_child_of_two_trees":
        r[inner[1]], left = l[inner[3]], True
    elif what == "a_cycle":
        leaf = inner[0]
        while l[leaf] >= 0:
            leaf = r[leaf]
        l[leaf], r[leaf], st = inner[0], inner[0], None
    elif what == "right_missing":
        r[inner[2]], st = -1, tdf.ERR_BAD_ARG
    elif what == "right_out_of_range":
        r[inner[2]], st = l.size, tdf.ERR_BAD_ARG
    elif what == "token_out_of_range":
        t[np.nonzero(l < 0)[0][7]], st = V, tdf.ERR_BAD_ARG
    elif what == "roots_in_another_order":
        roots = roots[[2, 0, 3, 1]]
    else:
        roots = roots[1::2]
    got = _same(programs.tree("lstm", True), (l, r, t, roots), left=left, max_tags=4 * l.size)[0]
    assert got == st if st is not None else got != tdf.OK


# ---- the same for every size of window, beside as many and as large trees as it takes; what is no piece is walked in the same launch (one
# wave a workgroup, or up to 512 instances of 4,096 nodes) or in one of its own
BESIDE = {
    "waves1": lambda rng: [_random(int(n), rng) for n in rng.integers(2, 40, 300)],
    "waves4": lambda rng: [_random(int(n), rng) for n in rng.integers(2, 40, 200)],
    "waves4_apart": lambda rng: [_random(int(n), rng) for n in rng.integers(100, 160, 520)],
    "waves16": lambda rng: [_random(3000, rng), _chain(1500), _complete(11)],
}


def _broken(what, forest, first):
    """-> forest, whether it is left to the lanes, status; the trees from `first` on stay as they are."""
    l, r, t, roots = [x.copy() for x in forest]
    inner = [next(v for v in (l[x], r[x]) if l[v] >= 0) for x in roots[:first]]
    left, st = False, tdf.OK
    if what == "a_child_before_its_parent":   # an inner node and the last of its subtree change places
        name = np.arange(l.size)
        v = inner[1]
        low = r[v] if l[r[v]] < 0 else l[v]
        name[[v, low]] = name[[low, v]]
        new = lambda x: np.where(x >= 0, name[np.maximum(x, 0)], -1)  # noqa: E731
        l2, r2, t2 = np.empty_like(l), np.empty_like(r), np.empty_like(t)
        l2[name], r2[name], t2[name] = new(l), new(r), t
        l, r, t, roots = l2, r2, t2, name[roots]
    elif what == "right_is_left":
        r[inner[1]], left = l[inner[1]], True
    elif what == "a_child_of_two_trees":
        r[inner[1]], left = l[inner[3]], True
    elif what == "a_root_inside_another_tree":
        roots[1], left = inner[0], True
    elif what == "a_cycle":
        leaf = inner[0]
        while l[leaf] >= 0:
            leaf = r[leaf]
        l[leaf], r[leaf], st = inner[0], inner[0], None
    elif what == "right_missing":
        r[inner[2]], st = -1, tdf.ERR_BAD_ARG
    elif what == "right_out_of_range":
        r[inner[2]], st = l.size, tdf.ERR_BAD_ARG
    elif what == "token_out_of_range":
        t[np.nonzero(l < 0)[0][7]], st = V, tdf.ERR_BAD_ARG
    elif what == "root_out_of_range":
        roots[2], st = l.size, tdf.ERR_BAD_ARG
    return (l, r, t, roots), left, st


@pytest.mark.parametrize("size", BESIDE)
@pytest.mark.parametrize("what", ["a_child_before_its_parent", "right_is_left", "a_child_of_two_trees", "a_root_inside_another_tree", "a_cycle",
                                  "right_missing", "right_out_of_range", "token_out_of_range", "root_out_of_range"])
def test_pieces_that_are_none_beside_others(what, size):
    rng = np.random.default_rng(11)
    some = [_chain(40), _random(30, rng), _complete(4), _random(25, rng)]
    forest, left, st = _broken(what, _in_pieces(some + BESIDE[size](rng), "depth", rng), 4)
    got = _same(programs.tree("lstm", True), forest, left=left, max_tags=4 * forest[0].size)[0]
    assert got == st if st is not None else got != tdf.OK


@pytest.mark.parametrize("size", BESIDE)
def test_forests_in_random_order(size):
    rng = np.random.default_rng(12)
    stats = _same(programs.tree("lstm", True), _trees([_chain(300), _complete(5)] + BESIDE[size](rng), rng))[3]
    assert stats.n_steps > 300


def test_what_the_statistics_say_of_pieces_and_walks():
    # include/tdf.h: the rounds of doubling and all nodes for trees in one piece, a wave's steps and its stack for trees that are walked
    rng = np.random.default_rng(13)
    shapes = [_chain(200), _complete(6), _random(90, rng)]
    piece = _same(programs.tree("lstm", True), _in_pieces(shapes, "depth", rng))[3]
    assert 2 ** piece.n_steps < 200 <= 2 ** (piece.n_steps + 1) and piece.peak_frames == piece.n_tags   # (200: the chain's height)
    walk = _same(programs.tree("lstm", True), _trees(shapes, rng))[3]
    assert walk.n_steps >= 200 and 64 * len(shapes) <= walk.peak_frames <= (512 + 64) * len(shapes)
