"""GPU parity of the depth-first lanes, which run the evaluations that keep no frames (statistics level 0):
values, tag and token counts and tag depth bit-exact against the oracle and against the step machine (the
same call with TDF_NO_LANES), with one wave (every hand-over inside it) and with as many as the library
takes (calls sent between waves).  Sizes: one instance, fewer instances than waves, more than a wave's lanes;
recursions deeper than the window and than several segments of a lane's stack; loops beyond the iterations of
one sweep; a call with an argument that is dead, which the lanes leave to the step machine."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2410_20225_amd import tdf, programs  # noqa: E402
import oracle  # noqa: E402
from oracle import programs as oprog  # noqa: E402
from tdf_workloads import make_config, SplitMix64  # noqa: E402
from tdf_workloads.trees import left_chain_tree, right_chain_tree, random_split_tree, build_forest  # noqa: E402
from gpu_util import DEV, TreeRun, run_oracle_tree, run_oracle_node_loss, rel_fro  # noqa: E402

INT = {
    "fib": (programs.fib, oprog.fib_program, [(n,) for n in list(range(16)) * 5]),
    "fib_one": (programs.fib, oprog.fib_program, [(19,)]),
    "ack": (programs.ack, oprog.ack_program, [(0, 0), (1, 2), (2, 3), (3, 3), (2, 0), (0, 7), (1, 90)]),
    "tak": (programs.tak, oprog.tak_program, [(7, 4, 2), (12, 8, 4), (1, 2, 3), (9, 5, 1)]),
    "sum_loop": (programs.sum_loop, oprog.sum_loop_program, [(n,) for n in (0, 1, 62, 63, 64, 65, 127, 128, 300)]),
    "gcd": (programs.gcd_loop, oprog.gcd_loop_program, [(a, b) for a in range(1, 20) for b in range(1, 8)]),
    "nested": (programs.nested_loop, oprog.nested_loop_program, [(n,) for n in (0, 1, 2, 5, 17, 30)]),
    "loop_of_calls": (programs.loop_of_calls, oprog.loop_of_calls_program, [(n,) for n in (0, 1, 3, 9, 12)]),
    "loop_in_function": (programs.loop_in_function, oprog.loop_in_function_program, [(n,) for n in (0, 1, 2, 6, 25, 40)]),
}


def _eval_int(g, args, n_args, max_tags):
    t_args = torch.tensor(args, dtype=torch.int64, device=DEV).reshape(-1)
    inp = tdf.make_inputs(len(args), args=t_args, n_args=n_args, max_tags=max_tags, stats_level=0)
    ws = torch.empty(tdf.workspace_size(g, inp), dtype=torch.uint8, device=DEV)
    out = torch.full((len(args),), -1, dtype=torch.int64, device=DEV)
    st, stats = tdf.eval(g, inp, ws, out_i64=out)
    return out.cpu().tolist(), (stats.n_tags, stats.n_tokens, stats.max_tag_depth), stats.repeats


@pytest.mark.parametrize("waves", ["1", "40", None], ids=["one_wave", "waves_40", "waves_default"])
@pytest.mark.parametrize("name", list(INT))
def test_integer_programs(name, waves, monkeypatch):
    gpu_prog, oracle_prog, args = INT[name]
    n_args = len(args[0])
    it = oracle.Interpreter(oracle.transform(oracle_prog()))
    want = it.run({("in", k): [a[k] for a in args] for k in range(n_args)}, len(args))[("out", 0)]
    n_tags = len(it.tags) + len(it.iter_tags)
    fns, r = gpu_prog()
    if waves:
        monkeypatch.setenv("TDF_LANE_WAVES", waves)
    g = tdf.graph_build(fns, r)
    got = [_eval_int(g, args, n_args, n_tags) for _ in range(2)]
    for out, counts, repeats in got:
        assert out == want and repeats == 0
        assert counts[0] == n_tags and counts[2] == it.max_tag_len
    monkeypatch.setenv("TDF_NO_LANES", "1")
    assert _eval_int(g, args, n_args, n_tags)[:2] == got[0][:2]


def test_a_recursion_of_a_million_tags_over_many_waves():
    F = [0, 1]
    while len(F) < 40:
        F.append(F[-1] + F[-2])
    ns = [26, 3, 25, 27]
    fns, r = programs.fib()
    g = tdf.graph_build(fns, r)
    n_tags = sum(2 * F[n + 1] - 1 for n in ns)
    for _ in range(3):
        out, counts, repeats = _eval_int(g, [(n,) for n in ns], 1, n_tags)
        assert out == [F[n] for n in ns] and counts == (n_tags, 2 * n_tags, 27) and repeats == 0


def test_a_call_with_a_dead_argument_goes_to_the_step_machine():
    # f(n) = if n < 1 then n else h(n - 1, 1); h(a, b) = f(a) + b: at the base case the call of h has one dead and one
    # constant argument, so its scope is opened but never completes
    T = tdf
    f = [(T.OP_IN, [], 0), (T.OP_CONST, [], 1), (T.OP_LT, [(0, 0), (1, 0)], 0), (T.OP_SWITCH, [(2, 0), (0, 0)], 0),
         (T.OP_SUB, [(3, 1), (1, 0)], 0), (T.OP_CALLFN, [(4, 0), (1, 0)], 2), (T.OP_ID, [(3, 0)], 0),
         (T.OP_MERGE, [(6, 0), (5, 0)], 0), (T.OP_OUT, [(7, 0)], 0)]
    h = [(T.OP_IN, [], 0), (T.OP_IN, [], 1), (T.OP_CALLFN, [(0, 0)], 1), (T.OP_ADD, [(2, 0), (1, 0)], 0), (T.OP_OUT, [(3, 0)], 0)]
    res = [(T.OP_IN, [], 0), (T.OP_CALLFN, [(0, 0)], 1), (T.OP_OUT, [(1, 0)], 0)]
    g = tdf.graph_build([("result", 1, res), ("f", 1, f), ("h", 2, h)], 0)
    ns = [0, 1, 5, 12]
    first = _eval_int(g, [(n,) for n in ns], 1, 200)
    again = _eval_int(g, [(n,) for n in ns], 1, 200)
    assert first[0] == again[0] == ns and first[1] == again[1]
    assert first[1][0] == sum(2 * n + 2 for n in ns)       # f n + 1 times, h n times, and the scope at the base case
    assert first[2] == 1 and again[2] == 0                 # found out in the first run, remembered by the graph


def _forest(cfg, shapes, **kw):
    c = make_config(cfg, n_trees=len(shapes), max_leaves=4, **kw)
    rng = SplitMix64(31)
    c["forest"] = build_forest(shapes, lambda n: rng.randint(0, c["V"] - 1, n))
    c["labels"] = rng.randint(0, 4, len(shapes))
    c["node_labels"] = rng.randint(0, 4, c["forest"].n_nodes)
    return c


TREES = {
    "single_leaves": lambda: _forest(3, [left_chain_tree(1)] * 70, hidden=32, vocab=50),
    "one_tree": lambda: _forest(4, [random_split_tree(60, SplitMix64(9))], hidden=32, vocab=50),
    "chains": lambda: _forest(3, [left_chain_tree(300), right_chain_tree(290), left_chain_tree(2), right_chain_tree(3)] +
                              [random_split_tree(10 + 5 * b, SplitMix64(b)) for b in range(8)], hidden=32, vocab=50),
    "many_small": lambda: make_config(4, n_trees=2500, max_leaves=6, hidden=24, vocab=60),
}


@pytest.mark.parametrize("waves", ["1", None, "walk"], ids=["one_wave", "waves_default", "walk"])
@pytest.mark.parametrize("name", list(TREES))
def test_tree_programs(name, waves, monkeypatch):
    # (recursions over the children of tree nodes are walked, unless that is switched off)
    c = TREES[name]()
    F = c["forest"]
    B = F.n_trees
    tag_phase = tdf.TAGS_WALK
    if waves != "walk":
        monkeypatch.setenv("TDF_NO_WALK", "1")
        tag_phase = tdf.TAGS_LANES
        if waves:
            monkeypatch.setenv("TDF_LANE_WAVES", waves)
    dy = np.full(B, 1.0 / B)
    ref = run_oracle_tree(c, head=True, grad=True, dy=dy)
    run = TreeRun(c, head=True, grad=True, stats_level=0)
    for _ in range(2):
        st, stats = run.run(dy)
        assert stats.tag_phase == tag_phase
        assert stats.repeats == 0 and stats.n_tags == F.n_nodes == len(ref["it"].tags) and stats.max_tag_depth == ref["it"].max_tag_len
        assert stats.n_leaf_rows == int(F.n_leaves.sum()) and stats.n_cell_rows == int(F.n_leaves.sum()) - B
        assert stats.n_grad_firings == F.n_nodes and stats.n_grad_not_once == 0
        assert rel_fro(run.out_f32.cpu().numpy(), np.array(ref["out"])) < 2e-2      # (the bars of the other bf16 parity tests)
        for k, t in (("dW", run.dW), ("db", run.db), ("dE", run.dE)):
            if k in ref["grads"]:
                assert rel_fro(t.cpu().numpy(), ref["grads"][k]) < 2e-2, k
    lab = c["node_labels"].copy()
    lab[::3] = -1
    dnode = np.full(F.n_nodes, 1.0 / F.n_nodes)
    ref = run_oracle_node_loss(c, lab, dnode)
    want = np.zeros(F.n_nodes)
    for v, loss in ref["node_loss"].items():
        want[v] = loss
    run = TreeRun(c, head=False, grad=True, node_labels=lab, stats_level=0)
    st, stats = run.run(None, dnode=dnode)
    got = run.out_node_loss.cpu().numpy()
    assert stats.tag_phase == tag_phase
    assert stats.repeats == 0 and np.array_equal(got == 0.0, want == 0.0) and rel_fro(got, want) < 2e-2


def test_max_tags_is_the_step_machines_limit(monkeypatch):
    # Without kept frames max_tags bounds the tags alive at once, as the step machine counts them; the lanes answer where
    # there are no more tags than that at all, and leave every other call to it.
    ns = [(n,) for n in [20] * 8]
    tags = 8 * (2 * 10946 - 1)
    fns, r = programs.fib()
    g = tdf.graph_build(fns, r)
    out, counts, repeats = _eval_int(g, ns, 1, tags)
    assert out == [6765] * 8 and counts[0] == tags and repeats == 0
    out, counts, repeats = _eval_int(g, ns, 1, tags - 1)
    assert out == [6765] * 8 and counts[0] == tags and repeats >= 1

    def status(max_tags):
        t_args = torch.tensor(ns, dtype=torch.int64, device=DEV).reshape(-1)
        inp = tdf.make_inputs(8, args=t_args, n_args=1, max_tags=max_tags, stats_level=0)
        ws = torch.empty(tdf.workspace_size(g, inp), dtype=torch.uint8, device=DEV)
        return tdf.eval(g, inp, ws, out_i64=torch.zeros(8, dtype=torch.int64, device=DEV), check=False)[0]
    got = [status(m) for m in (8, 64, 4096)]
    monkeypatch.setenv("TDF_NO_LANES", "1")
    assert got == [status(m) for m in (8, 64, 4096)] and got[0] == got[1] == tdf.ERR_TABLE_FULL


def test_the_lanes_are_tried_again_after_a_call_they_left_to_the_step_machine():
    # f(n) = if n < -5 then n else h(n, -5), h(a, b) = a + b: one argument of the call is dead below -5.  The lanes leave such
    # a call to the step machine, and the next eight evaluations with it; then they have their turn again
    T = tdf
    h = [(T.OP_IN, [], 0), (T.OP_IN, [], 1), (T.OP_ADD, [(0, 0), (1, 0)], 0), (T.OP_OUT, [(2, 0)], 0)]
    f = [(T.OP_IN, [], 0), (T.OP_CONST, [], -5), (T.OP_LT, [(0, 0), (1, 0)], 0), (T.OP_SWITCH, [(2, 0), (0, 0)], 0),
         (T.OP_CALLFN, [(3, 1), (1, 0)], 2), (T.OP_ID, [(3, 0)], 0), (T.OP_MERGE, [(5, 0), (4, 0)], 0), (T.OP_OUT, [(6, 0)], 0)]
    res = [(T.OP_IN, [], 0), (T.OP_CALLFN, [(0, 0)], 1), (T.OP_OUT, [(1, 0)], 0)]
    g = tdf.graph_build([("result", 1, res), ("f", 1, f), ("h", 2, h)], 0)
    good, bad = [(n,) for n in (3, 0, 9)], [(n,) for n in (3, -9, 9)]
    want = lambda ns: [n if n < -5 else n - 5 for n, in ns]  # noqa: E731
    for skipped in (8, 16):
        out, _, repeats = _eval_int(g, bad, 1, 200)
        assert out == want(bad) and repeats == 1
        for _ in range(skipped):
            out, _, repeats = _eval_int(g, bad, 1, 200)
            assert out == want(bad) and repeats == 0        # (the step machine from the start)
    out, _, repeats = _eval_int(g, bad, 1, 200)
    assert out == want(bad) and repeats == 1
    for _ in range(32):
        _eval_int(g, good, 1, 200)
    out, _, repeats = _eval_int(g, good, 1, 200)            # on the lanes, which makes eight of it again
    assert out == want(good) and repeats == 0
    out, _, repeats = _eval_int(g, bad, 1, 200)
    assert repeats == 1
    for _ in range(8):
        assert _eval_int(g, bad, 1, 200)[2] == 0
    assert _eval_int(g, bad, 1, 200)[2] == 1


@pytest.mark.parametrize("waves", ["1", None], ids=["one_wave", "waves_default"])
@pytest.mark.parametrize("name", ["fib_first", "chain_first", "every_third", "below"])
def test_chains_longer_than_a_wave_has_records(name, waves, monkeypatch):
    # chains with nothing to hand over, and chains whose frames are handed over and wait for one value each
    import lane_programs
    prog, ref = {"fib_first": lambda: lane_programs.fib_at_every_frame_of_a_chain(True),
                 "chain_first": lambda: lane_programs.fib_at_every_frame_of_a_chain(False),
                 "every_third": lane_programs.fibs_along_a_chain, "below": lane_programs.fib_below_a_chain}[name]()
    args = {"every_third": [(400, 2, 9), (90, 0, 12), (3, 1, 5)], "below": [(300, 18), (120, 14)]}.get(name, [(300, 12), (1000, 6), (5, 3)])
    if waves:
        monkeypatch.setenv("TDF_LANE_WAVES", waves)
    g = tdf.graph_build(*prog)
    for _ in range(3):
        out, counts, repeats = _eval_int(g, args, len(args[0]), 400000)
        assert out == [ref(*a) for a in args] and repeats == 0
