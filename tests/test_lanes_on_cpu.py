"""The depth-first lanes run on the CPU (tests/lane_cpu.py) against the oracle and plain Python references: the code that
is generated for a program, and the machine's hand-overs between lanes and waves in random orders of events."""
import os
import subprocess

import pytest

import oracle
from oracle import programs as oprog
import lane_random
from lane_cpu import CSRC, ROOT, Lanes, lane_source, needs_host_lanes
from lane_programs import BAD_INDEX, INTEGER, VECTOR, fib_at_every_frame_of_a_chain, fib_below_a_chain, fibs_along_a_chain

pytestmark = needs_host_lanes
tdf = pytest.importorskip("paper_2410_20225_amd.tdf")
from paper_2410_20225_amd import programs  # noqa: E402

INT = {
    "fib": (programs.fib, oprog.fib_program, [(n,) for n in [16, 3, 0, 11, 14, 1, 9]]),
    "tak": (programs.tak, oprog.tak_program, [(7, 4, 2), (12, 8, 4), (1, 2, 3), (9, 5, 1)]),
    "gcd": (programs.gcd_loop, oprog.gcd_loop_program, [(a, b) for a in range(1, 20) for b in range(1, 8)]),
    "loop_of_calls": (programs.loop_of_calls, oprog.loop_of_calls_program, [(n,) for n in (0, 1, 3, 9, 12)]),
}


@pytest.mark.parametrize("name", list(INT))
def test_integer_programs_against_the_oracle(name, tmp_path):
    prog, oracle_prog, args = INT[name]
    it = oracle.Interpreter(oracle.transform(oracle_prog()))
    want = it.run({("in", k): [a[k] for a in args] for k in range(len(args[0]))}, len(args))[("out", 0)]
    lanes = Lanes(prog(), tmp_path)
    for waves, queues, seed in [(1, 1, 1), (3, 1, 2), (16, 1, 3), (40, 2, 4)]:
        got = lanes.run(args, waves=waves, queues=queues, seed=seed)
        assert got["status"] == 0 and got["out"] == want
        assert got["tags"] == len(it.tags) + len(it.iter_tags) and got["depth"] == it.max_tag_len


def _loop_of_choices(n_choices, nested):
    """result(n, a) = { i = n; while 0 < i: i = i - 1; a = one choice after the other of a } a.  Choice k: a + k + 3 where
    a < 5 k, else a - 2 k - 1; nested: the first case has two of its own, by a < 2 k, that one Merge takes with the third."""
    T = tdf
    nodes = []

    def add(op, ins=(), imm=0):
        nodes.append((op, [r if isinstance(r, tuple) else (r, 0) for r in ins], imm))
        return len(nodes) - 1
    i0, a0 = add(T.OP_IN, imm=0), add(T.OP_IN, imm=1)
    p = add(T.OP_LT, [add(T.OP_CONST), i0])
    si, sa = add(T.OP_SWITCH, [p, i0]), add(T.OP_SWITCH, [p, a0])
    a = (sa, 0)
    for k in range(1, n_choices + 1):
        s = add(T.OP_SWITCH, [add(T.OP_LT, [a, add(T.OP_CONST, imm=5 * k)]), a])
        less, more = (s, 0), add(T.OP_SUB, [(s, 1), add(T.OP_CONST, imm=2 * k + 1)])
        if nested:
            s2 = add(T.OP_SWITCH, [add(T.OP_LT, [less, add(T.OP_CONST, imm=2 * k)]), less])
            a = add(T.OP_MERGE, [more, add(T.OP_MUL, [(s2, 1), add(T.OP_CONST, imm=3)]), add(T.OP_ADD, [(s2, 0), add(T.OP_CONST, imm=k + 3)])])
        else:
            a = add(T.OP_MERGE, [add(T.OP_ADD, [less, add(T.OP_CONST, imm=k + 3)]), more])
    add(T.OP_NEXT, [add(T.OP_SUB, [(si, 0), add(T.OP_CONST, imm=1)]), a])
    add(T.OP_OUT, [(sa, 1)])
    res = [(T.OP_IN, [], 0), (T.OP_IN, [], 1), (T.OP_LOOP, [(0, 0), (1, 0)], 1), (T.OP_OUT, [(2, 0)], 0)]

    def ref(n, a):
        for _ in range(n):
            for k in range(1, n_choices + 1):
                a = a - 2 * k - 1 if a >= 5 * k else a * 3 if nested and a >= 2 * k else a + k + 3
        return a
    return ([("result", 2, res), ("W", 2, nodes)], 0), ref


# (predicates: one for the loop, and one a choice, nested two; the truth tables hold six of them)
@pytest.mark.parametrize("n_choices,nested", [(1, False), (5, False), (6, False), (2, True), (3, True)])
def test_iterations_of_loops_with_choices(n_choices, nested, tmp_path):
    prog, ref = _loop_of_choices(n_choices, nested)
    lanes = Lanes(prog, tmp_path)
    # around the four iterations between two looks at who goes on, and around a sweep's share
    args = [(n, 7 * n % 31 - 9) for n in (0, 1, 2, 3, 4, 5, 7, 8, 9, 255, 256, 257, 258, 511, 512, 513, 700)]
    for waves in (1, 3):
        got = lanes.run(args, waves=waves)
        assert got["status"] == 0 and got["out"] == [ref(*a) for a in args]
        assert got["tags"] == sum(n + 1 for n, _ in args) and got["depth"] == 1


def _call_and_loop():
    """result(n, s) = down(n) + { i = s; a = 0; while 0 < i: a = a + i; i = i - 1 } a, down(n) = if n < 1 then n else down(n - 1) + 1"""
    T = programs.T
    r = programs._Fn("result", 2)
    n, s = r.add(T.OP_IN, imm=0), r.add(T.OP_IN, imm=1)
    r.add(T.OP_OUT, [r.add(T.OP_ADD, [r.add(T.OP_CALLFN, [n], imm=1), r.add(T.OP_LOOP, [s, r.add(T.OP_SUB, [s, s])], imm=2)])])
    d = programs._Fn("down", 1)
    v, one = d.add(T.OP_IN, imm=0), d.add(T.OP_CONST, imm=1)
    sw = d.add(T.OP_SWITCH, [d.add(T.OP_LT, [v, one]), v])
    low, high = (sw[0], 0), (sw[0], 1)
    rec = d.add(T.OP_CALLFN, [d.add(T.OP_SUB, [high, one])], imm=1)
    d.add(T.OP_OUT, [d.add(T.OP_MERGE, [d.add(T.OP_ID, [low]), d.add(T.OP_ADD, [rec, one])])])
    return [r.desc(), d.desc(), programs._counting_loop("S", 2, programs._sum_step).desc()], 0


def test_a_long_loop_leaves_the_wave_s_other_lanes_their_turns(tmp_path):
    # One lane's loop, alone in its wave, takes 256 iterations a sweep; beside a recursion of another lane 64: each of
    # the recursion's sweeps waits for that many, not for 256.
    lanes = Lanes(_call_and_loop(), tmp_path)
    iterations, depth = 6400, 20
    alone = lanes.run([(0, iterations)], waves=1)
    beside = lanes.run([(0, iterations), (depth, 0)], waves=1)
    for got, n in ((alone, 0), (beside, depth)):
        assert got["status"] == 0 and got["out"] == [iterations * (iterations + 1) // 2] + [n] * (n > 0)
    assert alone["sweeps"] <= iterations // 256 + 8
    # the recursion's sweeps (one down and one up a level, the last ones in place) are of 64 iterations each
    assert beside["sweeps"] >= 2 * (depth - 2) + (iterations - 64 * 2 * (depth + 2)) // 256


def _many_calls(n_calls, mutual, chained):
    """f(n) = n + 3 where n < 1, else the sum of k f(n - k) over k = 1 .. n_calls; mutual: f calls g, and g, the same, f;
    chained: the last call's argument is n - 2 plus what the first one returns times 0, so it is ready later than the others."""
    T = tdf
    bodies = [_body_of_calls(n_calls, callee, chained) for callee in ([2, 1] if mutual else [1])]
    res = [(T.OP_IN, [], 0), (T.OP_CALLFN, [(0, 0)], 1), (T.OP_OUT, [(1, 0)], 0)]

    def ref(n):   # value, tags, depth
        if n < 1:
            return n + 3, 1, 1
        below = [ref(n - (2 if chained and k == n_calls else k)) for k in range(1, n_calls + 1)]
        return sum((k + 1) * v[0] for k, v in enumerate(below)), 1 + sum(v[1] for v in below), 1 + max(v[2] for v in below)
    return ([("result", 1, res)] + [("fg"[i], 1, b) for i, b in enumerate(bodies)], 0), ref


def _body_of_calls(n_calls, callee, chained):
    T = tdf
    nodes = []

    def add(op, ins=(), imm=0):
        nodes.append((op, [r if isinstance(r, tuple) else (r, 0) for r in ins], imm))
        return len(nodes) - 1
    n, one = add(T.OP_IN, imm=0), add(T.OP_CONST, imm=1)
    s = add(T.OP_SWITCH, [add(T.OP_LT, [n, one]), n])
    total = first = None
    for k in range(1, n_calls + 1):
        if chained and k == n_calls:
            a = add(T.OP_ADD, [add(T.OP_SUB, [(s, 1), add(T.OP_CONST, imm=2)]), add(T.OP_MUL, [first, add(T.OP_CONST, imm=0)])])
        else:
            a = add(T.OP_SUB, [(s, 1), add(T.OP_CONST, imm=k)])
        call = add(T.OP_CALLFN, [a], imm=callee)
        first = call if first is None else first
        term = add(T.OP_MUL, [call, add(T.OP_CONST, imm=k)])
        total = term if total is None else add(T.OP_ADD, [total, term])
    add(T.OP_OUT, [add(T.OP_MERGE, [add(T.OP_ADD, [(s, 0), add(T.OP_CONST, imm=3)]), total])])
    return nodes


# (a state for each set of opened calls: two functions of four calls have more than get code of their own)
@pytest.mark.parametrize("n_calls,mutual", [(4, False), (7, False), (3, True), (4, True), (5, True)])
@pytest.mark.parametrize("chained", [False, True])
def test_functions_with_many_calls(n_calls, mutual, chained, tmp_path):
    prog, ref = _many_calls(n_calls, mutual, chained)
    assert ("bool known" in lane_source(prog)) == (mutual and n_calls > 3)
    lanes = Lanes(prog, tmp_path)
    args = [(n,) for n in (5, 0, 3, -1, 6, 1, 2, 4)]
    want = [ref(*a) for a in args]
    for waves, seed in [(1, 1), (3, 2), (16, 3)]:
        got = lanes.run(args, waves=waves, seed=seed)
        assert got["status"] == 0 and got["out"] == [w[0] for w in want]
        assert got["tags"] == sum(w[1] for w in want) and got["depth"] == max(w[2] for w in want)


@pytest.mark.parametrize("name", list(VECTOR))
def test_vector_results(name, tmp_path):
    prog, forest, args, ref = VECTOR[name]()
    lanes = Lanes(prog, tmp_path)
    for waves in (1, 4):
        got = lanes.run(args, waves=waves, log_cap=4096, vocab=50, **forest.arrays())
        log = [got["log"][k:k + 4] for k in range(0, len(got["log"]), 4)]
        leaves = [e for e in log if e[2] == 0]
        assert got["status"] == 0 and [log[r][0] for r in got["root"]] == [ref(*a) for a in args]
        # one leaf under every tag (of f)
        assert got["leaves"] == len(leaves) == got["tags"]


@pytest.mark.parametrize("name", list(INTEGER))
def test_integer_results(name, tmp_path):
    prog, forest, args, ref = INTEGER[name]()
    lanes = Lanes(prog, tmp_path)
    for waves in (1, 4):
        got = lanes.run(args, waves=waves, **forest.arrays())
        assert got["status"] == 0 and got["out"] == [ref(*a) for a in args]


@pytest.mark.parametrize("name", list(BAD_INDEX))
def test_nodes_that_do_not_exist_are_refused(name, tmp_path):
    # (the forest's arrays lie between inaccessible pages, so a read out of range would end the driver)
    prog, forest, bad = BAD_INDEX[name]()
    lanes = Lanes(prog, tmp_path)
    for v in bad:
        assert lanes.run([(v,)], **forest.arrays())["status"] == -tdf.ERR_BAD_ARG, v


@pytest.fixture(scope="module")
def fib_under_chain(tmp_path_factory):
    prog, ref = fib_below_a_chain()
    return Lanes(prog, tmp_path_factory.mktemp("lanes")), ref


def test_a_wave_whose_records_all_wait_takes_no_call(fib_under_chain):
    # six chains of 16 frames take the 96 records of a wave; the calls at their ends are in other waves when a call for
    # this wave comes
    lanes, ref = fib_under_chain
    args = [(14, 14)] * 6 + [(0, 1)] * 42
    for seed in range(1, 25):
        got = lanes.run(args, waves=8, seed=seed)
        assert got["status"] == 0 and got["out"] == [ref(*a) for a in args], seed
        assert got["records"] <= 8 * 96


@pytest.fixture(scope="module")
def fib(tmp_path_factory):
    return Lanes(programs.fib(), tmp_path_factory.mktemp("lanes"))


@pytest.mark.parametrize("slow", [0, 100, 1000])
def test_a_call_that_nobody_has_taken_yet_is_not_overwritten(fib, slow):
    # queues of few slots, which the tickets go round while a slow wave (one of `slow` turns) has not looked at its own
    for cap, waves, queues in [(8, 7, 1), (4, 3, 1), (4, 4, 2)]:
        for seed in range(1, 7):
            got = fib.run([(19,), (3,)], waves=waves, queues=queues, queue_cap=cap, slow=slow, seed=seed, max_turns=2000000)
            assert got["status"] == 0 and got["out"] == [4181, 2], (cap, waves, seed)


def test_frames_with_nothing_to_share_do_not_keep_a_wave_from_sharing(fib_under_chain):
    # a chain of calls above fib(18): every frame of it is pushed and popped, beyond that it costs nothing
    lanes, ref = fib_under_chain
    sweeps = {}
    for n in (0, 1, 4, 5, 16, 17, 20, 100, 200, 1000):
        got = [lanes.run([(n, 18)], waves=8, seed=seed) for seed in (1, 2, 3)]
        assert all(g["status"] == 0 and g["out"] == [ref(n, 18)] for g in got), n
        sweeps[n] = min(g["sweeps"] for g in got)
    for n in (100, 200, 1000):
        assert sweeps[n] - 2 * (n - 20) < 1.5 * sweeps[20], sweeps


@pytest.mark.parametrize("waves", [1, 2, 5, 16])
def test_stacks_between_frames_that_are_shared(waves, tmp_path):
    prog, ref = fibs_along_a_chain()
    lanes = Lanes(prog, tmp_path)
    args = [(70, 2, 9), (40, 0, 12), (3, 1, 5), (200, 2, 6), (0, 0, 10), (17, 1, 11)]
    for seed in range(1, 7):
        got = lanes.run(args, waves=waves, seed=seed)
        assert got["status"] == 0 and got["out"] == [ref(*a) for a in args], seed
        assert got["records"] <= 96 * waves


def test_a_run_beyond_max_tags_is_given_up(fib, tmp_path):
    # f(n) = 1 + f(n + 1) never ends: reports of the waves' tags end it soon after max_tags
    T = tdf
    f = [(T.OP_IN, [], 0), (T.OP_CONST, [], 1), (T.OP_ADD, [(0, 0), (1, 0)], 0), (T.OP_CALLFN, [(2, 0)], 1),
         (T.OP_ADD, [(3, 0), (1, 0)], 0), (T.OP_OUT, [(4, 0)], 0)]
    res = [(T.OP_IN, [], 0), (T.OP_CALLFN, [(0, 0)], 1), (T.OP_OUT, [(1, 0)], 0)]
    lanes = Lanes(([("result", 1, res), ("f", 1, f)], 0), tmp_path)
    got = lanes.run([(n,) for n in range(6)], waves=4, max_tags=5000)
    assert got["status"] == -tdf.ERR_TABLE_FULL and 2500 < got["tags"] < 15000
    # (as many tags as there may be are no reason)
    assert fib.run([(n,) for n in range(21)], waves=40, max_tags=57291)["status"] == 0


def test_a_run_without_stack_segments_is_given_up(fib_under_chain):
    # (an index that no segment has would end the driver)
    lanes, ref = fib_under_chain
    for segs in (1, 2, 5, 20):
        for args in ([(300, 14)] * 3 + [(20, 3)] * 9, [(150, 16)], [(40, 12)] * 60):
            for waves in (1, 3):
                got = lanes.run(args, waves=waves, segs=segs, seed=1)
                assert got["status"] == -tdf.ERR_TABLE_FULL, (segs, waves)


def test_a_long_run_is_not_given_up_while_waves_work(fib):
    # longer than the time in which nobody may work; waves that wait look at that all the time
    for seed in (1, 2, 3):
        got = fib.run([(24,)], waves=3, seed=seed, idle_ticks=50, dead_ticks=30000)
        assert got["status"] == 0 and got["out"] == [46368] and got["turns"] > 40000, seed


@pytest.mark.parametrize("node_loss", [False, True], ids=["roots", "node_losses"])
def test_the_schedule_of_tree_networks(node_loss, tmp_path):
    # chains of leaf-sided nodes above random trees: every cell of the log names the rows of its node's children, its level
    # is one above theirs, and with a loss term at every node every row is marked with its node
    import random
    rng = random.Random(3)
    left, right, token, roots = [], [], [], []

    def node(n, chain):
        v = len(left)
        left.append(-1), right.append(-1), token.append(rng.randrange(50))
        if n > 1:
            k = 1 if chain else rng.randrange(1, n)
            first = node(n - k, chain - 1 if chain else 0)
            second = node(k, 0)
            left[v], right[v] = (first, second) if chain % 2 else (second, first)
        return v

    for n, chain in [(1, 0), (2, 0), (140, 90), (40, 0), (130, 125), (60, 0), (17, 16), (64, 3)] * 2:
        roots.append(node(n, chain))
    lanes = Lanes(programs.tree("rnn", node_loss=node_loss), tmp_path)
    for waves, seed in [(1, 1), (6, 2), (20, 3)]:
        got = lanes.run([(v,) for v in roots], waves=waves, seed=seed, log_cap=16384, vocab=50, left=left, right=right, token=token,
                        node_loss=int(node_loss))
        n_leaf = sum(x < 0 for x in left)
        assert got["status"] == 0 and got["tags"] == len(left) and got["leaves"] == n_leaf and got["cells"] == len(left) - n_leaf
        log = [got["log"][k:k + 4] for k in range(0, len(got["log"]), 4)]

        def check(name, v, b):
            x, y, level, inst = log[name]
            assert inst == b and (not node_loss or got["marks"][name] == v)
            if left[v] < 0:
                assert (x, level) == (token[v], 0)
                return 0
            assert level == 1 + max(check(x, left[v], b), check(y, right[v], b))
            return level
        for b, v in enumerate(roots):
            check(got["root"][b], v, b)


@pytest.mark.parametrize("fib_first", [True, False], ids=["fib_first", "chain_first"])
def test_chains_in_which_every_frame_is_shared(fib_first, tmp_path):
    prog, ref = fib_at_every_frame_of_a_chain(fib_first)
    lanes = Lanes(prog, tmp_path)
    args = [(150, 8), (3, 12), (300, 5), (90, 10), (0, 5)]
    for waves in (1, 2, 5):
        for seed in range(1, 7):
            got = lanes.run(args, waves=waves, seed=seed)
            assert got["status"] == 0 and got["out"] == [ref(*a) for a in args], (waves, seed)
            assert got["records"] <= 96 * waves


def _random_case(seed):
    """What went wrong with the program of a seed, or None; whether it was one of the lanes' at all."""
    import random
    import tempfile
    rng = random.Random(seed)
    vector = seed % 2 == 1
    F, prog = lane_random.forest(rng), lane_random.program(rng, vector)
    source = lane_source(prog)
    cases = []
    for _ in range(40):
        args = (rng.randrange(12), rng.randint(-1, 9), rng.randint(-4, 9))
        try:
            cases.append((args, lane_random.evaluate(prog, F, args)))
        except lane_random.Skip:
            pass
    if source is None or not cases:
        return None, False
    with tempfile.TemporaryDirectory() as folder:
        lanes = Lanes(prog, folder, "-O0", source)
        for waves in (1, 3):
            got = lanes.run([a for a, _ in cases], waves=waves, log_cap=200000, vocab=9, **F)
            if got["status"] != 0 or [got[k] for k in ("tags", "leaves", "cells")] != [sum(r[i] for _, r in cases) for i in (1, 2, 3)]:
                return (seed, waves, "status or counts", {k: got[k] for k in ("status", "tags", "leaves", "cells")}), True

            def same(name, v):
                x, y, level, _ = got["log"][4 * name:4 * name + 4]
                return level == 0 and x == v[1] if v[0] == "E" else level > 0 and same(x, v[1]) and same(y, v[2])
            for k, (a, r) in enumerate(cases):
                if not (same(got["root"][k], r[0]) if vector else got["out"][k] == r[0]):
                    return (seed, waves, a), True
    return None, True


def test_random_programs():
    from concurrent.futures import ThreadPoolExecutor
    lane_source(programs.fib())   # (builds the generator before the threads use it)
    with ThreadPoolExecutor(6) as pool:
        results = list(pool.map(_random_case, range(48)))
    assert [r for r, _ in results if r] == []
    assert sum(ran for _, ran in results) >= 24   # (the others are too large, or none of the lanes')


def test_when_waves_look_after_every_sweep(tmp_path):
    # (waves, instances, tags a wave reports at once, entries of the log, busy lanes, sweeps of the wave, age of the run): max_tags
    # says what there is room for (tags_at_once is max_tags over twice the waves), so ample room alone must not break a run up
    # for good; and tree programs, which keep a log, are not broken up at all
    cases = {(2048, 1, 4096, 0, 60, 3, 5000): 1, (2048, 1, 4096, 0, 60, 3, 50000): 0,   # while the run is young
             (2048, 1, 256, 0, 60, 3, 5000): 0, (2048, 300, 4096, 0, 60, 3, 50000): 1,   # too small for it at any rate; many roots
             (2048, 1, 4096, 0, 60, 16, 5000): 0, (2048, 1, 4096, 0, 10, 3, 50000): 0,
             (2048, 300, 64, 0, 10, 47, 50000): 1, (2048, 300, 64, 0, 10, 48, 50000): 0,   # few lanes with all the work
             (8, 8, 64, 0, 10, 47, 50000): 1, (8, 8, 64, 0, 32, 3, 0): 0,
             (2048, 1, 4096, 1 << 20, 60, 3, 5000): 0, (8, 8, 64, 4096, 10, 3, 0): 0}
    src = tmp_path / "spreads.cpp"
    src.write_text("""#include "host_wave.h"
#include "lane_device.h"
int main() {
  unsigned w, n, t, l, r, i, age;
  while (scanf("%u %u %u %u %u %u %u", &w, &n, &t, &l, &r, &i, &age) == 7)
    printf("%d\\n", (int)tdf::lane_spreads(w, n, t, l, r, i, [&] { return age; }));
}
""")
    exe = tmp_path / "spreads"
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "tests"),
                    str(src), "-o", str(exe)], check=True)
    text = "".join("%d %d %d %d %d %d %d\n" % c for c in cases)
    got = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout.split()
    assert dict(zip(cases, map(int, got))) == cases
