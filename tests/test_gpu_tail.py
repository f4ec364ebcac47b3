"""The launches in which every die walks the narrow levels on its own (k_tail_fwd, k_tail_bwd): widths at which a
wave's share of the reduction, or where its weights are kept, changes; levels of one cell and of several row tiles;
NaNs, whose bit patterns these launches use for rows that are still to be written."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2410_20225_amd import tdf  # noqa: E402
from tdf_workloads import make_config  # noqa: E402
from gpu_util import TreeRun, run_oracle_tree, rel_fro  # noqa: E402

# (workload recipe, hidden, trees, most leaves): 2 TreeRNN fp32, 3 TreeRNN bf16, 4 TreeLSTM bf16.  The padded width is a
# multiple of 64; weights stay in registers up to 512 units (TreeRNN forward: 1024), and are fetched per tile beyond.
FORWARD = [(2, 33, 1, 9), (2, 256, 60, 12), (2, 520, 20, 10), (2, 1040, 6, 8), (3, 64, 300, 14), (3, 192, 40, 12), (3, 512, 9, 40),
           (3, 1056, 6, 8), (4, 60, 1, 30), (4, 150, 50, 12), (4, 320, 40, 10), (4, 512, 20, 9), (4, 580, 8, 8)]


@pytest.mark.parametrize("cfg,hidden,trees,leaves", FORWARD)
def test_forward_and_gradients_at_the_widths_where_the_tiles_change(cfg, hidden, trees, leaves):
    c = make_config(cfg, n_trees=trees, max_leaves=leaves, hidden=hidden, vocab=200)
    B = c["forest"].n_trees
    dy = np.full(B, 1.0 / B)
    ref = run_oracle_tree(c, head=True, grad=True, dy=dy)
    run = TreeRun(c, head=True, grad=True, stats_level=0)
    # fp32: sums over at most 2 x 1088 terms through at most 40 contracting levels; bf16: the suite's bar for rounded states
    tol = 1e-5 if cfg == 2 else 2e-2
    for _ in range(2):
        st, stats = run.run(dy)
        assert stats.n_waves < 4 or stats.tail_used == 1
        assert stats.n_grad_not_once == 0 and stats.n_grad_firings == c["forest"].n_nodes
        assert rel_fro(run.out_f32.cpu().numpy(), np.array(ref["out"])) < tol
        for name, t in (("dW", run.dW), ("db", run.db), ("dE", run.dE)):
            assert rel_fro(t.cpu().numpy(), ref["grads"][name]) < tol, name


# A die's level of more than 16 cells is several tiles for one workgroup, the last of which is not full: those behind the first find
# their rows looked for already.
@pytest.mark.parametrize("bf16", [True, False], ids=["bf16", "fp32"])
@pytest.mark.parametrize("hidden,trees,leaves", [(40, 8, 70), (64, 130, 12), (150, 190, 30)])
def test_gradients_of_levels_of_several_tiles(hidden, trees, leaves, bf16):
    c = make_config(4, n_trees=trees, max_leaves=leaves, hidden=hidden, vocab=200)
    c["bf16"] = bf16
    B = c["forest"].n_trees
    dy = np.full(B, 1.0 / B)
    ref = run_oracle_tree(c, head=True, grad=True, dy=dy)
    run = TreeRun(c, head=True, grad=True, stats_level=0)
    tol = 2e-2 if bf16 else 2e-5   # (the bars of the other gradient tests)
    for _ in range(2):
        st, stats = run.run(dy)
        assert stats.tail_used == 1 and stats.repeats == 0
        assert stats.n_grad_not_once == 0 and stats.n_grad_firings == c["forest"].n_nodes
        assert rel_fro(run.out_f32.cpu().numpy(), np.array(ref["out"])) < tol
        for name, t in (("dW", run.dW), ("db", run.db), ("dE", run.dE)):
            assert rel_fro(t.cpu().numpy(), ref["grads"][name]) < tol, name


# ... and where that is so on average of the levels, which takes the kernel that looks: cells of a level on a die in rows of
# 16, a row for a group of workgroups, one for each column tile, of which a die's 32 compute units hold 31 workgroups.
@pytest.mark.parametrize("hidden,trees,leaves,bf16", [(250, 300, 12, True), (180, 560, 10, True), (120, 800, 10, False)])
def test_gradients_where_a_workgroup_has_several_tiles_of_a_level(hidden, trees, leaves, bf16):
    c = make_config(4, n_trees=trees, max_leaves=leaves, hidden=hidden, vocab=200)
    c["bf16"] = bf16
    B = c["forest"].n_trees
    dy = np.full(B, 1.0 / B)
    ref = run_oracle_tree(c, head=True, grad=True, dy=dy)
    run = TreeRun(c, head=True, grad=True, stats_level=0)
    tol = 2e-2 if bf16 else 2e-5
    for _ in range(2):
        st, stats = run.run(dy)
        groups = 31 // (2 * ((hidden + 63) // 64 * 64) // 32)
        assert stats.tail_used == 1 and stats.n_wide_waves == 0 and stats.n_cell_rows > 8 * 16 * groups * stats.n_waves
        assert stats.n_grad_not_once == 0 and stats.n_grad_firings == c["forest"].n_nodes
        assert rel_fro(run.out_f32.cpu().numpy(), np.array(ref["out"])) < tol
        for name, t in (("dW", run.dW), ("db", run.db), ("dE", run.dE)):
            assert rel_fro(t.cpu().numpy(), ref["grads"][name]) < tol, name


@pytest.mark.parametrize("cfg", [3, 4])
def test_offsets_beyond_32_bits(cfg, monkeypatch):
    import os
    hooks = tdf.load_library(os.path.join(os.path.dirname(tdf.__file__), "libtdf_hooks.so"))
    monkeypatch.setenv("TDF_TEST_WIDE_OFFSETS", "1")
    c = make_config(cfg, n_trees=30, max_leaves=30, hidden=96, vocab=200)
    B = c["forest"].n_trees
    dy = np.full(B, 1.0 / B)
    ref = run_oracle_tree(c, head=True, grad=True, dy=dy)
    with tdf.use_library(hooks):
        run = TreeRun(c, head=True, grad=True, stats_level=0)
        st, stats = run.run(dy)
    assert stats.tail_used == 1
    assert rel_fro(run.out_f32.cpu().numpy(), np.array(ref["out"])) < 2e-2
    for name, t in (("dW", run.dW), ("db", run.db), ("dE", run.dE)):
        assert rel_fro(t.cpu().numpy(), ref["grads"][name]) < 2e-2, name


@pytest.mark.parametrize("cfg,hidden", [(2, 256), (3, 512), (4, 512)])
def test_offsets_beyond_32_bits_at_the_widest_rows_that_share_a_compute_unit(cfg, hidden, monkeypatch):
    # (rows that are there before the launch and rows that are waited for, in one tile; as many levels in the tail as with 32 bits)
    import os
    hooks = tdf.load_library(os.path.join(os.path.dirname(tdf.__file__), "libtdf_hooks.so"))
    c = make_config(cfg, n_trees=200, max_leaves=12, hidden=hidden, vocab=200)
    got = []
    for wide in (False, True):
        if wide:
            monkeypatch.setenv("TDF_TEST_WIDE_OFFSETS", "1")
        with tdf.use_library(hooks):
            run = TreeRun(c, head=True, grad=False, stats_level=0)
            for _ in range(2):
                st, stats = run.run()
                assert stats.tail_used == 1 and stats.repeats == 0
        got.append((run.out_f32.clone(), stats.n_wide_waves))
    assert torch.equal(got[0][0], got[1][0]) and got[0][1] == got[1][1]


@pytest.mark.parametrize("pattern", [-1, 0x7FC0])
@pytest.mark.parametrize("cfg", [3, 4])
def test_nans_pass_through(cfg, pattern):
    # an embedding row of NaNs (all bits set: the pattern that stands for a row that is still to be written, and another
    # one): nothing waits, and no other tree's loss is a NaN.  (The 16-bit path's tanh of a TreeRNN cell clamps its
    # argument, which makes a number of a NaN; the gates of a TreeLSTM cell keep it.)
    c = make_config(cfg, n_trees=40, max_leaves=16, hidden=64, vocab=60)
    F = c["forest"]
    B = F.n_trees
    run = TreeRun(c, head=True, grad=True, stats_level=0)
    run.t_E.view(torch.int16)[7].fill_(pattern)
    st, stats = run.run(np.full(B, 1.0 / B))
    assert stats.tail_used == 1 and stats.n_grad_not_once == 0
    roots = np.asarray(F.roots)
    tree_of = np.full(F.n_nodes, -1)
    for b in range(B):
        todo = [int(roots[b])]
        while todo:
            v = todo.pop()
            tree_of[v] = b
            if F.left[v] >= 0:
                todo += [int(F.left[v]), int(F.right[v])]
    has = np.zeros(B, bool)
    has[tree_of[np.asarray(F.token) == 7]] = True
    assert has.any() and not has.all()
    nan = np.isnan(run.out_f32.cpu().numpy())
    assert not nan[~has].any()
    assert cfg == 3 or nan[has].all()


@pytest.mark.parametrize("where", ["embedding", "dy"])
@pytest.mark.parametrize("cfg,bf16", [(2, False), (3, True), (4, False), (4, True)])
def test_nans_pass_through_both_passes(cfg, bf16, where):
    # A NaN with all bits set enters a tree, as a row of E or as the gradient of its loss, and flows through the states, dz and
    # dc that the tails wait for: nothing waits for good, and what no such tree has part in is a number.
    c = make_config(cfg, n_trees=40, max_leaves=16, hidden=64, vocab=400)
    c["bf16"] = bf16
    F = c["forest"]
    B, rnd = F.n_trees, np.random.default_rng(1)
    tree_of = np.full(F.n_nodes, -1)
    for b in range(B):   # (a tree's nodes are contiguous from its root)
        tree_of[F.roots[b]:F.roots[b] + 2 * F.n_leaves[b] - 1] = b
    leaf = F.token >= 0
    bad = np.zeros(B, bool)
    bad[np.flatnonzero(F.n_leaves >= 4)[:5]] = True
    # the bad trees' tokens are theirs alone
    F.token[leaf] = np.where(bad[tree_of[leaf]], rnd.integers(300, 400, leaf.sum()), rnd.integers(0, 300, leaf.sum()))
    run = TreeRun(c, head=True, grad=True, stats_level=0)
    dy = torch.full((B,), 1.0 / B, dtype=torch.float32, device="cuda:0")
    if where == "embedding":
        deepest = [int(F.token[(tree_of == b) & leaf][0]) for b in np.flatnonzero(bad)]
        run.t_E.view(torch.int16 if bf16 else torch.int32)[deepest] = -1
    else:
        dy.view(torch.int32)[torch.tensor(bad, device="cuda:0")] = -1
    for _ in range(2):   # (the second evaluation finds the first one's rows in the workspace)
        st, stats = tdf.eval_grad(run.graph, run.inputs, dy, run.ws, run.dW, run.db, run.dE, out_f32=run.out_f32)
        assert st == tdf.OK and stats.tail_used == 1 and stats.repeats == 0
        assert stats.n_grad_not_once == 0 and stats.n_grad_firings == F.n_nodes
        loss, dE = run.out_f32.cpu().numpy(), run.dE.cpu().numpy()
        assert not np.isnan(loss[~bad]).any() and not np.isnan(dE[:300]).any()
        # (the 16-bit tanh of a TreeRNN cell clamps its argument, which makes a number of a NaN)
        clamped = cfg == 3 and bf16
        if where == "embedding":
            assert clamped or np.isnan(loss[bad]).all()
        else:
            assert not np.isnan(loss).any()
        if where == "dy" or not clamped:   # every leaf of a bad tree gets its gradient through NaNs
            assert np.isnan(dE[np.unique(F.token[leaf & bad[tree_of]])]).all()
            assert np.isnan(run.dW.cpu().numpy()).any() and np.isnan(run.db.cpu().numpy()).any()
