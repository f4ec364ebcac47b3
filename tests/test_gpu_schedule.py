"""How the levels of a batch are dealt to launches (level launches, tails, the chain of deep instances), as tdf_stats
reports it, on batches whose levels lie unevenly: parity with the oracle at the bars of the other bf16 tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from paper_2410_20225_amd import tdf  # noqa: E402
from tdf_workloads import make_config, SplitMix64  # noqa: E402
from tdf_workloads.trees import complete_tree, left_chain_tree, random_split_tree, build_forest  # noqa: E402
from gpu_util import TreeRun, run_oracle_tree, rel_fro  # noqa: E402

FWD, BWD, TAIL_FWD, TAIL_BWD = (tdf.PHASES.index(n) for n in ("cells_fwd", "cells_bwd", "tail_fwd", "tail_bwd"))


def _case(cfg, shapes, hidden=64):
    c = make_config(cfg, n_trees=len(shapes), max_leaves=4, hidden=hidden, vocab=300)
    rng = SplitMix64(5)
    c["forest"] = build_forest(shapes, lambda n: rng.randint(0, c["V"] - 1, n))
    c["labels"] = rng.randint(0, 4, len(shapes))
    return c


def _train(c, times=1):
    """The statistics of the evaluations, whose results are the oracle's."""
    F = c["forest"]
    dy = np.full(F.n_trees, 1.0 / F.n_trees)
    ref = run_oracle_tree(c, head=True, grad=True, dy=dy)
    run = TreeRun(c, head=True, grad=True, stats_level=0)
    all_stats = []
    for _ in range(times):
        all_stats.append(run.run(dy)[1])
        assert rel_fro(run.out_f32.cpu().numpy(), np.array(ref["out"])) < 2e-2
        for name, t in (("dW", run.dW), ("db", run.db), ("dE", run.dE)):
            assert rel_fro(t.cpu().numpy(), ref["grads"][name]) < 2e-2, name
        assert all_stats[-1].n_grad_firings == F.n_nodes and all_stats[-1].n_grad_not_once == 0
    return all_stats


SHALLOW = [random_split_tree(12 + b % 13, SplitMix64(b)) for b in range(40)]


@pytest.mark.parametrize("cfg", [3, 4])
def test_both_tails_of_a_batch_with_deep_instances_are_in_the_phases(cfg):
    st, = _train(_case(cfg, SHALLOW + [left_chain_tree(60 + b) for b in range(4)]))
    assert st.deep_split and st.tail_used
    # the chain's launches, and the other instances' levels (here all of them a tail) beside or behind it
    assert st.phase_launches[TAIL_FWD] == 1 and st.phase_launches[TAIL_BWD] == 2
    assert st.phase_launches[FWD] == st.n_wide_waves + 1 and st.phase_launches[BWD] == 2 * st.n_wide_waves + 2
    assert st.phase_ms[FWD] > 0.005 and st.phase_ms[BWD] > 0.005   # (some ten levels of a microsecond and more)


@pytest.mark.parametrize("cfg", [3, 4])
@pytest.mark.parametrize("shallow,levels", [([], 0), ([left_chain_tree(1)], 0), ([left_chain_tree(2)] * 3, 1),
                                            ([left_chain_tree(5)], 4), ([left_chain_tree(9)], 8)])
def test_shallow_instances_that_end_early_beside_deep_ones(cfg, shallow, levels):
    # nothing is launched for levels that only deep instances have: level launches up to three levels, else a tail of its own
    st, = _train(_case(cfg, shallow + [left_chain_tree(50 + b) for b in range(9)]))
    assert st.deep_split and st.tail_used and st.n_waves == 57
    assert st.n_wide_waves == (levels if levels < 4 else 0)
    assert st.phase_launches[FWD] == (levels if levels < 4 else 1)
    assert st.phase_launches[BWD] == 2 * st.phase_launches[FWD]


@pytest.mark.parametrize("cfg", [3, 4])
def test_dies_without_a_cell_hold_nobody_up(cfg):
    # chains on one die of eight, and the same chains on all of them: the launches over all levels last as long
    times = []
    for deep in ([7], range(8)):
        shapes = [left_chain_tree(100) if b in deep else left_chain_tree(3) for b in range(8)]
        all_stats = _train(_case(cfg, shapes), times=5)
        assert all(st.n_machines == 8 and st.deep_split for st in all_stats)
        times.append([min(st.phase_ms[ph] for st in all_stats) for ph in (TAIL_FWD, TAIL_BWD)])
    for one, all_ in zip(*times):
        assert one < 1.5 * all_, times


@pytest.mark.parametrize("cfg,hidden,trees,wide", [
    (3, 512, 1, 2), (3, 512, 2, 1), (3, 512, 8, 0),   # 1,024 cells of the first level on a die, 512, 256: its three groups take 384
    (4, 256, 1, 3), (3, 64, 1, 0)])   # TreeLSTM, three groups that take 240; TreeRNN of 64 units: a die takes 1,024
def test_levels_that_lie_on_few_dies_are_launched_over_all_of_them(cfg, hidden, trees, wide):
    c = _case(cfg, [complete_tree(2048 if trees == 1 else 1024 if trees == 2 else 512)] * trees, hidden=hidden)
    run = TreeRun(c, head=True, grad=False, stats_level=0)
    st, stats = run.run()
    assert stats.n_machines == trees and stats.tail_used and stats.n_wide_waves == wide


@pytest.mark.parametrize("cfg,others", [(3, 0), (4, 0), (3, 7), (4, 7)])
def test_the_gradient_tail_may_begin_above_the_forward_one(cfg, others):
    # a complete tree's levels of 1,024 cells and fewer: all of them a tail forward, the first one (TreeRNN: none) launched
    # in the gradient pass, which has fewer workgroups for it; roots in that level too
    st, = _train(_case(cfg, [complete_tree(2048)] + [left_chain_tree(2)] * others))
    assert st.n_waves == 11 and st.tail_used and st.n_wide_waves == 0
    assert st.phase_launches[TAIL_FWD] == 1 and st.phase_launches[TAIL_BWD] == 2
    assert st.phase_launches[BWD] == (0 if cfg == 3 else 2)


def _on_top(shape, n):
    """The tree `shape` under a spine of n cells, each with a leaf on the right."""
    left, right = shape
    m = left.size
    up = np.arange(n)
    l = np.concatenate([np.append(up[1:], 2 * n), np.full(n, -1), np.where(left >= 0, left + 2 * n, -1)])
    r = np.concatenate([up + n, np.full(n, -1), np.where(right >= 0, right + 2 * n, -1)])
    assert l.size == m + 2 * n
    return l, r


@pytest.mark.parametrize("cfg,hidden,beside,fwd,bwd", [(3, 256, "0", 1, 2), (4, 128, "0", 1, 2), (3, 256, "1", 1, 2), (4, 128, "1", 2, 2)])
def test_wide_levels_of_deep_instances_are_launched_over_all_dies(cfg, hidden, beside, fwd, bwd, monkeypatch):
    # levels of 1,024 and 512 cells on one die: on 32 compute units a die a chain takes 896 and 480 (TreeRNN), 560 and 384; on the
    # 20 it has beside other instances 512 and 320, 320 and 256
    monkeypatch.setenv("TDF_DEEP_BESIDE", beside)
    st, = _train(_case(cfg, [_on_top(complete_tree(2048), 30)] + SHALLOW[:9], hidden=hidden))
    assert st.deep_split == 1 + int(beside) and st.n_waves == 41
    assert st.phase_launches[TAIL_FWD] == fwd + 1 and st.phase_launches[TAIL_BWD] == 2 * bwd + 2
