"""The programs of tests/lane_programs.py on the GPU: the depth-first lanes against plain Python references and against
the step machine (the same call with TDF_NO_LANES)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2410_20225_amd import tdf  # noqa: E402
from lane_programs import BAD_INDEX, INTEGER, VECTOR  # noqa: E402
from gpu_util import DEV  # noqa: E402


def _inputs(forest, args, **more):
    on = lambda v, d: torch.tensor(v, dtype=d, device=DEV)  # noqa: E731
    keep = {k: on(v, torch.int32) for k, v in forest.arrays().items()}
    if "E" in more:
        keep["E"] = more.pop("E")
    keep["args"] = on(args, torch.int64).reshape(-1)
    return keep, tdf.make_inputs(len(args), n_args=len(args[0]), max_tags=4096, stats_level=0, **keep, **more)


def _both_ways(prog, inp, out, monkeypatch, check):
    """The call on the lanes and on the step machine; check(stats) after each."""
    g = tdf.graph_build(*prog)
    seen = []
    for no_lanes in (False, True):
        if no_lanes:
            monkeypatch.setenv("TDF_NO_LANES", "1")
        for t in out.values():
            t.fill_(-77)
        ws = torch.empty(tdf.workspace_size(g, inp), dtype=torch.uint8, device=DEV)
        st, stats = tdf.eval(g, inp, ws, **out)
        assert stats.repeats == 0
        check()
        seen.append((stats.n_tags, stats.n_tokens, stats.n_leaf_rows, stats.n_cell_rows, stats.max_tag_depth))
    assert seen[0] == seen[1]


@pytest.mark.parametrize("name", list(VECTOR))
def test_vector_results(name, monkeypatch):
    prog, forest, args, ref = VECTOR[name]()
    E = torch.randn(50, 64, device=DEV)
    keep, inp = _inputs(forest, args, E=E, dtype=tdf.F32, hidden=64, vocab=50)
    out = torch.zeros(len(args), 64, device=DEV)
    want = E[[ref(*a) for a in args]]

    def check():
        assert torch.equal(out, want)
    _both_ways(prog, inp, dict(out_h=out), monkeypatch, check)


@pytest.mark.parametrize("name", list(INTEGER))
def test_integer_results(name, monkeypatch):
    prog, forest, args, ref = INTEGER[name]()
    keep, inp = _inputs(forest, args)
    out = torch.zeros(len(args), dtype=torch.int64, device=DEV)
    want = [ref(*a) for a in args]

    def check():
        assert out.cpu().tolist() == want
    _both_ways(prog, inp, dict(out_i64=out), monkeypatch, check)


@pytest.mark.parametrize("name", list(BAD_INDEX))
def test_nodes_that_do_not_exist_are_refused(name):
    # (every accessor checks its index before it reads: tests/test_lanes_on_cpu.py)
    prog, forest, bad = BAD_INDEX[name]()
    g = tdf.graph_build(*prog)
    for v in bad:
        keep, inp = _inputs(forest, [(v,)])
        ws = torch.empty(tdf.workspace_size(g, inp), dtype=torch.uint8, device=DEV)
        st, _ = tdf.eval(g, inp, ws, out_i64=torch.zeros(1, dtype=torch.int64, device=DEV), check=False)
        assert st == tdf.ERR_BAD_ARG, v
