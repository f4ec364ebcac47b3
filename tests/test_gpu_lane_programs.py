"""The programs of tests/lane_programs.py on the GPU: the depth-first lanes against plain Python references and against
the step machine (the same call with TDF_NO_LANES)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2410_20225_amd import tdf  # noqa: E402
from lane_programs import VECTOR  # noqa: E402
from gpu_util import DEV  # noqa: E402


@pytest.mark.parametrize("name", list(VECTOR))
def test_vector_results(name, monkeypatch):
    prog, forest, args, ref = VECTOR[name]()
    E = torch.randn(50, 64, device=DEV)
    on = lambda v, d: torch.tensor(v, dtype=d, device=DEV)  # noqa: E731
    keep = dict(args=on(args, torch.int64).reshape(-1), E=E, **{k: on(v, torch.int32) for k, v in forest.arrays().items()})
    inp = tdf.make_inputs(len(args), n_args=1, max_tags=4096, stats_level=0, dtype=tdf.F32, hidden=64, vocab=50, **keep)
    g = tdf.graph_build(*prog)
    seen = []
    for no_lanes in (False, True):
        if no_lanes:
            monkeypatch.setenv("TDF_NO_LANES", "1")
        out = torch.zeros(len(args), 64, device=DEV)
        ws = torch.empty(tdf.workspace_size(g, inp), dtype=torch.uint8, device=DEV)
        st, stats = tdf.eval(g, inp, ws, out_h=out)
        assert stats.repeats == 0 and torch.equal(out, E[[ref(*a) for a in args]])
        seen.append((stats.n_tags, stats.n_tokens, stats.n_leaf_rows, stats.n_cell_rows, stats.max_tag_depth))
    assert seen[0] == seen[1]
