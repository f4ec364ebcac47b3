"""The check that a level tail makes of rows that others write (unwritten.h): a row is complete when none of its elements is all
ones.  One element at a time, at every place of a row of one and of several chunks, with all 65,536 patterns of a 16-bit element, among
neighbours whose own patterns come close."""
import ctypes
import os

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2410_20225_amd import tdf  # noqa: E402

DEV = "cuda:0"


@pytest.fixture(scope="module")
def waiting():
    hooks = ctypes.CDLL(os.path.join(os.path.dirname(tdf.__file__), "libtdf_hooks.so"))
    fn = hooks.tdf_test_unwritten
    fn.argtypes = [ctypes.c_int, ctypes.c_void_p, ctypes.c_uint32, ctypes.c_uint32, ctypes.c_void_p, ctypes.c_void_p]

    def run(dtype, rows):   # rows: unsigned elements [n, chunks * elements of a chunk]
        t = torch.from_numpy(rows.view(np.int32)).to(DEV)
        out = torch.full((len(rows),), -1, dtype=torch.int32, device=DEV)
        torch.cuda.synchronize()
        assert fn(dtype, t.data_ptr(), t.numel() // len(rows) // 4, len(rows), out.data_ptr(), None) == tdf.OK
        torch.cuda.synchronize()
        return out.cpu().numpy()
    return run


@pytest.mark.parametrize("chunks", [1, 5])
@pytest.mark.parametrize("others", [0x0000, 0x7FFF, 0x8000, 0xFFFE, None])
def test_16_bit_elements(waiting, chunks, others):
    rng = np.random.default_rng(1)
    for place in range(8 * chunks):
        rows = rng.integers(0, 0xFFFF, (65536, 8 * chunks)).astype(np.uint16) if others is None else np.full((65536, 8 * chunks), others, np.uint16)
        rows[:, place] = np.arange(65536)
        got = waiting(tdf.BF16, np.ascontiguousarray(rows))
        assert np.array_equal(got, (rows == 0xFFFF).any(axis=1)), place


@pytest.mark.parametrize("chunks", [1, 5])
def test_32_bit_elements(waiting, chunks):
    rng = np.random.default_rng(2)
    some = np.array([0, 1, 0x7FFFFFFF, 0x80000000, 0xFFFF, 0xFFFF0000, 0xFFFFFFFE, 0xFFFEFFFF, 0xFFFFFFFF], np.uint32)
    for place in range(4 * chunks):
        rows = rng.integers(0, 0xFFFFFFFF, (len(some) * 50, 4 * chunks), dtype=np.uint32)
        rows[::2] = some[:-1][rng.integers(0, len(some) - 1, rows[::2].shape)]
        rows[:, place] = np.tile(some, 50)
        assert np.array_equal(waiting(tdf.F32, rows), (rows == 0xFFFFFFFF).any(axis=1)), place


def test_two_unwritten_halves_of_a_word(waiting):
    rows = np.full((16, 8), 0x1234, np.uint16)
    for k in range(8):
        rows[k, k] = 0xFFFF
        rows[8 + k, [k, k ^ 1]] = 0xFFFF
    assert waiting(tdf.BF16, rows).all()
