"""The kernels' mask arithmetic (csrc/mask.h), compiled for the host, against the definition of every mask: the key range of
a row, the row range of a key, and the ranges by which a wave of 32 keys skips a block of query rows or computes it
without a mask."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2603_11101_amd import binding as va

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_11101_amd", "csrc")
SOURCE = """
#include <algorithm>
#define VA_DEV inline
using std::max;
using std::min;
#include "mask.h"
extern "C" void bounds(int P, int P2, int L, int mode, int rows, int* lo, int* vis, int* first, int* end, int* blocks) {
    const va::MaskBounds m(P, P2, L, mode);
    for (int i = 0; i < L; ++i) { lo[i] = m.lo(i); vis[i] = m.vis(i); first[i] = m.first_row(i); end[i] = m.end_row(i); }
    for (int w = 0; w < rows / 32; ++w) {
        const va::KeyBlock k(m, 32 * w);
        const int b[4] = {k.some_from, k.some_end, k.all_from, k.all_end};
        for (int e = 0; e < 4; ++e) blocks[4 * w + e] = b[e];
    }
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("mask")
    (d / "mask.cpp").write_text(SOURCE)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", CSRC, str(d / "mask.cpp"), "-o", str(d / "mask.so")])
    return ctypes.CDLL(str(d / "mask.so"))


def visible_pairs(mode, L, P, P2):
    i, j = np.arange(L)[:, None], np.arange(L)[None, :]
    if mode == va.VA_MASK_CAUSAL:
        return j <= i
    if mode == va.VA_MASK_SLIDING_WINDOW:
        return (j <= i) & (j > i - P)
    if mode == va.VA_MASK_PREFIX_LM_CAUSAL:
        return np.where(i < P, j < P, j <= i)
    if mode == va.VA_MASK_PREFIX_LM:
        return np.where(i < P, j < P, j < L)
    return np.where(i < P, j < P, np.where(i < P2, j < P2, j < L))


@pytest.mark.parametrize("mode", [va.VA_MASK_CAUSAL, va.VA_MASK_PREFIX_LM, va.VA_MASK_PREFIX_LM_CAUSAL, va.VA_MASK_THREE_BLOCK,
                                  va.VA_MASK_SLIDING_WINDOW])
@pytest.mark.parametrize("L", [1, 31, 32, 33, 64, 65, 95, 128, 129, 200])
def test_bounds_are_those_of_the_definition(lib, mode, L):
    cuts = sorted({x for x in (0, 1, 17, 31, 32, 33, 64, 90, L // 2, L - 1, L) if 0 <= x <= L})
    if mode == va.VA_MASK_CAUSAL:
        ends = [(-1, -1)]
    elif mode == va.VA_MASK_SLIDING_WINDOW:
        ends = [(w, -1) for w in [*cuts, L + 1, 1000, 2 ** 31 - 1] if w >= 1]
    elif mode == va.VA_MASK_THREE_BLOCK:
        ends = [(a, b) for a in cuts for b in cuts if a <= b]
    else:
        ends = [(a, -1) for a in cuts]
    rows = (L + 127) // 128 * 128  # a key tile is 128 rows: its last waves may lie past the sample
    for P, P2 in ends:
        lo, vis, first, end = (np.zeros(L, dtype=np.int32) for _ in range(4))
        blocks = np.zeros((rows // 32, 4), dtype=np.int32)
        lib.bounds(P, P2, L, mode, rows, *(ctypes.c_void_p(x.ctypes.data) for x in (lo, vis, first, end, blocks)))
        seen = visible_pairs(mode, L, P, P2)
        r = np.arange(L)
        assert np.array_equal((r[None, :] >= lo[:, None]) & (r[None, :] < vis[:, None]), seen), (P, P2)
        assert np.array_equal((r[:, None] >= first[None, :]) & (r[:, None] < end[None, :]), seen), (P, P2)
        for w, (some_from, some_end, all_from, all_end) in enumerate(blocks):
            keys = seen[:, 32 * w:32 * w + 32]
            # exactly the rows that see a key: a block of rows is skipped if it holds none of them, not computed and dropped
            assert np.array_equal((r >= some_from) & (r < some_end), keys.any(axis=1)), (P, P2, w)
            if keys.shape[1]:
                assert np.array_equal((r >= all_from) & (r < all_end), keys.all(axis=1)), (P, P2, w)
