"""The view table and the bounds of its views, built by array operations for
batches of integer arrays, against the element-by-element forms (no GPU)."""
import numpy as np
import pytest

from paper_2603_08661_amd import _binding as B


def columns(n, seed, dtype):
    r = np.random.default_rng(seed)
    W, H = r.integers(3, 3000, n), r.integers(3, 2000, n)
    ino = r.permutation(np.cumsum(3 * W * H))
    return W.astype(dtype), H.astype(dtype), ino.astype(np.int64), (ino // 2).astype(np.int64)


@pytest.mark.parametrize("n", [1, B._FEW_VIEWS, B._FEW_VIEWS + 1, 300])
@pytest.mark.parametrize("dtype", [np.int32, np.int64, np.uint16])
@pytest.mark.parametrize("stride", [1, 2])
def test_table_and_extents_equal_the_loops(n, dtype, stride):
    cols = [np.repeat(c, stride)[::stride] for c in columns(n, 7 * n + stride, dtype)]
    tab, m = B.view_table(*cols)
    ref, k = B.view_table(*[[int(x) for x in c] for c in cols])
    assert m == k == n and bytes(tab) == bytes(ref)
    want = (max(v.in_offset + 3 * v.width * v.height for v in ref),
            max(v.out_offset + v.width * v.height for v in ref))
    assert B._extents(tab, n) == want


@pytest.mark.parametrize("bad", [(2 ** 31 - 1, 2 ** 31 - 1, 0, 0), (8, 8, 2 ** 62, 0), (8, 8, 0, 2 ** 62)])
def test_bounds_past_float64_are_exact(bad):
    cols = [np.append(c, b) for c, b in zip(columns(20, 3, np.int64), bad)]
    tab, n = B.view_table(*cols)
    assert B._extents(tab, n) == (max(v.in_offset + 3 * v.width * v.height for v in tab),
                                  max(v.out_offset + v.width * v.height for v in tab))
