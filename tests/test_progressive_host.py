"""The progressive driver's keep totals against the rule written out, on the CPU."""
import numpy as np
import pytest

from paper_2608_26806_amd.progressive import keep_totals


@pytest.mark.parametrize("pct", [0, 1, 33, 50, 99, 100])
def test_keep_totals_with_empty_sequences_and_images(pct):
    img_len = np.array([3, 0, 1 << 20, 7, 1, 0], dtype=np.int32)
    cu_img = np.array([0, 0, 3, 3, 5, 6], dtype=np.int32)
    got = keep_totals(img_len, cu_img, pct)
    assert got.dtype == np.int32
    want = [(pct * int(img_len[a:b].sum(dtype=np.int64)) + 50) // 100 for a, b in zip(cu_img[:-1], cu_img[1:])]
    assert got.tolist() == want
    assert keep_totals(np.zeros(0, np.int32), np.array([0, 0], np.int32), pct).tolist() == [0]
