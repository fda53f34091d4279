"""The progressive driver's host part, on the CPU: its keep totals against the
rule written out, and how the next layout is put together."""
import numpy as np
import pytest
import torch

from oracle import avtp_oracle as O
from paper_2608_26806_amd import avtp as A
from paper_2608_26806_amd.progressive import keep_totals
from paper_2608_26806_amd.workloads import build_layout


@pytest.mark.parametrize("pct", [0, 1, 33, 50, 99, 100])
def test_keep_totals_with_empty_sequences_and_images(pct):
    img_len = np.array([3, 0, 1 << 20, 7, 1, 0], dtype=np.int32)
    cu_img = np.array([0, 0, 3, 3, 5, 6], dtype=np.int32)
    got = keep_totals(img_len, cu_img, pct)
    assert got.dtype == np.int32
    want = [(pct * int(img_len[a:b].sum(dtype=np.int64)) + 50) // 100 for a, b in zip(cu_img[:-1], cu_img[1:])]
    assert got.tolist() == want
    assert keep_totals(np.zeros(0, np.int32), np.array([0, 0], np.int32), pct).tolist() == [0]


def test_the_next_layout_is_built_on_one_stream_only(monkeypatch):
    """The buffer, the kernel and the two copies of DeviceLayout.pruned depend
    on each other: no argument can put the kernel on another stream than torch's
    current one, which the copies run on (host tensors; the oracle stands for
    the kernel)."""
    lay = build_layout([[5, 3], [], [7]], 1, 2, 50)
    keep, cu = O.select(lay, np.arange(lay.N_tok, dtype=np.float32), np.array([2, 2, 4], np.int32))
    nxt = O.pruned_layout(lay, keep, cu, np.zeros(3, np.int32))
    streams = []

    def kernel(dl, keep_idx, cu_out, stream=None, out=None):
        streams.append(stream)
        for n, t in out.items():
            a = np.asarray(getattr(nxt, n), dtype=np.int32)
            t[:len(a)] = torch.from_numpy(a)

    monkeypatch.setattr(A, "pruned_layout", kernel)
    args = (A.DeviceLayout(lay, host_only=True), torch.from_numpy(np.asarray(keep, np.int32)),
            torch.from_numpy(np.asarray(cu, np.int32)), lambda n, c: keep_totals(n, c, 40))
    with pytest.raises(TypeError):
        A.DeviceLayout.pruned(*args, stream=object())
    got = A.DeviceLayout.pruned(*args)
    assert streams == [None]
    for n in A.DeviceLayout.NAMES[:-1]:
        assert got.host[n].tolist() == getattr(nxt, n).tolist(), n
        assert got.device_array(n).tolist() == getattr(nxt, n).tolist(), n
    assert got.device_array("keep_total").tolist() == keep_totals(nxt.img_len, nxt.cu_img, 40).tolist()
