"""The one-launch selection + compaction's row copy: every vector unit (16 to 1
bytes), planes, and odd numbers of units, against torch's row gather."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, say
from paper_2608_26806_amd import avtp as A
from paper_2608_26806_amd.workloads import build_layout

pytestmark = pytest.mark.gpu


# (images, width: rows `width` times as wide; the wide ones are copied row by row,
# the others as one run of units, all of them in one launch)
@pytest.mark.parametrize("imgs, width", [([[1]], 1), ([[49, 3]], 1), ([[65], [200, 31, 7]], 1),
                                         ([[1]], 39), ([[49, 3]], 39), ([[65], [200, 31, 7]], 7)], ids=str)
def test_rows_of_every_unit_width_and_planes(imgs, width):
    need_gpu()
    say(f"fused copy units {imgs}, width {width}")
    lay = build_layout(imgs, 1, 5, 50)
    dl = A.DeviceLayout(lay)
    g = torch.Generator(device="cuda").manual_seed(7)

    def draw(*s, dt=torch.uint8):
        """Every byte of every element drawn on its own."""
        es = dt.itemsize
        return torch.randint(0, 256, (*s, es), generator=g, device="cuda").to(torch.uint8).view(dt).view(s)

    N, w = dl.N_tok, width
    srcs = [(draw(N, w), 0), (draw(N, 3 * w, dt=torch.int16), 0), (draw(3, N, 5 * w, dt=torch.int32), 1),
            (draw(3, N, dt=torch.int64), 1), (draw(N, 8 * w, dt=torch.int16), 0),
            (draw(N, 2, 264 * w, dt=torch.int16), 0), (draw(2, N, 7 * w), 1), (draw(N, 34 * w, dt=torch.int32), 0)]
    row_bytes = sum(s.numel() * s.element_size() // N for s, _ in srcs)
    assert 2 * dl.N_out * row_bytes <= 4 << 20
    pairs = []
    for s, td in srcs:
        shape = list(s.shape)
        shape[td] = dl.N_out
        # 0xA5 in every byte: a part of a unit that is not copied shows
        fill = torch.full((*shape, s.element_size()), 0xA5, dtype=torch.uint8, device="cuda")
        pairs.append((s, fill.view(s.dtype).view(shape), td))
    scores = torch.rand(N, generator=g, device="cuda")
    budget = torch.tensor([n // 2 for seq in imgs for n in seq], dtype=torch.int32, device="cuda")
    # keep totals of the layout are rounded per sequence: give the rest to the last image
    lens = [n for seq in imgs for n in seq]
    i = 0
    for b, seq in enumerate(imgs):
        i += len(seq)
        used = sum(int(budget[j]) for j in range(i - len(seq), i))
        budget[i - 1] = min(lens[i - 1], int(budget[i - 1]) + int(lay.keep_total[b]) - used)
    keep, cu = A.select_compact(dl, scores, budget, pairs)
    n = int(cu[-1])
    idx = keep[:n].long()
    assert n == lay.T_tot + int(budget.sum()) and np.all(np.diff(idx.cpu().numpy()) > 0)
    for s, d, td in pairs:
        assert torch.equal(d.narrow(td, 0, n), s.index_select(td, idx)), (s.dtype, tuple(s.shape))


@pytest.mark.parametrize("n, row_bytes", [(64, 42816), (64, 42815), (729, 5393)])
def test_one_launch_is_not_slower_than_two_below_its_limit(n, row_bytes):
    """Rows of many vector units just below the 4 MiB that the one launch serves:
    it must not take longer than the selection and the compaction one after the
    other (row by row it takes less; with every unit looked up on its own it
    took up to six times as long)."""
    need_gpu()
    say(f"one launch against two, {n} tokens, rows of {row_bytes} bytes")
    lay = build_layout([[n]], 0, 16, 50)
    dl = A.DeviceLayout(lay)
    src = torch.randint(0, 256, (dl.N_tok, row_bytes), device="cuda").to(torch.uint8)
    dst = torch.zeros(dl.N_out, row_bytes, dtype=torch.uint8, device="cuda")
    assert 2 * dl.N_out * row_bytes <= 4 << 20
    scores = torch.rand(dl.N_tok, device="cuda")
    budget = torch.tensor(lay.keep_total, dtype=torch.int32, device="cuda")
    keep = torch.empty(dl.N_out, dtype=torch.int32, device="cuda")
    cu = torch.empty(2, dtype=torch.int32, device="cuda")
    ts = A.TensorSet([(src, dst, 0)])

    def one():
        A.select_compact(dl, scores, budget, ts, keep_idx=keep, cu_out=cu)

    def two():
        A.select(dl, scores, budget, keep_idx=keep, cu_out=cu)
        A.compact(dl, keep, ts)

    graphs = []
    for call in (one, two):
        call()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                call()
        graphs.append(g)

    def us(g):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        return a.elapsed_time(b) * 50

    runs = [[us(g) for g in graphs] for _ in range(15)]
    t = [min(r[i] for r in runs) for i in range(2)]
    say(f"one launch {t[0]:.1f} us, two {t[1]:.1f} us")
    assert torch.equal(dst, src[keep.long()])
    # (the best of 15 runs of 20 calls varies by a few per cent)
    assert t[0] < 1.25 * t[1]
