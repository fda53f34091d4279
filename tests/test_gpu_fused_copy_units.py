"""The one-launch selection + compaction's row copy: every vector unit (16 to 1
bytes), planes, and odd numbers of units, against torch's row gather."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, say
from paper_2608_26806_amd import avtp as A
from paper_2608_26806_amd.workloads import build_layout

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("imgs", [[[1]], [[49, 3]], [[65], [200, 31, 7]]], ids=str)
def test_rows_of_every_unit_width_and_planes(imgs):
    need_gpu()
    say(f"fused copy units {imgs}")
    lay = build_layout(imgs, 1, 5, 50)
    dl = A.DeviceLayout(lay)
    g = torch.Generator(device="cuda").manual_seed(7)
    draw = lambda *s, dt=torch.uint8: torch.randint(0, 255, s, generator=g, device="cuda").to(dt)  # noqa: E731
    N = dl.N_tok
    srcs = [(draw(N, 1), 0), (draw(N, 3, dt=torch.int16), 0), (draw(3, N, 5, dt=torch.int32), 1),
            (draw(3, N, dt=torch.int64), 1), (draw(N, 8, dt=torch.int16), 0), (draw(N, 2, 264, dt=torch.int16), 0),
            (draw(2, N, 7), 1), (draw(N, 34, dt=torch.int32), 0)]
    pairs = []
    for s, td in srcs:
        shape = list(s.shape)
        shape[td] = dl.N_out
        pairs.append((s, torch.full(shape, 99, dtype=s.dtype, device="cuda"), td))
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
