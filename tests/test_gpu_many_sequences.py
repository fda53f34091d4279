"""Batches of many sequences: the blocks that serve one image find its sequence
by looking 64 offsets up at a time, in one to three rounds.  Results against the
oracle around the edges of the rounds, empty sequences among them, and the time
against the same images in few sequences."""
import numpy as np
import pytest
import torch

from gpu_util import need_gpu, say
from oracle import avtp_oracle as O
from paper_2608_26806_amd import avtp as A
from paper_2608_26806_amd.workloads import build_layout

pytestmark = pytest.mark.gpu


def _images(B):
    """No images, one or two per sequence, of 1 to 5 tokens; the last has some."""
    return [[] if b % 3 == 1 and b + 1 < B else [1 + b % 5] if b % 2 else [2, 3] for b in range(B)]


@pytest.mark.parametrize("B", [1, 2, 63, 64, 65, 128, 4095, 4096, 4097, 4161])
def test_flags_sums_and_selection_go_to_the_right_sequence(B):
    need_gpu()
    say(f"many sequences, B={B}")
    lay = build_layout(_images(B), 0, 1, 60)
    dl = A.DeviceLayout(lay)
    rng = np.random.default_rng(B)
    h0 = rng.standard_normal((lay.N_tok, 8)).astype(np.float32)
    h1 = h0 + rng.standard_normal(h0.shape).astype(np.float32)
    marked = sorted({0, B // 2, B - 1} | {b for b in (63, 64, 4095, 4096) if b < B})
    marked = [b for b in marked if lay.cu_img[b + 1] > lay.cu_img[b]]
    for b in marked:                      # one visual token of these sequences is not a number
        h1[lay.img_start[lay.cu_img[b]]] = np.nan
    status = torch.zeros(B, dtype=torch.int32, device="cuda")
    s, isum = A.score_variation(dl, torch.from_numpy(h1).cuda(), torch.from_numpy(h0).cuda(), status=status)
    assert np.flatnonzero(status.cpu().numpy()).tolist() == marked
    sums = isum.cpu().numpy()
    assert np.flatnonzero(np.isnan(sums)).tolist() == [int(lay.cu_img[b]) for b in marked]
    s = s.cpu().numpy()
    for i in range(lay.n_img):
        a, n = int(lay.img_start[i]), int(lay.img_len[i])
        if not np.isnan(sums[i]):
            np.testing.assert_allclose(sums[i], s[a:a + n].sum(dtype=np.float64), rtol=1e-6, atol=1e-7)
    scores = rng.random(lay.N_tok).astype(np.float32)
    budget = np.array([int(rng.integers(0, n + 1)) for n in lay.img_len], np.int32)
    total = [int(budget[lay.cu_img[b]:lay.cu_img[b + 1]].sum()) for b in range(B)]
    arrays = {n: np.array(getattr(lay, n)) for n in A.DeviceLayout.NAMES}
    arrays["keep_total"] = np.array(total, np.int32)
    keep, cu = A.select(A.DeviceLayout(arrays), torch.from_numpy(scores).cuda(), torch.from_numpy(budget).cuda())
    keep_o, cu_o = O.select(lay, scores, budget)
    assert cu.tolist() == cu_o.tolist() and keep.tolist() == keep_o.tolist()


def test_many_sequences_take_no_longer_than_the_same_images_in_few():
    """4,096 images of 49 tokens and 4,096 text rows: in 4,096 sequences against
    16 (the lookup must not run through the sequences 64 at a time, each round
    waiting for the last: 2.5 times the time)."""
    need_gpu()
    say("4,096 images in 4,096 sequences and in 16")

    def call(B):
        lay = build_layout([[49] * (4096 // B)] * B, 0, 4096 // B, 50)
        dl = A.DeviceLayout(lay)
        h0, h1 = torch.randn(2, lay.N_tok, 64, device="cuda").unbind(0)
        out = torch.empty(lay.N_tok, device="cuda"), torch.empty(lay.n_img, device="cuda")
        run = lambda: A.score_variation(dl, h1, h0, scores=out[0], img_sum=out[1])  # noqa: E731
        run()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(10):
                run()
        return g, (dl, h0, h1, out)

    def us(g):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        return a.elapsed_time(b) * 100

    (many, _keep0), (few, _keep1) = call(4096), call(16)
    runs = [(us(many), us(few)) for _ in range(15)]
    t_many, t_few = min(a for a, _ in runs), min(b for _, b in runs)
    say(f"4,096 sequences {t_many:.1f} us, 16 sequences {t_few:.1f} us")
    # (the best of 15 runs of 10 calls varies by a few per cent)
    assert t_many < 1.4 * t_few
