"""The per-image epilogue of the scores in its two block sizes: at the edges of
the rule that picks them, against the oracle, and the cost of many short images."""
import numpy as np
import pytest
import torch

from gpu_util import TOL, need_gpu, say
from oracle import avtp_oracle as O
from paper_2608_26806_amd import avtp as A
from paper_2608_26806_amd.workloads import build_layout

pytestmark = pytest.mark.gpu

# images per sequence: the longest one of 255 to 2,100 tokens, and 512 or 513
# images, some empty, with a longest one beyond 256
LAYOUTS = {
    "len255": [[255, 1, 64]], "len256": [[256, 0, 3], [200]], "len257": [[257, 256], [1]],
    "len1025": [[1025, 1024, 1023]], "len2100": [[2100, 5]],
    "img512": [[300] + [3] * 127, [0, 1] * 64, [2] * 128, [7] * 128],
    "img513": [[300] + [3] * 128, [0, 1] * 64, [2] * 128, [7] * 128],
}


@pytest.mark.parametrize("name", sorted(LAYOUTS))
def test_scores_and_sums_match_the_oracle(name):
    need_gpu()
    say(f"finalize forms {name}")
    lay = build_layout(LAYOUTS[name], 1, 3, 50)
    rng = np.random.default_rng(4)
    q = rng.standard_normal((lay.T_tot, 6, 64), dtype=np.float32)
    k = rng.standard_normal((lay.N_tok, 3, 64), dtype=np.float32)
    dl = A.DeviceLayout(lay)
    s, isum = A.score_attn(dl, torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), 0.125)
    s_o, isum_o, _, _ = O.attn_scores(lay, q, k, 6, 3, 0.125, "fp32")
    s, vis = s.cpu().numpy(), lay.visual_mask()
    np.testing.assert_allclose(s[vis], s_o[vis], rtol=TOL["fp32"])
    assert np.isposinf(s[~vis]).all()
    np.testing.assert_allclose(isum.cpu().numpy(), isum_o, rtol=TOL["fp32"])
    h0 = rng.standard_normal((lay.N_tok, 16), dtype=np.float32)
    h1 = h0 + rng.standard_normal(h0.shape, dtype=np.float32)
    s, isum = A.score_variation(dl, torch.from_numpy(h1).cuda(), torch.from_numpy(h0).cuda())
    v_o, vsum_o = O.variation_scores(lay, h1, h0, "fp32")
    np.testing.assert_allclose(s.cpu().numpy()[vis], v_o[vis], rtol=TOL["fp32"], atol=1e-6)
    np.testing.assert_allclose(isum.cpu().numpy(), vsum_o, rtol=TOL["fp32"], atol=1e-5)


def test_many_short_images_cost_little_more_than_fewer_longer_ones():
    """131,072 visual tokens in 8,192 images of 16 and in 2,048 of 64: 1.2 times
    the time with blocks of 256 threads, 1.5 with 1,024 threads for 16 tokens."""
    need_gpu()
    say("8,192 images of 16 tokens and 2,048 of 64")

    def call(n, length):
        lay = build_layout([[length] * (n // 32)] * 32, 0, 8, 50)
        dl = A.DeviceLayout(lay)
        h0, h1 = torch.randn(2, lay.N_tok, 8, device="cuda").unbind(0)
        out = torch.empty(lay.N_tok, device="cuda"), torch.empty(lay.n_img, device="cuda")
        run = lambda: A.score_variation(dl, h1, h0, scores=out[0], img_sum=out[1])  # noqa: E731
        run()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            for _ in range(20):
                run()
        return g, (dl, h0, h1, out)

    def us(g):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        return a.elapsed_time(b) * 50

    (short, _keep0), (longer, _keep1) = call(8192, 16), call(2048, 64)
    runs = [(us(short), us(longer)) for _ in range(15)]
    t_short, t_longer = min(a for a, _ in runs), min(b for _, b in runs)
    say(f"8,192 images {t_short:.1f} us, 2,048 images {t_longer:.1f} us")
    # (the best of 15 runs of 20 calls varies by a few per cent)
    assert t_short < 1.35 * t_longer
