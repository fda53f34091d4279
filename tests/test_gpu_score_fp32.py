"""fp32 attention scores on the split bf16 MFMA path: stage and tile edges
against the float64 oracle, and infinite inputs whose logits are -inf."""
import numpy as np
import pytest
import torch

from gpu_util import TOL, need_gpu, say
from oracle import avtp_oracle as O
from paper_2608_26806_amd import avtp as A
from paper_2608_26806_amd.workloads import build_layout

pytestmark = pytest.mark.gpu

# head size, query heads, key heads, images, text before each, text at the end.
# Stages are 32 (d = 128) or 64 (d = 64) rows of 32-row tiles; key blocks are
# 128 or 256 keys; one to several sequences and query rows per key head.
CASES = [
    (128, 1, 1, [[31]], 0, 1), (128, 4, 2, [[32], [33]], 0, 8), (128, 3, 1, [[63, 65], [1]], 1, 10),
    (128, 8, 4, [[127, 129, 128]], 3, 17), (64, 2, 1, [[63]], 0, 16), (64, 7, 1, [[64, 65]], 1, 9),
    (64, 4, 4, [[255, 257], [513]], 2, 33), (64, 8, 2, [[700, 900], [31, 1]], 5, 64),
]


def _draw(case, seed):
    d, Hq, Hkv, imgs, pre, tail = case
    lay = build_layout(imgs, pre, tail, 50)
    rng = np.random.default_rng(seed)
    q = rng.standard_normal((lay.T_tot, Hq, d), dtype=np.float32)
    k = rng.standard_normal((lay.N_tok, Hkv, d), dtype=np.float32) * np.exp(
        0.5 * rng.standard_normal((lay.N_tok, 1, 1))).astype(np.float32)
    return lay, q, k


@pytest.mark.parametrize("case", CASES, ids=lambda c: f"d{c[0]}h{c[1]}-{c[2]}i{c[3]}t{c[4]}-{c[5]}")
def test_scores_match_the_oracle_at_the_edges(case):
    need_gpu()
    say(f"fp32 scores {case}")
    lay, q, k = _draw(case, 11)
    d, Hq, Hkv = case[:3]
    dl = A.DeviceLayout(lay)
    s, isum = A.score_attn(dl, torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), d ** -0.5)
    s_o, isum_o, _, _ = O.attn_scores(lay, q, k, Hq, Hkv, d ** -0.5, "fp32")
    vis = lay.visual_mask()
    np.testing.assert_allclose(s.cpu().numpy()[vis], s_o[vis], rtol=TOL["fp32"])
    np.testing.assert_allclose(isum.cpu().numpy(), isum_o, rtol=TOL["fp32"])


@pytest.mark.parametrize("d", [64, 128])
def test_an_infinite_key_value_with_negative_logits(d):
    """A key whose logits are all -inf scores 0 and leaves the others as they
    are without it (the split products of an infinity are not numbers)."""
    need_gpu()
    say(f"fp32 scores, infinite key value, d={d}")
    lay, q, k = _draw((d, 4, 2, [[200, 100]], 2, 20), 5)
    q[:, :, 3] = -np.abs(q[:, :, 3]) - 0.1
    j = int(lay.img_start[0]) + 40
    k[j, :, 3] = np.inf
    dl = A.DeviceLayout(lay)
    s, isum = A.score_attn(dl, torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), d ** -0.5)
    s, vis = s.cpu().numpy(), lay.visual_mask()
    kk = k.copy()
    kk[j] = 0.0
    kk[j, :, 3] = 1e6  # its logits below -1000: the same zero weight, in finite numbers
    s_o, _, _, _ = O.attn_scores(lay, q, kk, 4, 2, d ** -0.5, "fp32")
    assert s[j] == 0.0
    vis[j] = False
    np.testing.assert_allclose(s[vis], s_o[vis], rtol=TOL["fp32"])


def _check(lay, q, k, Hq, Hkv, d):
    dl = A.DeviceLayout(lay)
    s, isum = A.score_attn(dl, torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), d ** -0.5)
    s_o, isum_o, _, _ = O.attn_scores(lay, q, k, Hq, Hkv, d ** -0.5, "fp32")
    vis = lay.visual_mask()
    np.testing.assert_allclose(s.cpu().numpy()[vis], s_o[vis], rtol=TOL["fp32"])
    np.testing.assert_allclose(isum.cpu().numpy(), isum_o, rtol=TOL["fp32"])


@pytest.mark.parametrize("small", ["q", "k"])
@pytest.mark.parametrize("case", [CASES[3], CASES[5], CASES[7]], ids=lambda c: f"d{c[0]}h{c[1]}-{c[2]}")
def test_operands_at_both_ends_of_the_range(case, small):
    """Operands near 2^-122 against operands near 2^122: the third bf16 part of
    the small ones is below bf16's smallest step, their products are ordinary."""
    need_gpu()
    say(f"fp32 scores, {small} near 2^-122, {case}")
    lay, q, k = _draw(case, 13)
    lo, hi = np.float32(2.0 ** -122), np.float32(2.0 ** 122)
    q, k = (q * lo, k * hi) if small == "q" else (q * hi, k * lo)
    assert np.isfinite(q).all() and np.isfinite(k).all()
    d, Hq, Hkv = case[:3]
    _check(lay, q, k, Hq, Hkv, d)


@pytest.mark.parametrize("d", [64, 128])
def test_finite_values_that_round_to_infinity_in_bf16(d):
    need_gpu()
    say(f"fp32 scores, finite overflow of bf16, d={d}")
    lay, q, k = _draw((d, 4, 2, [[200, 100], [33]], 2, 20), 5)
    top = np.float32(3.4e38)                       # bf16 ends at 3.39e38
    assert torch.isinf(torch.tensor(top).bfloat16())
    q[:, :, 3] *= np.float32(1e-38)
    k[int(lay.img_start[0]) + 40, :, 3] = top
    k[int(lay.img_start[2]) + 32, :, 3] = -top
    _check(lay, q, k, 4, 2, d)


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf], ids=str)
@pytest.mark.parametrize("d", [64, 128])
def test_a_query_that_is_not_finite(d, value):
    """One text row before the second image whose logits are not numbers (or all
    infinite): the tokens it sees score NaN and are flagged, the others are as
    the oracle has them."""
    need_gpu()
    say(f"fp32 scores, a query of {value}, d={d}")
    lay, q, k = _draw((d, 4, 2, [[90, 150], [70]], 2, 20), 6)
    k[:, :, 3] = np.abs(k[:, :, 3]) + 0.1
    q_bad = q.copy()
    q_bad[3, 1, 3] = value                         # the second of the rows between the images
    dl = A.DeviceLayout(lay)
    status = torch.zeros(lay.B, dtype=torch.int32, device="cuda")
    s, _ = A.score_attn(dl, torch.from_numpy(q_bad).cuda(), torch.from_numpy(k).cuda(), d ** -0.5,
                        status=status)
    s_o, _, _, _ = O.attn_scores(lay, q, k, 4, 2, d ** -0.5, "fp32")
    s, vis = s.cpu().numpy(), lay.visual_mask()
    a, n = int(lay.img_start[0]), int(lay.img_len[0])
    assert int(lay.text_pos[3]) > a + n > int(lay.text_pos[1])
    assert np.isnan(s[a:a + n]).all()
    assert [x & 1 for x in status.tolist()] == [1, 0]
    vis[a:a + n] = False
    np.testing.assert_allclose(s[vis], s_o[vis], rtol=TOL["fp32"])


@pytest.mark.parametrize("d", [64, 128])
def test_a_key_that_is_not_a_number(d):
    """Every text row after it sees it, so the tokens of its sequence that those
    rows see score NaN; the other sequence is as the oracle has it."""
    need_gpu()
    say(f"fp32 scores, a key of NaN, d={d}")
    lay, q, k = _draw((d, 4, 2, [[90, 150], [70]], 2, 20), 8)
    k_bad = k.copy()
    k_bad[int(lay.img_start[0]) + 33, 0, 5] = np.nan
    dl = A.DeviceLayout(lay)
    status = torch.zeros(lay.B, dtype=torch.int32, device="cuda")
    s, _ = A.score_attn(dl, torch.from_numpy(q).cuda(), torch.from_numpy(k_bad).cuda(), d ** -0.5,
                        status=status)
    s_o, _, _, _ = O.attn_scores(lay, q, k, 4, 2, d ** -0.5, "fp32")
    s, vis = s.cpu().numpy(), lay.visual_mask()
    first = np.arange(lay.N_tok) < int(lay.cu_seqlens[1])
    assert np.isnan(s[vis & first]).all()
    assert [x & 1 for x in status.tolist()] == [1, 0]
    np.testing.assert_allclose(s[vis & ~first], s_o[vis & ~first], rtol=TOL["fp32"])


@pytest.mark.parametrize("d", [64, 128])
def test_partly_filled_row_tiles_cost_no_more_than_full_ones(d):
    """40 query rows per key head (a full row tile and one of 8 rows) against 64
    (two full tiles) over the same keys: the same tiles, so not slower.  The
    unused rows see no key, and must not send finite inputs to the fp32 MFMA
    (with that every tile of such a wave waits for d / 2 memory round trips:
    2 to 4 times the time)."""
    need_gpu()
    say(f"fp32 row tiles, d={d}")

    def call(rows):
        lay, q, k = _draw((d, 4, 1, [[1024, 1000]], 0, rows // 4), 3)
        dl = A.DeviceLayout(lay)
        q, k = torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda()
        out = torch.empty(4, lay.T_tot, device="cuda")
        ws = A.alloc_workspace(A.score_workspace_bytes(dl, A.SCORE_ATTN, A.FP32, 4, 1, d))
        A.row_lse(dl, q, k, d ** -0.5, out=out, ws=ws)
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):               # (the call's host part is as long as its kernels)
            for _ in range(20):
                A.row_lse(dl, q, k, d ** -0.5, out=out, ws=ws)
        return g, (dl, q, k, out, ws)

    def us(g):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        b.synchronize()
        return a.elapsed_time(b) * 50

    (part, _keep0), (full, _keep1) = call(40), call(64)
    runs = [(us(part), us(full)) for _ in range(15)]
    t_part, t_full = min(a for a, _ in runs), min(b for _, b in runs)
    say(f"40 rows {t_part:.1f} us, 64 rows {t_full:.1f} us")
    # the best of 15 runs of 20 calls varies by a few per cent
    assert t_part < 1.25 * t_full
