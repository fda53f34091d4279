"""The launch plan of the attention score, on the CPU: a host program linked
against libavtp.so prints it for a range of layouts."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIBDIR = os.path.join(ROOT, "paper_2608_26806_amd")

PROGRAM = r"""
#include <cstdio>
#include "avtp_internal.h"
// the pass-2 kernel's row -> token division against the integer one; wrong ones
static long long wrong_tokens() {
  long long bad = 0;
  for (uint64_t G = 3; G <= 256; ++G) {
    if ((G & (G - 1)) == 0) continue;
    const uint64_t m = avtp::group_mul((int)G), end = 1u << 25;
    for (uint64_t q = 0; q * G < end; q += q < 1000 || (q + 1000) * G > end ? 1 : 37)
      for (uint64_t r : {q * G, q * G + G - 1})
        if (r < end) bad += ((r * m) >> 32) >> 1 != r / G;
  }
  return bad;
}
int main() {
  std::printf("%lld\n", wrong_tokens());
  const int heads[][2] = {{4, 2}, {14, 2}, {16, 16}, {28, 4}, {32, 8}, {256, 1}};
  const int text[] = {0, 1, 7, 20, 37, 64, 71, 129, 200, 512, 1000}, batch[] = {1, 3, 8, 30};
  const int len[] = {33, 311, 1976, 4157, 16584};
  for (int B : batch) for (int L : len) for (int T : text) for (auto &h : heads)
    for (int d : {64, 128}) for (int dt : {AVTP_BF16, AVTP_FP32}) {
      if (T > L) continue;
      avtp::DevLayout lay{};
      lay.B = B; lay.N_tok = B * L; lay.T_tot = B * T; lay.max_seqlen = L; lay.max_text = T;
      const avtp::AttnPlan p = avtp::attn_plan(lay, h[0], h[1], d, dt);
      std::printf("%d %d %d %d %d %d %d %d %d %d\n", B, L, h[0], h[1], d, dt, p.rows_max, p.nqs, p.nkt2, p.nkb);
    }
}
"""


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """(B, longest sequence, Hq, Hkv, d, dtype, most query rows, query splits, key tiles,
    key blocks)"""
    assert shutil.which("g++")
    tmp = tmp_path_factory.mktemp("plan")
    src, exe = tmp / "plan.cpp", tmp / "plan"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(LIBDIR, "csrc"), str(src), "-L" + LIBDIR, "-lavtp",
                    "-Wl,-rpath," + LIBDIR, "-Wl,-rpath,/opt/rocm/lib", "-L/opt/rocm/lib",
                    "-lamdhip64", "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], check=True, capture_output=True, text=True).stdout
    return [tuple(map(int, line.split())) for line in out.splitlines()]


def test_rows_are_divided_by_every_group_size(plans):
    assert plans[0] == (0,)


def test_every_query_split_of_the_longest_sequence_holds_rows(plans):
    """Splits are whole stages: 128 rows in bf16, 24 KB of three bf16 planes in fp32."""
    assert len(plans) > 2000
    for p in plans[1:]:
        d, dtype, rows, nqs = p[4:8]
        stage = 128 if dtype == 0 else 24576 // (6 * d)
        per = -(-(-(-rows // nqs)) // stage) * stage
        assert nqs == 1 or (nqs - 1) * per < rows, p


def test_narrow_blocks_at_head_size_64_fill_the_chip_as_the_wide_ones_did(plans):
    """Where blocks of four key tiles give way to narrower ones there are 512
    blocks, two per CU, or every two stages of rows have a block of their own
    (fewer than 256 before the rows are split: 256 within the rounding of a split
    to stages, or a block for every stage)."""
    seen = 0
    for B, L, Hq, Hkv, d, dtype, rows, nqs, nkt2, nkb in plans[1:]:
        if d == 64 and dtype == 0 and nkt2 < 4 and rows:
            seen += 1
            blocks, stages = B * Hkv * nkb, -(-rows // 128)
            if blocks >= 256:
                assert blocks * nqs >= 512 or nqs >= stages // 2, (B, L, Hq, Hkv, rows, nqs, nkt2)
            else:
                assert blocks * nqs >= 256 or nqs == stages, (B, L, Hq, Hkv, rows, nqs, nkt2)
    assert seen > 200
