// The per-image epilogue of both score modes (Sec. 3.3.2 statistic per
// visual token, and the per-image sums that Sec. 3.3.3's budgets start from).
#include <hip/hip_runtime.h>

#include <stdint.h>

#include "avtp_internal.h"
#include "wave_ops.h"

namespace avtp {
namespace {

constexpr int kPlanesInFlight = 8;

// Per-image epilogue shared by both score modes: s_j from the column sums
// (attention mode) or as stored (variation mode), NaN / empty-row flags, and
// the per-image sum in a fixed reduction order.  Extra blocks write +inf at
// the text positions.  One block per image.
//
// A few hundred blocks of dependent loads: bound by latency, so a token has a
// thread of its own (kThreads = 1024) with eight planes' loads in flight, every
// wave finds the image's sequence itself (no barrier before the loads), and the
// text-row count runs while the planes arrive.  With 256 threads, four tokens
// each and the rest of a longer image one plane after the other: two sequences
// of 8 images of 256-1,536 tokens 8.7 -> 4.8 us, 8 x 16 images 8.1 -> 5.2, 4 x
// 729 tokens 4.5 -> 3.9.  Blocks of 256 threads serve short or many images, see
// launch_finalize.
template <int kThreads>
__global__ __launch_bounds__(kThreads) void finalize_kernel(
    const float *__restrict__ colsum, int Hq, int planes, int N_tok, int n_img, int T_tot,
    const int32_t *__restrict__ img_start, const int32_t *__restrict__ img_len,
    const int32_t *__restrict__ cu_img, const int32_t *__restrict__ cu_text,
    const int32_t *__restrict__ text_pos, int B, float *__restrict__ scores,
    float *__restrict__ img_sum, int32_t *__restrict__ status) {
  constexpr int kWaves = kThreads / 64;
  __shared__ float red[kWaves];
  __shared__ int cnt[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.x >= n_img) {
    const int t = (blockIdx.x - n_img) * kThreads + tid;
    if (t < T_tot) scores[text_pos[t]] = INFINITY;
    return;
  }
  const int i = blockIdx.x;
  const int s0 = img_start[i], n = img_len[i];
  const int b = wave::segment_of(cu_img, B, i).b;  // the sequence holding image i
  // the column sums of token j over the planes, in plane order
  auto plane_sum = [&](int j) __attribute__((always_inline)) {
    const float *p = colsum + s0 + j;
    float v = 0.f;
    for (int g0 = 0; g0 < planes; g0 += kPlanesInFlight) {
      float x[kPlanesInFlight];
#pragma unroll
      for (int u = 0; u < kPlanesInFlight; ++u)  // (a plane past the last re-reads it and is not added)
        x[u] = p[(size_t)min(g0 + u, planes - 1) * N_tok];
#pragma unroll
      for (int u = 0; u < kPlanesInFlight; ++u)
        if (g0 + u < planes) v += x[u];
    }
    return v;
  };
  float v = 0.f;  // the thread's first token, before the text-row count
  int nT = 0;
  if (colsum) {
    if (tid < n) v = plane_sum(tid);
    int c = 0;  // text rows after the image (their positions exceed s0)
    for (int t = cu_text[b] + tid; t < cu_text[b + 1]; t += kThreads) c += text_pos[t] > s0;
    c = wave::sum(c);
    if (lane == 0) cnt[wave] = c;
    __syncthreads();
    for (int w = 0; w < kWaves; ++w) nT += cnt[w];
  }
  float acc = 0.f;
  bool nan = false;
  for (int j = tid; j < n; j += kThreads) {
    float s;
    if (colsum) {
      if (j >= kThreads) v = plane_sum(j);
      s = nT > 0 ? v / (float)((long long)Hq * nT) : 0.f;
      scores[s0 + j] = s;
    } else {
      s = scores[s0 + j];
    }
    nan |= (s != s);
    acc += s;
  }
  // the image sum in a fixed order: each thread's tokens in order, the
  // wave's lanes in the DPP pattern, then the waves in order
  acc = wave::sum(acc);
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  if (tid == 0) {
    float sum = red[0];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) sum += red[w];
    img_sum[i] = sum;
  }
  if (status) {
    if (nan) atomicOr(status + b, AVTP_FLAG_NAN_SCORE);
    if (tid == 0 && colsum && nT == 0 && n > 0) atomicOr(status + b, AVTP_FLAG_NO_TEXT_AFTER);
  }
}

}  // namespace

hipError_t launch_finalize(hipStream_t st, const DevLayout &L, const float *colsum, int Hq,
                           int planes, float *scores, float *img_sum, int32_t *status) {
  clear_pending_error();
  // 1024 threads per image where most of them have a token and the blocks run at
  // once, two on a CU.  Else 256: the waves without a token cost their start and
  // the barriers, and with several rounds of blocks other images cover an
  // image's latency.  Score with a given LSE and variation score, 1024 against
  // 256 threads: 8,192 images of 49 tokens 76 and 106 -> 58 and 96 us, 512 of 64
  // tokens 23.0 and 10.0 -> 22.7 and 9.8; 2,048 of 729 tokens 222 -> 218
  // (variation); 512 of 1,024 tokens 271 -> 274 and 79.3 -> 79.8, 128 of 1,024
  // 61.2 -> 62.9 and 23.6 -> 24.2.
  const bool wide = L.max_img_len > 256 && L.n_img <= 512;
  const int threads = wide ? 1024 : 256;
  const int text_blocks = (L.T_tot + threads - 1) / threads;
  const int grid = L.n_img + text_blocks;
  if (grid == 0) return hipSuccess;
  const auto kernel = wide ? finalize_kernel<1024> : finalize_kernel<256>;
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, st, colsum, Hq, planes, L.N_tok,
                     L.n_img, L.T_tot, L.img_start, L.img_len, L.cu_img, L.cu_text, L.text_pos,
                     L.B, scores, img_sum, status);
  return hipGetLastError();
}

}  // namespace avtp
