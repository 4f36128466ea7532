// Scores of few bf16 queries (n_q <= 48) against many training rows: one read of
// Phi_train.  S = (Phi_q diag(d)) Phi_train^T is the projection of the training
// rows onto n_q columns, so the split form's row stream runs it with the
// queries as its packed map: pack_few_kernel writes them in fragment order
// (scaled by d in float32, rounded once), score_stream_kernel streams X by slabs
// of columns at the stream's rate (6.2 TB/s; the 128 x 128 tile kernel, which
// reads rows through registers, 5.6), and finish_few_kernel adds the slabs in
// order, transposes, and for cosines applies both norms, the training rows'
// taken from the same pass.  1 query x 4096 rows x 229376: 330 -> 302 us.
#include <algorithm>
#include <cmath>

#include "device_common.h"
#include "internal.h"
#include "split_stream.h"

namespace dattri {
using namespace dev;

// Fragment (kb, t): lane 16 g + n holds features kb KR + g EPL .. + EPL - 1 of
// query 16 t + n (zero past n_q and F).
__global__ __launch_bounds__(256) void pack_few_kernel(const uint8_t* __restrict__ Q, int64_t ldq,
                                                       const float* __restrict__ d, int n_q, int64_t F, int nt,
                                                       int64_t n_chunks, uint8_t* __restrict__ out) {
  constexpr int EPL = 8, KR = 32;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_chunks) return;
  const int lane = (int)(i & 63);
  const int64_t frag = i >> 6, kb = frag / nt;
  const int q = (int)(frag - kb * nt) * 16 + (lane & 15);
  const int64_t f = kb * KR + (lane >> 4) * EPL;
  i32x4 v = {0, 0, 0, 0};
  if (q < n_q && f < F) {  // F is a whole number of 16-byte chunks
    v = *(const i32x4*)(Q + ((int64_t)q * ldq + f) * 2);
    if (d) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t w = (uint32_t)(e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w);
        const uint32_t lo = f32_to_bf16_bits(bf16_bits_to_f32(w & 0xFFFFu) * d[f + 2 * e]);
        const uint32_t hi = f32_to_bf16_bits(bf16_bits_to_f32(w >> 16) * d[f + 2 * e + 1]);
        const int r = (int)(lo | (hi << 16));
        if (e == 0) v.x = r;
        if (e == 1) v.y = r;
        if (e == 2) v.z = r;
        if (e == 3) v.w = r;
      }
    }
  }
  *(i32x4*)(out + i * 16) = v;
}

template <int NT, bool kNorm>
__global__ __launch_bounds__(256, 1) void score_stream_kernel(const void* X, int64_t ldx, int rows,
                                                                             int64_t F, int nt, int slab_cols,
                                                                             const void* pack, float* out,
                                                                             float* norms) {
  __shared__ __align__(1024) uint8_t smem[split_lds<2, NT>()];
  SplitOp O;
  O.X = X;
  O.lengths = nullptr;
  O.T = 1;
  O.rows = rows;
  O.ld = (int)ldx;
  O.width = (int)F;
  O.slab_cols = slab_cols;
  O.out_ld = 16 * nt;
  O.once = 1;
  O.nt = nt;
  O.out_base = 0;
  // the slabs of one row block on one XCD each (workgroup i runs on XCD i mod 8):
  // a slab's queries then cross into one L2 per eight slabs
  const SplitItem it = {0, (int)blockIdx.y, (int)blockIdx.x, 0};
  auto map = [&](int t, const uint8_t** base, int64_t* stride) {
    *stride = (int64_t)nt * kFragBytes;
    *base = (const uint8_t*)pack + t * kFragBytes;
  };
  split_stream_body<2, NT, kNorm>(it, O, map, out, smem, norms);
}

// S[q][j] = sum over slabs of parts[slab][j][q], times iq[q] and 1 / |x_j| when
// norms are given.  Thread: one training row.
__global__ __launch_bounds__(256) void finish_few_kernel(const float* __restrict__ parts, int n_slabs, int n_q,
                                                         int64_t n_train, int ldo, const float* __restrict__ iq,
                                                         const float* __restrict__ norm_parts, float* __restrict__ S) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= n_train) return;
  float it = 1.f;
  if (norm_parts) {
    float s = 0.f;
    for (int y = 0; y < n_slabs; ++y) s += norm_parts[(int64_t)y * n_train + j];
    it = s > 0.f ? 1.f / sqrtf(s) : 0.f;
  }
  const int q0 = blockIdx.y * 4;
  const float* p = parts + j * ldo + q0;
  const int64_t step = n_train * ldo;
  f32x4 s = {0.f, 0.f, 0.f, 0.f};
  int y = 0;
  for (; y + 4 <= n_slabs; y += 4) {
    const f32x4 v0 = *(const f32x4*)(p + y * step), v1 = *(const f32x4*)(p + (y + 1) * step),
                v2 = *(const f32x4*)(p + (y + 2) * step), v3 = *(const f32x4*)(p + (y + 3) * step);
    s = (((s + v0) + v1) + v2) + v3;
  }
  for (; y < n_slabs; ++y) s += *(const f32x4*)(p + y * step);
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (q0 + e < n_q) S[(int64_t)(q0 + e) * n_train + j] = norm_parts ? s[e] * (iq[q0 + e] * it) : s[e];
}

int64_t score_stream_pack_bytes(int64_t n_q, int64_t F) { return (F + 31) / 32 * ((n_q + 15) / 16) * kFragBytes; }

// All items cost the same, so the slab count is the one that minimises rounds of
// resident workgroups (one per CU) times an item's bytes plus its fixed cost
// (prologue, partial scores written and read again).
StreamShape score_stream_shape(int64_t n_q, int64_t n_train, int64_t F) {
  StreamShape s;
  s.nt = (int)((n_q + 15) / 16);
  const int64_t rows = split_stream_rows(2), slots = 256;
  const int64_t rblocks = (n_train + rows - 1) / rows;
  const double fixed = 131072.0 + 2.0 * rows * s.nt * 16 * 4;
  double best = -1.0;
  s.slab_cols = kSplitSlabQuantum;
  s.n_slabs = 1;
  for (int64_t want = 1; want <= std::min<int64_t>(256, std::max<int64_t>(1, F / kSplitSlabQuantum)); ++want) {
    const int64_t cols = ((F + want - 1) / want + kSplitSlabQuantum - 1) / kSplitSlabQuantum * kSplitSlabQuantum;
    const int64_t n = (F + cols - 1) / cols, rounds = (rblocks * n + slots - 1) / slots;
    const double cost = (double)rounds * ((double)std::min(n_train, rows) * cols * 2 + fixed);
    if (best < 0 || cost < best) {
      best = cost;
      s.slab_cols = cols;
      s.n_slabs = (int)n;
    }
  }
  return s;
}

// The stream takes three launches where the tile kernel takes one or two, and
// pays from training rows that no cache holds: 8 queries x 2048 rows, 256 MB:
// 65 us against the tile kernel's 58; 512 MB: 100 against 101; 1 GB: 188 against
// 195.  With 48 queries x 100000 rows x 4096 it takes 250 us against the 256 x 256
// kernel's 256, with 64 264 against 258.  (float32 rows stay with their tile
// kernel, which splits fewer values: 8 x 20000 x 12288 190 us against 224.)
constexpr int64_t kStreamMinBytes = (int64_t)512 << 20, kStreamMaxQueries = 48;
ScorePath score_path(int elt, int64_t n_q, int64_t n_train, int64_t F) {
  const int64_t rblocks = (n_train + split_stream_rows(2) - 1) / split_stream_rows(2);
  if (elt == 2 && n_q > 0 && n_q <= kStreamMaxQueries && n_train * F * 2 >= kStreamMinBytes && rblocks <= 65535)
    return kScoreStream;
  return score_uses_big(elt, n_q, n_train) ? kScoreBig : kScoreTile;
}

template <bool kNorm>
static hipError_t launch_stream(const StreamShape& h, const void* X, int64_t ldx, int64_t n_train, int64_t F,
                                const void* pack, float* parts, float* norms, hipStream_t s) {
  const dim3 grid((unsigned)h.n_slabs, (unsigned)((n_train + split_stream_rows(2) - 1) / split_stream_rows(2)));
  if (h.nt <= 2)
    hipLaunchKernelGGL((score_stream_kernel<2, kNorm>), grid, dim3(256), 0, s, X, ldx, (int)n_train, F, h.nt,
                       (int)h.slab_cols, pack, parts, norms);
  else
    hipLaunchKernelGGL((score_stream_kernel<4, kNorm>), grid, dim3(256), 0, s, X, ldx, (int)n_train, F, h.nt,
                       (int)h.slab_cols, pack, parts, norms);
  return hipGetLastError();
}

hipError_t launch_score_stream(const void* Q, int64_t ldq, const float* d, const void* X, int64_t ldx, float* S,
                               int64_t n_q, int64_t n_train, int64_t F, void* pack, float* parts, const float* iq,
                               float* norm_parts, hipStream_t s) {
  if (n_q <= 0 || n_train <= 0) return hipSuccess;
  if (!pack || !parts || n_q > kStreamMaxQueries) return hipErrorInvalidValue;
  const StreamShape h = score_stream_shape(n_q, n_train, F);
  const int64_t chunks = score_stream_pack_bytes(n_q, F) / 16;
  hipLaunchKernelGGL(pack_few_kernel, dim3((unsigned)((chunks + 255) / 256)), dim3(256), 0, s, (const uint8_t*)Q, ldq, d,
                     (int)n_q, F, h.nt, chunks, (uint8_t*)pack);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess)
    e = norm_parts ? launch_stream<true>(h, X, ldx, n_train, F, pack, parts, norm_parts, s)
                   : launch_stream<false>(h, X, ldx, n_train, F, pack, parts, nullptr, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(finish_few_kernel, dim3((unsigned)((n_train + 255) / 256), (unsigned)((n_q + 3) / 4)), dim3(256), 0,
                     s, parts, h.n_slabs, (int)n_q, n_train, 16 * h.nt, iq, norm_parts, S);
  return hipGetLastError();
}

}  // namespace dattri
