// One item of the row streams: X[rows of a block, one slab of columns] times a
// packed map, float32, written as projected rows.  Shared by the split form's
// stage 1 (split.hip) and the scoring of few queries (score_few.hip), whose
// packed "map" is the queries.
#pragma once
#include "device_common.h"
#include "internal.h"
#include "project_rows.h"

namespace dattri {
namespace dev {

template <int ELT, int NT>
struct SplitShape {
  static constexpr int kRows = split_stream_rows(ELT), kRT = kRows / 64;
  static constexpr int D = NT <= 2 ? 4 : NT <= 6 ? 3 : 2;  // bf16: stages per wave
  static constexpr int kLoads = ELT == 2 ? kRT * 2 : kRT;  // row pieces a lane loads per stage
};

// Whether any thread of the workgroup has `v` set (w: a word of LDS that nothing else uses meanwhile).
__device__ inline bool block_any(bool v, uint32_t* w) {
  __syncthreads();
  if (threadIdx.x == 0) *w = 0u;
  __syncthreads();
  if (v) *w = 1u;  // every writer writes the same value
  __syncthreads();
  const bool any = *w != 0u;
  __syncthreads();
  return any;
}

// kNorm (bf16): also the sums of squares of the slab's columns of every row, one float
// per row at norms + slab * O.rows.
// map(t, &base, &stride): tile t's packed map (its fragment of k-block kb at
// base + kb * stride).
template <int ELT, int NT, bool kNorm, class Map>
__device__ inline void split_stream_body(const SplitItem& it, const SplitOp& O, const Map& map,
                                         float* __restrict__ out, uint8_t* smem, float* __restrict__ norms) {
  using S = SplitShape<ELT, NT>;
  constexpr int KR = 4 * (16 / ELT);  // rows of a packed k-block
  constexpr int RT = S::kRT, D = S::D, ROWS = S::kRows;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, m16 = lane & 15;
  const int row0 = it.row_block * ROWS;
  const int nrows = min(ROWS, O.rows - row0);
  const int col0 = it.slab * O.slab_cols;
  const int d = min(O.slab_cols, O.width - col0);
  const int r_wave = wave * RT * 16;
  // rows to read and to write: inside the block and their example's length.
  // bf16: load i of a stage takes row i * 8 + lane / 8; float32: row i * 16 + m16
  auto row_of = [&](int i) { return r_wave + (ELT == 4 ? i * 16 + m16 : i < S::kLoads ? i * 8 + (lane >> 3) : (i - S::kLoads) * 16 + m16); };
  constexpr int kNR = ELT == 2 ? S::kLoads + RT : RT;  // rows to check (float32 writes the rows it reads)
  uint32_t ok = 0;
#pragma unroll
  for (int i = 0; i < kNR; ++i) ok |= (row_of(i) < nrows ? 1u : 0u) << i;
  if (O.lengths) {  // uniform; every load before the first use
    int len[kNR], tok[kNR];
#pragma unroll
    for (int i = 0; i < kNR; ++i) {
      const int gr = min(row0 + row_of(i), O.rows - 1), ex = gr / O.T;
      len[i] = O.lengths[ex];
      tok[i] = gr - ex * O.T;
    }
#pragma unroll
    for (int i = 0; i < kNR; ++i) ok &= ~((tok[i] < len[i] ? 0u : 1u) << i);
    if (!block_any(ok != 0, (uint32_t*)smem)) return;  // every row of the block lies past its example's length
  }
  const uint32_t out_rows = ELT == 2 ? ok >> S::kLoads : ok;
  uint32_t rowoff[S::kLoads];
#pragma unroll
  for (int i = 0; i < S::kLoads; ++i) {
    const int row_l = row_of(i);
    const int chunk = ELT == 2 ? (lane & 7) ^ (row_l & 7) : g;
    rowoff[i] = (ok >> i) & 1u ? (uint32_t)((row_l - r_wave) * (int64_t)O.ld * ELT) + (chunk << 4) : kFarOff;
  }
  // descriptor over this wave's rows, starting at the slab's first column
  const int wrows = min(RT * 16, nrows - r_wave);
  const uint8_t* base = (const uint8_t*)O.X + ((int64_t)(row0 + r_wave) * O.ld + col0) * ELT;
  const rsrc_t r = make_rsrc(base, wrows > 0 ? (uint32_t)(((int64_t)(wrows - 1) * O.ld + O.width - col0) * ELT) : 0u);
  const int kb0 = col0 / KR;
  auto P = [&](int t, const uint8_t** fb, int64_t* fs) {
    map(t < O.nt ? t : 0, fb, fs);
    *fb += kb0 * *fs;
  };
  f32x4 acc[RT][NT];
  auto clear = [&] {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[rt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  clear();
  float nsq[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) nsq[rt] = 0.f;
  if constexpr (ELT == 2) {
    stream_rows<RT, NT, D, kNorm>(r, rowoff, d, O.nt, P, O.once != 0, acc, nsq, smem);
  } else {
    const bool bad = stream_rows_f32<RT, NT>(r, rowoff, d, O.nt, P, __any(ok != 0), acc, smem);
    if (__any(bad)) {  // infinities, NaN, overflow or values too small to split: float32 products
      clear();
      plain_rows_f32<RT, NT>(r, (uint32_t)(m16 * (int64_t)O.ld * ELT), O.ld, out_rows, d, O.nt, P, acc);
    }
  }

  // the map fragment is the first MFMA operand: lane (g, n) holds columns
  // 4g .. 4g + 3 of token row n, one 16-byte store per tile
  const int ldo = O.out_ld;
  float* dst = out + O.out_base + ((int64_t)it.slab * O.rows + row0) * ldo;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int row = r_wave + rt * 16 + m16;
    if ((out_rows >> rt) & 1u) {
#pragma unroll
      for (int t = 0; t < NT; ++t)
        if (t < O.nt) *(f32x4*)(dst + (int64_t)row * ldo + t * 16 + 4 * g) = acc[rt][t];
    }
  }
  if constexpr (kNorm) {  // lanes g = 0 .. 3 hold the row's four column quarters
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      float v = nsq[rt];
      v += __shfl_xor(v, 16, 64);
      v += __shfl_xor(v, 32, 64);
      if (g == 0 && ((out_rows >> rt) & 1u))
        norms[(int64_t)it.slab * O.rows + row0 + r_wave + rt * 16 + m16] = v;
    }
  }
}

template <int ELT, int NT>
constexpr int split_lds() {
  using S = SplitShape<ELT, NT>;
  if constexpr (ELT == 2)
    return StreamLds<S::kRT, NT, S::D>::kBytes;
  else
    return StreamF32Lds<NT>::kBytes;
}
constexpr int max_of(int a, int b) { return a > b ? a : b; }

}  // namespace dev
}  // namespace dattri
