// Scoring: S = (Phi_q diag(d)) Phi_train^T  (GradDot, Sec. 4.1, with an
// optional positive diagonal preconditioner applied once), float32 out.
//
// Both operands are row-major with the feature axis contiguous, which is the
// K-contiguous ("NT") form MFMA wants for both sides: a lane's 16-byte fragment
// is a contiguous slice of one row.  Workgroup tile 128 x 128, 4 waves in a
// 2 x 2 grid of 64 x 64 (4 x 4 MFMA tiles each), 128 bytes of K per stage, the
// next stage prefetched into registers while the current one is multiplied.
// bf16: double-buffered in LDS, rows XOR-swizzled by 16-byte chunk.  float32:
// values split into three bf16 terms on their way into LDS and multiplied on
// bf16 MFMA (score_gemm_split_kernel).
// Tiles are remapped so that each XCD walks a contiguous range of training
// tiles, all query tiles of one training tile back to back, so a Phi_train
// tile is fetched into that XCD's L2 once and reused by every query tile.
// When the tiles alone cannot fill the chip (few queries and training rows,
// long feature rows), the feature axis is split over grid.y: each split writes
// its partial tile, and the splits are summed in split order.
#include "device_common.h"
#include "internal.h"

namespace dattri {
using namespace dev;

// dst[r][f] = src[r][f] * d[f] for f < F; rows ld_src / ld_dst elements apart
// (the padding of dst rows is not written).
template <int ELT>
__global__ __launch_bounds__(256) void scale_rows_kernel(const uint8_t* __restrict__ src,
                                                         int64_t ld_src,
                                                         const float* __restrict__ d,
                                                         uint8_t* __restrict__ dst, int64_t ld_dst,
                                                         int64_t rows, int64_t F) {
  const int64_t n = rows * F;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / F, f = i - r * F;
    if constexpr (ELT == 2) {
      const float x = bf16_bits_to_f32(((const uint16_t*)src)[r * ld_src + f]) * d[f];
      ((uint16_t*)dst)[r * ld_dst + f] = f32_to_bf16_bits(x);
    } else {
      ((float*)dst)[r * ld_dst + f] = ((const float*)src)[r * ld_src + f] * d[f];
    }
  }
}

constexpr int kBM = 128, kBN = 128, kRowBytes = 128;  // tile rows, K bytes per stage

// XCD-aware tile order (dispatch round-robins workgroups over 8 XCDs)
__device__ inline void tile_of(int b, int n_qt, int n_xt, int* qt, int* xt) {
  const int n_full = n_qt * n_xt / 8 * 8;
  const int L = b < n_full ? (b % 8) * (n_full / 8) + b / 8 : b;
  *qt = L % n_qt;
  *xt = L / n_qt;
}

// norms (may be null): the tiles of the first query tile also write their
// training rows' sums of squares over this split's features.
__global__ __launch_bounds__(256) void score_gemm_kernel(const uint8_t* __restrict__ Q,
                                                         const uint8_t* __restrict__ X,
                                                         float* __restrict__ S, float* __restrict__ norms, int n_q,
                                                         int n_train, int F, int ldq, int ldx,
                                                         int n_qt, int n_xt, int sps) {
  constexpr int ELT = 2, EPL = 16 / ELT;
  constexpr int BK = kRowBytes / ELT;  // K elements per stage
  __shared__ __align__(16) uint8_t smem[2][2][kBM * kRowBytes];  // [stage][Q/X] 64 KiB
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, m16 = lane & 15, wm = wave >> 1, wn = wave & 1;

  int qt, xt;
  tile_of(blockIdx.x, n_qt, n_xt, &qt, &xt);
  const int q0 = qt * kBM, x0 = xt * kBN;
  const int rows_q = min(kBM, n_q - q0), rows_x = min(kBN, n_train - x0);
  // ranges end at the last row's F-th element (padding after it need not exist)
  const rsrc_t rq = make_rsrc(Q + (int64_t)q0 * ldq * ELT, (uint32_t)(((int64_t)(rows_q - 1) * ldq + F) * ELT));
  const rsrc_t rx = make_rsrc(X + (int64_t)x0 * ldx * ELT, (uint32_t)(((int64_t)(rows_x - 1) * ldx + F) * ELT));

  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk = (F + BK - 1) / BK;
  const int k0 = blockIdx.y * sps, k1 = min(nk, k0 + sps);  // this split's K steps
  S += (int64_t)blockIdx.y * n_q * n_train;                 // its partial tile (S itself when unsplit)
  i32x4 rqv[4], rxv[4];
  auto gload = [&](int kk) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = tid + 256 * i, row = c >> 3, ch = c & 7;
      const int col = kk * BK + ch * EPL;
      rqv[i] = load_frag_ld<ELT>(rq, row, rows_q, col, F, ldq);
      rxv[i] = load_frag_ld<ELT>(rx, row, rows_x, col, F, ldx);
    }
  };
  const bool sq = norms && qt == 0;  // uniform
  float nsq[4] = {0.f, 0.f, 0.f, 0.f};
  auto swrite = [&](int st) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (sq) nsq[i] = sum_sq<ELT>(rxv[i], nsq[i]);
      const int c = tid + 256 * i, row = c >> 3, ch = c & 7;
      const int off = row * kRowBytes + ((ch ^ (row & 7)) << 4);
      *(i32x4*)(smem[st][0] + off) = rqv[i];
      *(i32x4*)(smem[st][1] + off) = rxv[i];
    }
  };

  if (k0 < k1) {
    gload(k0);
    swrite(0);
  }
  __syncthreads();
  for (int kk = k0; kk < k1; ++kk) {
    const int st = (kk - k0) & 1;
    if (kk + 1 < k1) gload(kk + 1);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      i32x4 af[4], bf[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int row = wm * 64 + i * 16 + m16, ch = s * 4 + g;
        af[i] = *(const i32x4*)(smem[st][0] + row * kRowBytes + ((ch ^ (row & 7)) << 4));
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int row = wn * 64 + j * 16 + m16, ch = s * 4 + g;
        bf[j] = *(const i32x4*)(smem[st][1] + row * kRowBytes + ((ch ^ (row & 7)) << 4));
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = frag_mma<ELT>(af[i], bf[j], acc[i][j]);
    }
    if (kk + 1 < k1) swrite(st ^ 1);
    __syncthreads();
  }

#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int x = x0 + wn * 64 + j * 16 + m16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int q = q0 + wm * 64 + i * 16 + 4 * g + r;
        if (q < n_q && x < n_train) S[(int64_t)q * n_train + x] = acc[i][j][r];
      }
    }
  if (sq) {  // eight threads hold the pieces of a row
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float v = nsq[i];
      v += __shfl_xor(v, 1, 64);
      v += __shfl_xor(v, 2, 64);
      v += __shfl_xor(v, 4, 64);
      const int row = (tid + 256 * i) >> 3;
      if ((tid & 7) == 0 && x0 + row < n_train) norms[(int64_t)blockIdx.y * n_train + x0 + row] = v;
    }
  }
}

// float32: each thread loads 32 bytes of two rows per side, one stage ahead,
// splits them once and writes 16 bytes to each of the three planes of its side
// in LDS (64 bytes per row and plane; the 16-byte chunk c of row r at c XOR
// (r / 2) mod 4); the waves read operands from there: 24 reads for 96 MFMA per
// stage.  A value is split once per tile and used by 128 products.  Two
// workgroups share a CU (174 registers), so one's splitting runs beside the other's MFMA.  Blocks of 16
// query rows past n_q are not multiplied.  A wave's block with a result that
// the split may have cost bits (split_unsafe) is computed again in float32 MFMA from memory.  Bound by the issue of MFMA and
// splitting: the whole cosine call for 256 x 8192 x 12288 takes 0.30 ms (0.52 ms
// in float32 MFMA at 99 TFLOP/s, with a second read of both sides for the norms).
constexpr int kPlane = kBM * 64;
__device__ inline int plane_off(int row, int chunk) { return row * 64 + ((chunk ^ ((row >> 1) & 3)) << 4); }

__global__ __launch_bounds__(256, 2) void score_gemm_split_kernel(const uint8_t* __restrict__ Q,
                                                                  const uint8_t* __restrict__ X,
                                                                  float* __restrict__ S, float* __restrict__ norms,
                                                                  int n_q, int n_train, int F, int ldq, int ldx,
                                                                  int n_qt, int n_xt, int sps) {
  constexpr int BK = 32;
  __shared__ __align__(16) uint8_t lds[2 * 3 * kPlane];  // [Q, X][hi, mid, lo]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = lane >> 4, m16 = lane & 15, wm = wave >> 1, wn = wave & 1;
  int qt, xt;
  tile_of(blockIdx.x, n_qt, n_xt, &qt, &xt);
  const int q0 = qt * kBM, x0 = xt * kBN;
  const int rows_q = min(kBM, n_q - q0), rows_x = min(kBN, n_train - x0);
  const rsrc_t rq = make_rsrc(Q + (int64_t)q0 * ldq * 4, (uint32_t)(((int64_t)(rows_q - 1) * ldq + F) * 4));
  const rsrc_t rx = make_rsrc(X + (int64_t)x0 * ldx * 4, (uint32_t)(((int64_t)(rows_x - 1) * ldx + F) * 4));
  const int ni = min(4, max(0, (rows_q - wm * 64 + 15) / 16));  // this wave's blocks of query rows
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int nk = (F + BK - 1) / BK;
  const int k0 = blockIdx.y * sps, k1 = min(nk, k0 + sps);  // this split's K steps
  S += (int64_t)blockIdx.y * n_q * n_train;
  const int row = tid >> 2, pc = tid & 3;  // rows row and row + 64, features 8 pc .. + 7 of a stage
  i32x4 xq[2][2], xx[2][2];
  auto load = [&](int kk) {
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int col = kk * BK + pc * 8 + 4 * h;
        xq[t][h] = load_frag_ld<4>(rq, row + 64 * t, rows_q, col, F, ldq);
        xx[t][h] = load_frag_ld<4>(rx, row + 64 * t, rows_x, col, F, ldx);
      }
  };
  const bool sq = norms && qt == 0;  // uniform
  float nsq[2] = {0.f, 0.f};
  float big[2][2] = {{0.f, 0.f}, {0.f, 0.f}};  // [Q, X][row, row + 64]: largest magnitude of this thread's share
  auto put_one = [&](uint8_t* side, int r, const i32x4 (&v)[2]) {
    const Split3 s = split3(v[0], v[1]);
    uint8_t* w = side + plane_off(r, pc);
    *(bf16x8*)w = s.hi;
    *(bf16x8*)(w + kPlane) = s.mid;
    *(bf16x8*)(w + 2 * kPlane) = s.lo;
  };
  auto put = [&] {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      if (64 * t < rows_q) put_one(lds, row + 64 * t, xq[t]);  // uniform
      put_one(lds + 3 * kPlane, row + 64 * t, xx[t]);
      if (sq) nsq[t] = sum_sq<4>(xx[t][1], sum_sq<4>(xx[t][0], nsq[t]));
    }
#pragma unroll
    for (int t = 0; t < 2; ++t) {  // while the planes are written; query rows past the tile's are zero
      big[0][t] = max_abs(max_abs(big[0][t], xq[t][0]), xq[t][1]);
      big[1][t] = max_abs(max_abs(big[1][t], xx[t][0]), xx[t][1]);
    }
  };
  auto get = [&](const uint8_t* side, int r) {
    const uint8_t* w = side + plane_off(r, g);
    return Split3{*(const bf16x8*)w, *(const bf16x8*)(w + kPlane), *(const bf16x8*)(w + 2 * kPlane)};
  };
  if (k0 < k1) load(k0);
  for (int kk = k0; kk < k1; ++kk) {
    lds_barrier();  // the previous stage's operands are read
    put();
    load(kk + 1);  // past the last stage: never used
    lds_barrier();
    if (ni > 0) {
      Split3 b[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = get(lds + 3 * kPlane, wn * 64 + 16 * j + m16);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (i < ni) {  // uniform over the wave
          const Split3 a = get(lds, wm * 64 + 16 * i + m16);
#define DATTRI_TERM(p) _Pragma("unroll") for (int j = 0; j < 4; ++j) acc[i][j] = split_term<p>(a, b[j], acc[i][j]);
          DATTRI_TERM(0) DATTRI_TERM(1) DATTRI_TERM(2) DATTRI_TERM(3) DATTRI_TERM(4) DATTRI_TERM(5)
#undef DATTRI_TERM
        }
      }
    }
  }
  lds_barrier();  // the last stage's operands are read
  float* line = (float*)lds;  // [Q, X][128]: largest magnitude of each row
#pragma unroll
  for (int side = 0; side < 2; ++side)
#pragma unroll
    for (int t = 0; t < 2; ++t) {  // four threads hold the pieces of a row
      float m = big[side][t];
      m = fmaxf(m, __shfl_xor(m, 1, 64));
      m = fmaxf(m, __shfl_xor(m, 2, 64));
      if (pc == 0) line[side * kBM + row + 64 * t] = m;
    }
  lds_barrier();
  const bool bad = block_unsafe(acc, (float)((k1 - k0) * BK), line + wm * 64, line + kBM + wn * 64);
  // infinities, NaN, overflow or values too small to split: this wave's block
  // in float32 products, straight from memory
  if (__any(bad)) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int kk = k0; kk < k1; ++kk)
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int col = kk * BK + h * 16 + 4 * g;
        i32x4 a[4], b[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a[i] = load_frag_ld<4>(rq, wm * 64 + 16 * i + m16, rows_q, col, F, ldq);
          b[i] = load_frag_ld<4>(rx, wn * 64 + 16 * i + m16, rows_x, col, F, ldx);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = frag_mma<4>(a[i], b[j], acc[i][j]);
      }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int x = x0 + wn * 64 + j * 16 + m16;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int q = q0 + wm * 64 + i * 16 + 4 * g + r;
        if (q < n_q && x < n_train) S[(int64_t)q * n_train + x] = acc[i][j][r];
      }
    }
  if (sq) {  // four threads hold the pieces of a row
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      float v = nsq[t];
      v += __shfl_xor(v, 1, 64);
      v += __shfl_xor(v, 2, 64);
      if (pc == 0 && x0 + row + 64 * t < n_train) norms[(int64_t)blockIdx.y * n_train + x0 + row + 64 * t] = v;
    }
  }
}

// ------------------------------------------------------ cosine normalization
// inv[r] = 1 / |row r (times d, when given)|, 0 for a zero row.  One wave per
// row, 16-byte loads (rows are 16-byte aligned and F a multiple of 16 bytes).
template <int ELT>
__global__ __launch_bounds__(256) void row_inv_norms_kernel(const uint8_t* __restrict__ X, int64_t ld,
                                                            int64_t rows, int64_t F,
                                                            const float* __restrict__ d,
                                                            float* __restrict__ inv) {
  constexpr int EPL = 16 / ELT;
  const int lane = threadIdx.x & 63;
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (r >= rows) return;  // the whole wave leaves; no barrier below
  const uint8_t* row = X + r * ld * ELT;
  float s = 0.f;
  for (int64_t f = (int64_t)lane * EPL; f < F; f += 64 * EPL) {
    // elements named explicitly: bit-casting single vector elements inside an
    // unrolled loop was compiled to read element 0 for every index
    const i32x4 v = *(const i32x4*)(row + f * ELT);
    float x[EPL];
    if constexpr (ELT == 2) {
      const uint32_t w0 = (uint32_t)v.x, w1 = (uint32_t)v.y, w2 = (uint32_t)v.z, w3 = (uint32_t)v.w;
      x[0] = bf16_bits_to_f32(w0 & 0xFFFFu); x[1] = bf16_bits_to_f32(w0 >> 16);
      x[2] = bf16_bits_to_f32(w1 & 0xFFFFu); x[3] = bf16_bits_to_f32(w1 >> 16);
      x[4] = bf16_bits_to_f32(w2 & 0xFFFFu); x[5] = bf16_bits_to_f32(w2 >> 16);
      x[6] = bf16_bits_to_f32(w3 & 0xFFFFu); x[7] = bf16_bits_to_f32(w3 >> 16);
    } else {
      const f32x4 fv = __builtin_bit_cast(f32x4, v);
      x[0] = fv.x; x[1] = fv.y; x[2] = fv.z; x[3] = fv.w;
    }
#pragma unroll
    for (int j = 0; j < EPL; ++j) {
      const float y = d ? x[j] * d[f + j] : x[j];
      s = fmaf(y, y, s);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) inv[r] = s > 0.f ? 1.f / sqrtf(s) : 0.f;
}

// S[q][j] *= iq[q] * it[j] (rows of S dense, n_train apart).
__global__ __launch_bounds__(256) void scale_scores_kernel(float* __restrict__ S, int64_t n_q, int64_t n_train,
                                                           const float* __restrict__ iq,
                                                           const float* __restrict__ it) {
  for (int64_t q = blockIdx.x; q < n_q; q += gridDim.x) {
    const float a = iq[q];
    float* row = S + q * n_train;
    for (int64_t j = threadIdx.x; j < n_train; j += 256) row[j] *= a * it[j];
  }
}

// Inverse norms of few long rows: NW waves per row, four loads in flight per
// thread (one wave per row leaves a single query's 200k features to 450 round
// trips).
template <int ELT, int NW>
__global__ __launch_bounds__(64 * NW) void row_inv_norms_wide_kernel(const uint8_t* __restrict__ X, int64_t ld, int64_t F,
                                                                  const float* __restrict__ d,
                                                                  float* __restrict__ inv) {
  constexpr int EPL = 16 / ELT;
  __shared__ float red[NW];
  const uint8_t* row = X + (int64_t)blockIdx.x * ld * ELT;
  float s = 0.f;
#pragma unroll 4
  for (int64_t f = (int64_t)threadIdx.x * EPL; f < F; f += 64 * NW * EPL) {
    const i32x4 v = *(const i32x4*)(row + f * ELT);
    if (!d) {
      s = sum_sq<ELT>(v, s);
    } else if constexpr (ELT == 2) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t w = (uint32_t)(e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w);
        const float a = bf16_bits_to_f32(w & 0xFFFFu) * d[f + 2 * e], b = bf16_bits_to_f32(w >> 16) * d[f + 2 * e + 1];
        s = fmaf(b, b, fmaf(a, a, s));
      }
    } else {
      f32x4 x = __builtin_bit_cast(f32x4, v);
      x.x *= d[f]; x.y *= d[f + 1]; x.z *= d[f + 2]; x.w *= d[f + 3];
      s = sum_sq<4>(__builtin_bit_cast(i32x4, x), s);
    }
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) t += red[w];
    inv[blockIdx.x] = t > 0.f ? 1.f / sqrtf(t) : 0.f;
  }
}

template <int ELT>
static hipError_t launch_norms(const uint8_t* X, int64_t ld, int64_t rows, int64_t F, const float* d, float* inv,
                               hipStream_t s) {
  // Waves per row.  Short rows (up to 4 KB): one, as a workgroup each costs more
  // than it reads (2048 rows of 256 floats: 2.7 us, 16 waves 5.0).  Longer: four,
  // one load each in flight (100 rows of 4096 bf16: 2.4 us, one wave 4.0; 2048
  // rows of 12288 floats: 15.6 and 18.9), or 16 where that many have loads to
  // make and rows are too few to fill the chip with fewer (256 rows of 12288
  // floats, not in a cache: 5.2 us, 4 waves 8.1) or rows are very long (one of
  // 229376 floats: 7.9 us, 4 waves 14.1, one 98.9).  More than 2048 rows fill the
  // chip with a wave each (4096 rows of 12288: 28.8 us either way).
  const int64_t bytes = F * ELT;
  if (rows <= 2048 && (bytes > 131072 || (rows <= 512 && bytes > 16384))) {
    hipLaunchKernelGGL((row_inv_norms_wide_kernel<ELT, 16>), dim3((unsigned)rows), dim3(1024), 0, s, X, ld, F, d, inv);
  } else if (rows <= 2048 && bytes > 4096) {
    hipLaunchKernelGGL((row_inv_norms_wide_kernel<ELT, 4>), dim3((unsigned)rows), dim3(256), 0, s, X, ld, F, d, inv);
  } else {
    const int64_t b = (rows + 3) / 4;
    if (b > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(row_inv_norms_kernel<ELT>, dim3((unsigned)b), dim3(256), 0, s, X, ld, rows, F, d, inv);
  }
  return hipGetLastError();
}

hipError_t launch_row_inv_norms(int elt, const void* X, int64_t ld, int64_t rows, int64_t F, const float* d, float* inv,
                                hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  return elt == 2 ? launch_norms<2>((const uint8_t*)X, ld, rows, F, d, inv, s)
                  : launch_norms<4>((const uint8_t*)X, ld, rows, F, d, inv, s);
}

// S[q][j] = iq[q] / |x_j| sum over splits of part[y][q][j], |x_j|^2 the sum over
// splits of norm_parts[y][j].  Thread: one training row, qpt queries.
// part may be S itself (one split): every thread reads an element before it
// writes that element, and no other thread touches it.
__global__ __launch_bounds__(256) void finish_cosine_kernel(const float* part, int ks, int64_t n_q, int64_t n_train,
                                                            const float* __restrict__ iq,
                                                            const float* __restrict__ norm_parts, int qpt, float* S) {
  const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (j >= n_train) return;
  float s = 0.f;
  for (int y = 0; y < ks; ++y) s += norm_parts[(int64_t)y * n_train + j];
  const float it = s > 0.f ? 1.f / sqrtf(s) : 0.f;
  const int64_t step = n_q * n_train, q1 = min<int64_t>(n_q, ((int64_t)blockIdx.y + 1) * qpt);
  for (int64_t q = (int64_t)blockIdx.y * qpt; q < q1; ++q) {
    const float* p = part + q * n_train + j;
    float v = 0.f;
    int y = 0;
    for (; y + 4 <= ks; y += 4) {
      const float v0 = p[y * step], v1 = p[(y + 1) * step], v2 = p[(y + 2) * step], v3 = p[(y + 3) * step];
      v = (((v + v0) + v1) + v2) + v3;
    }
    for (; y < ks; ++y) v += p[y * step];
    S[q * n_train + j] = v * (iq[q] * it);
  }
}

hipError_t launch_finish_cosine(const float* part, int ks, int64_t n_q, int64_t n_train, const float* iq,
                                const float* norm_parts, float* S, hipStream_t s) {
  if (n_q <= 0 || n_train <= 0) return hipSuccess;
  // queries per thread: as many as leave about 1024 workgroups (each sums its
  // rows' norms once), and no more workgroups in y than a grid holds
  const int64_t gx = (n_train + 255) / 256;
  const int64_t qpt = std::max<int64_t>(std::min<int64_t>(32, n_q * gx / 1024), (n_q + 65534) / 65535);
  const int64_t per = std::max<int64_t>(qpt, 1), gy = (n_q + per - 1) / per;
  hipLaunchKernelGGL(finish_cosine_kernel, dim3((unsigned)gx, (unsigned)gy), dim3(256), 0, s, part, ks, n_q, n_train, iq,
                     norm_parts, (int)per, S);
  return hipGetLastError();
}

hipError_t launch_cosine_scale(int elt, const void* Q, int64_t ldq, const float* d, const void* X, int64_t ldx,
                               float* S, int64_t n_q, int64_t n_train, int64_t F, float* inv_q, float* inv_t,
                               hipStream_t s) {
  if (n_q <= 0 || n_train <= 0) return hipSuccess;
  hipError_t e = launch_row_inv_norms(elt, Q, ldq, n_q, F, d, inv_q, s);
  if (e == hipSuccess) e = launch_row_inv_norms(elt, X, ldx, n_train, F, nullptr, inv_t, s);
  if (e != hipSuccess) return e;
  const unsigned blocks = (unsigned)std::min<int64_t>(n_q, 4096);
  hipLaunchKernelGGL(scale_scores_kernel, dim3(blocks), dim3(256), 0, s, S, n_q, n_train, inv_q, inv_t);
  return hipGetLastError();
}

hipError_t launch_scale_rows(int elt, const void* src, int64_t ld_src, const float* d, void* dst,
                             int64_t ld_dst, int64_t rows, int64_t F, hipStream_t s) {
  const int64_t n = rows * F;
  if (n <= 0) return hipSuccess;
  const int blocks = (int)std::min<int64_t>((n + 255) / 256, 65536);
  if (elt == 2)
    hipLaunchKernelGGL(scale_rows_kernel<2>, dim3(blocks), dim3(256), 0, s, (const uint8_t*)src,
                       ld_src, d, (uint8_t*)dst, ld_dst, rows, F);
  else
    hipLaunchKernelGGL(scale_rows_kernel<4>, dim3(blocks), dim3(256), 0, s, (const uint8_t*)src,
                       ld_src, d, (uint8_t*)dst, ld_dst, rows, F);
  return hipGetLastError();
}

hipError_t launch_score_tiles(int elt, const void* Q, int64_t ldq, const float* d, const void* X, int64_t ldx,
                              float* S, int64_t n_q, int64_t n_train, int64_t F, void* qws, int64_t ld_ws,
                              float* partials, const float* iq, float* norm_parts, hipStream_t s) {
  if (n_q <= 0 || n_train <= 0) return hipSuccess;
  if (d && F > 0) {  // scaled queries, row-major in the workspace
    if (!qws) return hipErrorInvalidValue;
    hipError_t e = launch_scale_rows(elt, Q, ldq, d, qws, ld_ws, n_q, F, s);
    if (e != hipSuccess) return e;
    Q = qws;
    ldq = ld_ws;
  }
  const int n_qt = (int)((n_q + kBM - 1) / kBM), n_xt = (int)((n_train + kBN - 1) / kBN);
  const int64_t nb = (int64_t)n_qt * n_xt;
  if (nb > INT32_MAX) return hipErrorInvalidValue;
  const int64_t nk = (F + kRowBytes / elt - 1) / (kRowBytes / elt);
  const int ks = score_ksplit(elt, n_q, n_train, F);
  const int sps = ks > 1 ? (int)((nk + ks - 1) / ks) : (int)std::max<int64_t>(nk, 1);
  if (ks > 1 && !partials) return hipErrorInvalidValue;
  float* out = ks > 1 ? partials : S;
  if (elt == 2)
    hipLaunchKernelGGL(score_gemm_kernel, dim3((unsigned)nb, (unsigned)ks), dim3(256), 0, s, (const uint8_t*)Q,
                       (const uint8_t*)X, out, norm_parts, (int)n_q, (int)n_train, (int)F, (int)ldq, (int)ldx, n_qt,
                       n_xt, sps);
  else
    hipLaunchKernelGGL(score_gemm_split_kernel, dim3((unsigned)nb, (unsigned)ks), dim3(256), 0, s, (const uint8_t*)Q,
                       (const uint8_t*)X, out, norm_parts, (int)n_q, (int)n_train, (int)F, (int)ldq, (int)ldx, n_qt,
                       n_xt, sps);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (norm_parts) return launch_finish_cosine(out, ks, n_q, n_train, iq, norm_parts, S, s);
  return ks == 1 ? hipSuccess : launch_splitk_sum(partials, ks, n_q * n_train, S, s);
}

}  // namespace dattri
