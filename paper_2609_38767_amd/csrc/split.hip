// Factored route (Eq. (2), left side) in two stages, for captures with few
// examples or short sequences.
//
// The fused kernel's work items are (input group, example, token chunk); with
// few layers, examples or tokens there are too few of them, each streaming
// whole rows of width d_in + d_out, and most of the chip idles.  Here the
// projections themselves are split over the feature dimension:
//
//   stage 1  for every factor block X (a group's A, each member's B) viewed as
//            n*T token rows: out[s][row][:] = X[row, slab s] P[slab s, :],
//            float32, one workgroup per (block, 256-row block, slab; 128 rows
//            in float32 and at 8 unaligned tiles).  The aligned stream neither
//            reads nor writes rows past an example's length; the element loads
//            of unaligned blocks take them along, and stage 2 ignores them.
//   stage 2  per (layer, example, token chunk): Psi[c][r] = sum_t a~_t[c] g~_t[r]
//            with a~_t = sum_s outA[s][t] and g~_t = sum_s outB[s][t], over
//            the example's first T_i tokens (Eq. (4) allows T_i < T), written
//            into the layer block of phi, or as partial blocks summed by the
//            reduce kernel when an example's tokens span several chunks.
//
// Every sum runs in a fixed order, so results are bitwise reproducible.
#include "device_common.h"
#include "internal.h"
#include "project_rows.h"
#include "split_stream.h"

namespace dattri {
using namespace dev;

// ---------------------------------------------------------------- stage 1
// Blocks with 16-byte aligned rows: rows stream through LDS by direct loads
// (stream_rows, stream_rows_f32).  Bound by HBM: per 256-row item and 128-byte
// column stage a workgroup moves 32 KiB of X and 2 NT KiB of map fragments
// (from L2).  One launch serves every op of the call, whatever its tile count
// (the body is chosen per item), so the chip fills once per call and not once
// per tile count; bf16: one workgroup per CU, its ring as deep as 160 KiB of
// LDS allow; float32: three, whose splitting and MFMA interleave.  Measured
// against the register path it replaced: 4 Llama-8B-shaped blocks, 8 x 2048
// bf16 rows, k = 32: 2.07 -> 1.50 ms (6.1 TB/s); 24 Pythia-410M-shaped blocks,
// 8 ragged float32 examples of up to 512, k = 64: 2.27 -> 1.1 ms.  The loads of a
// block that no other op reads are non-temporal (1.69 -> 1.55 ms on the first).
template <int ELT>
__global__ __launch_bounds__(256, ELT == 2 ? 1 : 3) void split_stream_kernel(
    const SplitItem* __restrict__ items, const SplitOp* __restrict__ ops, float* __restrict__ out) {
  constexpr int kMax24 = max_of(split_lds<ELT, 2>(), split_lds<ELT, 4>());
  constexpr int kBytes = ELT == 2 ? max_of(kMax24, max_of(split_lds<2, 6>(), split_lds<2, 8>())) : kMax24;
  static_assert(kBytes <= 160 * 1024, "LDS of one CU");
  __shared__ __align__(1024) uint8_t smem[kBytes];
  const SplitItem it = items[blockIdx.x];
  if (it.op < 0) return;  // padding item of the XCD-interleaved order
  const SplitOp& O = ops[it.op];
  auto map = [&](int t, const uint8_t** base, int64_t* stride) {
    *stride = (int64_t)O.ptile_nt[t] * kFragBytes;
    *base = (const uint8_t*)O.ptile[t] + (int64_t)O.ptile_local[t] * kFragBytes;
  };
  if (O.nt <= 2) {
    split_stream_body<ELT, 2, false>(it, O, map, out, smem, nullptr);
  } else if (ELT == 4 || O.nt <= 4) {  // float32 ops hold at most 4 tiles (kSplitMaxTilesF32)
    split_stream_body<ELT, 4, false>(it, O, map, out, smem, nullptr);
  } else if constexpr (ELT == 2) {
    if (O.nt <= 6)
      split_stream_body<2, 6, false>(it, O, map, out, smem, nullptr);
    else
      split_stream_body<2, 8, false>(it, O, map, out, smem, nullptr);
  }
}

// Blocks whose rows are not 16-byte multiples: element loads into registers.
template <int ELT, int NT>
__global__ __launch_bounds__(256, 2) void split_project_kernel(const SplitItem* __restrict__ items,
                                                               const SplitOp* __restrict__ ops,
                                                               float* __restrict__ out) {
  constexpr bool AL = false;
  constexpr int KR = 4 * (16 / ELT);  // rows of a packed k-block
  constexpr int RT = split_rt_of(NT), ROWS = split_rows_of(NT);
  static_assert(kWaves * RT * 16 == ROWS, "row block");
  constexpr int PD = 2;  // measured: deeper prefetch does not pay with 4 row tiles
  __shared__ __align__(16) uint8_t pan[2][kPanel][NT][kFragBytes];
  const SplitItem it = items[blockIdx.x];
  if (it.op < 0) return;  // padding item of the XCD-interleaved order
  const SplitOp& O = ops[it.op];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int g = lane >> 4, m16 = lane & 15;
  const int row0 = it.row_block * ROWS;
  const int nrows = min(ROWS, O.rows - row0);
  const int col0 = it.slab * O.slab_cols;
  const int d = min(O.slab_cols, O.ld - col0);
  // descriptor over this row block, starting at the slab's first column
  const uint8_t* base = (const uint8_t*)O.X + ((int64_t)row0 * O.ld + col0) * ELT;
  const rsrc_t r = make_rsrc(base, (uint32_t)(((int64_t)nrows * O.ld - col0) * ELT));
  FragSrc<NT> P;
  P.nt = O.nt;
  const int kb0 = col0 / KR;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int tt = t < O.nt ? t : 0;
    P.stride[t] = (int64_t)O.ptile_nt[tt] * kFragBytes;
    P.base[t] = (const uint8_t*)O.ptile[tt] + (int64_t)O.ptile_local[tt] * kFragBytes + kb0 * P.stride[t];
  }
  f32x4 acc[RT][NT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[rt][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int r_wave = wave * RT * 16;
  project_rows<ELT, AL, RT, NT, NT, PD>(r, r_wave, nrows, d, O.ld, P, acc, pan);

  const int ldo = O.out_ld;
  float* dst = out + O.out_base + ((int64_t)it.slab * O.rows + row0) * ldo;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      if (t < O.nt) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = r_wave + rt * 16 + 4 * g + i;
          if (row < nrows) dst[(int64_t)row * ldo + t * 16 + m16] = acc[rt][t][i];
        }
      }
    }
}

// ---------------------------------------------------------------- stage 2
// Psi = A~^T B~ over the tokens of one (layer, example, token chunk), float32
// MFMA 16x16x4 straight from the projected rows: a lane of group g loads VA
// (VB) consecutive columns of token 4u + g, which are the K slots of VA x VB
// output tiles at once (tile i, j holds columns VA m + i and VB n + j), so one
// 64-byte to 512-byte row piece per token feeds VA * VB products and nothing
// passes through LDS.  The eight waves take every eighth 16-token step, the
// next step's rows loaded while the current one is multiplied; their blocks
// are added pairwise in LDS in a fixed order.  Slabs are added on load in slab
// order.  Bound by the row reads: 28 layers x 8 examples x 2048 tokens, k = 32,
// 0.032 ms (0.253 ms with rows copied to LDS and products on the vector ALU).  A task with one chunk per example writes phi; otherwise each chunk
// writes a padded partial block that the reduce kernel sums in chunk order.
constexpr int kConWaves = 8;

template <int V>
__device__ inline void load_cols(rsrc_t r, uint32_t off, float (&v)[V]) {
  if constexpr (V == 1) {
    v[0] = __builtin_bit_cast(float, load4(r, off));
  } else if constexpr (V == 2) {
    const i32x2 x = load8(r, off);
    v[0] = __builtin_bit_cast(float, (int)x.x);
    v[1] = __builtin_bit_cast(float, (int)x.y);
  } else {
#pragma unroll
    for (int q = 0; q < V / 4; ++q) {
      const f32x4 x = __builtin_bit_cast(f32x4, load16(r, off + 16 * q));
      v[4 * q] = x.x; v[4 * q + 1] = x.y; v[4 * q + 2] = x.z; v[4 * q + 3] = x.w;
    }
  }
}

template <int VA, int VB>
__global__ __launch_bounds__(64 * kConWaves, VA * VB >= 16 ? 2 : 4) void split_contract_kernel(
    const ContractTask* __restrict__ tasks, const float* __restrict__ proj, float* __restrict__ partials,
    void* __restrict__ phi, int phi_bf16, int64_t ld_phi) {
  constexpr int U = VA * VB > 16 ? 2 : 4;  // token quads per step
  constexpr int kStep = 4 * U;             // tokens per wave and step
  __shared__ f32x4 red[kConWaves / 2][VA * VB][64];
  const ContractTask t = tasks[blockIdx.z];
  const int chunk = blockIdx.x, ex = blockIdx.y, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (chunk >= t.n_tchunks) return;
  const int g = lane >> 4, m = lane & 15;
  int t_eff = t.T;
  if (t.lengths) t_eff = min(max(t.lengths[ex], 0), t.T);
  const int tok0 = chunk * t.tok_chunk, tok1 = min(t_eff, tok0 + t.tok_chunk);
  const int nt = max(tok1 - tok0, 0);
  const int ki16 = (t.k_in + 15) & ~15, ko16 = (t.k_out + 15) & ~15;
  // one descriptor per side over the chunk's rows of one slab; tokens past the
  // chunk and columns past the layer's tiles read as zero
  const int64_t row = (int64_t)ex * t.T + tok0;
  const int a_row = t.a_ld * 4, b_row = t.b_ld * 4;
  const uint32_t a_rng = nt > 0 ? (uint32_t)((nt - 1) * a_row + ki16 * 4) : 0u;
  const uint32_t b_rng = nt > 0 ? (uint32_t)((nt - 1) * b_row + ko16 * 4) : 0u;
  const uint32_t a0 = VA * m < ki16 ? (uint32_t)(g * a_row + VA * m * 4) : kFarOff;
  const uint32_t b0 = VB * m < ko16 ? (uint32_t)(g * b_row + VB * m * 4) : kFarOff;
  auto load = [&](int step, float (&a)[U][VA], float (&b)[U][VB]) {
    const float* pa = proj + t.a_base + row * t.a_ld + t.a_col0;
    const float* pb = proj + t.b_base + row * t.b_ld;
    const rsrc_t ra = make_rsrc(pa, a_rng), rb = make_rsrc(pb, b_rng);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int tok = step * kStep + 4 * u;
      load_cols<VA>(ra, tok + g < nt ? a0 + (uint32_t)(tok * a_row) : kFarOff, a[u]);
      load_cols<VB>(rb, tok + g < nt ? b0 + (uint32_t)(tok * b_row) : kFarOff, b[u]);
    }
    for (int sl = 1; sl < t.a_slabs; ++sl) {
      const rsrc_t rs = make_rsrc(pa + (int64_t)sl * t.rows * t.a_ld, a_rng);
      float x[U][VA];
#pragma unroll
      for (int u = 0; u < U; ++u)
        load_cols<VA>(rs, step * kStep + 4 * u + g < nt ? a0 + (uint32_t)((step * kStep + 4 * u) * a_row) : kFarOff, x[u]);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < VA; ++i) a[u][i] += x[u][i];
    }
    for (int sl = 1; sl < t.b_slabs; ++sl) {
      const rsrc_t rs = make_rsrc(pb + (int64_t)sl * t.rows * t.b_ld, b_rng);
      float x[U][VB];
#pragma unroll
      for (int u = 0; u < U; ++u)
        load_cols<VB>(rs, step * kStep + 4 * u + g < nt ? b0 + (uint32_t)((step * kStep + 4 * u) * b_row) : kFarOff, x[u]);
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < VB; ++i) b[u][i] += x[u][i];
    }
  };
  f32x4 psi[VA][VB];
#pragma unroll
  for (int i = 0; i < VA; ++i)
#pragma unroll
    for (int j = 0; j < VB; ++j) psi[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int steps = (nt + kStep - 1) / kStep;
  float a[U][VA], b[U][VB];
  if (wave < steps) load(wave, a, b);
  for (int s = wave; s < steps; s += kConWaves) {
    float an[U][VA], bn[U][VB];
    if (s + kConWaves < steps) load(s + kConWaves, an, bn);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < VA; ++i)
#pragma unroll
        for (int j = 0; j < VB; ++j) psi[i][j] = mfma_f32_4(a[u][i], b[u][j], psi[i][j]);
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int i = 0; i < VA; ++i) a[u][i] = an[u][i];
#pragma unroll
      for (int j = 0; j < VB; ++j) b[u][j] = bn[u][j];
    }
  }
  // waves w + h into w for h = 4, 2, 1
#pragma unroll
  for (int h = kConWaves / 2; h >= 1; h >>= 1) {
    if (wave >= h && wave < 2 * h) {
#pragma unroll
      for (int i = 0; i < VA; ++i)
#pragma unroll
        for (int j = 0; j < VB; ++j) red[wave - h][i * VB + j][lane] = psi[i][j];
    }
    __syncthreads();
    if (wave < h) {
#pragma unroll
      for (int i = 0; i < VA; ++i)
#pragma unroll
        for (int j = 0; j < VB; ++j) psi[i][j] += red[wave][i * VB + j][lane];
    }
    __syncthreads();
  }
  if (wave != 0) return;
  float* part = nullptr;
  if (t.n_tchunks > 1)
    part = partials + t.partial_base + ((int64_t)ex * t.n_tchunks + chunk) * ki16 * ko16;
#pragma unroll
  for (int i = 0; i < VA; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int c = VA * (4 * g + e) + i;
#pragma unroll
      for (int j = 0; j < VB; ++j) {
        const int r = VB * m + j;
        const float v = psi[i][j][e];
        if (part) {
          if (c < ki16 && r < ko16) part[c * ko16 + r] = v;
        } else if (c < t.k_in && r < t.k_out) {
          const int64_t o = (int64_t)ex * ld_phi + t.phi_offset + (int64_t)c * t.k_out + r;
          if (phi_bf16)
            ((uint16_t*)phi)[o] = f32_to_bf16_bits(v);
          else
            ((float*)phi)[o] = v;
        }
      }
    }
}

// ---------------------------------------------------------------- launch
int split_nt_instance(int nt_req) { return nt_req <= 1 ? 1 : nt_req <= 2 ? 2 : nt_req <= 4 ? 4 : 8; }

template <int ELT>
static hipError_t launch_split_unaligned(int nt, const SplitItem* items, int n_items, const SplitOp* ops, float* out,
                                         hipStream_t s) {
  const dim3 grid((unsigned)n_items), block(256);
  switch (nt) {
    case 1: hipLaunchKernelGGL((split_project_kernel<ELT, 1>), grid, block, 0, s, items, ops, out); break;
    case 2: hipLaunchKernelGGL((split_project_kernel<ELT, 2>), grid, block, 0, s, items, ops, out); break;
    case 4: hipLaunchKernelGGL((split_project_kernel<ELT, 4>), grid, block, 0, s, items, ops, out); break;
    case 8: hipLaunchKernelGGL((split_project_kernel<ELT, 8>), grid, block, 0, s, items, ops, out); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_split_project(int elt_bytes, int aligned, int nt, const SplitItem* items,
                                int n_items, const SplitOp* ops, float* out, hipStream_t s) {
  if (n_items <= 0) return hipSuccess;
  if (!aligned)
    return elt_bytes == 2 ? launch_split_unaligned<2>(nt, items, n_items, ops, out, s)
                          : launch_split_unaligned<4>(nt, items, n_items, ops, out, s);
  const dim3 grid((unsigned)n_items);
  if (elt_bytes == 2)
    hipLaunchKernelGGL(split_stream_kernel<2>, grid, dim3(256), 0, s, items, ops, out);
  else
    hipLaunchKernelGGL(split_stream_kernel<4>, grid, dim3(256), 0, s, items, ops, out);
  return hipGetLastError();
}

hipError_t launch_split_contract(int na, int nb, const ContractTask* tasks, int n_tasks, int n_examples,
                                 int max_tchunks, const float* proj, float* partials, void* phi,
                                 int phi_bf16, int64_t ld_phi, hipStream_t s) {
  if (n_tasks <= 0 || n_examples <= 0 || max_tchunks <= 0) return hipSuccess;
  if (n_examples > 65535 || n_tasks > 65535) return hipErrorInvalidValue;
  const dim3 grid(max_tchunks, n_examples, n_tasks), block(64 * kConWaves);
#define DATTRI_CON(A, B)                                                                                       \
  if (na <= A && nb <= B) {                                                                                    \
    hipLaunchKernelGGL((split_contract_kernel<A, B>), grid, block, 0, s, tasks, proj, partials, phi, phi_bf16, \
                       ld_phi);                                                                                \
    return hipGetLastError();                                                                                  \
  }
  DATTRI_CON(1, 1) DATTRI_CON(1, 2) DATTRI_CON(1, 4) DATTRI_CON(2, 1) DATTRI_CON(2, 2) DATTRI_CON(2, 4)
  DATTRI_CON(4, 1) DATTRI_CON(4, 2) DATTRI_CON(4, 4) DATTRI_CON(8, 4)
#undef DATTRI_CON
  return hipErrorInvalidValue;
}

}  // namespace dattri
