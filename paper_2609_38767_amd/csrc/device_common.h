// Device helpers for gfx950: MFMA wrappers, buffer-resource loads with
// hardware bounds checks, and bf16 conversion.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dattri {
namespace dev {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

// Raw buffer descriptor over [base, base + bytes).  Loads at byte offsets
// >= bytes return zero (CDNA buffer range checking), which masks ragged
// token rows and feature tails without branches.
// Every caller passes a wave-uniform base and size; readfirstlane makes that
// visible to the compiler so the descriptor lives in SGPRs (no per-lane
// "waterfall" loop around each buffer load).
__device__ inline rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t p = (uint64_t)base;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)p);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(p >> 32));
  const uint32_t n = __builtin_amdgcn_readfirstlane(bytes);
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), (short)0, (int)n,
                                           0x00020000);
}
constexpr uint32_t kOOB = 0xFFFFFFF0u;  // an offset no descriptor here covers

// LDS destination of a direct load (buffer_load ... lds): lane l's 16 bytes
// land at p + 16 l.
#define DATTRI_LDS_PTR(p) ((__attribute__((address_space(3))) void*)(p))

// Wait until at most N vector-memory operations of this wave are in flight
// (direct loads count until their data is in LDS); other counters untouched.
template <int N>
__device__ inline void wait_vmcnt_dma() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

__device__ inline i32x4 load16(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0);
}
typedef int i32x2 __attribute__((ext_vector_type(2)));
__device__ inline i32x2 load8(rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(i32x2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ inline uint32_t load4(rsrc_t r, uint32_t off) {
  return (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0);
}
__device__ inline uint32_t load2(rsrc_t r, uint32_t off) {
  return (uint32_t)(uint16_t)__builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0);
}

// One 16-byte operand fragment: EPL = 16 / ELT consecutive elements of row
// `row` starting at column `col` of a row-major [nrows, d] block.  Rows
// >= nrows and columns >= d read as zero (their offsets are sent out of the
// descriptor's range, so 32-bit offsets never wrap into valid rows).
// `aligned` means d*ELT and the base are multiples of 16, so a fragment is
// either wholly inside or wholly outside the row.
template <int ELT>
__device__ inline i32x4 load_frag(rsrc_t r, int row, int nrows, int col, int d, bool aligned) {
  constexpr int EPL = 16 / ELT;
  const int64_t row_off = (int64_t)row * d;
  const bool row_ok = row < nrows;
  if (aligned) {
    const uint32_t off = (row_ok && col < d) ? (uint32_t)((row_off + col) * ELT) : kOOB;
    return load16(r, off);
  }
  uint32_t w[EPL];
#pragma unroll
  for (int j = 0; j < EPL; ++j) {
    const uint32_t off = (row_ok && (col + j) < d) ? (uint32_t)((row_off + col + j) * ELT) : kOOB;
    w[j] = ELT == 2 ? load2(r, off) : load4(r, off);
  }
  i32x4 v;
  if (ELT == 2) {
    v[0] = (int)(w[0] | (w[1] << 16));
    v[1] = (int)(w[2] | (w[3] << 16));
    v[2] = (int)(w[4] | (w[5] << 16));
    v[3] = (int)(w[6] | (w[7] << 16));
  } else {
    v[0] = (int)w[0]; v[1] = (int)w[1]; v[2] = (int)w[2]; v[3] = (int)w[3];
  }
  return v;
}

// One 16-byte fragment of row `row` at column `col` of a block whose rows
// are `ld` elements apart and hold d valid elements; d*ELT, ld*ELT and the
// base are multiples of 16.  Rows >= nrows and columns >= d read as zero.
template <int ELT>
__device__ inline i32x4 load_frag_ld(rsrc_t r, int row, int nrows, int col, int d, int ld) {
  const uint32_t off = (row < nrows && col < d) ? (uint32_t)(((int64_t)row * ld + col) * ELT) : kOOB;
  return load16(r, off);
}

__device__ inline f32x4 mfma_f32_4(float a, float b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// acc[16x16] += A_frag (16 rows x K) * B_frag (K x 16 cols), where each lane's
// 16-byte fragment holds its K-slice: one 16x16x32 bf16 MFMA, or four
// 16x16x4 f32 MFMAs (element j of every lane forms the j-th K=4 step).  The
// same K-slot order is used for both operands, so the sum covers all K.
template <int ELT>
__device__ inline f32x4 frag_mma(i32x4 a, i32x4 b, f32x4 c);

template <>
__device__ inline f32x4 frag_mma<2>(i32x4 a, i32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                 __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The whole 16-byte fragment is reinterpreted as four floats first: taking
// __builtin_bit_cast(float, v[j]) of single vector elements inside an unrolled
// loop was compiled to read element 0 for every j.
template <>
__device__ inline f32x4 frag_mma<4>(i32x4 a, i32x4 b, f32x4 c) {
  const f32x4 fa = __builtin_bit_cast(f32x4, a);
  const f32x4 fb = __builtin_bit_cast(f32x4, b);
  c = mfma_f32_4(fa[0], fb[0], c);
  c = mfma_f32_4(fa[1], fb[1], c);
  c = mfma_f32_4(fa[2], fb[2], c);
  c = mfma_f32_4(fa[3], fb[3], c);
  return c;
}

// A float32 value as three bf16 terms, hi + mid + lo = v exactly (hi and mid
// rounded to nearest: |v - hi| <= 2^-9 |v|, and the remainder left for lo has at
// most 8 significant bits), for finite v whose rounded hi is finite and
// |v| >= 2^-103.  Products of two split values keep the six terms down to
// 2^-18: the three left out are at most 2^-26 of the product together, below
// the float32 rounding of the sum they are added to.  Non-finite values do not
// survive the split (inf - inf), and of smaller values up to 2^-125 is lost
// (mid and lo fall among the bf16 subnormals).  Kernels that use it therefore
// keep the largest magnitude of every row and column they split and recompute
// in float32 wherever split_unsafe says that a result may miss more than its
// own float32 rounding.
struct Split3 {
  bf16x8 hi, mid, lo;
};
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ inline uint32_t pack_bf16(float a, float b) {  // round to nearest even, a in the low half
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ inline void split_pair(float a, float b, uint32_t* hi, uint32_t* mid, uint32_t* lo) {
  const uint32_t h = pack_bf16(a, b);
  const float ra = a - __builtin_bit_cast(float, h << 16), rb = b - __builtin_bit_cast(float, h & 0xFFFF0000u);
  const uint32_t m = pack_bf16(ra, rb);
  const float sa = ra - __builtin_bit_cast(float, m << 16), sb = rb - __builtin_bit_cast(float, m & 0xFFFF0000u);
  *hi = h;
  *mid = m;
  *lo = pack_bf16(sa, sb);
}
// The eight values of two float32 fragments as the K slots of one bf16 operand.
__device__ inline Split3 split3(i32x4 u, i32x4 v) {
  const f32x4 a = __builtin_bit_cast(f32x4, u), b = __builtin_bit_cast(f32x4, v);
  uint32_t h0, h1, h2, h3, m0, m1, m2, m3, l0, l1, l2, l3;
  split_pair(a.x, a.y, &h0, &m0, &l0);
  split_pair(a.z, a.w, &h1, &m1, &l1);
  split_pair(b.x, b.y, &h2, &m2, &l2);
  split_pair(b.z, b.w, &h3, &m3, &l3);
  const i32x4 h = {(int)h0, (int)h1, (int)h2, (int)h3}, m = {(int)m0, (int)m1, (int)m2, (int)m3},
              l = {(int)l0, (int)l1, (int)l2, (int)l3};
  return Split3{__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}
__device__ inline f32x4 mfma_bf16_16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
// Term p (0 .. 5, smallest products first) of a split product.
template <int p>
__device__ inline f32x4 split_term(const Split3& a, const Split3& b, f32x4 c) {
  if constexpr (p == 0) return mfma_bf16_16(a.lo, b.hi, c);
  if constexpr (p == 1) return mfma_bf16_16(a.hi, b.lo, c);
  if constexpr (p == 2) return mfma_bf16_16(a.mid, b.mid, c);
  if constexpr (p == 3) return mfma_bf16_16(a.mid, b.hi, c);
  if constexpr (p == 4) return mfma_bf16_16(a.hi, b.mid, c);
  return mfma_bf16_16(a.hi, b.hi, c);
}
// max(m, |v.x|, |v.y|, |v.z|, |v.w|), NaN ignored: one instruction per two
// values (written out: fmaxf would first quiet each loaded value).
__device__ inline float max_abs(float m, i32x4 v) {
  asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(v.x), "v"(v.y));
  asm("v_max3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(v.z), "v"(v.w));
  return m;
}
// The magnitude from which a sum of K split products of a row of largest
// magnitude mr and a column of largest magnitude mc is safe, that is off by at
// most 2^-24 of itself: each of its values lost up to 2^-125, together K 2^-125
// (mr + mc) at most, and sums of products below 2^-126 round at 2^-150 in each
// of six terms.  An exact zero stands (zero rows and disjoint rows are common)
// unless a line is below kTinyLine: nothing but zeros and values too small to
// split.
constexpr float kTinyLine = 0x1p-101f;
__device__ inline float split_safe(float K, float mr, float mc) { return K * fmaf(0x1p-101f, mr + mc, 0x1p-123f); }
__device__ inline uint32_t split_unsafe(float s, float least) {
  const float a = fabsf(s);
  return a == 0.f || (a >= least && a <= 0x1.fffffep127f) ? 0u : 1u;
}
// The smallest nonzero magnitude among the values added, and the largest (NaN
// if any is): the test of a whole block against its largest split_safe in four
// instructions per two values, before any value is looked at by itself.
struct NonzeroRange {
  uint32_t lo = 0xFFFFFFFFu;  // 2 bits - 1 without the sign: zero comes out largest
  float hi = 0.f;
  __device__ void add(float a, float b) {
    lo = min(min(lo, 2u * __builtin_bit_cast(uint32_t, a) - 1u), 2u * __builtin_bit_cast(uint32_t, b) - 1u);
    asm("v_maximum3_f32 %0, |%1|, |%2|, %0" : "+v"(hi) : "v"(a), "v"(b));
  }
  __device__ void add(f32x4 v) { add(v.x, v.y); add(v.z, v.w); }
  __device__ bool unsafe(float least) const {
    return lo < 2u * __builtin_bit_cast(uint32_t, least) - 1u || !(hi <= 0x1.fffffep127f);
  }
};
// Whether a wave's 64 x 64 block of sums of K split products (4 x 4 tiles;
// rows, cols: the largest magnitudes of its 64 rows and 64 columns, in LDS) has
// an unsafe one among this lane's.
__device__ inline bool block_unsafe(const f32x4 (&acc)[4][4], float K, const float* rows, const float* cols) {
  const int lane = threadIdx.x & 63, g = lane >> 4, m16 = lane & 15;
  NonzeroRange lines, sums;
  float mr = 0.f, mc = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const f32x4 r = *(const f32x4*)(rows + 16 * i + 4 * g);  // acc[i]: rows 16 i + 4 g .. + 3, column m16
    const float c = cols[16 * i + m16];
    mr = max_abs(mr, __builtin_bit_cast(i32x4, r));
    mc = fmaxf(mc, c);
    lines.add(r);
    lines.add(c, c);
#pragma unroll
    for (int j = 0; j < 4; ++j) sums.add(acc[i][j]);
  }
  uint32_t bad = lines.unsafe(kTinyLine) ? 1u : 0u;
  if (__any(sums.unsafe(split_safe(K, mr, mc))))
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          bad |= split_unsafe(acc[i][j][r], split_safe(K, rows[16 * i + 4 * g + r], cols[16 * j + m16]));
  return bad != 0u;
}

// Workgroup barrier that orders LDS accesses only.  __syncthreads() also
// fences global memory, which makes the compiler wait for every outstanding
// global load (vmcnt(0)) and would drain register prefetch pipelines.
__device__ inline void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

__device__ inline float bf16_bits_to_f32(uint32_t h) { return __builtin_bit_cast(float, h << 16); }

__device__ inline uint16_t f32_to_bf16_bits(float f) {
  uint32_t u = __builtin_bit_cast(uint32_t, f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// acc + the sum of squares of a fragment's values.
template <int ELT>
__device__ inline float sum_sq(i32x4 v, float acc) {
  if constexpr (ELT == 2) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t w = (uint32_t)(i == 0 ? v.x : i == 1 ? v.y : i == 2 ? v.z : v.w);
      const float a = bf16_bits_to_f32(w & 0xFFFFu), b = __builtin_bit_cast(float, w & 0xFFFF0000u);
      acc = fmaf(b, b, fmaf(a, a, acc));
    }
  } else {
    const f32x4 f = __builtin_bit_cast(f32x4, v);
    acc = fmaf(f.w, f.w, fmaf(f.z, f.z, fmaf(f.y, f.y, fmaf(f.x, f.x, acc))));
  }
  return acc;
}

// Element (v, c) of a fragment-major packed projection map (see internal.h),
// converted to float; rows >= d or columns >= k read as zero.
template <int ELT>
__device__ inline float packed_elem(const uint8_t* P, int v, int c, int d, int k) {
  if (v >= d || c >= k) return 0.f;
  constexpr int EPL = 16 / ELT, KR = 4 * EPL;
  const int nt_all = (k + 15) >> 4;
  const int kb = v / KR, w = v % KR, g = w / EPL, j = w % EPL;
  const int64_t off = (((int64_t)kb * nt_all + (c >> 4)) * 64 + 16 * g + (c & 15)) * 16 + j * ELT;
  if (ELT == 2) return bf16_bits_to_f32(*(const uint16_t*)(P + off));
  return *(const float*)(P + off);
}

}  // namespace dev
}  // namespace dattri
