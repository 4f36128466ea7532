// Streaming projection of row blocks onto 16-column tiles of a packed
// projection map: the building block of the factored route's kernels.
#pragma once
#include "device_common.h"
#include "internal.h"

namespace dattri {
namespace dev {

constexpr int kPanel = 4;  // k-blocks per LDS panel of projection fragments

// k-blocks of factor fragments prefetched ahead: about 8 KiB in flight per
// wave where the register budget of two waves per SIMD allows it, else 4 KiB.
constexpr int pd_of(int rt, int na, int nb) { return (rt >= 4 || na * (rt + nb) >= 24) ? 2 : 4; }

// Projection fragment source of up to NT output tiles: fragment (kb, t) of the
// packed map lives at base[t] + kb * stride[t] (bytes).
template <int NT>
struct FragSrc {
  const uint8_t* base[NT];
  int64_t stride[NT];
  int nt;  // tiles in use
};

// One operand fragment of X: row `row` (zero if >= nrows), EPL consecutive
// columns from `col` (zero past d), rows ld elements apart.
template <int ELT>
__device__ inline i32x4 load_frag_ld(rsrc_t r, int row, int nrows, int col, int d, int64_t ld,
                                     bool aligned) {
  constexpr int EPL = 16 / ELT;
  const int64_t row_off = (int64_t)row * ld;
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
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (int32_t)(w[2 * j] | (w[2 * j + 1] << 16));
  } else {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] = (int32_t)w[j];
  }
  return v;
}

// acc[rt][t] += X[rows, 0:d] * P[0:d, tile t] over all k-blocks of the d
// columns.  X rows r_wave + rt*16 + (lane & 15) of descriptor `r`, ld elements
// apart (rows >= nrows and columns >= d read as zero).  All 256 threads must
// call this together.
template <int ELT, bool AL, int RT, int NT, int NTL, int kPD>
__device__ inline void project_rows(const rsrc_t r, int r_wave, int nrows, int d, int64_t ld,
                                    const FragSrc<NT>& P, f32x4 (&acc)[RT][NT],
                                    uint8_t (*pan)[kPanel][NTL][kFragBytes]) {
  constexpr int EPL = 16 / ELT, KR = 4 * EPL;
  static_assert(kPanel % kPD == 0, "ring slots must be static inside a panel");
  // A panel holds kPanel * NT fragments of 1 KiB; fragment f = w + 4*i is
  // copied by wave w (one 16-byte load per lane), so every index is static.
  constexpr int NF = kPanel * NT;
  constexpr int CPT = (NF + kWaves - 1) / kWaves;  // fragments per wave
  static_assert(NT <= NTL, "panel too small");
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, m16 = lane & 15;
  const int wave = tid >> 6;
  const int nkb = (d + KR - 1) / KR;
  const int npan = (nkb + kPanel - 1) / kPanel;

  auto load_panel = [&](int p, i32x4 (&st)[CPT]) {
#pragma unroll
    for (int i = 0; i < CPT; ++i)
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const int f = w + kWaves * i, t = f % NT, kbl = f / NT;
        if (f < NF && wave == w) {
          const int kb = min(p * kPanel + kbl, nkb - 1);
          st[i] = (t < P.nt) ? *(const i32x4*)(P.base[t] + kb * P.stride[t] + lane * 16)
                             : i32x4{0, 0, 0, 0};
        }
      }
  };
  auto store_panel = [&](int buf, const i32x4 (&st)[CPT]) {
#pragma unroll
    for (int i = 0; i < CPT; ++i)
#pragma unroll
      for (int w = 0; w < kWaves; ++w) {
        const int f = w + kWaves * i, t = f % NT, kbl = f / NT;
        if (f < NF && wave == w) *(i32x4*)(&pan[buf][kbl][t][lane * 16]) = st[i];
      }
  };
  auto load_x = [&](int kb, i32x4 (&x)[RT]) {
    const int col = kb * KR + g * EPL;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) x[rt] = load_frag_ld<ELT>(r, r_wave + rt * 16 + m16, nrows, col, d, ld, AL);
  };

  i32x4 stage[CPT];
  i32x4 ring[kPD][RT];
  load_panel(0, stage);
#pragma unroll
  for (int s = 0; s < kPD; ++s) load_x(s, ring[s]);
  store_panel(0, stage);
  lds_barrier();
  for (int p = 0; p < npan; ++p) {
    const int buf = p & 1;
    if (p + 1 < npan) load_panel(p + 1, stage);
#pragma unroll
    for (int kbl = 0; kbl < kPanel; ++kbl) {
      const int kb = p * kPanel + kbl;
      if (kb < nkb) {
        i32x4 x[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) x[rt] = ring[kbl % kPD][rt];
        load_x(kb + kPD, ring[kbl % kPD]);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t < P.nt) {
            const i32x4 pf = *(const i32x4*)(&pan[buf][kbl][t][lane * 16]);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt][t] = frag_mma<ELT>(x[rt], pf, acc[rt][t]);
          }
        }
      }
    }
    if (p + 1 < npan) store_panel(buf ^ 1, stage);
    lds_barrier();
  }
}

// ---------------------------------------------------------------------------
// The same projection for bf16 blocks with 16-byte aligned rows, streamed
// through LDS by direct loads (buffer_load ... lds, no registers): each load
// instruction moves 8 rows x 128 bytes (2 k-blocks of 8 rows), so every L2
// request carries 128 bytes of a row instead of the 64 a register operand
// load gets (16 rows x 64 bytes), and many more bytes can be in flight per CU.
//
// A stage is 2 k-blocks (64 columns).  Each wave streams only its own RT x 16
// rows, into a private double buffer (RT x 16 x 128 bytes per stage), rows
// 128 bytes apart with their 16-byte chunks XOR-swizzled by (row & 7) so the
// MFMA fragment reads (16 rows x 16 bytes per lane group) spread over the
// banks: each lane fetches the chunk that lands in its fixed LDS slot.  The
// stage's 2 x NT projection fragments (NT / 2 per wave; NT = 2, 4 or 6, so
// the maps of up to three layers that share the input block ride along) go by
// direct load into a 3-slot ring shared by the workgroup.  Every wave issues
// exactly kDmaOps loads per stage, so "stage s has landed" is vmcnt(kDmaOps) while
// stage s + 1 is in flight and vmcnt(0) otherwise (any extra load issued later
// would only make that wait longer); one barrier per stage then publishes the
// shared fragments.  The wave's reads of a buffer finish (lgkmcnt(0)) before
// the load of stage s + 2 into it is issued, and the map slot it refills was
// last read in stage s - 1, before every wave passed stage s's barrier.
// K-blocks are contracted in the order of project_rows, so results are
// bitwise those of the register path.
template <int RT, int NT>
struct DmaLds {
  static_assert((2 * NT) % kWaves == 0 && 2 * NT <= 3 * kWaves, "NT / 2 projection fragments per wave and stage");
  static constexpr int kRowBytes = 128;                      // 2 k-blocks of 32 bf16
  static constexpr int kWaveStage = RT * 16 * kRowBytes;     // bytes per wave and stage
  static constexpr int kLoads = RT * 16 / 8;                 // 1 KiB row-group loads per stage
  static constexpr int kMapLoads = 2 * NT / kWaves;          // this wave's fragments per stage
  static constexpr int kDmaOps = kLoads + kMapLoads;
  static constexpr int kMapOff = kWaves * 2 * kWaveStage;
  static constexpr int kMapStage = 2 * NT * kFragBytes;
  static constexpr int kBytes = kMapOff + 3 * kMapStage;
};

// kOnce: rows are streamed past L2's other lines (nt): right where no other
// workgroup of the same XCD reads them about the same time.  (The factor sums
// set it by size alone: layers that share an input are separate ops there,
// mostly on different XCDs.  4 Qwen-shaped blocks with shared inputs, 32 x 512
// rows: k = 64 1.95 ms with, 1.96 without; k = 16 2.20 both.)
template <int RT, int NT, bool kOnce>
__device__ inline void project_rows_dma(const rsrc_t r, int r_wave, int nrows, int d, int64_t ld,
                                        const FragSrc<NT>& P, f32x4 (&acc)[RT][NT], uint8_t* lds) {
  using C = DmaLds<RT, NT>;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, m16 = lane & 15;
  const int wave = tid >> 6;
  const int nkb = (d + 31) / 32;
  const int nst = (nkb + 1) / 2;
  uint8_t* own = lds + wave * 2 * C::kWaveStage;
  // this wave's projection fragments of every stage: fragment f = wave *
  // kMapLoads + i of the stage is k-block 2s + f / NT of tile f % NT
  int f_kbl[C::kMapLoads], f_t[C::kMapLoads];
  int64_t f_stride[C::kMapLoads];
  const uint8_t* f_base[C::kMapLoads];  // (descriptors are built per load: no arrays of rsrc_t)
#pragma unroll
  for (int i = 0; i < C::kMapLoads; ++i) {
    const int f = wave * C::kMapLoads + i;
    f_kbl[i] = f / NT;
    f_t[i] = f % NT;
    // a select chain, not P.base[f_t[i]]: a runtime index would put the
    // arrays in memory (the compiler promotes them to LDS)
    const uint8_t* base = P.base[0];
    int64_t stride = P.stride[0];
#pragma unroll
    for (int t = 1; t < NT; ++t)
      if (f_t[i] == t) {
        base = P.base[t];
        stride = P.stride[t];
      }
    f_stride[i] = stride;
    f_base[i] = base;
  }

  auto issue = [&](int s) {
    uint8_t* xs = own + (s & 1) * C::kWaveStage;
#pragma unroll
    for (int i = 0; i < C::kLoads; ++i) {
      const int row_l = i * 8 + (lane >> 3);
      const int c = (lane & 7) ^ (row_l & 7);  // the logical chunk that lands in this lane's slot
      const int row = r_wave + row_l, col = s * 64 + c * 8;
      const uint32_t off = (row < nrows && col < d) ? (uint32_t)(((int64_t)row * ld + col) * 2) : kOOB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(r, DATTRI_LDS_PTR(xs + i * 1024), 16, off, 0, 0, kOnce ? 2 : 0);
    }
#pragma unroll
    for (int i = 0; i < C::kMapLoads; ++i) {
      const int kb = 2 * s + f_kbl[i];
      uint8_t* ms = lds + C::kMapOff + (s % 3) * C::kMapStage + (f_kbl[i] * NT + f_t[i]) * kFragBytes;
      const uint32_t moff = (f_t[i] < P.nt && kb < nkb) ? (uint32_t)(kb * f_stride[i] + lane * 16) : kOOB;
      const rsrc_t rp = make_rsrc(f_base[i], (uint32_t)((int64_t)nkb * f_stride[i]));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rp, DATTRI_LDS_PTR(ms), 16, moff, 0, 0, 0);
    }
  };

  // the stage barrier: this wave's LDS reads done, then s_barrier.  An inline
  // barrier, because a fenced one (lds_barrier) makes the compiler wait for
  // every outstanding direct load (vmcnt(0)), the prefetched stage included.
  auto stage_barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
  if (nst > 0) issue(0);
  if (nst > 1) issue(1);
  for (int s = 0; s < nst; ++s) {
    if (s + 1 < nst)
      wait_vmcnt_dma<C::kDmaOps>();
    else
      wait_vmcnt_dma<0>();
    stage_barrier();
    const uint8_t* xs = own + (s & 1) * C::kWaveStage;
    const uint8_t* ms = lds + C::kMapOff + (s % 3) * C::kMapStage;
#pragma unroll
    for (int kbl = 0; kbl < 2; ++kbl) {
      if (2 * s + kbl < nkb) {  // uniform
        i32x4 x[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          const int row_l = rt * 16 + m16;
          x[rt] = *(const i32x4*)(xs + row_l * C::kRowBytes + (((kbl * 4 + g) ^ (row_l & 7)) << 4));
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t < P.nt) {
            const i32x4 pf = *(const i32x4*)(ms + (kbl * NT + t) * kFragBytes + lane * 16);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt][t] = frag_mma<2>(x[rt], pf, acc[rt][t]);
          }
        }
      }
    }
    if (s + 2 < nst) {
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this wave's reads of the buffer are done
      issue(s + 2);
    }
  }
  stage_barrier();  // every wave is done with the ring before the next call refills it
}

// ---------------------------------------------------------------------------
// The bf16 direct-load stream with per-row validity and a ring of D stages:
// acc[rt][t] += (X[rows, 0:d] P[0:d, tile t])^T, the map fragment as the first
// MFMA operand; stages, chunk swizzle and map fragments as in project_rows_dma.
// rowoff[i]: byte offset in `r` of the chunk this lane loads of row group i's
// stage 0 (row i * 8 + lane / 8 of the wave, chunk (lane % 8) ^ (row % 8)), or
// kFarOff for a row that must not be read (it reads as zero).  kNorm: nsq[rt]
// also gathers the squares of this lane's columns of row tile rt.  P(t, &base,
// &stride): the packed map's fragment (k-block kb, tile t) is at base + kb *
// stride; nt tiles are in use.  Stages s .. s +
// D - 1 are in flight or in use: the wait for stage s leaves the loads of the
// later stages already issued outstanding, the barrier publishes the
// shared map fragments, and stage s + D is issued into the wave's own buffer
// s % D once its reads of stage s are done.  A map slot is refilled D + 1
// stages later: its readers (stage s - 1) all passed stage s's barrier.
constexpr uint32_t kFarOff = 0x80000000u;  // + any column offset: past every descriptor used with it (< 2 GiB)

template <int RT, int NT, int D>
struct StreamLds {
  static_assert((2 * NT) % kWaves == 0, "NT / 2 projection fragments per wave and stage");
  static constexpr int kWaveStage = RT * 16 * 128;   // bytes per wave and stage
  static constexpr int kLoads = RT * 16 / 8;         // 1 KiB row-group loads per stage
  static constexpr int kMapLoads = 2 * NT / kWaves;  // this wave's fragments per stage
  static constexpr int kOps = kLoads + kMapLoads;
  static_assert((D - 1) * kOps < 64, "vmcnt range");
  static constexpr int kMapOff = kWaves * D * kWaveStage;
  static constexpr int kMapStage = 2 * NT * kFragBytes;
  static constexpr int kBytes = kMapOff + (D + 1) * kMapStage;
};

// One k-block's operand fragments from LDS: RT row tiles (2 KiB apart from
// byte address xa) and NT map fragments (1 KiB apart from pa), waited for in
// the same block.  Inline assembly, because the compiler cannot tell which LDS
// bytes a direct load in flight will write and would put vmcnt(0) before the
// reads, draining the ring each stage.
template <int RT, int NT>
__device__ inline void read_frags(i32x4 (&x)[RT], i32x4 (&p)[NT], uint32_t xa, uint32_t pa) {
  static_assert(RT == 4 && (NT == 2 || NT == 4 || NT == 6 || NT == 8), "row and map tiles");
  if constexpr (NT == 2)
    asm volatile("ds_read_b128 %0, %[xa] offset:0\n\t" "ds_read_b128 %1, %[xa] offset:2048\n\t"
                 "ds_read_b128 %2, %[xa] offset:4096\n\t" "ds_read_b128 %3, %[xa] offset:6144\n\t"
                 "ds_read_b128 %4, %[pa] offset:0\n\t" "ds_read_b128 %5, %[pa] offset:1024\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(p[0]), "=&v"(p[1])
                 : [xa] "v"(xa), [pa] "v"(pa)
                 : "memory");
  else if constexpr (NT == 4)
    asm volatile("ds_read_b128 %0, %[xa] offset:0\n\t" "ds_read_b128 %1, %[xa] offset:2048\n\t"
                 "ds_read_b128 %2, %[xa] offset:4096\n\t" "ds_read_b128 %3, %[xa] offset:6144\n\t"
                 "ds_read_b128 %4, %[pa] offset:0\n\t" "ds_read_b128 %5, %[pa] offset:1024\n\t"
                 "ds_read_b128 %6, %[pa] offset:2048\n\t" "ds_read_b128 %7, %[pa] offset:3072\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(p[3])
                 : [xa] "v"(xa), [pa] "v"(pa)
                 : "memory");
  else if constexpr (NT == 6)
    asm volatile("ds_read_b128 %0, %[xa] offset:0\n\t" "ds_read_b128 %1, %[xa] offset:2048\n\t"
                 "ds_read_b128 %2, %[xa] offset:4096\n\t" "ds_read_b128 %3, %[xa] offset:6144\n\t"
                 "ds_read_b128 %4, %[pa] offset:0\n\t" "ds_read_b128 %5, %[pa] offset:1024\n\t"
                 "ds_read_b128 %6, %[pa] offset:2048\n\t" "ds_read_b128 %7, %[pa] offset:3072\n\t"
                 "ds_read_b128 %8, %[pa] offset:4096\n\t" "ds_read_b128 %9, %[pa] offset:5120\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(p[3]), "=&v"(p[4]), "=&v"(p[5])
                 : [xa] "v"(xa), [pa] "v"(pa)
                 : "memory");
  else if constexpr (NT == 8)
    asm volatile("ds_read_b128 %0, %[xa] offset:0\n\t" "ds_read_b128 %1, %[xa] offset:2048\n\t"
                 "ds_read_b128 %2, %[xa] offset:4096\n\t" "ds_read_b128 %3, %[xa] offset:6144\n\t"
                 "ds_read_b128 %4, %[pa] offset:0\n\t" "ds_read_b128 %5, %[pa] offset:1024\n\t"
                 "ds_read_b128 %6, %[pa] offset:2048\n\t" "ds_read_b128 %7, %[pa] offset:3072\n\t"
                 "ds_read_b128 %8, %[pa] offset:4096\n\t" "ds_read_b128 %9, %[pa] offset:5120\n\t"
                 "ds_read_b128 %10, %[pa] offset:6144\n\t" "ds_read_b128 %11, %[pa] offset:7168\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]), "=&v"(p[0]), "=&v"(p[1]), "=&v"(p[2]), "=&v"(p[3]), "=&v"(p[4]), "=&v"(p[5]), "=&v"(p[6]), "=&v"(p[7])
                 : [xa] "v"(xa), [pa] "v"(pa)
                 : "memory");
}

template <int RT, int NT, int D, bool kNorm, class Frag>
__device__ inline void stream_rows(const rsrc_t r, const uint32_t (&rowoff)[StreamLds<RT, NT, D>::kLoads], int d,
                                   int nt, const Frag& P, bool once, f32x4 (&acc)[RT][NT], float (&nsq)[RT],
                                   uint8_t* lds) {
  using C = StreamLds<RT, NT, D>;
  constexpr int EPL = 8, KR = 4 * EPL;
  const int lane = threadIdx.x & 63, g = lane >> 4, m16 = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nkb = (d + KR - 1) / KR;
  const int nst = (nkb + 1) / 2;
  uint8_t* own = lds + wave * D * C::kWaveStage;
  // LDS addresses of this lane's reads of stage slot 0: row m16 of each row
  // tile (its chunk g of k-block 0; k-block 1 is 64 bytes across), and the maps
  typedef __attribute__((address_space(3))) uint8_t lds_u8;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lds_u8*)lds;
  const uint32_t x0 = lds0 + (uint32_t)(wave * D * C::kWaveStage + m16 * 128 + ((g ^ (m16 & 7)) << 4));
  const uint32_t m0 = lds0 + (uint32_t)(C::kMapOff + lane * 16);
  // fragment f = wave * kMapLoads + i of a stage is k-block 2s + f / NT of tile f % NT
  int f_kbl[C::kMapLoads], f_t[C::kMapLoads];
  int64_t f_stride[C::kMapLoads];
  const uint8_t* f_base[C::kMapLoads];
#pragma unroll
  for (int i = 0; i < C::kMapLoads; ++i) {
    const int f = wave * C::kMapLoads + i;
    f_kbl[i] = f / NT;
    f_t[i] = f % NT;
    P(f_t[i], &f_base[i], &f_stride[i]);
  }
  auto issue = [&](int s) {
    uint8_t* xs = own + (s % D) * C::kWaveStage;
    const uint32_t colb = (uint32_t)s * 128;
    const bool whole = (s + 1) * 2 * KR <= d;  // uniform: no column of the stage lies past d
#pragma unroll
    for (int i = 0; i < C::kLoads; ++i) {
      const int c = (lane & 7) ^ ((lane >> 3) & 7);  // row i * 8 + lane / 8: its low three bits are lane / 8
      uint32_t off = rowoff[i] + colb;
      if (!whole && s * 2 * KR + c * EPL >= d) off = kFarOff;
      if (once)  // uniform: streamed past L2's other lines (nt)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, DATTRI_LDS_PTR(xs + i * 1024), 16, off, 0, 0, 2);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, DATTRI_LDS_PTR(xs + i * 1024), 16, off, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < C::kMapLoads; ++i) {
      const int kb = 2 * s + f_kbl[i];
      uint8_t* ms = lds + C::kMapOff + (s % (D + 1)) * C::kMapStage + (f_kbl[i] * NT + f_t[i]) * kFragBytes;
      const uint32_t moff = (f_t[i] < nt && kb < nkb) ? (uint32_t)(kb * f_stride[i] + lane * 16) : kFarOff;
      const rsrc_t rp = make_rsrc(f_base[i], (uint32_t)((int64_t)nkb * f_stride[i]));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rp, DATTRI_LDS_PTR(ms), 16, moff, 0, 0, 0);
    }
  };
  auto stage_barrier = [] { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };
#pragma unroll
  for (int s = 0; s < D; ++s)
    if (s < nst) issue(s);
  for (int s = 0; s < nst; ++s) {
    const int later = nst - 1 - s;  // stages already issued behind stage s (at most D - 1)
    if (later >= D - 1)
      wait_vmcnt_dma<(D - 1) * C::kOps>();
    else if (D > 3 && later == 2)
      wait_vmcnt_dma<2 * C::kOps>();
    else if (D > 2 && later == 1)
      wait_vmcnt_dma<C::kOps>();
    else
      wait_vmcnt_dma<0>();
    stage_barrier();
    const uint32_t xs = x0 + (uint32_t)((s % D) * C::kWaveStage);
    const uint32_t ms = m0 + (uint32_t)((s % (D + 1)) * C::kMapStage);
#pragma unroll
    for (int kbl = 0; kbl < 2; ++kbl) {
      if (2 * s + kbl < nkb) {  // uniform
        i32x4 x[RT], pf[NT];
        read_frags<RT, NT>(x, pf, kbl ? xs ^ 64u : xs, ms + (uint32_t)(kbl * NT * kFragBytes));
        if constexpr (kNorm) {
#pragma unroll
          for (int rt = 0; rt < RT; ++rt) nsq[rt] = sum_sq<2>(x[rt], nsq[rt]);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (t < nt) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[rt][t] = frag_mma<2>(pf[t], x[rt], acc[rt][t]);
          }
        }
      }
    }
    if (s + D < nst) issue(s + D);  // this wave's reads of the buffer are done (read_frags waited)
  }
}

// ---------------------------------------------------------------------------
// The float32 stream: products on bf16 MFMA with both operands split into three
// bf16 terms (split3): 6 MFMA of 16 cycles per tile product where float32 MFMA
// takes 8 of 32, so maps of up to 4 tiles stay bound by the row stream.  A
// stage is 32 columns, one K = 32 step: its two float32 k-blocks give K slots
// 0-3 and 4-7 of every lane, for rows and maps alike.  A wave's rows go
// straight into registers, two stages ahead, and are split there; the map
// fragments are shared by the workgroup: wave t splits tile t of stage s + 1
// while stage s is multiplied, into double-buffered bf16 planes in LDS.
// Measured on 32 blocks of 4096 rows of 4096 (2.15 GB): 0.45 ms with k = 16
// (HBM-bound), 0.54 ms with k = 64, where the vector ALU (43% of cycles:
// splitting) and the matrix cores (40%) take turns on the issue port; float32
// MFMA with rows streamed through LDS took 1.3 times as long.  Rows staged in
// LDS by direct loads, and 256-row workgroups, measured the same at k = 64.
template <int NT>
struct StreamF32Lds {
  static_assert(NT <= kWaves, "one map tile per wave is split");
  static constexpr int kPlane = NT * kFragBytes;  // hi, mid, lo planes of NT fragments
  static constexpr int kColMax = 2 * 3 * kPlane;  // largest magnitude of each map column, floats
  static constexpr int kBytes = kColMax + NT * 16 * 4;
};

// rowoff[rt]: byte offset in `r` of this lane's 16 bytes of stage 0 in row
// m16 of row tile rt (chunk lane / 16), or kFarOff for a row not to be read.
// P, nt as for stream_rows; live: the wave has a row to read (uniform).
// Returns whether a result of this lane needs float32 products (split_unsafe).
template <int RT, int NT, class Frag>
__device__ inline bool stream_rows_f32(const rsrc_t r, const uint32_t (&rowoff)[RT], int d, int nt, const Frag& P,
                                       bool live, f32x4 (&acc)[RT][NT], uint8_t* lds) {
  using C = StreamF32Lds<NT>;
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nkb = (d + 15) / 16;
  const int nst = (nkb + 1) / 2;
  const uint8_t* m_base;
  int64_t m_stride;
  P(wave, &m_base, &m_stride);
  const bool splits = wave < nt;  // uniform over the wave
  const rsrc_t rm = make_rsrc(m_base, splits ? (uint32_t)((int64_t)nkb * m_stride) : 0u);
  // no branch around any load: behind one, the compiler's wait counts fall back to vmcnt(0)
  auto load_x = [&](int s, i32x4 (&x)[RT][2]) {
    const int col = s * 32 + g * 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const bool in = col + h * 16 < d;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) x[rt][h] = load16(r, in ? rowoff[rt] + (uint32_t)(s * 128 + h * 64) : kFarOff);
    }
  };
  auto load_m = [&](int s, i32x4 (&m)[2]) {  // k-blocks past the map read as zero
#pragma unroll
    for (int h = 0; h < 2; ++h) m[h] = load16(rm, 2 * s + h < nkb ? (uint32_t)((2 * s + h) * m_stride + lane * 16) : kFarOff);
  };
  float mcol = 0.f, mrow[RT];  // largest magnitudes of this lane's share of map column m16 and of its rows
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) mrow[rt] = 0.f;
  auto put_planes = [&](int buf, const i32x4 (&m)[2]) {
    if (splits) {
      mcol = max_abs(max_abs(mcol, m[0]), m[1]);
      const Split3 v = split3(m[0], m[1]);
      uint8_t* w = lds + buf * 3 * C::kPlane + wave * kFragBytes + lane * 16;
      *(bf16x8*)w = v.hi;
      *(bf16x8*)(w + C::kPlane) = v.mid;
      *(bf16x8*)(w + 2 * C::kPlane) = v.lo;
    }
  };
  i32x4 x[2][RT][2], m[2][2];
  load_m(0, m[0]);
  load_x(0, x[0]);
  load_m(1, m[1]);
  load_x(1, x[1]);
  put_planes(0, m[0]);
  load_m(2, m[0]);
  // stages by pairs (register arrays indexed statically); an odd last stage's
  // partner reads zeros
  for (int s0 = 0; s0 < nst; s0 += 2) {
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int s = s0 + q;
      lds_barrier();  // planes of stage s are written, those of stage s - 1 read
      put_planes(q ^ 1, m[q ^ 1]);
      load_m(s + 3, m[q ^ 1]);
      if (live) {
        Split3 pv[NT];
        const uint8_t* pl = lds + q * 3 * C::kPlane + lane * 16;
#pragma unroll
        for (int t = 0; t < NT; ++t) {  // tiles >= nt multiply whatever the planes hold and are dropped
          pv[t].hi = *(const bf16x8*)(pl + t * kFragBytes);
          pv[t].mid = *(const bf16x8*)(pl + C::kPlane + t * kFragBytes);
          pv[t].lo = *(const bf16x8*)(pl + 2 * C::kPlane + t * kFragBytes);
        }
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
          mrow[rt] = max_abs(max_abs(mrow[rt], x[q][rt][0]), x[q][rt][1]);
          const Split3 xv = split3(x[q][rt][0], x[q][rt][1]);
#define DATTRI_TERM(p) _Pragma("unroll") for (int t = 0; t < NT; ++t) acc[rt][t] = split_term<p>(pv[t], xv, acc[rt][t]);
          DATTRI_TERM(0) DATTRI_TERM(1) DATTRI_TERM(2) DATTRI_TERM(3) DATTRI_TERM(4) DATTRI_TERM(5)
#undef DATTRI_TERM
        }
      }
      load_x(s + 2, x[q]);
    }
  }
  // lanes 16 apart hold the four pieces of a row, or of a map column
  auto quad_max = [](float v) {
    v = fmaxf(v, __shfl_xor(v, 16, 64));
    return fmaxf(v, __shfl_xor(v, 32, 64));
  };
  float* cm = (float*)(lds + C::kColMax);
  if (splits) {
    mcol = quad_max(mcol);
    if (g == 0) cm[wave * 16 + lane] = mcol;
  }
  lds_barrier();
  if (!live) return false;
  const float K = (float)d;
  NonzeroRange lines, sums;
  float mr = 0.f, mc = 0.f;
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    mrow[rt] = quad_max(mrow[rt]);
    mr = fmaxf(mr, mrow[rt]);
    lines.add(mrow[rt], mrow[rt]);
  }
#pragma unroll
  for (int t = 0; t < NT; ++t)
    if (t < nt) {
      const f32x4 c = *(const f32x4*)(cm + t * 16 + 4 * g);  // acc: columns 4g .. 4g + 3 of row m16
      mc = max_abs(mc, __builtin_bit_cast(i32x4, c));
      lines.add(c);
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) sums.add(acc[rt][t]);
    }
  uint32_t bad = lines.unsafe(kTinyLine) ? 1u : 0u;
  if (__any(sums.unsafe(split_safe(K, mr, mc))))
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (t < nt)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            bad |= split_unsafe(acc[rt][t][e], split_safe(K, mrow[rt], cm[t * 16 + 4 * g + e]));
  return bad != 0u;
}

// The same product with float32 MFMA and operands loaded straight into
// registers: for blocks whose split products are unsafe.  row0: byte offset
// in `r` of this lane's row of row tile 0 (rows 16 ld floats apart per tile),
// rows: bit rt set where that row may be read.
template <int RT, int NT, class Frag>
__device__ inline void plain_rows_f32(const rsrc_t r, uint32_t row0, int64_t ld, uint32_t rows, int d,
                                      int nt, const Frag& P, f32x4 (&acc)[RT][NT]) {
  const int lane = threadIdx.x & 63, g = lane >> 4;
  const int nkb = (d + 15) / 16;
  for (int kb = 0; kb < nkb; ++kb) {
    const int col = kb * 16 + g * 4;
    i32x4 x[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
      x[rt] = load16(r, ((rows >> rt) & 1u) && col < d ? row0 + (uint32_t)((rt * 16 * ld + col) * 4) : kFarOff);
#pragma unroll
    for (int t = 0; t < NT; ++t)
      if (t < nt) {
        const uint8_t* pb;
        int64_t ps;
        P(t, &pb, &ps);
        const i32x4 pf = *(const i32x4*)(pb + kb * ps + lane * 16);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) acc[rt][t] = frag_mma<4>(pf, x[rt], acc[rt][t]);
      }
  }
}

}  // namespace dev
}  // namespace dattri
