// Device code of the gradient dA_t = X^T Gs (Adapter-Tuning: dD_t = z^T Gs), which runs in a launch of its own or rides in that
// of the backbone product, and what the adapter kernels share with it.
#pragma once
#include "mux_device_utils.h"

namespace mux {
namespace adapter {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __amdgpu_buffer_rsrc_t rsrc_t;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
constexpr uint32_t OOB = 0x80000000u;

__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ u32x4 buf_load16(rsrc_t r, uint32_t byte_off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, 0);
}
// The same past the caches (see kStreamBytes)
template <bool STREAM>
__device__ __forceinline__ u32x4 buf_load16_once(rsrc_t r, uint32_t byte_off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, STREAM ? 2 : 0);
}
__device__ __forceinline__ bf16x4 lds_read_tr(const bf16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)p);
}
__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// Validity bits of the rows of a row group of up to 1024 rows, fetched once: lane l keeps the 32-bit word that holds
// row row0 + 32 l (and the one after it); step s of the group then takes its 32 bits from lanes with two lane reads
// instead of a memory access of its own, on which the step's loads would have to wait.
struct GroupBits { uint32_t lo, hi; int sh; };
__device__ __forceinline__ GroupBits load_group_bits(const int32_t* __restrict__ dtab, int rowbits_off, int row0, int nrows, int T, int lane) {
  const uint32_t* bm = (const uint32_t*)(dtab + rowbits_off);
  const int w0 = row0 >> 5;
  const int last = (T + 31) >> 5;                        // the spare word after the last one exists
  const int nw = ((nrows + 31) >> 5) + 1;
  GroupBits g;
  g.lo = (lane < nw && w0 + lane <= last) ? bm[w0 + lane] : 0u;
  g.hi = (lane < nw && w0 + lane + 1 <= last) ? bm[w0 + lane + 1] : 0u;
  g.sh = row0 & 31;
  return g;
}
__device__ __forceinline__ uint32_t step_bits(const GroupBits& g, int s) {
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)g.lo, s), hi = (uint32_t)__builtin_amdgcn_readlane((int)g.hi, s);
  return (uint32_t)((((uint64_t)hi << 32) | lo) >> g.sh);
}

constexpr int GP = 72;   // LDS row pitch in elements (144 B): 16 consecutive rows of one 16-byte piece hit 64 different banks

// Per-row-group partials part[item][r][C] = sum over the rows of Gs[i][:]^T X[i][:].  Each wave owns 64 columns and walks the
// rows 32 at a time: the 32x64 slab of X and the 32xRP slab of Gs go through a wave-private LDS region in their natural
// layout and come back k-major per lane through ds_read_b64_tr_b16.  No workgroup barrier: the four waves are independent
// streams.
struct GradParams {
  const int32_t* dtab;
  const bf16_t* Gs;        // [T, RP]
  const bf16_t* X;         // [T, K]
  const bf16_t* Zc;        // TUNING items: saved x W, [z_rows, N], in the place of X
  float* part;             // [n_items][slot], a slot holds [RP][C] of the item's kind
  size_t slot;             // elements per item in part
  int K, N, RP;
  int items_off, rowbits_off, T;   // word offsets in dtab of the row-group list and of the row-validity bits; rows of the batch
  int direct, accumulate;  // direct: every task is one row group, whose sums are dA_t [C][r]: straight to the gradient
  int n_items, col_blocks; // row groups, blocks of 256 columns: a workgroup each
  int pieces;              // 16-wide rank pieces the code is built for: 1, 2 or 4
};
constexpr int kGradLdsElems = 4 * 2 * 32 * GP;

// DEPTH steps of loads in flight; the loop body has no branch and a fixed number of loads per step (what does not
// exist gets an out-of-range offset), so that the wait for one step's data leaves the younger loads in flight.
template <int NJM, int DEPTH, bool STREAM>
__device__ __forceinline__ void grad_rows(const GradParams& p, const TaskRef& tasks, const int item, const int cols, bf16_t* lds) {
  const int4 iw = *(const int4*)(p.dtab + p.items_off + item * DI_WORDS);
  const ItemView it = {iw.x, iw.y, iw.z, iw.w};
  if (it.task < 0 || it.nvalid == 0) return;
  const DevTask tk = get_task(tasks, it.task);
  if (tk.kind != MUX_ADAPTER_LORA && tk.kind != MUX_ADAPTER_TUNING) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const bool from_z = tk.kind == MUX_ADAPTER_TUNING;
  const int C = from_z ? p.N : p.K;
  const int cw0 = cols * 256 + wave * 64;
  if (cw0 >= C) return;
  const int rank = tk.rank, NJ = (rank + 15) >> 4;
  bf16_t* sBig = lds + wave * (2 * 32 * GP);
  bf16_t* sSm = sBig + 32 * GP;

  const bf16_t* big = from_z ? p.Zc + (size_t)(tk.zrow0 + it.row0 - tk.row_begin) * C : p.X + (size_t)it.row0 * C;
  const rsrc_t rB = make_rsrc(big, (uint32_t)it.nrows * (uint32_t)C * 2u);
  const rsrc_t rS = make_rsrc(p.Gs + (size_t)it.row0 * p.RP, (uint32_t)it.nrows * (uint32_t)p.RP * 2u);
  // Big slab: 4 loads per lane, row = 8q + lane/8, 16-byte piece = lane%8
  const int b_row = lane >> 3, b_pc = (lane & 7) * 8;
  const bool b_col_ok = cw0 + b_pc < C;
  // Small slab: pieces per row = RP/8 (RP <= 16 NJM); idx = lane + 64 q -> row = idx / ppr, piece = idx % ppr
  const int ppr = p.RP >> 3;
  int s_row[NJM], s_pc[NJM];
#pragma unroll
  for (int q = 0; q < NJM; ++q) { const int idx = lane + 64 * q; s_row[q] = idx / ppr; s_pc[q] = (idx % ppr) * 8; }

  u32x4 gb[DEPTH][4], gs[DEPTH][NJM];
  const int steps = (it.nrows + 31) >> 5;
  const GroupBits gbits = load_group_bits(p.dtab, p.rowbits_off, it.row0, it.nrows, p.T, lane);
  auto load_step = [&](int s, int buf) {       // a step past the end loads nothing (every offset out of range)
    const int base = s * 32;
    // validity of the 32 rows of this step, wave-uniform, from the words fetched once for the whole group
    const uint32_t vbits = s < steps ? step_bits(gbits, s) : 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = base + b_row + 8 * q;
      const bool ok = b_col_ok && m < it.nrows && ((vbits >> (b_row + 8 * q)) & 1u);
      gb[buf][q] = buf_load16_once<STREAM>(rB, ok ? (uint32_t)(((size_t)m * C + cw0 + b_pc) * 2) : OOB);
    }
#pragma unroll
    for (int q = 0; q < NJM; ++q) {
      const int m = base + s_row[q];
      const bool ok = s < steps && s_row[q] < 32 && m < it.nrows;
      gs[buf][q] = buf_load16(rS, ok ? (uint32_t)((m * p.RP + s_pc[q]) * 2) : OOB);
    }
  };
  auto store_step = [&](int buf) {
#pragma unroll
    for (int q = 0; q < 4; ++q) *(u32x4*)(sBig + (b_row + 8 * q) * GP + b_pc) = gb[buf][q];
#pragma unroll
    for (int q = 0; q < NJM; ++q)
      if (s_row[q] < 32) *(u32x4*)(sSm + s_row[q] * GP + s_pc[q]) = gs[buf][q];
  };

  f32x4 acc[NJM][4];
#pragma unroll
  for (int jt = 0; jt < NJM; ++jt)
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) acc[jt][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};

  const int l16 = lane & 15, g = lane >> 4;
  const int tr_off = (8 * g + (l16 >> 2)) * GP + 4 * (l16 & 3);
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load_step(d, d);
  for (int s0 = 0; s0 < steps; s0 += DEPTH) {
#pragma unroll
    for (int u = 0; u < DEPTH; ++u) {          // may run past the last step: zeros in
      store_step(u);
      load_step(s0 + u + DEPTH, u);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      bf16x8 a[NJM], b[4];
#pragma unroll
      for (int jt = 0; jt < NJM; ++jt) {
        const bf16x4 lo = lds_read_tr(sSm + tr_off + jt * 16), hi = lds_read_tr(sSm + tr_off + 4 * GP + jt * 16);
        a[jt] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        const bf16x4 lo = lds_read_tr(sBig + tr_off + ct * 16), hi = lds_read_tr(sBig + tr_off + 4 * GP + ct * 16);
        b[ct] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
#pragma unroll
      for (int jt = 0; jt < NJM; ++jt)
        if (jt < NJ)
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) acc[jt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[jt], b[ct], acc[jt][ct], 0, 0, 0);
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
  // acc[jt][ct][v] = part[j = jt*16 + 4g + v][c = cw0 + ct*16 + l16]
  if (p.direct) {
    if (tk.dA == nullptr) return;
    const bool runs = (rank & 3) == 0 && ((uintptr_t)tk.dA & 15) == 0;    // 16 bytes a lane, a column's ranks in one run
#pragma unroll
    for (int jt = 0; jt < NJM; ++jt)
#pragma unroll
      for (int ct = 0; ct < 4; ++ct) {
        const int c = cw0 + ct * 16 + l16, j0 = jt * 16 + 4 * g;
        if (j0 >= rank || c >= C) continue;
        float* d = tk.dA + (size_t)c * rank + j0;
        if (runs) {
          *(f32x4*)d = p.accumulate ? *(const f32x4*)d + acc[jt][ct] : acc[jt][ct];
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v)
            if (j0 + v < rank) d[v] = p.accumulate ? d[v] + acc[jt][ct][v] : acc[jt][ct][v];
        }
      }
    return;
  }
  float* dst = p.part + (size_t)item * p.slot;
#pragma unroll
  for (int jt = 0; jt < NJM; ++jt)
    if (jt < NJ)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int j = jt * 16 + 4 * g + v;
        if (j < rank)
#pragma unroll
          for (int ct = 0; ct < 4; ++ct) {
            const int c = cw0 + ct * 16 + l16;
            if (c < C) dst[(size_t)j * C + c] = acc[jt][ct][v];
          }
      }
}

}  // namespace adapter
}  // namespace mux
