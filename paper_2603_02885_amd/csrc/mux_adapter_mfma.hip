// Adapter kernels on the matrix cores (bf16 in, fp32 accumulate).  All of them stream a big
// activation matrix once from HBM and are bound by that stream; the MFMA only keeps the
// arithmetic (r FLOP per byte) off the vector ALUs.
//
//   down:  Out[T,RP] = s_t * In[T,C] A_t        S1: In = X; rows of A_t in whole 16-byte pieces (see rank_pieces)
//   s4:    one pass over dY for both of its products (the adapter's backward is computed "in a fused manner",
//          section 3.2): per (row group, 512-column slab) the slab's share of dY B_t^T (summed over the slabs and scaled
//          by gs_reduce -> Gs[T,RP]) and the row group's share of Hs^T dY (summed over the row groups by reduce -> dB_t)
//   grad:  part[item][r][C] = sum_{rows of item} Small[i][:]^T Big[i][:]
//                                               S6: Small = Gs, Big = X   -> dA_t[K][r] (transposed on reduce)
//   dl:    part[item][N] = sum_{rows of item} dY[i][:] * Z[i][:]          (IA3_OUT)
//   reduce: per task, partials summed in ascending item order (deterministic), optional accumulate.
//
// Padding rows are masked with out-of-range buffer offsets (the load returns zeros), never multiplied.
#include <type_traits>

#include "mux_grad_device.h"

namespace mux {
using namespace adapter;
namespace {

constexpr int TS64 = 0, TS256 = 2, TS1024 = 3;

// ------------------------------------------------------------------------------------------------
// down-projection.  One workgroup = 32 rows of one 64-row item; its waves split the contraction.
// A wave walks its share 64 columns at a time: the 32x64 slab of In and the rank x 64 slab of P_t are fetched with
// loads that cover whole 128-byte lines (8 rows x 128 B per wave instruction: rows of 64 B move at half the rate
// on this memory system), two slabs ahead in registers, pass through a wave-private LDS region in their natural
// layout and come back in the 16x16x32 MFMA operand layout.  No workgroup barrier in the loop.  The partial sums
// of the waves are combined through LDS in a fixed order.  A_t [C][r] is read in rows of rank_pieces(r) 16-byte
// pieces: the 64 rows of a slab are one contiguous run, laid into LDS row by row and read back with the contraction
// index contiguous through ds_read_b64_tr_b16.
//   DOWN_X     LoRA items: Out = s_t X A_t; rows of other kinds: zero.
//   DOWN_TUNE  TUNING items only (other rows are left alone): u = z D_t with z from the saved compact rows;
//              U2 = u, Out = s_t gelu(u)
// The work item and the validity bits of its rows come from two lists whose offsets are launch arguments, so the
// first loads of X wait for one memory latency, not for a chain of them.
enum : int { DOWN_X = 0, DOWN_TUNE = 2 };
struct DownParams {
  const int32_t* dtab;
  const bf16_t* In;    // [T, C]  (DOWN_TUNE: [z_rows, C], rows numbered like the saved x W)
  bf16_t* Out;         // [T, RP]
  bf16_t* U2;          // [T, RP] pre-activations of the TUNING rows: written by DOWN_TUNE
  int C, RP, mode;
  int items_off, bits_off;   // word offsets in dtab: 64-row items, and two words of row-validity bits per item
  TaskRef tasks;
};

__device__ __forceinline__ float gelu_f(float u) { return 0.5f * u * (1.f + erff(u * 0.70710678f)); }
__device__ __forceinline__ float gelu_slope_f(float u) {
  return 0.5f * (1.f + erff(u * 0.70710678f)) + u * __expf(-0.5f * u * u) * 0.39894228f;
}

template <int NJM, int NWV, int DEPTH, bool STREAM>
__global__ __launch_bounds__(64 * NWV) void k_down(const DownParams p) {
  constexpr int ROWS = 32, NTHR = 64 * NWV;
  constexpr int PP = NJM * 16 + 8;                              // LDS pitch of the [64][r] slab of A_t (elements)
  constexpr int PSLAB = 64 * PP;
  constexpr int SLAB = ROWS * GP + PSLAB;                      // elements per wave: In slab, then P slab
  constexpr int REDW = NJM * 16 * (ROWS + 4) * 2;              // the same region later holds the partial sums (floats)
  constexpr int REGION = SLAB > REDW ? SLAB : REDW;
  __shared__ __attribute__((aligned(16))) bf16_t lds[NWV][REGION];
  const int item = blockIdx.x >> 1, sub = blockIdx.x & 1;
  const int4 iw = *(const int4*)(p.dtab + p.items_off + item * DI_WORDS);
  const uint32_t vbits = ((const uint32_t*)(p.dtab + p.bits_off))[2 * item + sub];
  const ItemView it = {iw.x, iw.y, iw.z, iw.w};
  const int r0 = sub * ROWS;
  if (r0 >= it.nrows) return;
  const int nr = it.nrows - r0 < ROWS ? it.nrows - r0 : ROWS;
  const int row0 = it.row0 + r0;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int kind = it.task >= 0 ? get_task_kind(p.tasks, it.task) : MUX_ADAPTER_NONE;
  const bool mine = p.mode == DOWN_TUNE ? kind == MUX_ADAPTER_TUNING : kind == MUX_ADAPTER_LORA;
  if (!mine && p.mode == DOWN_TUNE) return;
  if (!mine || vbits == 0u) {
    for (int e = tid; e < nr * p.RP; e += NTHR) {
      const size_t o = (size_t)(row0 + e / p.RP) * p.RP + e % p.RP;
      p.Out[o] = 0;
      if (p.mode == DOWN_TUNE) p.U2[o] = 0;
    }
    return;
  }
  const DevTask tk = get_task(p.tasks, it.task);
  const int rank = tk.rank, NJ = (rank + 15) >> 4;
  const int ppr = rank_pieces(rank);                 // 16-byte pieces in a row of A_t
  const int per = ((p.C + NWV - 1) / NWV + 63) & ~63;
  const int cbeg = wave * per, cend = cbeg + per < p.C ? cbeg + per : p.C;
  bf16_t* sX = lds[wave];
  bf16_t* sP = lds[wave] + ROWS * GP;

  const size_t in_row0 = p.mode == DOWN_TUNE ? (size_t)(tk.zrow0 + row0 - tk.row_begin) : (size_t)row0;
  const rsrc_t rIn = make_rsrc(p.In + in_row0 * p.C, (uint32_t)nr * (uint32_t)p.C * 2u);
  const rsrc_t rP = make_rsrc(tk.A, (uint32_t)p.C * (uint32_t)ppr * 16u);
  // one wave instruction: 8 rows x 128 B; lane -> row lane/8 (+ 8 q), 16-byte piece lane%8
  const int b_row = lane >> 3, b_pc = (lane & 7) * 8;
  uint32_t x_off[4], p_off[2 * NJM];
  int p_lds[2 * NJM];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int m = b_row + 8 * q;
    x_off[q] = (m < nr && ((vbits >> m) & 1u)) ? ((uint32_t)m * (uint32_t)p.C + (uint32_t)b_pc) * 2u : OOB;
  }
  // the slab is 64 ppr 16-byte pieces in a row; piece -> (row, piece of the row)
#pragma unroll
  for (int q = 0; q < 2 * NJM; ++q) {
    const int piece = q * 64 + lane;
    p_off[q] = q < ppr ? (uint32_t)piece * 16u : OOB;
    p_lds[q] = (piece / ppr) * PP + (piece % ppr) * 8;
  }
  // columns of the LDS slab beyond the last piece are never written: they read as zero
  for (int e = lane; e < 64 * (PP / 8); e += 64) *(u32x4*)(sP + (e / (PP / 8)) * PP + (e % (PP / 8)) * 8) = (u32x4){0u, 0u, 0u, 0u};

  f32x4 acc[2][NJM];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int jt = 0; jt < NJM; ++jt) acc[rt][jt] = (f32x4){0.f, 0.f, 0.f, 0.f};

  u32x4 gx[DEPTH][4], gp[DEPTH][2 * NJM];
  // Every slab issues the same number of loads, whatever the rank and wherever the share ends (a piece that does not
  // exist gets an out-of-range offset, costs no memory access and reads as zeros): the compiler can then count the
  // loads still in flight when it waits for a slab, instead of waiting for all of them.
  auto load = [&](int c, int buf) {          // a slab that starts past the end of this wave's share reads as zeros
    const bool in = c < cend;                 // the share ends on a multiple of 64 or at C, where the buffer ends
    const uint32_t kx = (c + b_pc < cend) ? (uint32_t)c * 2u : OOB;     // OOB + OOB wraps into range: mask on k only
    const uint32_t kp = in ? (uint32_t)c * (uint32_t)ppr * 16u : OOB;
#pragma unroll
    for (int q = 0; q < 4; ++q) gx[buf][q] = buf_load16_once<STREAM>(rIn, (x_off[q] == OOB || kx == OOB) ? OOB : x_off[q] + kx);
#pragma unroll
    for (int q = 0; q < 2 * NJM; ++q) {
      const bool ok = p_off[q] != OOB && kp != OOB;
      gp[buf][q] = buf_load16(rP, ok ? p_off[q] + kp : OOB);
    }
  };
  const int i = lane & 15, g = lane >> 4;
  const int tr_off = (8 * g + (i >> 2)) * PP + 4 * (i & 3);     // transposed reads of the [k][j] slab
  // DEPTH slabs in flight while one is multiplied
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) {
    load(cbeg + 64 * d, d);
    __builtin_amdgcn_sched_barrier(0);       // in the order in which the loop uses them
  }
  for (int c = cbeg; c < cend; c += 64 * DEPTH) {
#pragma unroll
    for (int buf = 0; buf < DEPTH; ++buf) {
      {                                      // also for a slab past the end (zeros): no branch around the loads
#pragma unroll
        for (int q = 0; q < 4; ++q) *(u32x4*)(sX + (b_row + 8 * q) * GP + b_pc) = gx[buf][q];
#pragma unroll
        for (int q = 0; q < 2 * NJM; ++q)
          if (q < ppr) *(u32x4*)(sP + p_lds[q]) = gp[buf][q];
        load(c + 64 * buf + 64 * DEPTH, buf);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        bf16x8 a[2][2], b[NJM][2];
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
          for (int rt = 0; rt < 2; ++rt) a[rt][s] = *(const bf16x8*)(sX + (rt * 16 + i) * GP + s * 32 + 8 * g);
#pragma unroll
          for (int jt = 0; jt < NJM; ++jt)
            if (jt < NJ) {
              const bf16x4 lo = lds_read_tr(sP + s * 32 * PP + tr_off + jt * 16);
              const bf16x4 hi = lds_read_tr(sP + s * 32 * PP + tr_off + 4 * PP + jt * 16);
              b[jt][s] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            }
        }
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int jt = 0; jt < NJM; ++jt)
              if (jt < NJ) acc[rt][jt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[rt][s], b[jt][s], acc[rt][jt], 0, 0, 0);
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }

  // acc[rt][jt][v] = partial of Out[row0 + rt*16 + 4g + v][jt*16 + i]; staged column-major, one 16-byte store each
  float* red = (float*)lds[wave];
#pragma unroll
  for (int rt = 0; rt < 2; ++rt)
#pragma unroll
    for (int jt = 0; jt < NJM; ++jt)
      if (jt < NJ) *(f32x4*)&red[(jt * 16 + i) * (ROWS + 4) + rt * 16 + 4 * g] = acc[rt][jt];
  __syncthreads();
  for (int e = tid; e < ROWS * p.RP; e += NTHR) {
    const int orow = e / p.RP, j = e % p.RP;
    if (orow >= nr) continue;
    float s = 0.f;
    if (j < NJ * 16) {
#pragma unroll
      for (int w = 0; w < NWV; ++w) s += ((const float*)lds[w])[j * (ROWS + 4) + orow];
    }
    const bool ok = ((vbits >> orow) & 1u) && j < rank;
    const size_t o = (size_t)(row0 + orow) * p.RP + j;
    float v = ok ? tk.scale * s : 0.f;
    if (p.mode == DOWN_TUNE) {
      p.U2[o] = f32_to_bf16(ok ? s : 0.f);
      v = ok ? tk.scale * gelu_f(s) : 0.f;
    }
    p.Out[o] = f32_to_bf16(v);
  }
}

// Bytes of the rows of the LoRA tasks, `lora` columns wide, and of the Adapter-Tuning tasks, `tuning` columns wide: what a
// kernel of these kinds reads (see kStreamBytes), however large the batch.  20000 tokens, 4096 x 4096, 6000 of them LoRA, forward and
// backward, by the rows of all tasks 1130 us, by these 1124; 3000 Adapter-Tuning, tune_up 17.7 us and 16.0, tune_dz 17.5 and 15.6.
size_t ranked_bytes(const mux_segtab* st, int lora, int tuning) {
  size_t n = 0;
  for (const HostTask& ht : st->tasks)
    n += (size_t)ht.row_count * 2 * (ht.kind == MUX_ADAPTER_LORA ? lora : ht.kind == MUX_ADAPTER_TUNING ? tuning : 0);
  return n;
}

void launch_down(const CallCtx& c, const char* name, DownParams p) {
  p.items_off = c.st->dev_image[DH_NITEMS0 + 3 * TS64 + 1];
  p.bits_off = c.st->dev_image[DH_OFF_ITEM_BITS];
  p.tasks = *c.tref;
  const unsigned items = (unsigned)c.st->items[TS64].size();
  // Eight waves split the contraction; two slabs in flight.  Ranks above 32 need LDS regions of 14 KB a wave: eight waves
  // leave room for one workgroup a compute unit, four for two.  So they take eight where a unit has one workgroup or none
  // (84 items at 4096: 18.6 -> 15.1 us) and four beyond (324 items: 61.7 us, eight waves 63.6).
  const dim3 grid(items * 2);
  const bool stream = p.mode == DOWN_X && past_caches(c, ranked_bytes(c.st, p.C, 0));     // (k_tune_add reads the x W of DOWN_TUNE again)
  auto launch = [&](auto STREAM) {
    constexpr bool S = decltype(STREAM)::value;
    if (c.st->r_max <= 16) MUX_LAUNCH(name, (k_down<1, 8, 2, S>), grid, dim3(512), 0, c.stream, p);
    else if (c.st->r_max <= 32) MUX_LAUNCH(name, (k_down<2, 8, 2, S>), grid, dim3(512), 0, c.stream, p);
    else if (items * 2 <= (unsigned)kComputeUnits) MUX_LAUNCH(name, (k_down<4, 8, 2, S>), grid, dim3(512), 0, c.stream, p);
    else MUX_LAUNCH(name, (k_down<4, 4, 2, S>), grid, dim3(256), 0, c.stream, p);
  };
  if (stream) launch(std::true_type{}); else launch(std::false_type{});
}

// ------------------------------------------------------------------------------------------------
// The pass over dY of the backward (LoRA: Gs = s_t dY B_t^T and dB_t = Hs^T dY; Adapter-Tuning: the same two products
// with U_t in the place of B_t).  grid = (row groups of the chosen size, ceil(N / 512)); each of the eight waves owns
// 64 columns and walks the group's rows 32 at a time: the 32x64 slab of dY and the 32xRP slab of Hs go through a
// wave-private LDS region; dY is read from it twice, row-major as the A operand of the slab's share of dY B_t^T
// (B_t's [r][64] piece stays in registers for the whole group), and with the rows contiguous, through
// ds_read_b64_tr_b16, as the B operand of Hs^T dY, whose sums stay in the accumulators until the group ends.
// The shares of dY B_t^T of the eight waves are added up through LDS (two barriers a step) and go out as one fp32
// partial per (column slab, row); k_gs_reduce adds the slabs.
struct S4Params {
  const int32_t* dtab;
  const bf16_t* dY;     // [T, N]
  const bf16_t* Hs;     // [T, RP]
  float* gpart;         // [n_slabs][T][RP]: dY B_t^T over the columns of one slab, unscaled
  float* bpart;         // [n_items][RP][N]: Hs^T dY over the rows of one group
  int N, RP, ts, T;
  int items_off, rowbits_off;   // word offsets in dtab of the row-group list and of the row-validity bits
  int direct, accumulate;       // direct: every task is one row group, whose sums are dB_t: no partial, straight to the gradient
  const bf16_t* U2;             // ONE: pre-activations of the TUNING rows
  bf16_t* Gs;                   // ONE: [T, RP]
  TaskRef tasks;
};

// ONE: the launch has one column slab, whose shares are all of dY B_t^T: they go out as Gs, scaled, masked and rounded as
// gs_reduce does it, which such a launch does without (256 x 256, two tasks, 3 us of 34).
// BATCH: steps whose shares of dY B_t^T wait in registers before the waves meet to add them up; DEPTH: steps of loads
// in flight.  The loop body has no branch and a fixed number of loads and stores per step (what does not exist gets an
// out-of-range offset), so that the waits for one step's data leave the younger loads in flight.
__device__ __forceinline__ void buf_store4(rsrc_t r, uint32_t byte_off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, (int)byte_off, 0, 0);
}
__device__ __forceinline__ void lds_barrier() {     // LDS traffic of every wave done; loads from memory stay in flight
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);               // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

template <int NJM, int BATCH, int DEPTH, bool ONE, bool STREAM>
__global__ __launch_bounds__(512) void k_s4(const S4Params p) {
  constexpr int NWV = 8, NTHR = 512, BROWS = BATCH * 32, RPITCH = BROWS + 4;   // RPITCH: floats between two columns of a staged share
  constexpr int UNR = BATCH > DEPTH ? BATCH : DEPTH;
  constexpr int RPJ = NJM * 16;                                   // columns of a staged share
  constexpr int NRED = BROWS * RPJ / NTHR;                        // sums a thread forms when the waves meet
  static_assert(RPJ * RPITCH * 4 <= 2 * 32 * GP * 2, "a wave's share of dY B_t^T fits its own LDS region");
  static_assert(UNR % BATCH == 0 && UNR % DEPTH == 0 && BROWS * RPJ % NTHR == 0, "powers of two");
  __shared__ __attribute__((aligned(16))) bf16_t lds[NWV][2][32 * GP];
  const int4 iw = *(const int4*)(p.dtab + p.items_off + blockIdx.x * DI_WORDS);   // the lists' offsets are launch arguments:
  const ItemView it = {iw.x, iw.y, iw.z, iw.w};                                    // one memory latency before the first load
  if (it.task < 0 || (!ONE && it.nvalid == 0)) return;
  const DevTask tk = get_task(p.tasks, it.task);
  if (tk.kind != MUX_ADAPTER_LORA && tk.kind != MUX_ADAPTER_TUNING) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (ONE && it.nvalid == 0) {                   // (row groups of another size may read these rows of Gs)
    for (int e = tid; e < it.nrows * (p.RP >> 3); e += NTHR) *(u32x4*)(p.Gs + (size_t)it.row0 * p.RP + 8 * (size_t)e) = (u32x4){0u, 0u, 0u, 0u};
    return;
  }
  const int cw0 = blockIdx.y * (64 * NWV) + wave * 64;           // may lie beyond N: such a wave adds zeros
  const int rank = tk.rank, NJ = (rank + 15) >> 4;
  bf16_t* sBig = lds[wave][0];
  bf16_t* sSm = lds[wave][1];

  const rsrc_t rB = make_rsrc(p.dY + (size_t)it.row0 * p.N, (uint32_t)it.nrows * (uint32_t)p.N * 2u);
  const rsrc_t rS = make_rsrc(p.Hs + (size_t)it.row0 * p.RP, (uint32_t)it.nrows * (uint32_t)p.RP * 2u);
  const rsrc_t rP = make_rsrc(tk.B, (uint32_t)rank * (uint32_t)p.N * 2u);
  // the partial sums of this slab for the rows of this group
  const rsrc_t rG = make_rsrc(p.gpart + ((size_t)blockIdx.y * p.T + it.row0) * p.RP, (uint32_t)it.nrows * (uint32_t)p.RP * 4u);
  const int b_row = lane >> 3, b_pc = (lane & 7) * 8;
  const bool b_col_ok = cw0 + b_pc < p.N;
  const int ppr = p.RP >> 3;                   // 16-byte pieces in a row of Hs; RP <= 16 NJM, so a lane loads at most NJM of them
  const int l16 = lane & 15, g = lane >> 4;

  // B_t[j][columns of this wave], as the B operand of dY B_t^T: lane (j = l16, g) holds 8 consecutive columns
  bf16x8 bt[NJM][2];
#pragma unroll
  for (int jt = 0; jt < NJM; ++jt)
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int j = jt * 16 + l16, col = cw0 + s * 32 + 8 * g;
      bt[jt][s] = as_bf16x8(buf_load16(rP, (j < rank && col < p.N) ? (uint32_t)(((size_t)j * p.N + col) * 2) : OOB));
    }

  u32x4 gb[DEPTH][4], gs[DEPTH][NJM];
  const int steps = (it.nrows + 31) >> 5;
  const GroupBits gbits = load_group_bits(p.dtab, p.rowbits_off, it.row0, it.nrows, p.T, lane);
  // per-lane pieces of the Hs slab: idx = lane + 64 q -> row idx / ppr, piece idx % ppr
  int s_row[NJM], s_pc[NJM];
#pragma unroll
  for (int q = 0; q < NJM; ++q) { const int idx = lane + 64 * q; s_row[q] = idx / ppr; s_pc[q] = (idx % ppr) * 8; }
  auto load_step = [&](int s, int buf) {       // a step past the end loads nothing (every offset out of range)
    const int base = s * 32;
    const uint32_t vbits = s < steps ? step_bits(gbits, s) : 0u;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int m = base + b_row + 8 * q;
      const bool ok = b_col_ok && m < it.nrows && ((vbits >> (b_row + 8 * q)) & 1u);
      gb[buf][q] = buf_load16_once<STREAM>(rB, ok ? (uint32_t)(((size_t)m * p.N + cw0 + b_pc) * 2) : OOB);
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

  f32x4 accb[NJM][4];
#pragma unroll
  for (int jt = 0; jt < NJM; ++jt)
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) accb[jt][ct] = (f32x4){0.f, 0.f, 0.f, 0.f};
  f32x4 accg[BATCH][2][NJM];

  const int tr_off = (8 * g + (l16 >> 2)) * GP + 4 * (l16 & 3);
  float* red = (float*)lds[wave];
#pragma unroll
  for (int d = 0; d < DEPTH; ++d) load_step(d, d);
  for (int s0 = 0; s0 < steps; s0 += UNR) {
#pragma unroll
    for (int u = 0; u < UNR; ++u) {
      const int s = s0 + u;                       // may run past the last step: zeros in, nothing out
      store_step(u % DEPTH);
      load_step(s + DEPTH, u % DEPTH);
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      {
        // the slab's share of dY B_t^T first, one 16-row half at a time (its operands are dead before the next are read)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
          bf16x8 ay[2];
#pragma unroll
          for (int ks = 0; ks < 2; ++ks) ay[ks] = *(const bf16x8*)(sBig + (rt * 16 + l16) * GP + ks * 32 + 8 * g);
#pragma unroll
          for (int jt = 0; jt < NJM; ++jt) {
            f32x4 v = (f32x4){0.f, 0.f, 0.f, 0.f};
            if (jt < NJ)
#pragma unroll
              for (int ks = 0; ks < 2; ++ks) v = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ay[ks], bt[jt][ks], v, 0, 0, 0);
            accg[u % BATCH][rt][jt] = v;
          }
        }
        bf16x8 a[NJM];
#pragma unroll
        for (int jt = 0; jt < NJM; ++jt) {
          const bf16x4 lo = lds_read_tr(sSm + tr_off + jt * 16), hi = lds_read_tr(sSm + tr_off + 4 * GP + jt * 16);
          a[jt] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        }
#pragma unroll
        for (int ct = 0; ct < 4; ++ct) {
          const bf16x4 lo = lds_read_tr(sBig + tr_off + ct * 16), hi = lds_read_tr(sBig + tr_off + 4 * GP + ct * 16);
          const bf16x8 b = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
          for (int jt = 0; jt < NJM; ++jt)
            if (jt < NJ) accb[jt][ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[jt], b, accb[jt][ct], 0, 0, 0);
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      if ((u % BATCH) == BATCH - 1) {
        // The waves meet: accg[bi][rt][jt][v] = this wave's share of (dY B_t^T)[row of the batch 32 bi + 16 rt + 4 g + v]
        // [16 jt + l16], staged over the slabs just read, added up in wave order, one fp32 partial per row and column out.
#pragma unroll
        for (int bi = 0; bi < BATCH; ++bi)
#pragma unroll
          for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int jt = 0; jt < NJM; ++jt) *(f32x4*)&red[(jt * 16 + l16) * RPITCH + bi * 32 + rt * 16 + 4 * g] = accg[bi][rt][jt];
        lds_barrier();
        const int base = (s - (BATCH - 1)) * 32;                // first row of the batch inside the group
#pragma unroll
        for (int i = 0; i < NRED; ++i) {
          const int e = tid + NTHR * i, m = e / RPJ, j = e % RPJ;
          float v = 0.f;
#pragma unroll
          for (int w = 0; w < NWV; ++w) v += ((const float*)lds[w])[j * RPITCH + m];
          const bool ok = base + m < it.nrows && j < 16 * NJ;     // (the reduction reads the task's rank pieces only)
          uint32_t bits = 0;
          if (ONE) bits = (uint32_t)__shfl((int)gbits.lo, (base + m + gbits.sh) >> 5);      // (every lane takes part)
          if (!ONE) {
            buf_store4(rG, ok ? (uint32_t)(((base + m) * p.RP + j) * 4) : OOB, v);
          } else if (base + m < it.nrows && j < p.RP) {           // columns beyond the rank and padding rows: zeros
            const size_t o = (size_t)(it.row0 + base + m) * p.RP + j;
            float g = 0.f;
            if (j < rank && ((bits >> ((base + m + gbits.sh) & 31)) & 1u)) {
              g = tk.scale * v;
              if (tk.kind == MUX_ADAPTER_TUNING) g *= gelu_slope_f(bf16_to_f32(p.U2[o]));
            }
            p.Gs[o] = f32_to_bf16(g);
          }
        }
        lds_barrier();
      }
    }
  }
  if (cw0 >= p.N) return;
  // accb[jt][ct][v] = bpart[j = jt*16 + 4g + v][c = cw0 + ct*16 + l16]
  float* dst = p.direct ? tk.dB : p.bpart + (size_t)blockIdx.x * ((size_t)p.RP * p.N);
  if (dst == nullptr) return;                    // (no gradient asked for)
  auto put = [&](auto ADD) {
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
              float* d = dst + (size_t)j * p.N + c;
              if (c < p.N) *d = decltype(ADD)::value ? *d + accb[jt][ct][v] : accb[jt][ct][v];
            }
        }
  };
  if (p.direct && p.accumulate) put(std::true_type{});
  else put(std::false_type{});
}

// ------------------------------------------------------------------------------------------------
// IA3_OUT: part[item][n] = sum_{rows} g[i][n] * z[i][n], and dYs[i][n] = g[i][n] * l_t[n] (the operand of the
// backbone backward for these rows).  grid = (64-row items, ceil(N/1024)), 512 threads: 128 column threads of 8
// columns, times four quarters of the item's rows (16 rows each, all 32 loads of a thread issued before the first
// sum), the quarters' sums added through LDS in the order of the rows.
constexpr int kDlCols = 1024;
struct DlParams {
  const bf16_t *dY, *Z;
  float* part;
  bf16_t* dYs;
  int N, items_off, bits_off;
};
__device__ __forceinline__ void dl_rows(const int32_t* dtab, const TaskRef& tasks, const DlParams& q, int item, int block,
                                        float (*sq)[128][9]) {
  const bf16_t* const dY = q.dY;
  const bf16_t* const Z = q.Z;
  const int N = q.N;
  const int4 iw = *(const int4*)(dtab + q.items_off + item * DI_WORDS);
  const int task = iw.x, row0 = iw.y, nrows = iw.z;
  if (task < 0 || iw.w == 0) return;
  if (get_task_kind(tasks, task) != MUX_ADAPTER_IA3_OUT) return;
  const DevTask tk = get_task(tasks, task);
  const uint32_t* bw = (const uint32_t*)(dtab + q.bits_off) + 2 * item;
  const int ct = threadIdx.x & 127, rq = threadIdx.x >> 7;
  const uint32_t bits = (rq < 2 ? bw[0] : bw[1]) >> (16 * (rq & 1)) & 0xffffu;    // validity of this quarter's 16 rows
  const int n0 = (block * 128 + ct) * 8;
  const bool cols = n0 < N;
  constexpr int RQ = 16;
  float s[8], lv[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) { s[e] = 0.f; lv[e] = 0.f; }
  if (cols) {
    const uint4 l4 = *(const uint4*)((const bf16_t*)tk.L + n0);
    const uint32_t* pl = (const uint32_t*)&l4;
#pragma unroll
    for (int e = 0; e < 4; ++e) { lv[2 * e] = __uint_as_float(pl[e] << 16); lv[2 * e + 1] = __uint_as_float(pl[e] & 0xffff0000u); }
    // every thread issues the same 2 RQ loads (a row that does not count reads the item's first row instead and is
    // dropped afterwards)
    uint4 gv[RQ], zv[RQ];
#pragma unroll
    for (int u = 0; u < RQ; ++u) {
      const int m = rq * RQ + u;
      const int row = row0 + (m < nrows ? m : 0);
      gv[u] = *(const uint4*)(dY + (size_t)row * N + n0);
      zv[u] = *(const uint4*)(Z + (size_t)(tk.zrow0 + row - tk.row_begin) * N + n0);
    }
#pragma unroll
    for (int u = 0; u < RQ; ++u) {
      const int m = rq * RQ + u;
      if (!(m < nrows && ((bits >> u) & 1u))) continue;
      const uint32_t* pg = (const uint32_t*)&gv[u];
      const uint32_t* pz = (const uint32_t*)&zv[u];
      uint4 sv;
      uint32_t* ps = (uint32_t*)&sv;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float g0 = __uint_as_float(pg[e] << 16), g1 = __uint_as_float(pg[e] & 0xffff0000u);
        s[2 * e] = fmaf(g0, __uint_as_float(pz[e] << 16), s[2 * e]);
        s[2 * e + 1] = fmaf(g1, __uint_as_float(pz[e] & 0xffff0000u), s[2 * e + 1]);
        ps[e] = pack_bf16x2(g0 * lv[2 * e], g1 * lv[2 * e + 1]);
      }
      *(uint4*)(q.dYs + (size_t)(tk.zrow0 + row0 + m - tk.row_begin) * N + n0) = sv;
    }
  }
  if (rq > 0) {
#pragma unroll
    for (int e = 0; e < 8; ++e) sq[rq - 1][ct][e] = s[e];
  }
  __syncthreads();
  if (rq == 0 && cols) {
    float* dst = q.part + (size_t)item * N + n0;
#pragma unroll
    for (int e = 0; e < 8; ++e) dst[e] = ((s[e] + sq[0][ct][e]) + sq[1][ct][e]) + sq[2][ct][e];
  }
}

__global__ __launch_bounds__(512) void k_dl(const int32_t* __restrict__ dtab, const TaskRef tasks, const DlParams q) {
  __shared__ float sq[3][128][9];
  dl_rows(dtab, tasks, q, blockIdx.x, blockIdx.y, sq);
}

// Ranks that are not multiples of 8: A_t [K, r] (Adapter-Tuning: D_t [N, r]) once more with its rows padded to
// round_up(r, 8) elements (zeros), so that every kernel of the matrix-core path reads rows of whole 16-byte pieces.
// tk.L is the caller's matrix, tk.A the padded copy in the workspace; piece e of the copy by one thread.  A copy of a few
// hundred KB, bound by its launch (4 us at 1608 x 12); before it, such ranks sent the whole backward product to a
// register-staged GEMM at a third of the pipelined one's rate.
__device__ __forceinline__ void pad_rank_piece(const TaskRef& tasks, int task, int e, int K, int N) {
  const DevTask tk = get_task(tasks, task);
  if ((tk.kind != MUX_ADAPTER_LORA && tk.kind != MUX_ADAPTER_TUNING) || tk.L == nullptr) return;
  const int rows = tk.kind == MUX_ADAPTER_LORA ? K : N;
  const int pieces = rank_pieces(tk.rank);
  if (e >= rows * pieces) return;
  const int row = e / pieces, j0 = (e % pieces) * 8;
  const uint16_t* src = (const uint16_t*)tk.L + (size_t)row * tk.rank;
  uint32_t w[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int j = j0 + 2 * i;
    w[i] = (j < tk.rank ? (uint32_t)src[j] : 0u) | (j + 1 < tk.rank ? (uint32_t)src[j + 1] << 16 : 0u);
  }
  *(uint4*)((uint16_t*)tk.A + (size_t)e * 8) = make_uint4(w[0], w[1], w[2], w[3]);
}

__global__ __launch_bounds__(256) void k_pad_rank(const TaskRef tasks, int K, int N) {
  pad_rank_piece(tasks, blockIdx.x, blockIdx.y * 256 + threadIdx.x, K, N);
}

// Gs[T,RP] = s_t * (sum over the column slabs of the shares k_s4 left, ascending), times gelu'(u) for the TUNING rows;
// zero on padding rows, beyond the rank and on the rows of the other kinds.  One workgroup per 64-row item.  Behind these
// the launch has the workgroups of two small jobs that need nothing of it and that the next launches wait for, as
// launches of their own 4-9 us each: the padded copies of A_t (n_pad a task) and, in the build with DL, the IA3 rows
// (1608 x 6424, ranks 4 and 12, two micro-batches forward and backward: 391 us, 384 with the copies, 376 with both).
template <bool DL>
__global__ __launch_bounds__(DL ? 512 : 256) void k_gs_reduce(const int32_t* __restrict__ dtab, const TaskRef tasks,
                                                  const float* __restrict__ gpart, int n_slabs, int T, int RP,
                                                  const bf16_t* __restrict__ U2, bf16_t* __restrict__ Gs, int items_off,
                                                  int bits_off, int n_items, int n_dl, int n_pad, int K, const DlParams q) {
  constexpr int NTHR = DL ? 512 : 256;
  int b = blockIdx.x;
  if constexpr (DL) {                  // the longest first: n_dl column blocks an item
    __shared__ float sq[3][128][9];
    if (b < n_items * n_dl) {
      dl_rows(dtab, tasks, q, b / n_dl, b % n_dl, sq);
      return;
    }
    b -= n_items * n_dl;
  }
  if (b >= n_items) {
    b -= n_items;
    pad_rank_piece(tasks, b / n_pad, (b % n_pad) * NTHR + threadIdx.x, K, q.N);
    return;
  }
  const int item = b;
  const int4 iw = *(const int4*)(dtab + items_off + item * DI_WORDS);
  const uint32_t* bw = (const uint32_t*)(dtab + bits_off) + 2 * item;
  const uint32_t bits0 = bw[0], bits1 = bw[1];
  const int task = iw.x, row0 = iw.y, nrows = iw.z;
  const int kind = task >= 0 ? get_task_kind(tasks, task) : MUX_ADAPTER_NONE;
  const bool mine = (kind == MUX_ADAPTER_LORA || kind == MUX_ADAPTER_TUNING) && (bits0 | bits1) != 0u;
  float scale = 0.f;
  int rank = 0;
  if (mine) { const DevTask tk = get_task(tasks, task); scale = tk.scale; rank = tk.rank; }
  const int q4 = RP >> 2;                        // groups of four columns a row
  for (int e = threadIdx.x; e < nrows * q4; e += NTHR) {
    const int m = e / q4, j = (e % q4) * 4;
    const size_t o = (size_t)(row0 + m) * RP + j;
    const bool valid = mine && (((m < 32 ? bits0 >> m : bits1 >> (m - 32)) & 1u) != 0u) && j < rank;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (valid) {
      for (int q = 0; q < n_slabs; q += 4) {     // four slabs in flight; the sum runs in ascending slab order
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
          v[u] = q + u < n_slabs ? *(const float4*)(gpart + ((size_t)(q + u) * T + row0 + m) * RP + j) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 4; ++u) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
      }
      s.x *= scale; s.y *= scale; s.z *= scale; s.w *= scale;
      if (kind == MUX_ADAPTER_TUNING) {
        s.x *= gelu_slope_f(bf16_to_f32(U2[o])); s.y *= gelu_slope_f(bf16_to_f32(U2[o + 1]));
        s.z *= gelu_slope_f(bf16_to_f32(U2[o + 2])); s.w *= gelu_slope_f(bf16_to_f32(U2[o + 3]));
      }
      if (j + 1 >= rank) s.y = 0.f;
      if (j + 2 >= rank) s.z = 0.f;
      if (j + 3 >= rank) s.w = 0.f;
    }
    uint2 out;
    out.x = pack_bf16x2(s.x, s.y);
    out.y = pack_bf16x2(s.z, s.w);
    *(uint2*)(Gs + o) = out;
  }
}

// ------------------------------------------------------------------------------------------------
// The gradient partials of dA_t (dD_t), a workgroup of four waves a (row group, 256 columns), in a launch of their own.
template <int NJM, int DEPTH, bool STREAM>
__global__ __launch_bounds__(256) void k_grad(const GradParams p, const TaskRef tasks) {
  __shared__ __attribute__((aligned(16))) bf16_t lds[kGradLdsElems];
  grad_rows<NJM, DEPTH, STREAM>(p, tasks, blockIdx.x, blockIdx.y, lds);
}

// ------------------------------------------------------------------------------------------------
// Adapter-Tuning: Out = In + Small P for the rows of TUNING items (forward: P = U_t [r][N] as stored, Y = z + Hs U_t,
// In = the saved compact z rows, Out = Y; backward: P = D_t^T, dYs = dY + Gs D_t^T, In = dY, Out = the compact dYs
// rows).  grid = (64-row items, ceil(N/256)); each wave owns 64 columns: its [r][64] slab of U_t goes through a
// wave-private LDS region in natural layout and comes back k-major with ds_read_b64_tr_b16; of D_t [N][r] a lane
// loads the eight consecutive r of one column (a 16-byte piece of a row) straight from memory; the products are staged 16 rows at a time in fp32 so that In is read and Out is written in whole 128-byte lines.
struct TuneAddParams {
  const int32_t* dtab;
  const bf16_t* In;
  const bf16_t* Small;   // [T, RP]
  bf16_t* Out;
  int N, RP, backward;
  TaskRef tasks;
};

template <int NKS>      // k-steps of 32 over the rank pitch (1 or 2)
__global__ __launch_bounds__(256) void k_tune_add(const TuneAddParams p) {
  constexpr int SP = 68;                                       // fp32 staging pitch
  __shared__ __attribute__((aligned(16))) bf16_t sP[4][NKS * 32 * GP];
  __shared__ __attribute__((aligned(16))) float sC[4][16 * SP];
  const ItemView it = load_item(p.dtab, TS64, blockIdx.x);
  if (it.task < 0 || get_task_kind(p.tasks, it.task) != MUX_ADAPTER_TUNING) return;
  const DevTask tk = get_task(p.tasks, it.task);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int cw0 = blockIdx.y * 256 + wave * 64;
  if (cw0 >= p.N) return;
  const int rank = tk.rank;
  bf16_t* sp = sP[wave];
  float* sc = sC[wave];

  // slab [NKS*32][64] of U_t -> LDS, natural layout; rows beyond the rank read as zero
  const int b_row = lane >> 3, b_pc = (lane & 7) * 8;
  if (!p.backward) {
    const rsrc_t rP = make_rsrc(tk.B, (uint32_t)rank * (uint32_t)p.N * 2u);
#pragma unroll
    for (int q = 0; q < NKS * 4; ++q) {
      const int j = b_row + 8 * q;
      const bool ok = j < rank && cw0 + b_pc < p.N;
      const u32x4 v = buf_load16(rP, ok ? (uint32_t)(((size_t)j * p.N + cw0 + b_pc) * 2) : OOB);
      *(u32x4*)(sp + j * GP + b_pc) = v;
    }
  }
  // Small rows in the A-operand layout straight from global memory: row = 16 rt + lane%16, k = 32 ks + 8 (lane/16)
  const int i = lane & 15, g = lane >> 4;
  const rsrc_t rS = make_rsrc(p.Small + (size_t)it.row0 * p.RP, (uint32_t)it.nrows * (uint32_t)p.RP * 2u);
  bf16x8 a[4][NKS];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int m = rt * 16 + i, k = ks * 32 + 8 * g;
      a[rt][ks] = as_bf16x8(buf_load16(rS, (m < it.nrows && k < p.RP) ? (uint32_t)((m * p.RP + k) * 2) : OOB));
    }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  const int tr_off = (8 * g + (i >> 2)) * GP + 4 * (i & 3);
  bf16x8 b[4][NKS];
  if (p.backward) {
    const uint32_t pitch = 16u * (uint32_t)rank_pieces(rank);       // bytes in a row of D_t
    const rsrc_t rD = make_rsrc(tk.A, (uint32_t)p.N * pitch);
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const int col = cw0 + ct * 16 + i, k = ks * 32 + 8 * g;
        b[ct][ks] = as_bf16x8(buf_load16(rD, (col < p.N && k < rank) ? (uint32_t)col * pitch + (uint32_t)k * 2u : OOB));
      }
  } else {
#pragma unroll
    for (int ct = 0; ct < 4; ++ct)
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) {
        const bf16x4 lo = lds_read_tr(sp + ks * 32 * GP + tr_off + ct * 16), hi = lds_read_tr(sp + ks * 32 * GP + tr_off + 4 * GP + ct * 16);
        b[ct][ks] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
  }

  const uint32_t vbits_lo = row_valid_bits32(p.dtab, it.row0);
  const uint32_t vbits_hi = it.nrows > 32 ? row_valid_bits32(p.dtab, it.row0 + 32) : 0u;
  const size_t zrow0 = (size_t)(tk.zrow0 + it.row0 - tk.row_begin);
  const bf16_t* in = p.In + (p.backward ? (size_t)it.row0 : zrow0) * p.N;
  bf16_t* out = p.Out + (p.backward ? zrow0 : (size_t)it.row0) * p.N;
  // the eight pieces of `In` this lane adds to are fetched up front (fetched where they are used, each cost the wave
  // a memory latency)
  uint4 xin[4][2];
  bool xok[4][2];
#pragma unroll
  for (int rt = 0; rt < 4; ++rt)
#pragma unroll
    for (int ps = 0; ps < 2; ++ps) {
      const int m = rt * 16 + b_row + 8 * ps, c = cw0 + b_pc;
      xok[rt][ps] = m < it.nrows && c < p.N && ((m < 32 ? vbits_lo >> m : vbits_hi >> (m - 32)) & 1u) != 0;
      xin[rt][ps] = xok[rt][ps] ? *(const uint4*)(in + (size_t)m * p.N + c) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
  for (int rt = 0; rt < 4; ++rt) {
    if (rt * 16 >= it.nrows) break;
    // operands exchanged: acc[ct][v] = product[row 16 rt + i][column 16 ct + 4 g + v]
#pragma unroll
    for (int ct = 0; ct < 4; ++ct) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks) acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[ct][ks], a[rt][ks], acc, 0, 0, 0);
      *(f32x4*)(sc + i * SP + ct * 16 + 4 * g) = acc;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int ps = 0; ps < 2; ++ps) {
      const int ml = b_row + 8 * ps, m = rt * 16 + ml, c = cw0 + b_pc;
      if (m < it.nrows && c < p.N) {
        uint4 o = make_uint4(0, 0, 0, 0);
        if (xok[rt][ps]) {
          const uint4 x = xin[rt][ps];
          const f32x4 p0 = *(const f32x4*)(sc + ml * SP + b_pc), p1 = *(const f32x4*)(sc + ml * SP + b_pc + 4);
          const uint32_t* px = (const uint32_t*)&x;
          o.x = pack_bf16x2(__uint_as_float(px[0] << 16) + p0[0], __uint_as_float(px[0] & 0xffff0000u) + p0[1]);
          o.y = pack_bf16x2(__uint_as_float(px[1] << 16) + p0[2], __uint_as_float(px[1] & 0xffff0000u) + p0[3]);
          o.z = pack_bf16x2(__uint_as_float(px[2] << 16) + p1[0], __uint_as_float(px[2] & 0xffff0000u) + p1[1]);
          o.w = pack_bf16x2(__uint_as_float(px[3] << 16) + p1[2], __uint_as_float(px[3] & 0xffff0000u) + p1[3]);
        }
        *(uint4*)(out + (size_t)m * p.N + c) = o;
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
  }
}

// ------------------------------------------------------------------------------------------------
// out_t = (accumulate ? out_t : 0) + sum over the task's items, ascending.  grid = (tasks, blocks).
// LoRA and Adapter-Tuning tasks: the first blocks take 1024 elements of dB_t [r][N] each, from part0; the blocks after
// them dA_t, whose partials in part1 are [r][K] and which is stored [K][r]: such a block takes all r of
// reduce_cols(r) columns, so that it writes one contiguous run of dA_t.  IA3_OUT tasks: dl_t [N] from part_ia3 (one row
// per 64-row item).
// Bound by the latency of a few dependent loads and, before blocks wrote whole runs of dA_t, by stores of 4 bytes at a
// stride of r floats: 32 tasks of rank 16, 8192 x 1024 and 1024 x 8192, 29.2 -> 14.7 us a launch; 16 tasks of rank 8 to
// 64 at 4096 x 4096, 31.4 -> 18.4 us; two tasks at 256 x 256, 4.1 -> 2.9 us.
static_assert(MUX_MAX_RANK <= 256, "reduce_cols: a block takes four columns at least");
__host__ __device__ __forceinline__ int reduce_cols(int rank) { return (1024 / rank) & ~3; }   // columns of dA_t a block takes
struct ReduceParams {
  const int32_t* dtab;
  const float *part0, *part1, *part_ia3;
  int N, K, accumulate;
  int ranked;                                // 0: the LoRA and Adapter-Tuning gradients are there already
  int items_off[3], task_items_off[3];       // word offsets in dtab of the row groups of part0, part1 and part_ia3
  size_t slot0, slot1;                       // elements per row group in part0, part1
  TaskRef tasks;
};
__global__ __launch_bounds__(256) void k_reduce(const ReduceParams p) {
  __shared__ float sT[2048];                 // the block's piece of dA_t, [columns][r + 1]
  const int t = blockIdx.x;
  const DevTask tk = get_task(p.tasks, t);
  const bool ranked = tk.kind == MUX_ADAPTER_LORA || tk.kind == MUX_ADAPTER_TUNING;
  if (ranked ? !p.ranked : tk.kind != MUX_ADAPTER_IA3_OUT) return;
  const int rows = ranked ? tk.rank : 1, N = p.N;
  const int nb0 = (int)(((size_t)rows * N + 1023) / 1024);
  const bool transposed = (int)blockIdx.y >= nb0;
  if (transposed && !ranked) return;
  const int which = !ranked ? 2 : (transposed ? 1 : 0);
  const int C = (transposed && tk.kind != MUX_ADAPTER_TUNING) ? p.K : N;    // the first gradient of Adapter-Tuning is dD_t [N][r]
  float* out = !ranked ? tk.dL : (transposed ? tk.dA : tk.dB);
  const float* part = which == 0 ? p.part0 : (which == 1 ? p.part1 : p.part_ia3);
  const size_t slot = which == 0 ? p.slot0 : (which == 1 ? p.slot1 : (size_t)N);
  const int cols = transposed ? reduce_cols(rows) : 0, c0 = transposed ? ((int)blockIdx.y - nb0) * cols : 0;
  if (!out || (transposed && c0 >= C)) return;
  // four consecutive elements of one row of the partials a thread (N, K multiples of 4)
  const int tid = threadIdx.x;
  const size_t e = ((size_t)blockIdx.y * 256 + tid) * 4;                    // in dB_t or dl_t
  const int j_t = transposed ? tid / (cols >> 2) : 0, ct = transposed ? (tid % (cols >> 2)) * 4 : 0;
  const bool mine = transposed ? (j_t < rows && c0 + ct < C) : e < (size_t)rows * C;
  const size_t at = transposed ? (size_t)j_t * C + c0 + ct : e;             // in a row group's partials
  const int32_t* ti = p.dtab + p.task_items_off[which] + 2 * t;
  const int ib = ti[0], ic = ti[1];
  const int32_t* items = p.dtab + p.items_off[which];
  // four items in flight (a thread that fetched them one by one would wait a memory latency per item); an item
  // without valid rows holds no partial and adds an exact zero; the sum runs in ascending item order
  float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
  if (mine)
    for (int q = 0; q < ic; q += 4) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool has = q + u < ic && items[(ib + q + u) * DI_WORDS + DI_NVALID] != 0;
        v[u] = has ? *(const float4*)(part + (size_t)(ib + q + u) * slot + at) : make_float4(0.f, 0.f, 0.f, 0.f);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) { s.x += v[u].x; s.y += v[u].y; s.z += v[u].z; s.w += v[u].w; }
    }
  if (transposed) {
    const int pitch = rows + 1;
    if (mine) {
      sT[ct * pitch + j_t] = s.x;
      sT[(ct + 1) * pitch + j_t] = s.y;
      sT[(ct + 2) * pitch + j_t] = s.z;
      sT[(ct + 3) * pitch + j_t] = s.w;
    }
    __syncthreads();
    const int n = (C - c0 < cols ? C - c0 : cols) * rows;
    float* dst = out + (size_t)c0 * rows;
    for (int i = tid; i < n; i += 256) {
      const float v = sT[(i / rows) * pitch + i % rows];
      dst[i] = p.accumulate ? dst[i] + v : v;
    }
    return;
  }
  if (!mine) return;
  if (((uintptr_t)out & 15) == 0) {
    float4* dst = (float4*)(out + e);
    float4 o = s;
    if (p.accumulate) { const float4 d = *dst; o.x += d.x; o.y += d.y; o.z += d.z; o.w += d.w; }
    *dst = o;
  } else {                                     // a gradient buffer of the caller that is only 4-byte aligned
    float* dst = out + e;
    dst[0] = p.accumulate ? dst[0] + s.x : s.x;
    dst[1] = p.accumulate ? dst[1] + s.y : s.y;
    dst[2] = p.accumulate ? dst[2] + s.z : s.z;
    dst[3] = p.accumulate ? dst[3] + s.w : s.w;
  }
}

// Row groups of 1024 mean 1/4 of the partial bytes of groups of 256; they are taken when the launch still has
// `enough` workgroups to occupy the chip.
int choose_group(const mux_segtab* st, int col_blocks, int enough) {
  return st->items[TS1024].size() * (size_t)col_blocks >= (size_t)enough ? TS1024 : TS256;
}
constexpr int kS4Cols = 512;                          // columns of one workgroup of the dY pass
int s4_slabs(int N) { return (N + kS4Cols - 1) / kS4Cols; }
int s4_group(const mux_segtab* st, int N) { return choose_group(st, s4_slabs(N), 192); }
int da_group(const mux_segtab* st, int C) { return choose_group(st, (C + 255) / 256, 384); }
int grad_width(const CallCtx& c) { return (c.st->n_tuning > 0 && c.N > c.K) ? c.N : c.K; }   // columns of the widest dA_t (dD_t)

// Is every LoRA and Adapter-Tuning task one row group, of size `ts_b` in the pass over dY and `ts_a` in the one over X?  Then
// their sums are the gradients, and no partials and no reduction are needed (256 x 256, two tasks of 100 and 150 tokens, 4 us
// of 34).  Not where a gradient goes over an input: the reduction writes after the last read of X, dY and the saved activations,
// the passes themselves do not.
bool single_groups(const CallCtx& c, int ts_b, int ts_a) {
  const mux_segtab* const st = c.st;
  if (!c.grads_apart) return false;
  for (int t = 0; t < st->n_tasks; ++t) {
    if (st->tasks[t].kind != MUX_ADAPTER_LORA && st->tasks[t].kind != MUX_ADAPTER_TUNING) continue;
    if (st->tasks[t].valid == 0 || st->task_item_count[ts_b][t] != 1 || st->task_item_count[ts_a][t] != 1) return false;
  }
  return true;
}

// 16-byte pieces of the largest padded copy of an A_t (D_t); 0: no rank needs one
size_t padded_pieces(const CallCtx& c) {
  size_t most = 0;
  for (const HostTask& ht : c.st->tasks)
    if (rank_is_padded(ht)) {
      const size_t n = (size_t)rank_pieces(ht.rank) * (ht.kind == MUX_ADAPTER_LORA ? c.K : c.N);
      if (n > most) most = n;
    }
  return most;
}

int dl_blocks(int N) { return (N + kDlCols - 1) / kDlCols; }
// The IA3 rows ride in the launch of gs_reduce where they have no more than a few rounds of workgroups.  Forward and
// backward, a launch of their own against riding: 512 rows of 2048 x 2048 81.4 -> 79.6 us (64 workgroups), 3072 of
// 4096 x 4096 396 -> 392 (384), 4096 of 4096 x 4096 326.5 -> 323 (288); 4096 of 4096 x 8192, 1280 workgroups,
// 1147 and 1148: the 174 registers of that build then cost the reduction what the launch gains.
bool dl_rides_along(const CallCtx& c) {
  return c.st->n_ia3 > 0 && c.st->n_lora + c.st->n_tuning > 0 && s4_slabs(c.N) > 1 &&
         c.st->items[TS64].size() * (size_t)dl_blocks(c.N) <= 4 * (size_t)kComputeUnits;
}

struct PartLayout { size_t gpart, part0, part1, ia3, total; };
PartLayout part_layout(int K, int N, const mux_segtab* st) {
  PartLayout o{};
  const int RP = rank_pitch(st);
  const int K1 = (st->n_tuning > 0 && N > K) ? N : K;       // a TUNING item's second partial is [RP][N]
  if (RP > 0) {
    o.gpart = align256((size_t)s4_slabs(N) * st->T * RP * 4);
    o.part0 = align256((size_t)st->items[TS256].size() * RP * N * 4);      // sized for the smaller row groups
    o.part1 = align256((size_t)st->items[TS256].size() * RP * K1 * 4);
  }
  o.ia3 = st->n_ia3 > 0 ? align256((size_t)st->items[TS64].size() * N * 4) : 0;
  o.total = o.gpart + o.part0 + o.part1 + o.ia3;     // the IA3 partials lie behind the others: one reduction takes both
  return o;
}

}  // namespace

size_t adapter_partial_bytes(int K, int N, const mux_segtab* st) { return part_layout(K, N, st).total; }

namespace {
DlParams dl_params(const CallCtx& c, const void* dY, const void* Z, void* part) {
  const PartLayout pl = part_layout(c.K, c.N, c.st);
  return DlParams{(const bf16_t*)dY, (const bf16_t*)Z, (float*)((char*)part + pl.gpart + pl.part0 + pl.part1), (bf16_t*)c.dYs,
                  c.N, c.st->dev_image[DH_NITEMS0 + 3 * TS64 + 1], c.st->dev_image[DH_OFF_ITEM_BITS]};
}
}  // namespace

void adapter_pad_ranks(const CallCtx& c) {
  const size_t most = padded_pieces(c);
  if (most > 0)
    MUX_LAUNCH("pad_rank", k_pad_rank, dim3((unsigned)c.st->n_tasks, (unsigned)((most + 255) / 256)), dim3(256), 0, c.stream,
               *c.tref, c.K, c.N);
}

mux_status adapter_down_x(const CallCtx& c, const void* X, void* Hs) {
  if (c.st->n_lora == 0) return MUX_OK;
  DownParams p{c.dtab, (const bf16_t*)X, (bf16_t*)Hs, nullptr, c.K, c.RP, DOWN_X};
  launch_down(c, "down_x", p);
  return MUX_OK;
}

// The pass over dY: Gs (LoRA: s_t dY B_t^T; Adapter-Tuning: s_t (dY U_t^T) * gelu'(u)) and the partial sums of
// dB_t = Hs^T dY (dU_t), which adapter_reduce brings together.
mux_status adapter_dy_pass(const CallCtx& c, const void* dY, const void* Hs, const void* Z, void* Gs, void* part, int accumulate) {
  if (c.st->n_lora + c.st->n_tuning == 0) return MUX_OK;
  const PartLayout pl = part_layout(c.K, c.N, c.st);
  float* gpart = (float*)part;
  float* part0 = (float*)((char*)part + pl.gpart);
  const int ts = s4_group(c.st, c.N), slabs = s4_slabs(c.N);
  S4Params p{c.dtab, (const bf16_t*)dY, (const bf16_t*)Hs, gpart, part0, c.N, c.RP, ts, c.st->T,
             c.st->dev_image[DH_NITEMS0 + 3 * ts + 1], c.st->dev_image[DH_OFF_ROWBITS]};
  p.tasks = *c.tref;
  p.direct = single_groups(c, ts, da_group(c.st, grad_width(c))) ? 1 : 0;
  p.accumulate = accumulate;
  p.U2 = (const bf16_t*)c.U2;
  p.Gs = (bf16_t*)Gs;
  const dim3 grid((unsigned)c.st->items[ts].size(), (unsigned)slabs);
  // (rank pieces, steps between two meetings of the waves, steps of loads in flight)
  if (slabs == 1) {
    adapter_pad_ranks(c);
    if (c.st->r_max <= 16) MUX_LAUNCH("s4_dy_pass", (k_s4<1, 2, 2, true, false>), grid, dim3(512), 0, c.stream, p);
    else if (c.st->r_max <= 32) MUX_LAUNCH("s4_dy_pass", (k_s4<2, 2, 1, true, false>), grid, dim3(512), 0, c.stream, p);
    else MUX_LAUNCH("s4_dy_pass", (k_s4<4, 1, 1, true, false>), grid, dim3(512), 0, c.stream, p);
    return MUX_OK;
  }
  auto launch = [&](auto STREAM) {
    constexpr bool S = decltype(STREAM)::value;
    if (c.st->r_max <= 16) MUX_LAUNCH("s4_dy_pass", (k_s4<1, 2, 2, false, S>), grid, dim3(512), 0, c.stream, p);
    else if (c.st->r_max <= 32) MUX_LAUNCH("s4_dy_pass", (k_s4<2, 2, 1, false, S>), grid, dim3(512), 0, c.stream, p);
    else MUX_LAUNCH("s4_dy_pass", (k_s4<4, 1, 1, false, S>), grid, dim3(512), 0, c.stream, p);
  };
  if (past_caches(c, ranked_bytes(c.st, c.N, c.N))) launch(std::true_type{}); else launch(std::false_type{});
  // moved: the partials of every slab once in (a task's real tokens, its rank rounded up to four columns), Gs once out
  double moved = (double)c.st->T * c.RP * 2;
  for (const HostTask& ht : c.st->tasks)
    if (ht.kind == MUX_ADAPTER_LORA || ht.kind == MUX_ADAPTER_TUNING) moved += (double)slabs * ht.valid * round_up(ht.rank, 4) * 4;
  const bool dl = dl_rides_along(c);
  // and what rides along: the IA3 rows of dY and of the saved x W in, their scaled copies and the partial sums out; A_t in, its copy out
  for (const HostTask& ht : c.st->tasks) {
    if (dl && ht.kind == MUX_ADAPTER_IA3_OUT) moved += 6.0 * ht.valid * c.N + 4.0 * c.N * ((ht.row_count + 63) / 64);
    if (rank_is_padded(ht)) moved += 2.0 * (ht.rank + round_up(ht.rank, 8)) * (ht.kind == MUX_ADAPTER_LORA ? c.K : c.N);
  }
  prof_note_bytes(moved);
  const unsigned items = (unsigned)c.st->items[TS64].size(), threads = dl ? 512 : 256;
  const unsigned n_pad = (unsigned)((padded_pieces(c) + threads - 1) / threads), n_dl = dl ? (unsigned)dl_blocks(c.N) : 0;
  auto reduce = [&](auto DL) {
    MUX_LAUNCH("gs_reduce", (k_gs_reduce<decltype(DL)::value>), dim3(items * (1 + n_dl) + (unsigned)c.st->n_tasks * n_pad),
               dim3(threads), 0, c.stream, c.dtab, *c.tref, (const float*)gpart, slabs, c.st->T, c.RP, (const bf16_t*)c.U2,
               (bf16_t*)Gs, c.st->dev_image[DH_NITEMS0 + 3 * TS64 + 1], c.st->dev_image[DH_OFF_ITEM_BITS], (int)items,
               (int)n_dl, (int)n_pad, c.K, dl_params(c, dY, Z, part));
  };
  if (dl) reduce(std::true_type{}); else reduce(std::false_type{});
  return MUX_OK;
}

// Adapter-Tuning: Y = z + Hs U_t (forward) or dYs = dY + Gs D_t^T (backward)
mux_status adapter_tune_add(const CallCtx& c, const void* In, const void* Small, void* Out, int backward) {
  if (c.st->n_tuning == 0) return MUX_OK;
  TuneAddParams p{c.dtab, (const bf16_t*)In, (const bf16_t*)Small, (bf16_t*)Out, c.N, c.RP, backward};
  p.tasks = *c.tref;
  const dim3 grid((unsigned)c.st->items[TS64].size(), (c.N + 255) / 256);
  if (c.RP <= 32) MUX_LAUNCH(backward ? "tune_dz" : "tune_up", (k_tune_add<1>), grid, dim3(256), 0, c.stream, p);
  else MUX_LAUNCH(backward ? "tune_dz" : "tune_up", (k_tune_add<2>), grid, dim3(256), 0, c.stream, p);
  return MUX_OK;
}

// Adapter-Tuning forward, after the backbone GEMM saved z = x W: u = z D_t, Hs = s_t gelu(u).
mux_status adapter_down_tune(const CallCtx& c, const void* Z, void* Hs) {
  if (c.st->n_tuning == 0) return MUX_OK;
  DownParams p{c.dtab, (const bf16_t*)Z, (bf16_t*)Hs, (bf16_t*)c.U2, c.N, c.RP, DOWN_TUNE};
  launch_down(c, "tune_down", p);
  return MUX_OK;
}

// dA_t = X^T Gs (Adapter-Tuning: dD_t = z^T Gs) in partial sums per row group, after adapter_dy_pass: the description of the
// work, for adapter_grad_da or for the launch of the backbone product that takes it along.  n_items = 0: nothing to do.
GradParams adapter_grad_job(const CallCtx& c, const void* X, const void* Gs, const void* Z, void* part, int accumulate) {
  GradParams p{};
  if (c.st->n_lora + c.st->n_tuning == 0) return p;
  const PartLayout pl = part_layout(c.K, c.N, c.st);
  const int K1 = grad_width(c), ts = da_group(c.st, K1);
  p.dtab = c.dtab; p.Gs = (const bf16_t*)Gs; p.X = (const bf16_t*)X; p.Zc = (const bf16_t*)Z;
  p.part = (float*)((char*)part + pl.gpart + pl.part0);
  p.slot = (size_t)c.RP * K1;
  p.K = c.K; p.N = c.N; p.RP = c.RP; p.T = c.st->T;
  p.items_off = c.st->dev_image[DH_NITEMS0 + 3 * ts + 1];
  p.rowbits_off = c.st->dev_image[DH_OFF_ROWBITS];
  p.direct = single_groups(c, s4_group(c.st, c.N), ts) ? 1 : 0;
  p.accumulate = accumulate;
  p.n_items = (int)c.st->items[ts].size();
  p.col_blocks = (K1 + 255) / 256;
  p.pieces = c.st->r_max <= 16 ? 1 : (c.st->r_max <= 32 ? 2 : 4);
  return p;
}

void adapter_grad_da(const CallCtx& c, const GradParams& p) {
  if (p.n_items == 0) return;
  const dim3 grid((unsigned)p.n_items, (unsigned)p.col_blocks);
  // two steps of loads in flight where the registers still allow four waves a SIMD
  auto launch = [&](auto STREAM) {
    constexpr bool S = decltype(STREAM)::value;
    if (p.pieces == 1) MUX_LAUNCH("grad_da", (k_grad<1, 2, S>), grid, dim3(256), 0, c.stream, p, *c.tref);
    else if (p.pieces == 2) MUX_LAUNCH("grad_da", (k_grad<2, 2, S>), grid, dim3(256), 0, c.stream, p, *c.tref);
    else MUX_LAUNCH("grad_da", (k_grad<4, 1, S>), grid, dim3(256), 0, c.stream, p, *c.tref);
  };
  if (past_caches(c, ranked_bytes(c.st, c.K, c.N))) launch(std::true_type{}); else launch(std::false_type{});
}

// IA3_OUT: the partial sums of dl_t and the scaled rows the backbone backward reads.
void adapter_dl(const CallCtx& c, const void* dY, const void* Z, void* part) {
  if (c.st->n_ia3 == 0 || dl_rides_along(c)) return;
  MUX_LAUNCH("grad_dl", k_dl, dim3((unsigned)c.st->items[TS64].size(), (unsigned)dl_blocks(c.N)), dim3(512), 0, c.stream,
             c.dtab, *c.tref, dl_params(c, dY, Z, part));
}

// The partial sums of every gradient brought together, after all of the above.
void adapter_reduce(const CallCtx& c, void* part, int accumulate) {
  const int M = c.st->n_tasks;
  const PartLayout pl = part_layout(c.K, c.N, c.st);
  const int K1 = grad_width(c);
  const int ts_b = s4_group(c.st, c.N), ts_a = da_group(c.st, K1);
  const bool ranked = c.st->n_lora + c.st->n_tuning > 0 && !single_groups(c, ts_b, ts_a);
  float* part0 = (float*)((char*)part + pl.gpart);
  float* part1 = (float*)((char*)part + pl.gpart + pl.part0);
  float* part_ia3 = (float*)((char*)part + pl.gpart + pl.part0 + pl.part1);
  double moved = 0.0;       // what the reduction moves: every row group's partials once in, the gradients once out
  int blocks = 0;           // of the reduction, the most a task has
  if (ranked)
    for (const HostTask& ht : c.st->tasks)
      if (ht.kind == MUX_ADAPTER_LORA || ht.kind == MUX_ADAPTER_TUNING) {
        const int kk = ht.kind == MUX_ADAPTER_TUNING ? c.N : c.K;
        const int nb = (int)(((size_t)ht.rank * c.N + 1023) / 1024) + (kk + reduce_cols(ht.rank) - 1) / reduce_cols(ht.rank);
        if (nb > blocks) blocks = nb;
        const double gb = (ht.row_count + kTileRows[ts_b] - 1) / kTileRows[ts_b], ga = (ht.row_count + kTileRows[ts_a] - 1) / kTileRows[ts_a];
        moved += 4.0 * ht.rank * (gb * c.N + ga * kk) + 4.0 * ht.rank * ((double)c.N + kk) * (accumulate ? 2 : 1);
      }
  if (c.st->n_ia3 > 0) {
    if ((c.N + 1023) / 1024 > blocks) blocks = (c.N + 1023) / 1024;
    for (const HostTask& ht : c.st->tasks)
      if (ht.kind == MUX_ADAPTER_IA3_OUT) moved += 4.0 * c.N * ((ht.row_count + 63) / 64) + 4.0 * c.N * (accumulate ? 2 : 1);
  }
  if (blocks == 0) return;
  // one reduction for every kind: a task's workgroups take the sums its kind has
  ReduceParams p{c.dtab, part0, part1, part_ia3, c.N, c.K, accumulate, ranked ? 1 : 0, {}, {}, (size_t)c.RP * c.N, (size_t)c.RP * K1};
  const int ts[3] = {ts_b, ts_a, TS64};
  for (int i = 0; i < 3; ++i) {
    p.items_off[i] = c.st->dev_image[DH_NITEMS0 + 3 * ts[i] + 1];
    p.task_items_off[i] = c.st->dev_image[DH_NITEMS0 + 3 * ts[i] + 2];
  }
  p.tasks = *c.tref;
  prof_note_bytes(moved);
  MUX_LAUNCH("reduce_grads", k_reduce, dim3(M, (unsigned)blocks), dim3(256), 0, c.stream, p);
}

}  // namespace mux
