// Backbone GEMM, pipelined version: global -> LDS by direct buffer loads (no register staging),
// operand reads software-pipelined one MFMA step ahead.
//
//   forward  (NN):  Y[T,N]  = mask * ( X[T,K] W[K,N]      + Hs[T,r] B_t[r,N] )      Eq. 1 + LoRA + Add
//   backward (NT):  dX[T,K] = mask * ( dY[T,N] W[K,N]^T   + Gs[T,r] A_t[K,r]^T )    Eq. 2 + LoRA
//
// 256x256 output tile per workgroup of eight waves (two per SIMD), 128x64 per wave as 4x2
// v_mfma_f32_32x32x16_bf16.
//   * `buffer_load_dwordx4 ... lds` writes each lane's 16 bytes at LDS base + 16*lane, so a wave
//     instruction fills 1 KB of a stage.  A masked piece gets an out-of-range offset and lands as zeros.
//   * K-tiles are 64 deep: a row of a [rows][64] tile is one whole 128-byte line of X, dY or W.  Measured on this
//     part, the L2 -> LDS path moves half-lines (the 64-byte rows of a 32-deep tile) at half the rate of whole
//     lines, at every level of the hierarchy, and that rate, not the matrix cores, was the limit of a 32-deep
//     version.  Two stages of 64 KB; the loads of tile kt+2 go out right after the barrier that frees the stage of
//     tile kt.  A contraction length that is no multiple of 64 ends in a tile whose 16-byte pieces past the end are
//     parked out of range (zeros land): 1608 x 6424 on 2378 rows took 173 us forward and 282 us backward in a
//     register-staged kernel that masked its loads, 83 and 123 us here (a template flag: the test for the last tile in the
//     loop of launches without one cost them 1 %).
//   * LDS rows cannot be padded under the DMA rule, so 16-byte pieces are XOR-swizzled instead:
//     [rows][64] tiles by row bits, the forward's [64][256] tile of W by k bits.
//   * one workgroup barrier per K-tile, placed before the last MFMA step: by then every read of
//     the current stage is done (it may be refilled) and the next tile has landed (it may be read).
//   * one workgroup per compute unit at a time; the tiles left over after the last full round of workgroups are
//     cut into two 256x128 halves or four 128x128 quarters (four waves, four 32 KB stages) at the end of the
//     same launch, so that they occupy the compute units once more instead of a fraction of them for a whole
//     tile time.
//   * padding costs no products: the tiles are those of row groups with real tokens (a list on the host's side of the
//     table), dealt to the XCDs by their number; a row group with tokens in its first 128 rows only runs as two quarters, and
//     the groups without any are cleared by workgroups at the end of the launch.  32 tasks of about 1024 rows, aligned to
//     1024 (a quarter of the row groups is padding, and fell on the XCDs unevenly), 8192 x 1024 and 1024 x 8192, both
//     directions: 2984 -> 2667 us for the whole pass; 18 k rows aligned to 512, 5120-wide: 6095 -> 5849 us.
// Every stage is its own __shared__ array so that the compiler's wait-count insertion can tell
// the stage being filled from the stage being read.
#include <atomic>
#include <cstdlib>
#include <type_traits>

#include "mux_grad_device.h"

namespace mux {
namespace {

using adapter::bf16x4;
using adapter::bf16x8;
using adapter::lds_read_tr;
using adapter::OOB;
using adapter::u32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((address_space(3))) void* lds_void_ptr;

constexpr int BM = 256;
constexpr int BK = 64;                          // depth of a K-tile
constexpr int TILE_N = 256;                     // width of a tile in the launch's tile index space
// Columns of a row group without tokens that a workgroup clears.  In a launch of a few pieces the clearing must not outlast
// them: 2048 columns, 1 MB a workgroup, did (704 x 2496, two tasks of 88 and 62 tokens aligned to 512, forward 13.0 us so, 12.7
// now).
constexpr int CLEAR_N = 512;
// Bytes of an output, and of it and the activations that it is formed from, beyond which it is written past the caches
constexpr size_t kStreamOut = (size_t)64 << 20, kStreamBoth = (size_t)144 << 20;
constexpr int kStreamDepth = 512;               // contraction up to which the former alone decides

// A workgroup reads these one after the other as it finds out what it computes, from lines of 64 bytes that are cold at the
// start of a launch: what it needs first lies in the first line, what comes next in the second.  (Spread over three lines,
// 4096 x 4096, four tasks of 37 to 129 tokens, forward 40.4 us, so 40.0; 40.2 before there were two kinds of row groups.)
struct GemmParams {
  const int32_t* dtab;
  unsigned long long* clk;  // diagnostic: counters workgroup 0 adds its elapsed cycles and 100 MHz ticks to (null: off)
  int n_full;              // workgroups that compute full tiles (a multiple of 8); the rest compute pieces of tiles
  int tail_split;          // pieces per tile after the full ones: 2 (halves) or 4 (quarters)
  int n_m;                 // row groups with tokens past their first 128 rows
  int n_mh;                // those with tokens in their first 128 rows only
  int half0, clear0;       // first workgroups of the pieces of the latter, and of those that clear the groups without tokens
  int below;               // and, before these, the rows past the first 128 of the n_mh groups
  int n_n;                 // column tiles
  int items_off;           // word offset in dtab of the row groups' list (DH_OFF_GEMM_ITEMS)
  int Kc, Nc, RP;
  int splits;              // pieces of the contraction, each a workgroup of its own (1: none)
  int start_h[9];          // of the tiles of the n_mh groups, the first one of every XCD (start_h[8]: how many there are)
  int quarters;            // of a launch whose contraction is split
  int grad0;               // first workgroup of the gradient dA_t (launches of pieces, backward)
  const bf16_t* Ain;   // [T, Kc]  activations (X or dY)
  const bf16_t* W;     // [K, ldw]
  int64_t ldw;
  const bf16_t* Ext;   // [T, RP]  Hs or Gs
  bf16_t* Out;         // [T, Nc]
  bf16_t* Zsave;       // forward: x W of IA3_OUT rows (may be null)
  bf16_t* HsOut;       // forward with the down-projection in the tile loop: Hs [T, RP] is written here (else null)
  float* Part;             // partial tiles of a split contraction: [splits][quarters][128 * 128] fp32, in accumulator order
  float* PartH;            // and of X A_t with it (forward): [splits][rows of the quarters, 128 each][32] fp32
  const uint32_t* DiffPack; // entries of the Diff-Pruning masks packed for this launch (index << 16 | bf16 value), or null
  const bf16_t* Wdiff;      // merged weights W + M_t * delta_t of the Diff-Pruning tasks, `wdiff_stride` elements apart (or null)
  int64_t wdiff_stride;
  const bf16_t* AinScaled;  // backward: prepared input rows (IA3_OUT: dY * l_t; TUNING: dY + p D_t^T), [z_rows, Kc], indexed like the saved x W
  TaskRef tasks;
};

// Raw buffer descriptor (stride 0) over `bytes` bytes starting at p, as four dwords.
typedef __attribute__((ext_vector_type(4))) int rsrc_t;
__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  const uint64_t a = (uint64_t)p;
  // wave-uniform by construction; said explicitly so that the descriptor always lives in scalar registers
  return (rsrc_t){__builtin_amdgcn_readfirstlane((int)(uint32_t)a), __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32)),
                  __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
}
// One direct-to-LDS load: lane l's 16 bytes from buffer offset byte_off land at lds_dst_uniform + 16*l.
// Written as inline assembly on purpose: the wait counts of these loads are managed by hand (vmcnt) around
// the workgroup barrier, and the compiler must not pair them with the LDS reads of other stages.
__device__ __forceinline__ void dma16(rsrc_t r, bf16_t* lds_dst_uniform, uint32_t byte_off) {
  const uint32_t lds_addr = (uint32_t)(uintptr_t)(lds_void_ptr)lds_dst_uniform;
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(lds_addr), "v"(byte_off), "s"(r)
               : "m0");
}
// The same with 4 bytes a lane: lane l's dword lands at LDS byte address lds_addr + 4*l.
__device__ __forceinline__ void dma4(rsrc_t r, uint32_t lds_addr, uint32_t byte_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
               :
               : "s"(lds_addr), "v"(byte_off), "s"(r)
               : "m0");
}
// s_waitcnt vmcnt(n) only (gfx9 encoding: vmcnt[3:0] | expcnt[6:4] | lgkmcnt[11:8] | vmcnt_hi[15:14])
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  __builtin_amdgcn_s_waitcnt((N & 15) | 0x70 | 0xF00 | ((N >> 4) << 14));
}
__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// Swizzle of the 16-byte piece index inside a 128-byte row of a [rows][64] tile: sixteen consecutive rows read the
// same logical piece with one ds_read_b128 and must land in sixteen different 16-byte bank groups.
__device__ __forceinline__ int swz_row(int r) { return (r >> 1) & 7; }
// Swizzle of the 32-byte segments of a k-row of the forward's [64][BN] tile of W: the four k-rows that sixteen lanes read
// across, two segments wide, must land in 256 different bytes of the banks.  Rows of 128 bytes: two of them do as they lie.
template <int BN>
__device__ __forceinline__ int swz_k(int kk) { return BN >= 128 ? (kk & 3) << 1 : kk & 2; }

// LDS of a workgroup: the stages (see gemm_tile), the per-row validity flags, and with DIFFP, per K-tile, where the entries
// of this tile's buckets begin, split and end.
struct Smem {
  bf16_t* base;
  int* row;
  int* off;
};

// Stages of a piece of 64 MI x 64 NI: as many as the LDS holds, eight at most.
constexpr int kSlabElems = 2048;                  // FUSE: [64][rank <= 32] slab of A_t, 4 KB a stage
constexpr int kPackElems = 512;                   // DIFFP: 256 packed entries of the masks, 1 KB a stage
constexpr int piece_elems(int MI, int NI, bool FUSE, bool DIFFP) {
  return 64 * (MI + NI) * BK + (FUSE ? kSlabElems : 0) + (DIFFP ? kPackElems : 0);
}
constexpr int piece_stages(int MI, int NI, bool FUSE, bool DIFFP) {
  const int room = (160 * 1024 - 1024 - (DIFFP ? 12288 : 0)) / 2, n = room / piece_elems(MI, NI, FUSE, DIFFP);
  return n < 8 ? n : 8;
}

// Number of the tile in slot `j` of an XCD, of `total` tiles; -1: the XCD has no such slot.  An XCD takes a contiguous
// range of the tiles, and the first `total % 8` XCDs one tile more than the others.
__device__ __forceinline__ int tile_of_slot(int total, int xcd, int j) {
  const int q = total >> 3, r = total & 7;
  return j < q + (xcd < r ? 1 : 0) ? xcd * q + (xcd < r ? xcd : r) + j : -1;
}

// Row group tm and column tile tn of tile L: groups of four row groups, the row group running fastest.
__device__ __forceinline__ void tile_at(int n_m, int n_n, int L, int& tm, int& tn) {
  constexpr int GROUP = 4;
  const int width = GROUP * n_n;
  const int first_m = (L / width) * GROUP;
  const int gsize = n_m - first_m < GROUP ? n_m - first_m : GROUP;
  tm = first_m + (L % width) % gsize;
  tn = (L % width) / gsize;
}

// Zeros on the rows past the first 128 of a row group that has tokens in those only (256 threads): 128 columns of
// the output, and with the first of them the rows of Hs.
__device__ __forceinline__ void clear_below(const GemmParams& p, int row0, int nrows, int c0) {
  if (nrows <= 128) return;
  const int tid = threadIdx.x & 255, c = c0 + (tid & 15) * 8;
  if (c < p.Nc)
    for (int m = 128 + (tid >> 4); m < nrows; m += 16) *(uint4*)(p.Out + (size_t)(row0 + m) * p.Nc + c) = make_uint4(0, 0, 0, 0);
  if (c0 == 0 && p.HsOut != nullptr)
    for (int e = tid; e < (nrows - 128) * (p.RP / 8); e += 256)
      *(uint4*)(p.HsOut + (size_t)(row0 + 128 + e / (p.RP / 8)) * p.RP + (e % (p.RP / 8)) * 8) = make_uint4(0, 0, 0, 0);
}

// Quarter q of a split launch: true: of a row group with tokens in its first 128 rows only.
__device__ __forceinline__ bool quarter_of(const GemmParams& p, int q, int& L, int& half, int& mhalf) {
  const int q0 = 4 * p.n_m * p.n_n;
  const bool hg = q >= q0;
  half = q & 1;
  mhalf = hg ? 0 : (q >> 1) & 1;
  L = hg ? (q - q0) >> 1 : q >> 2;
  return hg;
}

// One output tile.  WNW = waves along N, MI x NI = 32x32 MFMA tiles per wave; 2*WNW waves on a
// BMT x BN tile with BMT = 2*MI*32 and BN = WNW*NI*32:
//   <4,4,2> eight waves (two per SIMD), 128x64 per wave, the full 256x256 tile;
//   <4,4,1> eight waves, 128x32 per wave, a 256x128 half of a tile beside full ones;
//   <2,2,2> and <2,4,2> four waves (one per SIMD), 64x64 or 128x64 per wave: a 128x128 quarter beside full tiles, a half in
//           a launch without them;
//   <1,MI,NI> four waves, a piece of 64 MI x 64 NI in a launch without full tiles: each wave forms the whole piece from a
//           quarter of the contraction, one of the four MFMA steps of every K-tile, and the four sums are added at the end.
// L = number of the tile among those of the `n_m` row groups from `item0` on; `half` selects the 128 columns of a
// half-width tile, `mhalf` the 128 rows of a quarter.  MI = 1: the list holds groups of 64 rows, L is the group and `half`
// the column piece.
// FUSE (forward, pieces): the down-projection Hs = s_t X A_t of the tile's rows is
// computed in the same K loop -- the [64][rank] slab of A_t of every K-tile is staged beside the tile of W, the two waves
// of a row half multiply it with the X fragments of half of its row blocks each (MI = 1: each wave its step) -- and goes, scaled and
// rounded to bf16, straight into the A side of the adapter K-tile (and, from the tiles of the first column, to
// memory for the backward): no separate pass over X, no launch for it.  Every column tile redoes the product for
// its rows, which is why this is for launches that do not fill the compute units anyway.
// DIFFP: the rows of a Diff-Pruning task meet W + M_t * delta_t without a copy of W: once a tile of W
// has landed in LDS, the masked entries that fall into it are added in place (one bf16 read-modify-write each) and a
// second barrier follows before the tile is read.  The mask lists its entries by tiles -- buckets of 64 of the
// contraction index by 128 lines of the W side, numbered so that the one or two buckets of a tile are neighbours --
// and the launch brings them packed, (contraction index % 64) << 23 | (line % 128) << 16 | bf16 value.  The entries
// of a K-tile travel with it: every loading wave fetches 64 of them straight into LDS with the tile's other loads
// (256 a tile; a bucket pair with more reads the rest from memory when the tile is patched).
// SPLITK (quarters): the tile's `split`-th share of its K-tiles only; the accumulators go to p.Part as they lie in the
// registers (slot: the quarter's number), for k_gemm_sum.
// STREAM: the output is written past the caches.
template <bool NT, int WAVES_N, int MI, int NI, bool FUSE = false, bool DIFFP = false, bool TAIL = false, bool SPLITK = false,
          bool STREAM = false>
__device__ __forceinline__ void gemm_tile(const GemmParams& p, const int item0, const int n_m, const int L,
                                          const int half, const int mhalf, const Smem sm, const int split = 0,
                                          const int slot = 0, const bool clear = false) {
  static_assert(!SPLITK || (!DIFFP && MI == 2 && NI == 2), "SPLITK: quarters, the plain loop");
  static_assert(WAVES_N == 4 || WAVES_N == 2 || WAVES_N == 1, "eight waves or four");
  static_assert(!FUSE || (!NT && WAVES_N <= 2), "FUSE: forward, pieces");
  constexpr bool KS = WAVES_N == 1;               // the waves share out the contraction in the loop, the tile after it
  constexpr int WNW = KS ? 2 : WAVES_N;
  static_assert(!DIFFP || !KS, "DIFFP: tiles and their halves and quarters");
  static_assert(!DIFFP || !FUSE, "DIFFP: not with FUSE");
  constexpr int BN = WNW * NI * 32;
  constexpr int BMT = 2 * MI * 32;
  constexpr bool PIECE = WNW == 2, ROW64 = MI == 1;
  static_assert(KS == ROW64, "row groups of 64: one wave a step");
  // LDS stages.  A stage of a full or half tile takes 64 or 48 KB: two of 64 KB fit.  A piece's takes less and has less
  // MFMA time, which is below the latency of the loads: as many stages as there is room for, so many tiles less one in flight.
  constexpr int NST = PIECE ? piece_stages(MI, NI, FUSE, DIFFP) : 2;
  constexpr int NW = 2 * WNW, NTHR = 64 * NW;
  constexpr int A_ELEMS = BMT * BK;               // elements of one A stage
  // The loads are issued by the first half of the waves only.  Each SIMD hosts waves w and w + NW/2 and serves the
  // older one first, so wave w runs ahead and then idles at the barrier; a wave that cannot issue a load (the
  // vector memory pipeline takes 16 cycles per instruction, 1 KB) cannot issue the MFMA behind it either.
  // Giving wave w all the loads uses its slack and leaves wave w + NW/2 a pure MFMA / LDS-read stream.
  constexpr int LW = NW == 8 ? NW / 2 : NW;       // four waves: one per SIMD, all of them load
  constexpr int ACH = (A_ELEMS / 512) / LW, BCH = (BN * BK / 512) / LW;   // 1 KB chunks a loading wave fetches per K-tile
  constexpr int ECH = FUSE ? 1 : 0;               // FUSE: and one of the (up to) 4 KB of the slab of A_t
  constexpr int DCH = DIFFP ? 1 : 0;              // DIFFP: and 64 packed entries of the mask
  constexpr int NLD = ACH + BCH + ECH + DCH;      // loads a loading wave issues per K-tile
  static_assert(ACH >= 1 && BCH >= 1, "every loading wave fetches at least one chunk of each tile");
  static_assert(!FUSE || LW == 4, "FUSE: four loading waves bring the four chunks of a slab");
  constexpr int LPR = BK / 8;                     // [rows][BK] tiles: lanes (16-byte pieces) per row
  constexpr int RPC = 64 / LPR;                   //                   rows per 1 KB chunk
  constexpr int PPRB = BN / 8;                    // forward: 16-byte pieces per k-row of the [BK][BN] tile
  constexpr int RPCB = 64 / PPRB;                 // forward: k-rows per 1 KB chunk
  constexpr int WCOLS = NI * 32;                  // columns of the wave tile
  constexpr int EPW = WCOLS + 8;                  // epilogue staging pitch (elements)
  constexpr int STAGE = PIECE ? piece_elems(MI, NI, FUSE, DIFFP) : 2 * BM * BK;      // elements
  int* const sRow = sm.row;

  int tm, tn;
  if (ROW64) { tm = L; tn = half; } else tile_at(n_m, p.n_n, L, tm, tn);
  const int4 iw = *(const int4*)(p.dtab + p.items_off + (item0 + tm) * DI_WORDS);
  const ItemView it = {iw.x, iw.y, iw.z, iw.w};   // (nvalid: rows up to the last real token)
  const int mrow0 = mhalf * BMT;                  // first row of the item this tile covers
  const int nrows = it.nrows - mrow0 < BMT ? it.nrows - mrow0 : BMT;   // rows of the item inside this tile
  const int row0 = it.row0 + mrow0;
  const int c0 = ROW64 ? tn * BN : tn * TILE_N + half * BN;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (wave >= NW) return;                         // a piece beside full tiles: the other waves end here, before any barrier
  const int wm = wave / WNW, wn = wave % WNW;
  const bool loader = wave < LW;
  const int lw = wave % LW;                       // chunk owner index (meaningful for loading waves)

  if (tid < BMT) sRow[tid] = (tid < nrows && row_is_valid(p.dtab, row0 + tid)) ? 1 : 0;

  // Rows of the tile up to its last token: at least one.  A group with tokens past its first 128 rows has some in each of
  // its pieces, one without them runs its upper pieces only, and a group without any token makes no tile.
  const int nlive = it.nvalid - mrow0 < nrows ? it.nvalid - mrow0 : nrows;

  const DevTask tk = get_task(p.tasks, it.task);
  const bool lora = tk.kind == MUX_ADAPTER_LORA;
  const bool ia3 = tk.kind == MUX_ADAPTER_IA3_OUT;
  const bool tuning = tk.kind == MUX_ADAPTER_TUNING;   // forward: only x W is produced here (saved); backward: prepared rows
  const int rank = lora ? tk.rank : 0;
  const bf16_t* adapterB = NT ? (const bf16_t*)tk.A : (const bf16_t*)tk.B;
  const bf16_t* Lvec = (const bf16_t*)tk.L;

  const int KT = (p.Kc + BK - 1) / BK;
  const int k_tail = p.Kc - (KT - 1) * BK;          // TAIL: contraction indices in the last backbone tile (a multiple of 8)
  const int KT_ext = lora && !(FUSE && SPLITK) ? (rank + BK - 1) / BK : 0;
  // this tile forms Hs of its rows in the K loop (SPLITK: only those of the first column, whose share k_gemm_sum adds up)
  const bool fuse_h = FUSE && lora && (!SPLITK || c0 == 0);
  const int KT_total = KT + KT_ext;
  const int kt_first = SPLITK ? (int)((unsigned)(split * KT_total) / (unsigned)p.splits) : 0;
  const int kt_end = SPLITK ? (int)((unsigned)((split + 1) * KT_total) / (unsigned)p.splits) : KT_total;
  // DIFFP: the bucket offsets of this task's listing for this direction, the buckets of this tile in a K-tile's row
  // of buckets, and per stage the entries of the tile it holds: first, first of the second bucket, end
  const bool patch = DIFFP && tk.kind == MUX_ADAPTER_DIFF && tk.rank >= 0 && p.DiffPack != nullptr && c0 < p.Nc;
  static_assert(!DIFFP || BN >= 128, "DIFFP: whole buckets");
  constexpr int SPAN = BN >= 128 ? BN / 128 : 1;
  const int32_t* bptr = (const int32_t*)tk.dB;
  const int nbk = (p.Nc + 127) >> 7, bcol = c0 >> 7;
  const int bspan = bcol + SPAN <= nbk ? SPAN : nbk - bcol;      // a ragged last tile may hold one bucket only
  const uint32_t* dlist = p.DiffPack + (patch ? tk.rank : 0);
  const rsrc_t rPk = make_rsrc(patch ? (const void*)dlist : (const void*)p.Ain, patch ? (uint32_t)tk.at_off * 4u : 0u);
  int ps0[NST], ps1[NST], ps2[NST];
#pragma unroll
  for (int q = 0; q < NST; ++q) { ps0[q] = 0; ps1[q] = 0; ps2[q] = 0; }
  int nx0 = 0, nx1 = 0, nx2 = 0;                   // the same for the tile after the ones in flight
  // The offsets of every K-tile's entries go to LDS once (a load from the listing inside the loop would have the loop
  // wait for it, and for the tiles in flight with it, at every K-tile).
  if (DIFFP && patch) {
    for (int t = tid; t < KT; t += NTHR) {
      const int32_t* q = bptr + (size_t)t * nbk + bcol;
      sm.off[3 * t] = q[0];
      sm.off[3 * t + 1] = q[1];
      sm.off[3 * t + 2] = q[bspan];
    }
    __syncthreads();
  }
  // offsets of the entries of K-tile t (none past the backbone tiles, none without a mask)
  auto bucket_offsets = [&](int t, int& o0, int& o1, int& o2) {
    o0 = 0; o1 = 0; o2 = 0;
    if (DIFFP && patch && t < KT) {
      o0 = __builtin_amdgcn_readfirstlane(sm.off[3 * t]);
      o1 = __builtin_amdgcn_readfirstlane(sm.off[3 * t + 1]);
      o2 = __builtin_amdgcn_readfirstlane(sm.off[3 * t + 2]);
    }
  };

  // ---- DMA geometry.  A wave instruction fills 1 KB: RPC rows x 2 BK bytes of a [rows][BK] tile
  // (lane -> row lane/LPR, physical piece lane%LPR), or RPCB k-rows of the forward's [BK][BN] tile of W
  // (lane -> k-row lane/PPRB, physical piece lane%PPRB).  Loading wave w owns chunks w*ACH .. of A and w*BCH .. of B.
  const int r_in = lane / LPR;                                  // row inside the chunk
  const uint32_t a_rows_bytes = (uint32_t)nlive * (uint32_t)p.Kc * 2u;     // (rows past the last token are not fetched)
  const bf16_t* a_base = (NT && (ia3 || tuning)) ? p.AinScaled + (size_t)(tk.zrow0 + row0 - tk.row_begin) * p.Kc
                                     : p.Ain + (size_t)row0 * p.Kc;
  const rsrc_t rA = make_rsrc(a_base, a_rows_bytes);
  const rsrc_t rW = make_rsrc(task_weight(tk, p.W, p.Wdiff, p.wdiff_stride), (uint32_t)((size_t)(NT ? p.Nc : p.Kc) * p.ldw * 2));
  const rsrc_t rE = make_rsrc(lora ? p.Ext + (size_t)row0 * p.RP : p.Ain, lora ? (uint32_t)nrows * (uint32_t)p.RP * 2u : 0u);
  const int a_pitch = 8 * rank_pieces(rank);         // elements in a row of A_t
  const rsrc_t rP = make_rsrc(lora ? adapterB : p.Ain, lora ? (uint32_t)(NT ? (size_t)p.Nc * a_pitch : (size_t)rank * p.Nc) * 2u : 0u);

  // FUSE: A_t [K][a_pitch]; the slab of K-tile kt is the 128 a_pitch bytes from byte kt * 128 a_pitch on, loading wave
  // w brings its w-th KB (lane l the 16 bytes at 1024 w + 16 l), so the slab lies in LDS as in memory, [64][a_pitch]
  const rsrc_t rAt = make_rsrc(fuse_h ? tk.A : (const void*)p.Ain, fuse_h ? (uint32_t)p.Kc * (uint32_t)a_pitch * 2u : 0u);
  const uint32_t offE = (fuse_h && (uint32_t)(lw * 1024 + lane * 16) < 128u * (uint32_t)a_pitch) ? (uint32_t)(lw * 1024 + lane * 16) : OOB;
  const uint32_t stepE = 128u * (uint32_t)a_pitch;
  uint32_t kE = (uint32_t)kt_first * stepE;

  // row of the [rows][BK] tile chunk q of this wave puts this lane on, and the logical k-piece it fetches there
  auto a_row_of = [&](int q) { return lw * (RPC * ACH) + RPC * q + r_in; };
  auto b_row_of = [&](int q) { return lw * (RPC * BCH) + RPC * q + r_in; };   // backward: row of W inside the tile
  auto piece_of = [&](int row) { return (lane % LPR) ^ swz_row(row); };
  // forward W tile: k-row = (lw*BCH + q)*RPCB + lane/PPRB, physical piece lane%PPRB -> logical n
  const int nk_in = lane / PPRB;
  const int n_pp = lane % PPRB;

  // Per-thread byte offsets of the pieces this lane fetches per tile, without the K-tile term.
  // A piece that must read as zero is parked out of range.
  uint32_t offA[ACH], offB[BCH];
#pragma unroll
  for (int q = 0; q < ACH; ++q)
    offA[q] = ((uint32_t)a_row_of(q) * (uint32_t)p.Kc + (uint32_t)(piece_of(a_row_of(q)) * 8)) * 2u;
#pragma unroll
  for (int q = 0; q < BCH; ++q) {
    if (NT) {
      offB[q] = (uint32_t)(((size_t)(c0 + b_row_of(q)) * p.ldw + piece_of(b_row_of(q)) * 8) * 2);
    } else {
      const int kk = (lw * BCH + q) * RPCB + nk_in;          // k-row inside the tile
      const int seg = (n_pp >> 1) ^ swz_k<BN>(kk);           // logical 32-byte segment
      const int n = seg * 16 + (n_pp & 1) * 8;
      offB[q] = (c0 + n < p.Nc) ? (uint32_t)(((size_t)kk * p.ldw + c0 + n) * 2) : OOB;
    }
  }
  // K-tile term: advances by one tile per issue (scalar).  After the last backbone tile the sources switch
  // to the adapter operands (Ext rows and B_t / A_t), whose offsets restart from zero; past the last tile
  // everything is parked out of range (zeros land in a stage nobody reads).
  rsrc_t curA = rA, curB = rW;
  uint32_t stepA = BK * 2u, stepB = NT ? BK * 2u : (uint32_t)((size_t)BK * p.ldw * 2);
  uint32_t kA = (uint32_t)kt_first * stepA, kB = (uint32_t)kt_first * stepB;
  int next_tile = kt_first;                                          // index of the tile the next issue() fetches

  // uniform, rarely taken: everything that changes at a tile-kind boundary
  const int odd_tile = TAIL ? KT - 1 : KT;                    // the first tile that is not like the ones before it
  const int special = SPLITK && kt_end < odd_tile ? kt_end : odd_tile;
  auto prepare = [&]() {
    if (next_tile < special) return;
    if (PIECE && next_tile >= kt_end) {
      curA[2] = 0; curB[2] = 0;                               // past the end, or the next share's: zeros, whatever the offset
      if (FUSE) kE = OOB;
    } else if (TAIL && next_tile == KT - 1) {                                // the last backbone tile is not full: pieces past the end
#pragma unroll
      for (int q = 0; q < ACH; ++q)
        if (piece_of(a_row_of(q)) * 8 >= k_tail) offA[q] = OOB;
      if (NT) {                                               // (the forward's rows of W past the end lie behind its buffer)
#pragma unroll
        for (int q = 0; q < BCH; ++q)
          if (piece_of(b_row_of(q)) * 8 >= k_tail) offB[q] = OOB;
      }
    } else {
      if (FUSE) kE = OOB;                                     // no slab of A_t past the backbone tiles
      if (next_tile >= KT_total) {
        kA = OOB; kB = OOB;
      } else {
        const int j0 = (next_tile - KT) * BK;        // first contraction index of this adapter tile
        curB = rP; kB = 0; stepA = 0; stepB = 0;
        if (FUSE) {
          curA[2] = 0;                                        // the A side of the adapter tile comes from the accumulators
        } else {
          curA = rE; kA = 0;
#pragma unroll
          for (int q = 0; q < ACH; ++q) {
            const int j = j0 + piece_of(a_row_of(q)) * 8;
            offA[q] = (j < p.RP) ? ((uint32_t)a_row_of(q) * (uint32_t)p.RP + (uint32_t)j) * 2u : OOB;
          }
        }
#pragma unroll
        for (int q = 0; q < BCH; ++q) {
          if (NT) {
            const int c = c0 + b_row_of(q);
            const int j = j0 + piece_of(b_row_of(q)) * 8;
            offB[q] = (c < p.Nc && j < a_pitch) ? (uint32_t)(((size_t)c * a_pitch + j) * 2) : OOB;
          } else {
            const int kk = (lw * BCH + q) * RPCB + nk_in;
            const int seg = (n_pp >> 1) ^ swz_k<BN>(kk);
            const int n = seg * 16 + (n_pp & 1) * 8;
            offB[q] = (c0 + n < p.Nc && j0 + kk < rank) ? (uint32_t)(((size_t)(j0 + kk) * p.Nc + c0 + n) * 2) : OOB;
          }
        }
      }
    }
  };
  // one load of the tile being fetched: i = 0 .. NLD-1, the A pieces first, then W, then (FUSE) the slab of A_t
  // (DIFFP: the last load brings entries o0 + 64 lw .. of the tile's buckets, below o2, into the stage's entry slots)
  auto issue_one = [&](bf16_t* dA, bf16_t* dB, bf16_t* dE, int i, uint32_t dP = 0, int o0 = 0, int o2 = 0) {
    if (!loader) return;
    if (i < ACH) dma16(curA, dA + (lw * ACH + i) * 512, offA[i] + kA);
    else if (i < ACH + BCH) dma16(curB, dB + (lw * BCH + (i - ACH)) * 512, offB[i - ACH] + kB);
    else if (DIFFP) dma4(rPk, dP + lw * 256, (o0 + lw * 64 + lane < o2) ? (uint32_t)(o0 + lw * 64 + lane) * 4u : OOB);
    else dma16(rAt, dE + lw * 512, (offE == OOB || kE == OOB) ? OOB : offE + kE);
  };
  auto issue_done = [&]() { kA += stepA; kB += stepB; if (FUSE && kE != OOB) kE += stepE; ++next_tile; };
  auto issue = [&](bf16_t* dA, bf16_t* dB, bf16_t* dE, uint32_t dP = 0, int o0 = 0, int o2 = 0) {
#pragma unroll
    for (int i = 0; i < NLD; ++i) issue_one(dA, dB, dE, i, dP, o0, o2);
    issue_done();
  };

  // ---- operand read geometry
  const int li = lane & 31, lg = lane >> 5;
  const int l16 = lane & 15, lhalf = (lane >> 4) & 1;
  // [rows][BK] tiles: row = (wm|wn)*128 + t*32 + li; logical piece 2*ks + lg (the swizzle depends on li only)
  const int swz = swz_row(li);
  const int a_rd = (wm * (32 * MI) + li) * BK;  // elements; + t*32*BK + ((2ks+lg)^swz)*8
  const int bt_rd = (wn * WCOLS + li) * BK;
  // forward W tile: k = ks*16 + 8 lg + 4 h + l16/4 ; logical seg = wn*8 + 2 t + lhalf ; + 4*(l16%4) elements
  const int kq = l16 >> 2;                      // k & 3 of the rows this lane addresses
  const int bn_col = 4 * (l16 & 3);

  auto read_ops = [&](const bf16_t* cA, const bf16_t* cB, int ks, bf16x8 (&a)[MI], bf16x8 (&b)[NI]) {
    const int pa = ((2 * ks + lg) ^ swz) * 8;
#pragma unroll
    for (int t = 0; t < MI; ++t) a[t] = *(const bf16x8*)(cA + a_rd + t * 32 * BK + pa);
    if (NT) {
#pragma unroll
      for (int t = 0; t < NI; ++t) b[t] = *(const bf16x8*)(cB + bt_rd + t * 32 * BK + pa);
    } else {
      const int krow = ks * 16 + 8 * lg + kq;
#pragma unroll
      for (int t = 0; t < NI; ++t) {
        const int seg = (wn * (2 * NI) + 2 * t + lhalf) ^ swz_k<BN>(kq);
        const bf16x4 lo = lds_read_tr(cB + krow * BN + seg * 16 + bn_col);
        const bf16x4 hi = lds_read_tr(cB + (krow + 4) * BN + seg * 16 + bn_col);
        b[t] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    }
  };

  // KS: step `wave` of a K-tile, all 2 MI + 2 NI fragments of the tile
  auto read_step = [&](const bf16_t* cA, const bf16_t* cB, int r, bf16x8 (&a)[2 * MI], bf16x8 (&b)[2 * NI]) {
    const int pa = ((2 * wave + lg) ^ swz) * 8;
    if (r < 2 * NI) {
      if (NT) {
        b[r] = *(const bf16x8*)(cB + (r * 32 + li) * BK + pa);
      } else {
        const int krow = wave * 16 + 8 * lg + kq;
        const int seg = (2 * r + lhalf) ^ swz_k<BN>(kq);
        const bf16x4 lo = lds_read_tr(cB + krow * BN + seg * 16 + bn_col);
        const bf16x4 hi = lds_read_tr(cB + (krow + 4) * BN + seg * 16 + bn_col);
        b[r] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    } else {
      a[r - 2 * NI] = *(const bf16x8*)(cA + ((r - 2 * NI) * 32 + li) * BK + pa);
    }
  };

  // Accumulators.  The MFMAs are issued with the operands exchanged, so acc[mi][ni] holds the transposed 32x32
  // block: this lane has row 32 mi + li and the four consecutive columns 32 ni + 8 j + 4 lg .. + 3 in registers
  // 4j .. 4j+3, which the epilogue packs into one 8-byte LDS store.
  f32x16 acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mi][ni][v] = 0.f;

  auto mma = [&](const bf16x8 (&a)[MI], const bf16x8 (&b)[NI]) {
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[ni], a[mi], acc[mi][ni], 0, 0, 0);
  };

  auto mma_one = [&](const bf16x8 (&a)[MI], const bf16x8 (&b)[NI], int m) {
    const int mi = m / NI, ni = m % NI;
    acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[ni], a[mi], acc[mi][ni], 0, 0, 0);
  };
  // One operand fragment of step ks: r = 0, 1 .. in the order the next step's MFMAs first need them
  // (A0, B0 .. B(NI-1), A1 .. A(MI-1)).
  auto read_one = [&](const bf16_t* cA, const bf16_t* cB, int ks, int r, bf16x8 (&a)[MI], bf16x8 (&b)[NI]) {
    const int pa = ((2 * ks + lg) ^ swz) * 8;
    if (r == 0 || r > NI) {
      const int t = r == 0 ? 0 : r - NI;
      a[t] = *(const bf16x8*)(cA + a_rd + t * 32 * BK + pa);
    } else {
      const int t = r - 1;
      if (NT) {
        b[t] = *(const bf16x8*)(cB + bt_rd + t * 32 * BK + pa);
      } else {
        const int krow = ks * 16 + 8 * lg + kq;
        const int seg = (wn * (2 * NI) + 2 * t + lhalf) ^ swz_k<BN>(kq);
        const bf16x4 lo = lds_read_tr(cB + krow * BN + seg * 16 + bn_col);
        const bf16x4 hi = lds_read_tr(cB + (krow + 4) * BN + seg * 16 + bn_col);
        b[t] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
      }
    }
  };
  // FUSE: the accumulators of this wave's 32 x 32 blocks of X A_t (row blocks HB wn .. of the wave's rows, transposed like
  // acc), and the fragment of the slab of A_t for step ks (lane (li, lg): column li of the slab, 8 consecutive k).
  constexpr int HB = MI / 2 > 0 ? MI / 2 : 1;
  f32x16 hacc[HB];
#pragma unroll
  for (int i = 0; i < HB; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) hacc[i][v] = 0.f;
  auto read_e = [&](const bf16_t* cE, int ks) -> bf16x8 {
    const int krow = ks * 16 + 8 * lg + kq;
    const bf16x4 lo = lds_read_tr(cE + krow * a_pitch + lhalf * 16 + bn_col);
    const bf16x4 hi = lds_read_tr(cE + (krow + 4) * a_pitch + lhalf * 16 + bn_col);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  // the products of this step's slab fragment with the X fragments of this wave's row blocks, picked by selects on the
  // (uniform) wn: an index would send the fragments through scratch memory, and a branch per row block makes the compiler
  // copy the accumulator behind each MFMA
  auto mma_h = [&](const bf16x8& e, const bf16x8 (&a)[MI]) {
#pragma unroll
    for (int i = 0; i < HB; ++i) {
      u32x4 x = __builtin_bit_cast(u32x4, a[i]);
      if (MI > 1) {
        const u32x4 y = __builtin_bit_cast(u32x4, a[MI > 1 ? HB + i : 0]);
#pragma unroll
        for (int c = 0; c < 4; ++c) x[c] = wn == 1 ? y[c] : x[c];
      }
      hacc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(e, __builtin_bit_cast(bf16x8, x), hacc[i], 0, 0, 0);
    }
  };
  // One MFMA step from (a, b) with the operand reads of step ks_next of (cA, cB) into (an, bn) issued one per
  // MFMA in its shadow, and, when LOADS, the loads of one tile into (dA, dB) spread over the MFMAs after them.
  auto fused_step = [&](const bf16x8 (&a)[MI], const bf16x8 (&b)[NI], const bf16_t* cA, const bf16_t* cB, int ks_next,
                        bf16x8 (&an)[MI], bf16x8 (&bn)[NI], auto LOADS, bf16_t* dA, bf16_t* dB, uint32_t dP = 0,
                        int o0 = 0, int o2 = 0) {
    constexpr bool loads = decltype(LOADS)::value;
    constexpr int NM = MI * NI, NR = MI + NI, NL = NLD;
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      mma_one(a, b, m);
      if (m < NR) read_one(cA, cB, ks_next, m, an, bn);
      if (m == NM - 1) {                                     // a narrower tile has more fragments than MFMAs
#pragma unroll
        for (int r = NM; r < NR; ++r) read_one(cA, cB, ks_next, r, an, bn);
      }
      if (loads) {
#pragma unroll
        for (int d = (m * NL) / NM; d < ((m + 1) * NL) / NM; ++d) issue_one(dA, dB, nullptr, d, dP, o0, o2);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  auto stA = [&](int st) -> bf16_t* { return sm.base + st * STAGE; };
  auto stB = [&](int st) -> bf16_t* { return sm.base + st * STAGE + (PIECE ? A_ELEMS : BM * BK); };
  auto stE = [&](int st) -> bf16_t* { return sm.base + st * STAGE + A_ELEMS + BN * BK; };
  auto tile_barrier = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // DIFFP: LDS byte address of a stage's packed entries (eight waves: behind the two stages)
  auto ldsP = [&](int st) -> uint32_t {
    return (uint32_t)(uintptr_t)(lds_void_ptr)(PIECE ? sm.base + st * STAGE + A_ELEMS + BN * BK : sm.base + 2 * STAGE + st * kPackElems);
  };
  typedef __attribute__((address_space(3))) uint32_t lds_u32;
  // DIFFP: the entries o0 .. o2 - 1 of a tile (o1: the first of its second bucket), the first 256 of them in cP, added to
  // the W side of the tile in stage cB (landed, visible to the workgroup)
  auto patch_tile = [&](bf16_t* cB, uint32_t cP, int o0, int o1, int o2) {
    auto add_entry = [&](uint32_t w, int pos) {
      const int j = (int)(w >> 23), line = (int)((w >> 16) & 127u) + ((SPAN == 2 && o0 + pos >= o1) ? 128 : 0);
      bf16_t* e = NT ? cB + line * BK + (((j >> 3) ^ swz_row(line)) * 8) + (j & 7)
                     : cB + j * BN + (((line >> 4) ^ swz_k<BN>(j)) * 16) + (line & 15);
      // (the packed bf16 add of the LDS atomic unit in place of this read-modify-write was 5 % slower)
      *e = f32_to_bf16(bf16_to_f32(*e) + __uint_as_float(w << 16));
    };
    static_assert(NTHR >= 256, "one entry a thread covers what was staged");
    if (tid < o2 - o0 && tid < 256) add_entry(*(const lds_u32*)(uintptr_t)(cP + 4u * (uint32_t)tid), tid);   // (an LDS address, said as such)
    // a bucket pair with more entries than were staged: the rest from memory, in a loop of its own so that the usual case
    // holds no memory load whose wait would also wait for the tiles in flight
    if (o2 - o0 > 256)
      for (int pos = 256 + tid; pos < o2 - o0; pos += NTHR) add_entry(dlist[o0 + pos], pos);
  };
  // ---- prologue: tiles 0 .. PRE-1 in flight; tile 0 landed and visible; its first operands in registers
  constexpr int PRE = NST;
#pragma unroll
  for (int s0 = 0; s0 < PRE; ++s0) {
    prepare();
    if (DIFFP) bucket_offsets(s0, ps0[s0], ps1[s0], ps2[s0]);
    issue(stA(s0), stB(s0), stE(s0), ldsP(s0), ps0[s0], ps2[s0]);
  }
  if (DIFFP) bucket_offsets(PRE, nx0, nx1, nx2);
  // (here, its stores wait for nothing and, younger than the loads, nothing waits for them: before the loads or behind the tile
  // they cost a launch of short contractions 2 us of 11, 448 x 10496 with three tasks)
  // (its group's rows are known here: looked up once more, the call took 0.3 us of 11 also where there was nothing to clear)
  if (clear) clear_below(p, row0, it.nrows, c0);
  wait_vmcnt<(PRE - 1) * NLD>();
  wait_lgkm0();
  tile_barrier();
  if (DIFFP && patch && ps2[0] > ps0[0]) {
    patch_tile(stB(0), ldsP(0), ps0[0], ps1[0], ps2[0]);
    wait_lgkm0();
    tile_barrier();
  }

  // FUSE: the K loop ends with the backbone; the adapter tile (its B_t side is fetched like any tile) follows below
  // The loops of pieces take two K-tiles a turn.  The last of an odd number follows the loop, as products alone: a way out in the
  // middle of a turn made the compiler copy all accumulators at every turn, and a K-tile of zeros in its place took as long as any
  // (448 x 10496, three tasks of 95, 92 and 29 tokens, forward 12.3 us so, 11.3 now; 832 x 4096, the same, 12.0 and 10.9).
  const int KT_loop = fuse_h && !SPLITK ? KT : kt_end - kt_first;

  if constexpr (KS) {
    // Each wave takes one of the four MFMA steps of every K-tile: every operand is read from LDS once (waves that each own a
    // quarter of the piece read all of them twice, and FUSE's slab four times), and the four sums meet in LDS once, at the end.
    // All operands are read one K-tile ahead (there is one wave a SIMD: nothing hides an LDS read but the wave's own
    // products); one barrier a K-tile, at its start: by then every wave has read this tile into registers (its stage may be
    // refilled) and the next one has landed.
    // Bound by the direct-to-LDS loads, about 24 cycles for each 1 KB instruction of a compute unit, whatever their depth
    // (a stage less changes nothing) and place in the loop: 0.27 us a K-tile of 64 x 128 (the loads alone 0.27, the rest
    // 0.15), 0.175 of 64 x 64 (0.165 and 0.10), 0.335 of 128 x 128.
    constexpr int NSLOT = 4 * MI * NI, RT = 2 * (MI + NI), HW = 2 * MI;
    f32x16 accf[2 * MI][2 * NI], haccf[FUSE ? HW : 1];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
#pragma unroll
      for (int t = 0; t < 2 * MI; ++t)
#pragma unroll
        for (int q = 0; q < 2 * NI; ++q) accf[t][q][v] = 0.f;
#pragma unroll
      for (int t = 0; t < (FUSE ? HW : 1); ++t) haccf[t][v] = 0.f;
    }
    bf16x8 ra[2][2 * MI], rb[2][2 * NI], re[2] = {};
#pragma unroll
    for (int r = 0; r < RT; ++r) read_step(stA(0), stB(0), r, ra[0], rb[0]);
    if (FUSE) re[0] = read_e(stE(0), wave);            // (a tile that forms no Hs multiplies zeros: no branch in the loop)
    int su = 0;                                      // stage of tile kt
    prepare();
    for (int kt2 = 0; kt2 + 1 < KT_loop; kt2 += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        {
          const int un = su + 1 == NST ? 0 : su + 1;
          wait_vmcnt<(NST - 2) * NLD>();
          wait_lgkm0();
          tile_barrier();
          __builtin_amdgcn_sched_barrier(0);
          // past the last tile: read, unused
#pragma unroll
          for (int i = 0; i < NSLOT; ++i) {
            const int t = i / (2 * NI), q = i % (2 * NI);
            accf[t][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rb[u][q], ra[u][t], accf[t][q], 0, 0, 0);
            if (FUSE && q == 2 * NI - 1)
              haccf[FUSE ? t : 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(re[u], ra[u][t], haccf[FUSE ? t : 0], 0, 0, 0);
#pragma unroll
            for (int r = i * RT / NSLOT; r < (i + 1) * RT / NSLOT; ++r) read_step(stA(un), stB(un), r, ra[u ^ 1], rb[u ^ 1]);
            if (FUSE && i == 0) re[u ^ 1] = read_e(stE(un), wave);
#pragma unroll
            for (int d = 2 * i * NLD / NSLOT; d < 2 * (i + 1) * NLD / NSLOT && d < NLD; ++d) issue_one(stA(su), stB(su), stE(su), d);
            if (i == NSLOT / 2) { issue_done(); prepare(); }      // all loads are out: what the next tile's need
            __builtin_amdgcn_sched_barrier(0);
          }
          su = un;
        }
      }
    }
    if (KT_loop & 1) {                               // its operands are there: products alone
#pragma unroll
      for (int i = 0; i < NSLOT; ++i) {
        const int t = i / (2 * NI), q = i % (2 * NI);
        accf[t][q] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rb[0][q], ra[0][t], accf[t][q], 0, 0, 0);
        if (FUSE && q == 2 * NI - 1)
          haccf[FUSE ? t : 0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(re[0], ra[0][t], haccf[FUSE ? t : 0], 0, 0, 0);
      }
    }
    // the refills issued past the last tile (zeros) must have landed before the stages are reused below
    wait_vmcnt<0>();
    wait_lgkm0();
    tile_barrier();
    if (FUSE && fuse_h) {
      // The adapter tile.  Its W-side operand (rows of B_t) was fetched like any K-tile into the stage after the last
      // backbone tile's; its A side is Hs = s_t (X A_t) of the tile's rows, of which every wave holds a share in haccf.
      // The shares meet in two other stages, wave w brings row block w together (lane: row li of it, columns 8 j + 4 lg ..
      // + 3).  Scaled, masked, rounded to bf16, it goes into the adapter tile's stage in the layout the operand reads expect
      // (pieces 4..7 of a row, contraction indices 32..63, are zero), and from the tiles of the first column to memory.
      const int sK = KT % NST;
      static_assert(HW * 4 * 1024 <= 2 * STAGE / 2 && NST >= 4, "the shares of Hs fit two stages");
      float4* red = (float4*)stA(sK < 2 ? 2 : 0);
#pragma unroll
      for (int t = 0; t < HW; ++t)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          red[((t * 4 + wave) * 4 + j) * 64 + lane] = make_float4(haccf[FUSE ? t : 0][4 * j], haccf[FUSE ? t : 0][4 * j + 1], haccf[FUSE ? t : 0][4 * j + 2], haccf[FUSE ? t : 0][4 * j + 3]);
      wait_lgkm0();
      tile_barrier();
      bf16_t* hA = stA(sK);
      if (wave < HW) {
        const int row_l = wave * 32 + li;
        const bool keep = row_l < nrows && sRow[row_l] != 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const float4 x = red[((wave * 4 + w) * 4 + j) * 64 + lane];
            v[0] += x.x; v[1] += x.y; v[2] += x.z; v[3] += x.w;
          }
          const int col = 8 * j + 4 * lg;
#pragma unroll
          for (int c4 = 0; c4 < 4; ++c4) v[c4] = (keep && col + c4 < rank) ? tk.scale * v[c4] : 0.f;
          uint2 pk;
          pk.x = pack_bf16x2(v[0], v[1]);
          pk.y = pack_bf16x2(v[2], v[3]);
          *(uint2*)(hA + row_l * BK + ((j ^ swz) * 8) + 4 * lg) = pk;
          if (c0 == 0 && p.HsOut != nullptr && row_l < nrows && col < p.RP)
            *(uint2*)(p.HsOut + (size_t)(row0 + row_l) * p.RP + col) = pk;
        }
#pragma unroll
        for (int q = 0; q < 2; ++q)
          *(uint4*)(hA + row_l * BK + (((4 + 2 * lg + q) ^ swz) * 8)) = make_uint4(0, 0, 0, 0);
      }
      wait_lgkm0();
      tile_barrier();
      if (wave < ((rank + 15) >> 4)) {               // steps that carry data (rank <= 32: one or two)
#pragma unroll
        for (int r = 0; r < RT; ++r) read_step(hA, stB(sK), r, ra[0], rb[0]);
#pragma unroll
        for (int i = 0; i < NSLOT; ++i)
          accf[i / (2 * NI)][i % (2 * NI)] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rb[0][i % (2 * NI)], ra[0][i / (2 * NI)], accf[i / (2 * NI)][i % (2 * NI)], 0, 0, 0);
      }
      wait_lgkm0();
      tile_barrier();
    }
    // The four sums of every 32x32 block meet in LDS, a row of blocks of each wave's part at a time: added in the order of the
    // steps, so that an element's sum does not depend on the shape of the piece.
    static_assert(16 * NI * 4 * 1024 <= NST * STAGE * 2, "the shares of one row of blocks fit the stages");
    float4* red = (float4*)sm.base;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
      for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni) {
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const f32x16& x = accf[(o >> 1) * MI + mi][(o & 1) * NI + ni];
            red[(((o * 4 + wave) * NI + ni) * 4 + j) * 64 + lane] = make_float4(x[4 * j], x[4 * j + 1], x[4 * j + 2], x[4 * j + 3]);
          }
          __builtin_amdgcn_sched_barrier(0);         // (a block at a time out of the accumulation registers)
        }
      wait_lgkm0();
      tile_barrier();
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          float4 s4 = red[((wave * 4 * NI + ni) * 4 + j) * 64 + lane];
#pragma unroll
          for (int w = 1; w < 4; ++w) {
            const float4 x = red[(((wave * 4 + w) * NI + ni) * 4 + j) * 64 + lane];
            s4.x += x.x; s4.y += x.y; s4.z += x.z; s4.w += x.w;
          }
          acc[mi][ni][4 * j] = s4.x; acc[mi][ni][4 * j + 1] = s4.y; acc[mi][ni][4 * j + 2] = s4.z; acc[mi][ni][4 * j + 3] = s4.w;
        }
      wait_lgkm0();
      tile_barrier();
    }
  } else if constexpr (PIECE && !DIFFP) {
    // One wave a SIMD: nothing hides an LDS read but the wave's own products, so all operands of the next K-tile are read
    // under those of this one (read one step of 16 ahead, as the eight-wave loop does, a quarter took 0.367 us a K-tile, 0.335
    // so; the loads alone take 0.31, see above).  One barrier a K-tile, as above.
    constexpr int NM = MI * NI, NR = MI + NI, NSLOT = 4 * NM, RT = 4 * NR;
    bf16x8 ra[2][4][MI], rb[2][4][NI], re[2][4] = {};
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      read_ops(stA(0), stB(0), ks, ra[0][ks], rb[0][ks]);
      if (FUSE) re[0][ks] = read_e(stE(0), ks);
    }
    int su = 0;                                      // stage of tile kt
    prepare();
    for (int kt2 = 0; kt2 + 1 < KT_loop; kt2 += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        {
          const int un = su + 1 == NST ? 0 : su + 1;
          wait_vmcnt<(NST - 2) * NLD>();
          wait_lgkm0();
          tile_barrier();
          __builtin_amdgcn_sched_barrier(0);
          // past the last tile: read, unused
#pragma unroll
          for (int i = 0; i < NSLOT; ++i) {
            const int ks = i / NM;
            mma_one(ra[u][ks], rb[u][ks], i % NM);
#pragma unroll
            for (int r = i * RT / NSLOT; r < (i + 1) * RT / NSLOT; ++r)
              read_one(stA(un), stB(un), r / NR, r % NR, ra[u ^ 1][r / NR], rb[u ^ 1][r / NR]);
            if (FUSE) {
              if (i % NM == 0) re[u ^ 1][ks] = read_e(stE(un), ks);
              if (i % NM == NM - 1) mma_h(re[u][ks], ra[u][ks]);
            }
#pragma unroll
            for (int d = 2 * i * NLD / NSLOT; d < 2 * (i + 1) * NLD / NSLOT && d < NLD; ++d) issue_one(stA(su), stB(su), stE(su), d);
            if (i == NSLOT / 2) { issue_done(); prepare(); }      // all loads are out: what the next tile's need
            __builtin_amdgcn_sched_barrier(0);
          }
          su = un;
        }
      }
    }
    if (KT_loop & 1) {                               // its operands are there: products alone
#pragma unroll
      for (int i = 0; i < NSLOT; ++i) {
        mma_one(ra[0][i / NM], rb[0][i / NM], i % NM);
        if (FUSE && i % NM == NM - 1) mma_h(re[0][i / NM], ra[0][i / NM]);
      }
    }
  } else {
    bf16x8 a0[MI], b0[NI], a1[MI], b1[NI];
    read_ops(stA(0), stB(0), 0, a0, b0);
    // Steps 0..2 run from registers read one step ahead; before the last step every wave has read all of this
    // stage and tile kt+1 has landed (the loads of the NST-2 tiles after it may stay in flight): barrier; then, under the
    // last step's MFMAs, the first operands of tile kt+1 are read and all loads of tile kt+NST are issued into the stage just
    // freed.
    for (int kt2 = 0; kt2 < KT_loop; kt2 += NST) {
#pragma unroll
      for (int u = 0; u < NST; ++u) {
        const int kt = kt2 + u;
        if (kt < KT_loop) {
          bf16_t* cA = stA(u);
          bf16_t* cB = stB(u);
          prepare();
          __builtin_amdgcn_sched_barrier(0);
          fused_step(a0, b0, cA, cB, 1, a1, b1, std::false_type{}, nullptr, nullptr);
          fused_step(a1, b1, cA, cB, 2, a0, b0, std::false_type{}, nullptr, nullptr);
          fused_step(a0, b0, cA, cB, 3, a1, b1, std::false_type{}, nullptr, nullptr);
          wait_vmcnt<(NST - 2) * NLD>();
          wait_lgkm0();
          tile_barrier();
          __builtin_amdgcn_sched_barrier(0);
          if (DIFFP) {
            // Tile kt + 1 has landed: its masked entries, then a second barrier, then it may be read.  (Waiting for the
            // tile one step earlier and adding the entries under the MFMAs of the third step was slower.)
            const int un = (u + 1) % NST;
            if (patch && ps2[un] > ps0[un]) {
              patch_tile(stB(un), ldsP(un), ps0[un], ps1[un], ps2[un]);
              wait_lgkm0();
              tile_barrier();
            }
            // this stage is refilled with tile kt + NST (PRE == NST here): its entries, and the offsets of the tile after
            ps0[u] = nx0; ps1[u] = nx1; ps2[u] = nx2;
            bucket_offsets(kt + NST + 1, nx0, nx1, nx2);
            __builtin_amdgcn_sched_barrier(0);
          }
          fused_step(a1, b1, stA((u + 1) % NST), stB((u + 1) % NST), 0, a0, b0, std::true_type{}, cA, cB, ldsP(u), ps0[u],
                     ps2[u]);                        // past the last tile: read, unused
          issue_done();
        }
      }
    }
  }
  if (!KS) {
    // the refills issued past the last tile (zeros) must have landed before the stages are reused below
    wait_vmcnt<0>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  }

  if (SPLITK) {                                     // 16 bytes a lane, 1 KB a store
    float4* part = (float4*)(p.Part + ((size_t)split * p.quarters + slot) * (BMT * BN)) + wave * (MI * NI * 4 * 64) + lane;
#pragma unroll
    for (int mi = 0; mi < MI; ++mi)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          part[((mi * NI + ni) * 4 + j) * 64] = make_float4(acc[mi][ni][4 * j], acc[mi][ni][4 * j + 1], acc[mi][ni][4 * j + 2], acc[mi][ni][4 * j + 3]);
    if (fuse_h) {                                   // this wave's rows of the share of X A_t, 32 columns a row
      const int row = (slot < 4 * p.n_m * p.n_n ? 2 * tm + mhalf : 2 * p.n_m + tm) * BMT + (wm * MI + wn) * 32 + li;
      float* hp = p.PartH + ((size_t)split * (2 * p.n_m + p.n_mh) * BMT + row) * 32 + 4 * lg;
#pragma unroll
      for (int j = 0; j < 4; ++j) *(float4*)(hp + 8 * j) = make_float4(hacc[0][4 * j], hacc[0][4 * j + 1], hacc[0][4 * j + 2], hacc[0][4 * j + 3]);
    }
    return;
  }
  if (!KS && FUSE && fuse_h) {
    // The adapter tile.  Its W-side operand (rows of B_t) was fetched like any K-tile into the stage after the last
    // backbone tile's; its A side is Hs = s_t (X A_t) of the tile's rows, which the waves hold in hacc: this lane has
    // row wn*32 + li of the wave's row half and columns 8 j + 4 lg .. + 3.  Scaled, masked beyond the rank, rounded to
    // bf16, it goes into that stage in the layout the operand reads expect (pieces 4..7 of a row, contraction
    // indices 32..63, are zero), and from the tiles of the first column to memory.
    const int sK = KT % NST;
    bf16_t* hA = stA(sK);
    const bf16_t* hB = stB(sK);
#pragma unroll
    for (int i = 0; i < HB; ++i) {
      const int row_l = wm * (32 * MI) + (wn * HB + i) * 32 + li;
      const bool keep = row_l < nrows && sRow[row_l] != 0;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int col = 8 * j + 4 * lg;
        float v[4];
#pragma unroll
        for (int c4 = 0; c4 < 4; ++c4) v[c4] = (keep && col + c4 < rank) ? tk.scale * hacc[i][4 * j + c4] : 0.f;
        uint2 pk;
        pk.x = pack_bf16x2(v[0], v[1]);
        pk.y = pack_bf16x2(v[2], v[3]);
        *(uint2*)(hA + row_l * BK + ((j ^ swz) * 8) + 4 * lg) = pk;
        if (c0 == 0 && p.HsOut != nullptr && row_l < nrows && col < p.RP)
          *(uint2*)(p.HsOut + (size_t)(row0 + row_l) * p.RP + col) = pk;
      }
#pragma unroll
      for (int q = 0; q < 2; ++q)
        *(uint4*)(hA + row_l * BK + (((4 + 2 * lg + q) ^ swz) * 8)) = make_uint4(0, 0, 0, 0);
    }
    wait_lgkm0();
    tile_barrier();
    const int nks = (rank + 15) >> 4;               // steps that carry data (rank <= 32: one or two)
    bf16x8 a0[MI], b0[NI];
    for (int ks = 0; ks < nks; ++ks) {
      read_ops(hA, hB, ks, a0, b0);
      mma(a0, b0);
    }
    wait_lgkm0();
    tile_barrier();                                 // the stages are reused as staging below
  }

  // ---- epilogue: aggregate, mask, store; 32 rows of the wave tile at a time through this wave's own array.
  constexpr int AREA = NI == 2 ? 2560 : 1280;     // elements of a staging area (5 KB or 2.5 KB)
  constexpr int AREAS = PIECE ? NW : A_ELEMS / AREA;   // staging areas per stage (eight waves: in its A side)
  static_assert(32 * EPW <= AREA && NW <= AREAS * NST && (!PIECE || NW * AREA <= NST * STAGE), "every wave has its own staging area");
  bf16_t* stage = stA(wave / AREAS) + (wave % AREAS) * AREA;
  constexpr int PPR = WCOLS / 8;                 // 16-byte pieces per staged row
  constexpr int RPI = 64 / PPR;                  // rows one wave instruction moves
  const int e_row = lane / PPR, e_pc = (lane % PPR) * 8;
  const bool scale_out = !NT && ia3;             // IA3 forward: Z = x W is saved first, then Y = Z * l_t
  const int passes = (scale_out && p.Zsave) ? 2 : 1;
  const bool z_only = !NT && tuning && p.Zsave;  // TUNING forward: x W goes to the saved region, Y is written by the bottleneck kernels
  for (int pass = 0; pass < passes; ++pass) {
    const bool to_z = z_only || pass + 1 < passes;
    bf16_t* dst = to_z ? p.Zsave + (size_t)(tk.zrow0 - tk.row_begin) * p.Nc : p.Out;   // indexed by the row in the batch
    if (scale_out && !to_z) {
      // (all loads before the first product: a column past the end reads the first ones and is not stored)
      float lv[NI][4][4];
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int c = c0 + wn * WCOLS + ni * 32 + 8 * j + 4 * lg;
          const bf16_t* l = Lvec + (c < p.Nc ? c : 0);        // Nc is a multiple of 8: the four columns together
#pragma unroll
          for (int e = 0; e < 4; ++e) lv[ni][j][e] = bf16_to_f32(l[e]);
        }
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int mi = 0; mi < MI; ++mi)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[mi][ni][4 * j + e] *= lv[ni][j][e];
    }
#pragma unroll
    for (int mi = 0; mi < MI; ++mi) {
#pragma unroll
      for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          uint2 v;
          v.x = pack_bf16x2(acc[mi][ni][4 * j + 0], acc[mi][ni][4 * j + 1]);
          v.y = pack_bf16x2(acc[mi][ni][4 * j + 2], acc[mi][ni][4 * j + 3]);
          *(uint2*)(stage + li * EPW + ni * 32 + 8 * j + 4 * lg) = v;
        }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int rr = 0; rr < 32 / RPI; ++rr) {
        const int ml = rr * RPI + e_row;
        const int m = wm * (32 * MI) + mi * 32 + ml;
        const int c = c0 + wn * WCOLS + e_pc;
        if (m < nrows && c < p.Nc) {
          uint4 v = *(const uint4*)(stage + ml * EPW + e_pc);
          if (sRow[m] == 0) v = make_uint4(0, 0, 0, 0);
          uint4* d = (uint4*)(dst + (size_t)(row0 + m) * p.Nc + c);
          if (STREAM) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, v), (u32x4*)d);
          else *d = v;
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  }
}

// A row group without tokens: CLEAR_N columns of its output rows (d: its number times the slabs of CLEAR_N columns, plus the
// slab), a wave a row, and with the first of them the rows of Hs.  With `below`, first the same of the rows past the first 128
// of the groups that have tokens in those only.
template <int NTHR>
__device__ __forceinline__ void clear_group(const GemmParams& p, int d) {
  const int slabs = (p.Nc + CLEAR_N - 1) / CLEAR_N;
  const int g = d / slabs + (p.below ? 0 : p.n_mh), m0 = g < p.n_mh ? 128 : 0;
  int4 iw = *(const int4*)(p.dtab + p.items_off + (p.n_m + g) * DI_WORDS);
  iw.y += m0;
  iw.z -= m0;
  const int c = (d % slabs) * CLEAR_N + (threadIdx.x & 63) * 8;
  if (c < p.Nc)
    for (int m = threadIdx.x >> 6; m < iw.z; m += NTHR / 64) *(uint4*)(p.Out + (size_t)(iw.y + m) * p.Nc + c) = make_uint4(0, 0, 0, 0);
  if (d % slabs == 0 && p.HsOut != nullptr)
    for (int e = threadIdx.x; e < iw.z * (p.RP / 8); e += NTHR)
      *(uint4*)(p.HsOut + (size_t)(iw.y + e / (p.RP / 8)) * p.RP + (e % (p.RP / 8)) * 8) = make_uint4(0, 0, 0, 0);
}

// Stamps of the diagnostic counters; the start stamps wait in the buffer itself (words 2, 3), so that nothing stays live
// across the tile.
__device__ __forceinline__ void clock_start(const GemmParams& p) {
  if (p.clk != nullptr && blockIdx.x == 0 && threadIdx.x == 0) { p.clk[2] = clock64(); p.clk[3] = wall_clock64(); }
}
__device__ __forceinline__ void clock_end(const GemmParams& p) {
  if (p.clk != nullptr && blockIdx.x == 0 && threadIdx.x == 0) {
    atomicAdd(p.clk, (unsigned long long)clock64() - p.clk[2]);
    atomicAdd(p.clk + 1, (unsigned long long)wall_clock64() - p.clk[3]);
  }
}

// Workgroup b's quarter of a tile left over, or (from half0 on) of one whose row group has tokens in its first 128 rows only.
struct Quarter { int L, half, mhalf; bool hg; };
__device__ __forceinline__ Quarter quarter_piece(const GemmParams& p, int b) {
  Quarter q;
  q.hg = b >= p.half0;
  const int t = b - (q.hg ? p.half0 : p.n_full);
  q.half = (t >> 3) & 1;
  q.mhalf = q.hg ? 0 : (t >> 4) & 1;
  if (q.hg) {
    q.L = p.start_h[t & 7] + (t >> 4);
    if (q.L >= p.start_h[(t & 7) + 1]) q.L = -1;
  } else {
    q.L = tile_of_slot(p.n_m * p.n_n, t & 7, (p.n_full >> 3) + (t >> 5));
  }
  return q;
}

// Launches with full tiles, those that add masked entries, and halves of short contractions.  Workgroups 0 .. n_full-1 compute full tiles, slot by slot with the XCD in the low three bits of
// the index (the hardware deals consecutive workgroups round-robin to the eight XCDs, so one XCD's L2 sees neighbouring tiles).
// The workgroups after them compute the remaining tiles in pieces (tail_split = 2: two half-width tiles each;
// 4: four 128 x 128 quarters each); all pieces of a tile run on the same XCD.  The dispatcher hands out workgroups
// in index order, so the pieces start as the compute units finish their last full tile.
template <bool NT, bool DIFFP, bool TAIL, bool STREAM>
__global__ __launch_bounds__(512, 1) void k_gemm_dma(const GemmParams p) {
  __shared__ __attribute__((aligned(1024))) bf16_t smem[4 * (BM * BK + (DIFFP ? kPackElems : 0))];   // two stages of 64 KB, or four of 32 KB
  static_assert(piece_stages(2, 2, false, DIFFP) == 4, "four stages of a quarter");
  __shared__ int sOff[DIFFP ? 3 * 1024 : 2];                                      // DIFFP: K < 65536, so at most 1023 K-tiles
  __shared__ int sRow[256];
  const Smem sm = {smem, sRow, sOff};
  const int b = blockIdx.x;
  if (b >= p.clear0) return clear_group<512>(p, b - p.clear0);
  clock_start(p);
  if (b < p.n_full) {
    const int L = tile_of_slot(p.n_m * p.n_n, b & 7, b >> 3);
    if (L < 0) return;
    gemm_tile<NT, 4, 4, 2, false, DIFFP, TAIL, false, STREAM>(p, 0, p.n_m, L, 0, 0, sm);
  } else if (b < p.half0 && p.tail_split == 2) {
    const int t = b - p.n_full;                                       // n_full is a multiple of 8
    const int L = tile_of_slot(p.n_m * p.n_n, t & 7, (p.n_full >> 3) + (t >> 4));
    if (L < 0) return;
    gemm_tile<NT, 4, 4, 1, false, DIFFP, TAIL, false, STREAM>(p, 0, p.n_m, L, (t >> 3) & 1, 0, sm);
  } else {
    const Quarter q = quarter_piece(p, b);
    if (q.L < 0) return;
    if (q.hg && threadIdx.x >= 256) {              // the four waves that a quarter does not need clear the padding below it
      int tm, tn;
      tile_at(p.n_mh, p.n_n, q.L, tm, tn);
      const int4 iw = *(const int4*)(p.dtab + p.items_off + (p.n_m + tm) * DI_WORDS);
      clear_below(p, iw.y, iw.z, tn * TILE_N + q.half * 128);
      return;
    }
    gemm_tile<NT, 2, 2, 2, false, DIFFP, TAIL, false, STREAM>(p, q.hg ? p.n_m : 0, q.hg ? p.n_mh : p.n_m, q.L, q.half, q.mhalf, sm);
  }
  clock_end(p);
}

// The other launches: four waves a workgroup, one a SIMD, with all of its registers.
//   PIECES_HALF     256 x 128, quarters for the row groups with tokens in their first 128 rows only
//   PIECES_QUARTER  128 x 128 (or such quarters alone)
//   PIECES_64X128, PIECES_64X64   of row groups of 64; an XCD takes a run of pieces, the row group running fastest, so that
//                   the pieces that read the same columns of W do it through one L2
// SPLITK (quarters): p.splits workgroups share the contraction of each; the (share, quarter) pairs, share by
// share, go to the XCDs in eight equal runs (dealt by whole tiles, 10 tiles of 6 quarters left three XCDs idle and gave
// the others two rounds: 20.8 us, 14.8 so, for 60 quarters of 2560 x 2560 in four shares).
enum : int { PIECES_HALF = 0, PIECES_QUARTER, PIECES_64X128, PIECES_64X64 };
// The backward takes the gradient dA_t along (workgroups from p.grad0 on, four waves that each walk a row group as in a launch of
// its own): such launches leave compute units idle, and a launch of its own costs 4 to 10 us before and behind it.
template <int PIECES, bool NT, bool FUSE, bool SPLITK>
__global__ __launch_bounds__(256, 1) void k_gemm_pieces(const GemmParams p, const adapter::GradParams job) {
  constexpr int MI = PIECES == PIECES_HALF ? 4 : (PIECES == PIECES_QUARTER ? 2 : 1), NI = PIECES == PIECES_64X64 ? 1 : 2;
  constexpr int ELEMS = piece_stages(MI, NI, FUSE, false) * piece_elems(MI, NI, FUSE, false);
  constexpr int QUART = PIECES == PIECES_HALF ? piece_stages(2, 2, FUSE, false) * piece_elems(2, 2, FUSE, false) : 0;
  __shared__ __attribute__((aligned(1024))) bf16_t smem[ELEMS > QUART ? ELEMS : QUART];
  __shared__ int sRow[256];
  const Smem sm = {smem, sRow, nullptr};
  const int b = blockIdx.x;
  if constexpr (NT) {
    static_assert(sizeof(smem) >= adapter::kGradLdsElems * sizeof(bf16_t), "the gradient's slabs");
    if (b >= p.grad0) {
      const int g = b - p.grad0, item = g % job.n_items, cols = g / job.n_items;
      if (job.pieces == 1) adapter::grad_rows<1, 2, false>(job, p.tasks, item, cols, smem);
      else if (job.pieces == 2) adapter::grad_rows<2, 2, false>(job, p.tasks, item, cols, smem);
      else adapter::grad_rows<4, 1, false>(job, p.tasks, item, cols, smem);
      return;
    }
  }
  if (b >= p.clear0) return clear_group<256>(p, b - p.clear0);
  clock_start(p);
  if constexpr (SPLITK) {
    const int id = (b & 7) * (p.clear0 >> 3) + (b >> 3), split = id / p.quarters, q = id % p.quarters;
    int L, half, mhalf;
    if (split >= p.splits) return;
    const bool hg = quarter_of(p, q, L, half, mhalf);
    gemm_tile<NT, 2, 2, 2, FUSE, false, true, true>(p, hg ? p.n_m : 0, hg ? p.n_mh : p.n_m, L, half, mhalf, sm, split, q, hg && split == 0 && !p.below);
  } else if constexpr (PIECES >= PIECES_64X128) {
    const int id = tile_of_slot(p.n_m * p.n_n, b & 7, b >> 3);
    if (id < 0) return;
    gemm_tile<NT, 1, 1, NI, FUSE, false, true>(p, 0, p.n_m, id % p.n_m, id / p.n_m, 0, sm);
  } else if (PIECES == PIECES_HALF && b < p.half0) {
    const int L = tile_of_slot(p.n_m * p.n_n, b & 7, b >> 4);
    if (L < 0) return;
    gemm_tile<NT, 2, 4, 2, FUSE, false, true>(p, 0, p.n_m, L, (b >> 3) & 1, 0, sm);
  } else {
    const Quarter q = quarter_piece(p, b);
    if (q.L < 0) return;
    gemm_tile<NT, 2, 2, 2, FUSE, false, true>(p, q.hg ? p.n_m : 0, q.hg ? p.n_mh : p.n_m, q.L, q.half, q.mhalf, sm, 0, 0, q.hg && !p.below);
  }
  clock_end(p);
}

// The shares of a split contraction, summed in ascending order, then the epilogue of gemm_tile (scale, mask, round, store).
// Bound by latency: there are few outputs, and a wave's time is its chain of loads.  So a workgroup takes one 32 x 64 block of
// a wave tile, eight a quarter, a wave a quarter of the block's accumulator registers (1 KB a wave instruction, as the tiles
// stored them), four shares in flight; the block turns in LDS into rows, one 16-byte piece a thread.
template <bool NT, bool FUSE>
__global__ __launch_bounds__(256) void k_gemm_sum(const GemmParams p) {
  constexpr int EPW = 72;
  __shared__ __attribute__((aligned(16))) bf16_t stage[32 * EPW];
  __shared__ __attribute__((aligned(16))) bf16_t sH[FUSE ? 32 * 40 : 8];      // FUSE: Hs of the block's rows
  __shared__ __attribute__((aligned(16))) bf16_t sB[FUSE ? 32 * 64 : 8];      //       and the block's columns of B_t
  const int b = blockIdx.x >> 3, wave_t = (blockIdx.x >> 1) & 3, mi = blockIdx.x & 1;    // quarter, its wave tile, row block
  int L, half, mhalf, tm, tn;
  const bool hg = quarter_of(p, b, L, half, mhalf);
  tile_at(hg ? p.n_mh : p.n_m, p.n_n, L, tm, tn);
  const int4 iw = *(const int4*)(p.dtab + p.items_off + ((hg ? p.n_m : 0) + tm) * DI_WORDS);
  const ItemView it = {iw.x, iw.y, iw.z, iw.w};
  const int mrow0 = mhalf * 128, row0 = it.row0 + mrow0;
  const int cw0 = tn * TILE_N + half * 128 + (wave_t & 1) * 64;
  const int nrows = it.nrows - mrow0 < 128 ? it.nrows - mrow0 : 128;
  const int m0 = (wave_t >> 1) * 64 + mi * 32;                         // first row of the block inside the quarter
  if (m0 >= nrows || cw0 >= p.Nc) return;
  const DevTask tk = get_task(p.tasks, it.task);
  const bool ia3 = !NT && tk.kind == MUX_ADAPTER_IA3_OUT, z_only = !NT && tk.kind == MUX_ADAPTER_TUNING && p.Zsave;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 31, lg = lane >> 5;
  const size_t share = (size_t)p.quarters * (128 * 128 / 4);
  const float4* part = (const float4*)(p.Part + (size_t)b * (128 * 128)) + (wave_t * 16 + mi * 8 + wave * 2) * 64 + lane;
  float4 s[2] = {make_float4(0.f, 0.f, 0.f, 0.f), make_float4(0.f, 0.f, 0.f, 0.f)};
  for (int k = 0; k < p.splits; k += 4) {
    float4 v[4][2];
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i) v[u][i] = k + u < p.splits ? part[(k + u) * share + i * 64] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i) { s[i].x += v[u][i].x; s[i].y += v[u][i].y; s[i].z += v[u][i].z; s[i].w += v[u][i].w; }
  }
  if (FUSE && tk.kind == MUX_ADAPTER_LORA) {
    // Hs = s_t (X A_t) of the block's rows from the shares, four columns a thread, to memory from the blocks of the first
    // column; then the adapter's product, on the vector units (rank <= 32): a thread's row times its two runs of columns.
    const int hr = threadIdx.x >> 3, hc = (threadIdx.x & 7) * 4, hm = m0 + hr;        // row, column of Hs
    const bool hin = hm < nrows && row_is_valid(p.dtab, row0 + hm);
    const int qrows = 2 * p.n_m + p.n_mh, prow = (hg ? 2 * p.n_m + tm : 2 * tm + mhalf) * 128 + hm;
    float4 h = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int k = 0; k < p.splits; k += 4) {
      float4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u)
        v[u] = k + u < p.splits ? *(const float4*)(p.PartH + ((size_t)(k + u) * qrows * 128 + prow) * 32 + hc) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int u = 0; u < 4; ++u) { h.x += v[u].x; h.y += v[u].y; h.z += v[u].z; h.w += v[u].w; }
    }
    const int rank = tk.rank;
    uint2 pk;
    pk.x = pack_bf16x2(hin && hc < rank ? tk.scale * h.x : 0.f, hin && hc + 1 < rank ? tk.scale * h.y : 0.f);
    pk.y = pack_bf16x2(hin && hc + 2 < rank ? tk.scale * h.z : 0.f, hin && hc + 3 < rank ? tk.scale * h.w : 0.f);
    *(uint2*)(sH + hr * 40 + hc) = pk;
    if (cw0 == 0 && hm < nrows && hc < p.RP) *(uint2*)(p.HsOut + (size_t)(row0 + hm) * p.RP + hc) = pk;
    const int bc = cw0 + (int)(threadIdx.x & 7) * 8;
    *(uint4*)(sB + hr * 64 + (threadIdx.x & 7) * 8) = hr < rank && bc < p.Nc ? *(const uint4*)((const bf16_t*)tk.B + (size_t)hr * p.Nc + bc) : make_uint4(0, 0, 0, 0);
    __syncthreads();
    for (int k = 0; k < rank; ++k) {
      const float hk = bf16_to_f32(sH[li * 40 + k]);
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int r = 2 * wave + i;
        const uint2 w = *(const uint2*)(sB + k * 64 + 32 * (r >> 2) + 8 * (r & 3) + 4 * lg);
        s[i].x = fmaf(hk, __uint_as_float(w.x << 16), s[i].x); s[i].y = fmaf(hk, __uint_as_float(w.x & 0xffff0000u), s[i].y);
        s[i].z = fmaf(hk, __uint_as_float(w.y << 16), s[i].z); s[i].w = fmaf(hk, __uint_as_float(w.y & 0xffff0000u), s[i].w);
      }
    }
  }
  const int m = m0 + (int)(threadIdx.x >> 3), c = cw0 + (int)(threadIdx.x & 7) * 8;      // the piece this thread stores
  const bool out = m < nrows && c < p.Nc, keep = out && row_is_valid(p.dtab, row0 + m);
  const int passes = (ia3 && p.Zsave) ? 2 : 1;
  for (int pass = 0; pass < passes; ++pass) {
    const bool to_z = z_only || pass + 1 < passes;
    bf16_t* dst = to_z ? p.Zsave + (size_t)(tk.zrow0 - tk.row_begin) * p.Nc : p.Out;
    // s[i], with 2 wave + i = 4 ni + j: row li of the block, columns 32 ni + 8 j + 4 lg .. + 3
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = 2 * wave + i, col = 32 * (r >> 2) + 8 * (r & 3) + 4 * lg;
      if (ia3 && !to_z && cw0 + col < p.Nc) {
        const bf16_t* l = (const bf16_t*)tk.L + cw0 + col;
        s[i].x *= bf16_to_f32(l[0]); s[i].y *= bf16_to_f32(l[1]); s[i].z *= bf16_to_f32(l[2]); s[i].w *= bf16_to_f32(l[3]);
      }
      uint2 v;
      v.x = pack_bf16x2(s[i].x, s[i].y);
      v.y = pack_bf16x2(s[i].z, s[i].w);
      *(uint2*)(stage + li * EPW + col) = v;
    }
    __syncthreads();
    if (out) {
      uint4 v = *(const uint4*)(stage + (threadIdx.x >> 3) * EPW + (threadIdx.x & 7) * 8);
      if (!keep) v = make_uint4(0, 0, 0, 0);
      *(uint4*)(dst + (size_t)(row0 + m) * p.Nc + c) = v;
    }
    __syncthreads();
  }
}

// Number of compute units of the current device, asked once; while it cannot be told, that of the part the kernels are made for.
int compute_units() {
  static std::atomic<int> n{0};
  if (const int known = n.load(std::memory_order_relaxed)) return known;
  int dev = 0, v = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || v <= 0)
    return kComputeUnits;
  n.store(v, std::memory_order_relaxed);
  return v;
}

// The tile plan of a launch: whole tiles for the full rounds of workgroups, the rest as halves or quarters, then the
// quarters of the row groups with tokens in their first 128 rows only, then the clearing of those without any.
struct TilePlan { int n_m, n_mh, n_n, n_full, tail_split, start_h[9], half0, clear0, grid, pieces; };
TilePlan plan_tiles(const mux_segtab* st, int Nc) {
  TilePlan t{};
  t.n_m = st->n_gemm[0];
  t.n_mh = st->n_gemm[1];
  t.n_n = (Nc + TILE_N - 1) / TILE_N;
  const int ncu = compute_units();
  // Where no pieces fit behind the last full round, its tiles run whole.  If those of the groups with tokens in their first 128
  // rows fit that round as whole tiles too, but not as the pairs of quarters that they would be else, and are few beside the
  // others, they run whole with them: next to whole tiles a quarter takes 0.6 of their time, so that a second round of
  // quarters ends after them.  As pairs, whole, forward: 640 x 2304, 198 tiles and 45 such, 35.6 us, 30.3; 4096 x 1536, 240 and 12,
  // 146, 122; 2560 x 1536, 216 and 30, 77.7, 79.7.  Where they are many the products saved count for more: 1280 x 1536, 186 and
  // 54, 44.8, 46.3; 2560 x 3584, 70 and 154, 58.3, 67.1; but 2560 x 1536, 162 and 84, 79.1, 75.6.
  {
    const int total = t.n_m * t.n_n, rem = total % ncu, lower = t.n_mh * t.n_n;
    if (rem + lower <= ncu && rem + 2 * lower > ncu && 2 * (rem + lower) > ncu && rem >= 4 * lower) { t.n_m += t.n_mh; t.n_mh = 0; }
  }
  const int total = t.n_m * t.n_n, total_h = t.n_mh * t.n_n;
  const int slots = (total + 7) / 8;                         // of the XCDs with most tiles
  // One workgroup per compute unit at a time: the tiles left after the last full round would keep a fraction of
  // the units busy for a whole tile time.  When they fit four times (beside the quarters that follow), they run as
  // quarters, when twice, as half-width tiles.
  static const bool no_halves = getenv("MUX_GEMM_NO_HALF_TILES") != nullptr;
  static const bool no_quarters = getenv("MUX_GEMM_NO_QUARTER_TILES") != nullptr;
  const int full_slots = (total / ncu) * (ncu / 8);          // per-XCD slots covered by whole rounds
  const int rem = total - full_slots * 8, more = 2 * total_h;
  int tail_slots = 0;
  if (!no_halves && ncu % 8 == 0 && rem > 0 && 2 * rem + more <= ncu) tail_slots = slots - full_slots;
  t.tail_split = (!no_quarters && 4 * rem + more <= ncu) ? 4 : 2;
  t.n_full = 8 * (slots - tail_slots);
  // The pairs of quarters go to the XCDs so that these have as many pieces as each other, to within one pair: the XCDs
  // without a tile more of the others (from `odd` on) first get as many pairs as such a tile has pairs of pieces, then all of
  // them equal shares.  So pieces that fit the compute units fit those of every XCD.  Ranges of ceil(tiles / 8) for both left
  // the last XCDs idle and gave the others a second round: 35 tiles and 49 pairs, 238 pieces for 256 units, were 34 on each of
  // seven XCDs of 32 units (1280 x 1792, forward: 33.1 us so, 19.0 now; 42 tiles and 42 pairs, 1280 x 5376: 33.0 and 20.4).
  const int odd = total % 8, ahead = tail_slots > 0 ? t.tail_split / 2 * (8 - odd) : 0;
  const int lead = odd == 0 ? 0 : (total_h < ahead ? total_h : ahead), rest = total_h - lead;
  int slots_h = 0;
  for (int x = 0; x < 8; ++x) {
    int n = rest / 8 + (((x - odd) & 7) < rest % 8 ? 1 : 0);
    if (x >= odd) n += lead / (8 - odd) + (x - odd < lead % (8 - odd) ? 1 : 0);
    t.start_h[x + 1] = t.start_h[x] + n;
    if (n > slots_h) slots_h = n;
  }
  t.half0 = t.n_full + 8 * t.tail_split * tail_slots;
  t.clear0 = t.half0 + 16 * slots_h;
  t.grid = t.clear0 + st->n_gemm[2] * ((Nc + CLEAR_N - 1) / CLEAR_N);
  t.pieces = t.tail_split == 4 ? PIECES_QUARTER : PIECES_HALF;
  return t;
}

// Pieces of a launch that quarters would not fill: of row groups of 64, where all of them find a compute unit at once.  A
// unit's loads bound a piece, 16 KB a K-tile for 64 x 64, 24 for 64 x 128, 32 for a quarter, so that smaller pieces on idle
// units take less time although they read more in all.  4096 x 4096, tasks of 37, 129, 64 and 90 tokens, forward: 160 quarters
// 41 us, 224 pieces of 64 x 128 27.2, 448 of 64 x 64 40; 512 x 1024, 1000 tokens, 256 pieces of 64 x 64 8.7 us, quarters 10.6; 1000 x 1000, 800
// tokens, forward and backward 31.6 us, quarters 41.1, 64 x 128 36.7.
int choose_pieces(const mux_segtab* st, int Nc, int units) {
  if (st->n_gemm64[0] * ((Nc + 63) / 64) <= units) return PIECES_64X64;
  if (st->n_gemm64[0] * ((Nc + 127) / 128) <= units) return PIECES_64X128;
  return PIECES_QUARTER;
}

// How many workgroups share the contraction of a quarter.  A launch that leaves compute units without a piece spends its
// time walking all of K on the rest; with S shares the walk of a quarter is 1 / S as long.  Estimate, in us, for weights that
// come from memory, as they do where a step goes through many layers (60 layers of 4096 x 640, three tasks of 64 to 100 tokens,
// forward: 26.4 us a call whole, 20.3 in eight shares; one layer over and over, its W in the last-level cache, 20.0 and 18.7): a
// K-tile 0.45 of a quarter, 0.40 of 64 x 128, 0.30 of 64 x 64, with the down-projection in the loop 0.04 more; 9 for the second
// launch and the shares' stores, 0.01 a share of a quarter.  A share keeps eight K-tiles, twice what is in flight.
// Weights from memory, whole -> shared: 640 x 4096, three tasks, forward and backward 31.2 -> 25.6 us a call, with a fourth of
// 440 tokens 33.8 -> 31.6; 4096 x 4096, 100 tokens, forward 28.8 -> 23.5.  From the cache: 8000 x 1000, 300 tokens, 34.5 -> 23.6,
// 11008 x 4096, 64 tokens, 47.0 -> 28.2; near the line 2048 x 512, 64 tokens, 13.5 -> 14.4.
// Arithmetic on the host alone: sizes are asked for in processes without a device too.
int count_quarters(const mux_segtab* st, int Nc) {
  return (4 * st->n_gemm[0] + 2 * st->n_gemm[1]) * ((Nc + TILE_N - 1) / TILE_N);
}
// Bytes of one share: its quarters' partial tiles, and where the forward forms Hs, its part of X A_t
size_t share_bytes(const mux_segtab* st, int Nc, bool nt) {
  const size_t q = (size_t)count_quarters(st, Nc) * (128 * 128 * 4);
  return q + (nt ? 0 : (size_t)(2 * st->n_gemm[0] + st->n_gemm[1]) * (128 * 32 * 4));
}
int plan_splits(const mux_segtab* st, int Kc, int Nc, bool nt, size_t room, int units) {
  const int quarters = count_quarters(st, Nc), kt = (Kc + BK - 1) / BK;
  if (quarters == 0 || st->n_diff > 0) return 1;
  const double fused = !nt && st->n_lora > 0 && st->n_tuning == 0 && st->r_max <= 32 ? 0.04 : 0.0;
  const size_t share = share_bytes(st, Nc, nt);
  int most = units / quarters < kt / 8 ? units / quarters : kt / 8;
  if ((size_t)most * share > room) most = (int)(room / share);
  const int pieces = choose_pieces(st, Nc, units);
  int best = 1;
  double best_us = kt * (fused + (pieces == PIECES_64X64 ? 0.30 : (pieces == PIECES_64X128 ? 0.40 : 0.45)));
  for (int s = 2; s <= most; ++s) {
    const double us = (kt + s - 1) / s * (0.45 + fused) + 0.01 * s * quarters + 9.0;
    if (us < best_us) { best_us = us; best = s; }
  }
  return best;
}
// The shares of a launch: only a launch of nothing but quarters is split.  MUX_GEMM_NO_SPLIT (read once): none is.
int launch_splits(const CallCtx& c, int Kc, int Nc, bool nt) {
  static const bool off = getenv("MUX_GEMM_NO_SPLIT") != nullptr;
  const TilePlan t = plan_tiles(c.st, Nc);
  if (off || t.n_full != 0 || t.tail_split != 4) return 1;
  return plan_splits(c.st, Kc, Nc, nt, c.split_room, compute_units());
}
size_t split_bytes(const mux_segtab* st, int Kc, int Nc, bool nt) {
  const int s = plan_splits(st, Kc, Nc, nt, ~(size_t)0, kComputeUnits);
  return s > 1 ? (size_t)s * share_bytes(st, Nc, nt) : 0;
}

// The plan of a launch of pieces of row groups of 64.
TilePlan plan_rows64(const mux_segtab* st, int Nc, int pieces) {
  TilePlan t{};
  t.pieces = pieces;
  t.n_m = st->n_gemm64[0];
  t.n_n = (Nc + (pieces == PIECES_64X64 ? 63 : 127)) / (pieces == PIECES_64X64 ? 64 : 128);
  t.half0 = t.clear0 = (t.n_m * t.n_n + 7) / 8 * 8;
  t.grid = t.clear0 + st->n_gemm64[1] * ((Nc + CLEAR_N - 1) / CLEAR_N);
  return t;
}
template <int PIECES, bool NT>
void launch_pieces(const char* name, dim3 grid, hipStream_t stream, const GemmParams& p, const adapter::GradParams& job) {
  if constexpr (!NT) {
    if (p.HsOut != nullptr) {
      MUX_LAUNCH(name, (k_gemm_pieces<PIECES, NT, true, false>), grid, dim3(256), 0, stream, p, job);
      return;
    }
  }
  MUX_LAUNCH(name, (k_gemm_pieces<PIECES, NT, false, false>), grid, dim3(256), 0, stream, p, job);
}

template <bool NT>
mux_status launch(const CallCtx& c, const bf16_t* Ain, const bf16_t* Ext, bf16_t* Out, bf16_t* Zsave, int Kc, int Nc,
                  bool fuse_down, const adapter::GradParams* take = nullptr) {
  GemmParams p;
  p.dtab = c.dtab; p.tasks = *c.tref; p.Ain = Ain; p.W = (const bf16_t*)c.W; p.ldw = c.ldw; p.Ext = Ext; p.Out = Out;
  p.Zsave = Zsave; p.Kc = Kc; p.Nc = Nc; p.RP = c.RP;
  p.HsOut = fuse_down ? (bf16_t*)Ext : nullptr;
  p.DiffPack = (const uint32_t*)c.diffPack;
  p.splits = launch_splits(c, Kc, Nc, NT);
  TilePlan t = plan_tiles(c.st, Nc);
  p.items_off = c.st->dev_image[DH_OFF_GEMM_ITEMS];
  if (p.splits == 1) {
    // (masked entries are listed by buckets of 128 lines)
    if (t.n_full == 0 && t.tail_split == 4 && p.DiffPack == nullptr) t.pieces = choose_pieces(c.st, Nc, compute_units());
    if (t.pieces >= PIECES_64X128) {
      t = plan_rows64(c.st, Nc, t.pieces);
      p.items_off = c.st->dev_image[DH_OFF_GEMM_ITEMS64];
    }
  }
  p.n_m = t.n_m; p.n_n = t.n_n; p.n_full = t.n_full; p.tail_split = t.tail_split;
  p.n_mh = t.n_mh; p.half0 = t.half0; p.clear0 = t.clear0;
  for (int x = 0; x < 9; ++x) p.start_h[x] = t.start_h[x];
  p.AinScaled = (const bf16_t*)c.dYs;
  p.Wdiff = (const bf16_t*)c.diffW; p.wdiff_stride = c.diffW_stride;
  p.clk = diag_clock_buffer();
  if (t.grid == 0) return MUX_OK;
  // An output of whole cache lines goes past the last-level cache where that would not hold it for its reader beside the
  // activations: it would push them, and the operands of the tiles to come, out.  Two projections, each one's output the next one's input, LoRA,
  // forward and backward, through the caches and past them (MB of the two activations): 4096 and 11008 columns (32, 86) 1259 and
  // 1271 us, 2048 and 5504 (32, 85) 720 and 731, 4096 and 4096 (64, 64) 1101 and 1106, (70, 70) 1134 and 1143; 3072 and 3072
  // (80, 80) 1062 and 1053, 4096 and 2048 (102, 51) 917 and 903, 2560 and 2560 (88, 88) 991 and 970, 4096 and 4096 (125, 125)
  // 1949 and 1921, 5120 and 5120 (176, 176) 3346 and 3288.  Behind a contraction of up to 512 an output goes past them from kStreamOut on:
  // such a launch is bound by what it writes, and crowds its operands out of the L2s.  Six projections in a row, 448 and 8384 columns, 4096
  // tokens (4, 69), forward and backward, through the caches and past them: LoRA 879 and 861 us, IA3 919 and 855, no adapter 589 and 554;
  // 256 and 8384 714 and 689, 755 and 706, 456 and 416; 640 and 8384, 6144 tokens, 1450 and 1461, 1490 and 1471, 1095 and 1137; 1280 and
  // 8384, 4096, 1456 and 1474, 1431 and 1449, 1146 and 1219.  Lines that tiles share (6424 columns) would be written twice.  Not the
  // forward of a batch of Adapter-Tuning for the most part: it writes x W, which the next two launches read (9000 tokens of rank
  // 64, 4096 x 4096, tune_down 40.3 us past the caches, 31.5 through them).
  const size_t out_bytes = (size_t)c.st->T * Nc * 2, in_bytes = (size_t)c.st->T * Kc * 2;
  int64_t tuning = 0;
  for (const HostTask& ht : c.st->tasks) tuning += !NT && ht.kind == MUX_ADAPTER_TUNING ? ht.row_count : 0;
  const bool stream = out_bytes >= kStreamOut && (Kc <= kStreamDepth || out_bytes + in_bytes > kStreamBoth) && 2 * tuning <= c.st->T && Nc % 64 == 0;
  p.Part = (float*)c.split;
  if (fuse_down && (NT || t.n_full != 0)) return fail(MUX_ERR_UNSUPPORTED, "gemm: this launch cannot carry the down-projection");
  if (p.DiffPack != nullptr && fuse_down) return fail(MUX_ERR_UNSUPPORTED, "gemm: this launch cannot add masked entries in the tile loop");
  const adapter::GradParams job = take ? *take : adapter::GradParams{};
  const int n_grads = job.n_items * job.col_blocks;
  const bool tail = Kc % BK != 0;                 // (masked entries are added only where there is none)
  // Halves of a short contraction that carry nothing else: eight waves bring the outputs out in half the time, four walk a long
  // contraction faster.  Forward, eight waves, four: 1024 columns, 4616 tokens, IA3, K = 320 12.1 us, 14.3, 768 17.2, 19.0, 1024 19.8,
  // 21.1, 1536 26.6, 26.2, 2048 31.3, 30.5; LoRA of rank 16 with its down_x, 320 14.6, 16.4, 1024 23.8, 23.8, 1280 28.7, 28.3, 2048 37.1, 34.8.
  const bool eight_waves = t.pieces == PIECES_HALF && Kc <= 1024 && !fuse_down && n_grads == 0;
  const bool four_waves = t.n_full == 0 && p.DiffPack == nullptr && !eight_waves;
  // The rows past the first 128 of a group with tokens in those only: where there are units left for it, workgroups of their own
  // clear them; else the quarters do, behind their first loads.  Thirteen tasks of 41 to 176 tokens aligned to 256, forward,
  // quarters, own workgroups: 768 x 1280 14.2 us, 13.4, 2048 x 1280 23.5, 22.8; 448 x 10496, three tasks, 246 quarters, 12.2 and 13.3.
  const int below = t.n_mh * ((Nc + CLEAR_N - 1) / CLEAR_N), pieces = p.splits > 1 ? p.splits * count_quarters(c.st, Nc) : t.clear0;
  p.below = four_waves && c.st->n_gemm_below > 0 && below > 0 && pieces + below <= compute_units();
  if (p.below) t.grid += below;
  const char* name = NT ? (n_grads > 0 ? "gemm_nt_da" : "gemm_nt") : "gemm_nn";
  if (n_grads > 0 && (t.n_full != 0 || p.DiffPack != nullptr)) return fail(MUX_ERR_UNSUPPORTED, "gemm: this launch cannot take the gradients along");
  const dim3 grid(t.grid + n_grads), block(512);
  p.grad0 = t.grid;
  if (p.splits > 1) {
    p.quarters = count_quarters(c.st, Nc);
    p.clear0 = (p.splits * p.quarters + 7) / 8 * 8;
    p.PartH = p.Part + (size_t)p.splits * p.quarters * (128 * 128);
    p.grad0 = t.grid - t.clear0 + p.clear0;
    const dim3 sgrid(p.grad0 + n_grads), sums(8 * p.quarters);
    const double moved = ((double)p.splits * 4 + 2) * c.st->valid_total * Nc;
    if (!NT && fuse_down) {
      MUX_LAUNCH(name, (k_gemm_pieces<PIECES_QUARTER, false, true, true>), sgrid, dim3(256), 0, c.stream, p, job);
      prof_note_bytes(moved);
      MUX_LAUNCH("gemm_sum", (k_gemm_sum<false, true>), sums, dim3(256), 0, c.stream, p);
    } else {
      MUX_LAUNCH(name, (k_gemm_pieces<PIECES_QUARTER, NT, false, true>), sgrid, dim3(256), 0, c.stream, p, job);
      prof_note_bytes(moved);
      MUX_LAUNCH("gemm_sum", (k_gemm_sum<NT, false>), sums, dim3(256), 0, c.stream, p);
    }
    return MUX_OK;
  }
  if (p.DiffPack != nullptr) {
    MUX_LAUNCH(name, (k_gemm_dma<NT, true, false, false>), grid, block, 0, c.stream, p);
  } else if (four_waves) {
    if (t.pieces == PIECES_HALF) launch_pieces<PIECES_HALF, NT>(name, grid, c.stream, p, job);
    else if (t.pieces == PIECES_QUARTER) launch_pieces<PIECES_QUARTER, NT>(name, grid, c.stream, p, job);
    else if (t.pieces == PIECES_64X128) launch_pieces<PIECES_64X128, NT>(name, grid, c.stream, p, job);
    else launch_pieces<PIECES_64X64, NT>(name, grid, c.stream, p, job);
  } else if (stream && tail) MUX_LAUNCH(name, (k_gemm_dma<NT, false, true, true>), grid, block, 0, c.stream, p);
  else if (stream) MUX_LAUNCH(name, (k_gemm_dma<NT, false, false, true>), grid, block, 0, c.stream, p);
  else if (tail) MUX_LAUNCH(name, (k_gemm_dma<NT, false, true, false>), grid, block, 0, c.stream, p);
  else MUX_LAUNCH(name, (k_gemm_dma<NT, false, false, false>), grid, block, 0, c.stream, p);
  return MUX_OK;
}

}  // namespace

size_t gemm_split_bytes(int K, int N, const mux_segtab* st) {
  const size_t f = split_bytes(st, K, N, false), b = split_bytes(st, N, K, true);
  return align256(f > b ? f : b);
}

// 16-byte loads need rows of X, dY, W, Hs and B_t to start 16-byte aligned (rows of A_t: see rank_pieces), and the
// 32-bit buffer offsets need W and the largest row group a kernel builds one descriptor over (1024 rows of
// activations; rows parked at offset 2^31 must stay out of range) below 2 GiB.
bool gemm_dma_supported(const CallCtx& c) {
  const int64_t big = (int64_t)1 << 31;
  return (c.K % 8 == 0) && (c.N % 8 == 0) && (c.ldw % 8 == 0) && (((uintptr_t)c.W & 15) == 0) &&
         ((int64_t)c.K * c.ldw * 2 < big) && ((int64_t)1024 * (c.K > c.N ? c.K : c.N) * 2 < big);
}

// Can the forward of this call form Hs = s_t X A_t inside the backbone tile loop?  The kernel can when the launch is
// made of pieces only, with LoRA ranks up to 32 and no Adapter-Tuning task.  It is chosen for launches of quarters and of pieces of
// row groups of 64 (at most a quarter of the compute units' worth of 256 x 256 tiles): there the loop waits on loads, and the launch
// that it saves costs more than the extra product; not in launches of halves.  Forward, four LoRA tasks of rank 16, separate and
// fused, six layers in turn (their weights come from memory): 4096 x 4096, 128 tokens 29.5 us, 23.3, 512 40.8, 36.9, 1024 51.3, 51.7;
// 2560 x 2560, 512 25.6, 20.5; 11008 x 4096, 512 89.0, 72.5, 1024 130.2, 119.3; 8192 x 1024, 2048 68.8, 58.6; halves: 4096 x 4096, 1536
// 64.3, 73.5; 2560 x 2560, 1536 32.3, 33.0; 11008 x 4096, 2048 170.8, 195.8.  One layer over and over, its weights in the last-level cache,
// loses where the quarters fill the units: 4096 x 4096, 1024 44.0, 48.8; 11008 x 4096, 1024 98.2, 114.7.
// MUX_GEMM_FUSE_DOWN (read once): 0 never, 2 in launches of halves as well.
bool gemm_dma_fuses_down(const CallCtx& c) {
  static const int mode = [] { const char* e = getenv("MUX_GEMM_FUSE_DOWN"); return e == nullptr ? 1 : atoi(e); }();
  if (mode == 0) return false;
  if (c.st->n_lora == 0 || c.st->n_tuning > 0 || c.st->r_max > 32 || c.diffPack != nullptr) return false;
  const TilePlan t = plan_tiles(c.st, c.N);
  if (t.n_full != 0 || (t.n_m + t.n_mh) * t.n_n == 0) return false;
  return t.tail_split == 4 || mode == 2;
}

mux_status gemm_dma_forward(const CallCtx& c, const void* X, const void* Hs, void* Y, void* Z, bool fuse_down) {
  return launch<false>(c, (const bf16_t*)X, (const bf16_t*)Hs, (bf16_t*)Y, (bf16_t*)Z, c.K, c.N, fuse_down);
}

// Launches of pieces only (their workgroups have four waves), of at most two rounds of them: those have compute units to spare,
// or nearly so.  Behind more rounds the gradient runs at the end, one workgroup a unit with the pieces' LDS, where a launch of its
// own has four.  Forward and backward, a launch of its own -> riding: 256 x 256, 250 tokens, 29.0 -> 25.1 us; 2048 x 3000, 300
// tokens, 58.9 -> 50.8; 2560 x 2560, 900 tokens, 81 -> 77.2; 1608 x 6424, 2400 tokens in two micro-batches, 402 -> 393; tasks of 40
// to 128 tokens, N = 1024, 512 pieces: 4096, 16 tasks 82.6 -> 80.7, 8192, 8 tasks of rank 64 114.5 -> 112.0; 768 and more: 4096, 24
// tasks 103.0 -> 104.9, 8192, 32 tasks 208.3 -> 213.1, 2048, 64 tasks of rank 64 159.6 -> 160.8.
bool gemm_dma_takes_grads(const CallCtx& c) {
  const TilePlan t = plan_tiles(c.st, c.K);
  return t.n_full == 0 && t.grid > 0 && t.clear0 <= 2 * compute_units() && c.diffPack == nullptr;
}

mux_status gemm_dma_backward(const CallCtx& c, const void* dY, const void* Gs, void* dX, const adapter::GradParams* job) {
  return launch<true>(c, (const bf16_t*)dY, (const bf16_t*)Gs, (bf16_t*)dX, nullptr, c.N, c.K, false, job);
}

}  // namespace mux
