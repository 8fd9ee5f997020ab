// Attention step of a chunk-aligned batch (section 3.5): causal softmax attention of every sequence on its own,
// forward and backward, bf16 storage, fp32 accumulation on the matrix cores (v_mfma_f32_32x32x16_bf16).
//
// Work item = a block of 128 tokens of one sequence x one head; four waves, 32 tokens each.  All three kernels keep
// the wave's own tokens on the N side of every product (lane l owns token l % 32; its two half-waves split the
// other index), so that softmax statistics, log-sum-exp and the dO.O term are per-lane scalars and a probability
// tile leaves the accumulators already in the layout of the next product's B operand:
//   forward   S^T = K Q^T (keys x queries)      -> P^T -> O^T  += V^T P^T          online softmax over key tiles
//   dQ        S^T, dP^T = V dO^T                -> dS^T -> dQ^T += K^T dS^T
//   dK, dV    S = Q K^T, dP = dO V^T (queries x keys, the wave owns keys) -> dV^T += dO^T P, dK^T += Q^T dS
// The operand that has to be read across rows (V^T, K^T, dO^T, Q^T) comes from a row-major LDS tile through
// ds_read_b64_tr_b16.  A sum over 16 tokens may take them in any order as long as both operands agree; the order
// used is the one the accumulator layout gives: slot i of half-wave h <-> token 8 (i / 4) + 4 h + i % 4.
// Every output element has one owner; nothing is accumulated across workgroups, results repeat bit for bit.
#include "mux_attn.h"
#include "mux_device_utils.h"

namespace mux {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int BLK = kAttnBlockRows;
constexpr int TILE = 64;        // tokens of the other side staged per step
// What follows from the head dimension D (a multiple of 16 up to 128; built for 64, 80, 96 and 128).
template <int D>
struct Dim {
  static_assert(D % 16 == 0 && D >= 32 && D <= 128, "head dimension");
  static constexpr int KS = D / 16;          // contraction steps of 16 over the head dimension
  static constexpr int DT = (D + 31) / 32;   // 32-column tiles of an output row (the last may be half used)
  static constexpr int DP = 32 * DT;         // columns of a staged tile; those from D on stay zero
  static constexpr int KP = DP + 8;          // LDS row pitch (elements) of a tile that is only read along rows
  static constexpr int TP = DP + 16;         // ... of a tile that is also read across rows
};
constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;

// A wave in a run of matrix products is served before the other wave of its SIMD, whose vector instructions then
// fill the issue slots between the products (forward and dQ: 2 % faster; dK/dV: no change, not used there).
#define ATTN_PRIO_HIGH() __builtin_amdgcn_s_setprio(2)
#define ATTN_PRIO_LOW() __builtin_amdgcn_s_setprio(0)

struct AttnParams {
  const int32_t* dtab;
  const bf16_t *Q, *K, *V, *O, *dO;
  bf16_t *Out, *dQ, *dK, *dV;
  float* lse;         // [H][T], natural log
  float* delta;       // [H][T]
  int64_t ldq, ldk, ldv, ldo;
  int T, H, Hkv;      // query heads, key/value heads (H = group * Hkv: query head h reads key/value head h / group)
  int short_map;      // forward: the pairs are dealt to the XCDs as in the kernel of the short sequences
  int list_off;       // word offset of the launch's block list in dtab
  int block0, n_blocks;   // the launch covers the entries block0 .. block0 + n_blocks - 1 of its list
  float scale;        // (comes with the arguments before it: behind the next two, a load of its own that the loops waited for, 41.9 us, 41.6)
  int n_blocks64, grid128;   // one-kernel backward: then as many of at most 64 tokens, from workgroup grid128 on
};

__device__ __forceinline__ bf16x4 lds_read_tr(const bf16_t* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4bf16((__attribute__((address_space(3))) bf16x4*)p);
}
__device__ __forceinline__ f32x16 mma(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// 2^x by the hardware instruction (arguments here are <= 0 or masked afterwards; denormal results may flush to zero)
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ bf16x8 zero8() { return __builtin_bit_cast(bf16x8, uint4{0u, 0u, 0u, 0u}); }
// accumulator elements 8u .. 8u+7 as a B operand
__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int u) {
  uint4 r;
  r.x = pack_bf16x2(v[8 * u + 0], v[8 * u + 1]);
  r.y = pack_bf16x2(v[8 * u + 2], v[8 * u + 3]);
  r.z = pack_bf16x2(v[8 * u + 4], v[8 * u + 5]);
  r.w = pack_bf16x2(v[8 * u + 6], v[8 * u + 7]);
  return __builtin_bit_cast(bf16x8, r);
}
// A operand read across the rows of a row-major tile: column c0 + lane % 32, the 8 rows 4h + {0..3}, 8 + 4h + {0..3} from row0
template <int TP>
__device__ __forceinline__ bf16x8 read_across(const bf16_t* tile, int row0, int c0, int lane) {
  const int j = lane & 15, grp = lane >> 4;
  const bf16_t* p = tile + (row0 + 4 * (grp >> 1) + (j >> 2)) * TP + c0 + 16 * (grp & 1) + 4 * (j & 3);
  const bf16x4 lo = lds_read_tr(p), hi = lds_read_tr(p + 8 * TP);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
// token of accumulator element j for half-wave h inside a 32-token tile
__device__ __forceinline__ int tok(int j, int half) { return 8 * (j >> 2) + 4 * half + (j & 3); }

// Work item of a workgroup: (block of the list, head).  Workgroups go to the eight XCDs round-robin; with a multiple of
// eight heads every XCD takes its own heads and walks the list in order, so that the blocks running on an XCD at one
// time belong to two or three sequences of one head and find their keys and values in that XCD's L2.
__device__ __forceinline__ void work_item(int n_blocks, int n_heads, int& block, int& head) {
  const unsigned id = blockIdx.x;
  if ((n_heads & 7) == 0) {
    const unsigned j = id >> 3;
    head = (int)(id & 7) + 8 * (int)(j / (unsigned)n_blocks);
    block = (int)(j % (unsigned)n_blocks);
  } else {
    head = (int)(id / (unsigned)n_blocks);
    block = (int)(id % (unsigned)n_blocks);
  }
}

__host__ __device__ __forceinline__ bool short_deals_blocks(int D, int n_blocks) { return D % 64 != 0 && n_blocks >= 32; }
// The same for launches of short sequences.  With a multiple of eight heads every XCD takes its own run of neighbouring
// heads of every block, the head running fastest.  Other numbers of heads: where the row segments of neighbouring heads
// share cache lines (160 bytes at D = 80) the blocks are dealt to the XCDs in turn, each with all of its heads, so that these
// meet in one L2; else, and with few blocks, the block runs fastest.  (A contiguous run of the pairs an XCD gives the first
// XCDs the long sequences: 53 heads of 96, 20 x 128 and 20 x 70 tokens, backward 131 us so, 116 now; 28 heads of 128, 200 x 50
// and 200 x 10, 427 and 317; 53 heads of 96, 128 x 128, dealt in turn 380, the block fastest 404.)
// false = nothing to do.
template <int D>
__device__ __forceinline__ bool short_item(unsigned id, int n_blocks, int n_heads, int& block, int& head) {
  const unsigned xcd = id & 7, j = id >> 3, nb = (unsigned)n_blocks, nh = (unsigned)n_heads;
  if ((n_heads & 7) == 0) {
    const unsigned hx = nh >> 3;
    block = (int)(j / hx);
    head = (int)(xcd * hx + j % hx);
  } else if (short_deals_blocks(D, n_blocks)) {
    block = (int)(xcd + 8 * (j / nh));
    head = (int)(j % nh);
  } else {
    block = (int)(id % nb);
    head = (int)(id / nb);
  }
  return block < n_blocks && head < n_heads;
}

// ROWS rows x D columns of one head from global memory (rows past `limit` read as zero) into registers, then LDS.
// The tile is cut into 16-byte pieces, D / 8 a row.  Where the pieces of a row divide evenly among the NTHR / ROWS
// threads that a row can have, a thread takes consecutive pieces of one row (one address, constant offsets);
// otherwise the NTHR threads take the pieces of the tile in order, NTHR at a time.
template <int ROWS, int D, int NTHR = 256>
struct TileLoadT {
  static constexpr int PPR = D / 8, NP = ROWS * PPR, TPR = NTHR / ROWS;
  static constexpr bool RUNS = PPR % TPR == 0;
  static constexpr int N = RUNS ? PPR / TPR : (NP + NTHR - 1) / NTHR;
  uint4 r[N];
  __device__ __forceinline__ void load(const bf16_t* base, int64_t ld, int first, int row0, int limit, int hc, int tid) {
    if (RUNS) {
      const int row = row0 + tid / TPR;
      const uint4* src = (const uint4*)(base + (size_t)(first + row) * ld + hc + (tid % TPR) * (8 * N));
#pragma unroll
      for (int i = 0; i < N; ++i) r[i] = row < limit ? src[i] : uint4{0u, 0u, 0u, 0u};
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int e = tid + NTHR * i, row = row0 + e / PPR, pc = e % PPR;
        const bool ok = (NP % NTHR == 0 || e < NP) && row < limit;
        r[i] = ok ? *(const uint4*)(base + (size_t)(first + row) * ld + hc + pc * 8) : uint4{0u, 0u, 0u, 0u};
      }
    }
  }
  __device__ __forceinline__ void store(bf16_t* tile, int pitch, int tid) const {
    if (RUNS) {
      uint4* dst = (uint4*)(tile + (tid / TPR) * pitch + (tid % TPR) * (8 * N));
#pragma unroll
      for (int i = 0; i < N; ++i) dst[i] = r[i];
    } else {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        const int e = tid + NTHR * i;
        if (NP % NTHR == 0 || e < NP) *(uint4*)(tile + (e / PPR) * pitch + (e % PPR) * 8) = r[i];
      }
    }
  }
};
// Zero in the columns D .. DP-1 of a staged tile of `rows` rows (nothing is ever stored there afterwards).
template <int D, int DP, int NTHR = 256>
__device__ __forceinline__ void zero_pad_columns(bf16_t* tile, int rows, int pitch, int tid) {
  if constexpr (DP > D) {
    constexpr int PIECES = (DP - D) / 8;       // 16-byte pieces a row
    for (int e = tid; e < rows * PIECES; e += NTHR)
      *(uint4*)(tile + (e / PIECES) * pitch + D + (e % PIECES) * 8) = uint4{0u, 0u, 0u, 0u};
  }
}

// ------------------------------------------------------------------------------------------------ forward
template <int D>
__global__ __launch_bounds__(256, 2) void k_attn_fwd(AttnParams p) {
  constexpr int KS = Dim<D>::KS, DT = Dim<D>::DT, DP = Dim<D>::DP, KP = Dim<D>::KP, TP = Dim<D>::TP;
  __shared__ __align__(16) bf16_t sK[TILE * KP];
  __shared__ __align__(16) bf16_t sV[TILE * TP];
  int wi_block, wi_head;
  if (p.short_map) { if (!short_item<D>(blockIdx.x, p.n_blocks, p.H, wi_block, wi_head)) return; }
  else work_item(p.n_blocks, p.H, wi_block, wi_head);
  const int32_t* blk = p.dtab + p.list_off + (p.block0 + wi_block) * DA_WORDS;
  const int first = blk[DA_FIRST_ROW], len = blk[DA_LEN], q0 = blk[DA_BLOCK0];
  const int hc = wi_head * D;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, half = lane >> 5;
  const int ql = q0 + 32 * wave + li;          // this lane's query inside the sequence
  const bool qok = ql < len;
  zero_pad_columns<D, DP>(sV, TILE, TP, tid);
  bf16x8 qf[KS];
  {
    const bf16_t* qrow = p.Q + (size_t)(first + ql) * p.ldq + hc + 8 * half;
#pragma unroll
    for (int s = 0; s < KS; ++s) qf[s] = qok ? *(const bf16x8*)(qrow + 16 * s) : zero8();
  }
  f32x16 o[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[dt][j] = 0.f;
  float m = -INFINITY, m_prev = -INFINITY, l = 0.f;
  const float c = p.scale * LOG2E;
  const float lazy = 8.f / c;                   // 8 in the exponent, in units of the raw score
  const int kend = min(len, q0 + BLK);          // keys [0, kend) are visible to some query of the block
  const int wq_first = q0 + 32 * wave, wq_last = wq_first + 31;
  TileLoadT<TILE, D> tk, tv;
  const int hck = wi_head / (p.H / p.Hkv) * D;  // this head's key/value columns
  tk.load(p.K, p.ldk, first, 0, len, hck, tid);
  tv.load(p.V, p.ldv, first, 0, len, hck, tid);
  for (int kb = 0; kb < kend; kb += TILE) {
    __syncthreads();
    tk.store(sK, KP, tid);
    tv.store(sV, TP, tid);
    __syncthreads();
    if (kb + TILE < kend) {
      tk.load(p.K, p.ldk, first, kb + TILE, len, hck, tid);
      tv.load(p.V, p.ldv, first, kb + TILE, len, hck, tid);
    }
    if (kb > wq_last) continue;                 // no key of this tile is visible to this wave's queries
    f32x16 s[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int j = 0; j < 16; ++j) s[kt][j] = 0.f;
    {
      // the K fragments of the first 32 keys are fetched up front; each is refilled for the second 32 keys as
      // soon as its product is issued, so that an LDS read has the other products to land behind
      const bf16_t* kp = sK + li * KP + 8 * half;
      bf16x8 kf[KS];
#pragma unroll
      for (int st = 0; st < KS; ++st) kf[st] = *(const bf16x8*)(kp + 16 * st);
      __builtin_amdgcn_sched_barrier(0);        // (the scheduler would otherwise sink every read next to its use)
      ATTN_PRIO_HIGH();
#pragma unroll
      for (int st = 0; st < KS; ++st) {
        s[0] = mma(kf[st], qf[st], s[0]);
        kf[st] = *(const bf16x8*)(kp + 32 * KP + 16 * st);
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int st = 0; st < KS; ++st) s[1] = mma(kf[st], qf[st], s[1]);
      ATTN_PRIO_LOW();
    }
    const bool diag = kb + TILE - 1 > wq_first;
    // running maximum on the raw scores (the scale is positive), then one fused multiply-add per element: m is kept in
    // units of the raw score, exp2 arguments are s c - m c
    float mx = -INFINITY;
    if (diag) {                                 // only the tiles on the diagonal pay for the mask
      const int rel = ql - kb - 4 * half;       // key 32 kt + 8 (j / 4) + j % 4 is hidden iff it exceeds rel
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (32 * kt + 8 * (j >> 2) + (j & 3) > rel) s[kt][j] = -INFINITY;
    }
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int j = 0; j < 16; ++j) mx = fmaxf(mx, s[kt][j]);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    // The reference point of the exponentials follows the running maximum lazily: it moves only when the maximum
    // has grown by more than 8 in the exponent (probabilities then stay below 2^8, harmless in fp32 and bf16, and
    // the final division by the row sum cancels the choice), so the rescaling of the output is rare.
    if (!(mx <= m + lazy)) m = mx;              // also the first tile (m = -inf) and never for mx = -inf
    const float ms = m == -INFINITY ? 0.f : m;
    const float alpha = fast_exp2((m_prev - ms) * c);
    m_prev = m;
    const float msc = ms * c;
    float rs = 0.f;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        const float e = fast_exp2(fmaf(s[kt][j], c, -msc));
        s[kt][j] = e;
        rs += e;
      }
    l = l * alpha + rs;
    if (__any(alpha != 1.f)) {                  // the running maximum of some query moved
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[dt][j] *= alpha;
    }
    ATTN_PRIO_HIGH();
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bf16x8 pb = pack8(s[kt], u);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[dt] = mma(read_across<TP>(sV, 32 * kt + 16 * u, 32 * dt, lane), pb, o[dt]);
      }
    ATTN_PRIO_LOW();
  }
  l += __shfl_xor(l, 32);
  if (qok) {
    const float inv = 1.f / l;
    bf16_t* orow = p.Out + (size_t)(first + ql) * p.ldo + hc;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int jg = 0; jg < 4; ++jg) {
        if (32 * dt + 8 * jg >= D) continue;      // the unused half of the last 32 columns
        uint2 v;
        v.x = pack_bf16x2(o[dt][4 * jg + 0] * inv, o[dt][4 * jg + 1] * inv);
        v.y = pack_bf16x2(o[dt][4 * jg + 2] * inv, o[dt][4 * jg + 3] * inv);
        *(uint2*)(orow + 32 * dt + 8 * jg + 4 * half) = v;
      }
    if (p.lse && half == 0) p.lse[(size_t)wi_head * p.T + first + ql] = (m * c + log2f(l)) * LN2;
  }
}

// Rows that belong to no sequence: zero in `n_out` outputs.  grid = (64-row items, slabs of 2048 elements).
struct ZeroParams {
  const int32_t* dtab;
  bf16_t* out[3];
  int64_t ld[3];
  int n_out;
  int width[3];
};
__global__ __launch_bounds__(256) void k_attn_zero_pad(ZeroParams p) {
  const ItemView it = load_item(p.dtab, 0, blockIdx.x);
  if (it.task >= 0 && it.nvalid == it.nrows) return;
  // wave w takes the rows w, w + 4, ..; the workgroup covers a slab of 256 vectors (4 KB) of the row width
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int slab = (int)blockIdx.y * 256 + lane;
  for (int r = wave; r < it.nrows; r += 4) {
    if (it.task >= 0 && row_is_valid(p.dtab, it.row0 + r)) continue;
    for (int o = 0; o < p.n_out; ++o) {
      uint4* dst = (uint4*)(p.out[o] + (size_t)(it.row0 + r) * p.ld[o]);
#pragma unroll
      for (int k = 0; k < 4; ++k)
        if (slab + 64 * k < p.width[o] / 8) dst[slab + 64 * k] = uint4{0u, 0u, 0u, 0u};
    }
  }
}

// delta[h][row] = sum_d dO[row][h, d] * O[row][h, d] for the rows of sequences.  Sixteen lanes per (row, head), a
// 16-byte piece each (a wave instruction then reads whole runs of the row); a group of sixteen takes four
// consecutive heads, all loads issued before the sums.
template <int D>
__global__ __launch_bounds__(256) void k_attn_delta(AttnParams p) {
  constexpr int PPR = D / 8, U = 4;
  const int l16 = threadIdx.x & 15;
  const size_t group = ((size_t)blockIdx.x * 256 + threadIdx.x) >> 4;
  const size_t n = (size_t)p.T * p.H;
  uint4 x[U], y[U];
  bool ok[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const size_t idx = group * U + u;
    const int row = idx < n ? (int)(idx / p.H) : 0, h = (int)(idx % p.H);
    ok[u] = idx < n && l16 < PPR && row_is_valid(p.dtab, row);
    x[u] = y[u] = uint4{0u, 0u, 0u, 0u};
    if (ok[u]) {
      x[u] = *(const uint4*)(p.dO + (size_t)row * p.ldo + h * D + 8 * l16);
      y[u] = *(const uint4*)(p.O + (size_t)row * p.ldo + h * D + 8 * l16);
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t xs[4] = {x[u].x, x[u].y, x[u].z, x[u].w}, ys[4] = {y[u].x, y[u].y, y[u].z, y[u].w};
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      s = fmaf(__uint_as_float(xs[q] << 16), __uint_as_float(ys[q] << 16), s);
      s = fmaf(__uint_as_float(xs[q] & 0xffff0000u), __uint_as_float(ys[q] & 0xffff0000u), s);
    }
    s += __shfl_xor(s, 8);
    s += __shfl_xor(s, 4);
    s += __shfl_xor(s, 2);
    s += __shfl_xor(s, 1);
    const size_t idx = group * U + u;
    if (idx < n && l16 == 0) p.delta[(size_t)(idx % p.H) * p.T + idx / p.H] = s;
  }
}

// ------------------------------------------------------------------------------------------------ dQ
template <int D>
__global__ __launch_bounds__(256, 2) void k_attn_bwd_q(AttnParams p) {
  constexpr int KS = Dim<D>::KS, DT = Dim<D>::DT, DP = Dim<D>::DP, KP = Dim<D>::KP, TP = Dim<D>::TP;
  __shared__ __align__(16) bf16_t sK[TILE * TP];
  __shared__ __align__(16) bf16_t sV[TILE * KP];
  int wi_block, wi_head;
  work_item(p.n_blocks, p.H, wi_block, wi_head);
  const int32_t* blk = p.dtab + p.list_off + (p.block0 + wi_block) * DA_WORDS;
  const int first = blk[DA_FIRST_ROW], len = blk[DA_LEN], q0 = blk[DA_BLOCK0];
  const int hc = wi_head * D;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, half = lane >> 5;
  const int ql = q0 + 32 * wave + li;
  const bool qok = ql < len;
  zero_pad_columns<D, DP>(sK, TILE, TP, tid);
  bf16x8 qf[KS], df[KS];
  {
    const bf16_t* qrow = p.Q + (size_t)(first + ql) * p.ldq + hc + 8 * half;
    const bf16_t* drow = p.dO + (size_t)(first + ql) * p.ldo + hc + 8 * half;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      qf[s] = qok ? *(const bf16x8*)(qrow + 16 * s) : zero8();
      df[s] = qok ? *(const bf16x8*)(drow + 16 * s) : zero8();
    }
  }
  const float c = p.scale * LOG2E;
  const float lse2 = qok ? p.lse[(size_t)wi_head * p.T + first + ql] * LOG2E : INFINITY;    // exp2(x - inf) = 0
  const float dl = qok ? p.delta[(size_t)wi_head * p.T + first + ql] : 0.f;
  f32x16 dq[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int j = 0; j < 16; ++j) dq[dt][j] = 0.f;
  const int kend = min(len, q0 + BLK);
  const int wq_first = q0 + 32 * wave, wq_last = wq_first + 31;
  TileLoadT<TILE, D> tk, tv;
  const int hck = wi_head / (p.H / p.Hkv) * D;  // this head's key/value columns
  tk.load(p.K, p.ldk, first, 0, len, hck, tid);
  tv.load(p.V, p.ldv, first, 0, len, hck, tid);
  for (int kb = 0; kb < kend; kb += TILE) {
    __syncthreads();
    tk.store(sK, TP, tid);
    tv.store(sV, KP, tid);
    __syncthreads();
    if (kb + TILE < kend) {
      tk.load(p.K, p.ldk, first, kb + TILE, len, hck, tid);
      tv.load(p.V, p.ldv, first, kb + TILE, len, hck, tid);
    }
    if (kb > wq_last) continue;
    const bool diag = kb + TILE - 1 > wq_first;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt) {            // one half of the tile at a time keeps the live registers down
      f32x16 s, dp;
#pragma unroll
      for (int j = 0; j < 16; ++j) { s[j] = 0.f; dp[j] = 0.f; }
      ATTN_PRIO_HIGH();
#pragma unroll
      for (int st = 0; st < KS; ++st) {
        s = mma(*(const bf16x8*)(sK + (32 * kt + li) * TP + 16 * st + 8 * half), qf[st], s);
        dp = mma(*(const bf16x8*)(sV + (32 * kt + li) * KP + 16 * st + 8 * half), df[st], dp);
      }
      ATTN_PRIO_LOW();
#pragma unroll
      for (int j = 0; j < 16; ++j) s[j] = fast_exp2(fmaf(s[j], c, -lse2));        // P^T (zero for a lane without query)
      if (diag) {                               // only the tiles on the diagonal pay for the mask
        const int rel = ql - kb - 32 * kt - 4 * half;
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (8 * (j >> 2) + (j & 3) > rel) s[j] = 0.f;
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) s[j] *= dp[j] - dl;                           // dS^T
      ATTN_PRIO_HIGH();
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bf16x8 ds = pack8(s, u);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) dq[dt] = mma(read_across<TP>(sK, 32 * kt + 16 * u, 32 * dt, lane), ds, dq[dt]);
      }
      ATTN_PRIO_LOW();
    }
  }
  if (qok) {
    bf16_t* orow = p.dQ + (size_t)(first + ql) * p.ldq + hc;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int jg = 0; jg < 4; ++jg) {
        if (32 * dt + 8 * jg >= D) continue;      // the unused half of the last 32 columns
        uint2 v;
        v.x = pack_bf16x2(dq[dt][4 * jg + 0] * p.scale, dq[dt][4 * jg + 1] * p.scale);
        v.y = pack_bf16x2(dq[dt][4 * jg + 2] * p.scale, dq[dt][4 * jg + 3] * p.scale);
        *(uint2*)(orow + 32 * dt + 8 * jg + 4 * half) = v;
      }
  }
}

// ------------------------------------------------------------------------------------------------ dK, dV
template <int D>
__global__ __launch_bounds__(256, 2) void k_attn_bwd_kv(AttnParams p) {
  constexpr int KS = Dim<D>::KS, DT = Dim<D>::DT, DP = Dim<D>::DP, KP = Dim<D>::KP, TP = Dim<D>::TP;
  constexpr int QT = 32;                       // queries staged per step
  __shared__ __align__(16) bf16_t sQ[QT * TP];
  __shared__ __align__(16) bf16_t sD[QT * TP];
  __shared__ __align__(16) bf16_t sVf[BLK * KP];   // the block's own V rows (B operand of dO V^T), kept here to save registers
  __shared__ float sLse[QT], sDelta[QT];
  int wi_block, wi_head;                       // wi_head: a key/value head
  work_item(p.n_blocks, p.Hkv, wi_block, wi_head);
  const int32_t* blk = p.dtab + p.list_off + (p.block0 + wi_block) * DA_WORDS;
  const int first = blk[DA_FIRST_ROW], len = blk[DA_LEN], k0 = blk[DA_BLOCK0];
  const int hc = wi_head * D;
  const int group = p.H / p.Hkv;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, li = lane & 31, half = lane >> 5;
  const int kl = k0 + 32 * wave + li;          // this lane's key inside the sequence
  const bool kok = kl < len;
  zero_pad_columns<D, DP>(sQ, QT, TP, tid);
  zero_pad_columns<D, DP>(sD, QT, TP, tid);
  bf16x8 kf[KS];
  {
    const bf16_t* krow = p.K + (size_t)(first + kl) * p.ldk + hc + 8 * half;
#pragma unroll
    for (int s = 0; s < KS; ++s) kf[s] = kok ? *(const bf16x8*)(krow + 16 * s) : zero8();
    TileLoadT<TILE, D> t;
    t.load(p.V, p.ldv, first, k0, len, hc, tid);
    t.store(sVf, KP, tid);
    t.load(p.V, p.ldv, first, k0 + TILE, len, hc, tid);
    t.store(sVf + TILE * KP, KP, tid);
  }
  const bf16_t* vfrag = sVf + (32 * wave + li) * KP + 8 * half;
  const float c = p.scale * LOG2E;
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int j = 0; j < 16; ++j) { dk[dt][j] = 0.f; dv[dt][j] = 0.f; }
  const int wk_first = k0 + 32 * wave;
  TileLoadT<QT, D> tq, td;
  float r_lse = 0.f, r_delta = 0.f;
  for (int g = 0; g < group; ++g) {             // every query head that reads this key/value head
  const int hq = wi_head * group + g, hcq = hq * D;
  auto load_stats = [&](int qb) {
    if (tid < QT) {
      const bool ok = qb + tid < len;
      r_lse = ok ? p.lse[(size_t)hq * p.T + first + qb + tid] * LOG2E : INFINITY;   // exp2(x - inf) = 0
      r_delta = ok ? p.delta[(size_t)hq * p.T + first + qb + tid] : 0.f;
    }
  };
  tq.load(p.Q, p.ldq, first, k0, len, hcq, tid);
  td.load(p.dO, p.ldo, first, k0, len, hcq, tid);
  load_stats(k0);
  for (int qb = k0; qb < len; qb += QT) {       // queries before the block see none of its keys
    __syncthreads();
    tq.store(sQ, TP, tid);
    td.store(sD, TP, tid);
    if (tid < QT) { sLse[tid] = r_lse; sDelta[tid] = r_delta; }
    __syncthreads();
    if (qb + QT < len) {
      tq.load(p.Q, p.ldq, first, qb + QT, len, hcq, tid);
      td.load(p.dO, p.ldo, first, qb + QT, len, hcq, tid);
      load_stats(qb + QT);
    }
    if (qb + QT - 1 < wk_first) continue;     // every query of the tile lies before this wave's keys
    const bool diag = qb < wk_first + 32;        // some query of the tile lies before some key of the wave
    {
      constexpr int qt = 0;
      f32x16 s, dp;
#pragma unroll
      for (int j = 0; j < 16; ++j) { s[j] = 0.f; dp[j] = 0.f; }
#pragma unroll
      for (int st = 0; st < KS; ++st) {
        s = mma(*(const bf16x8*)(sQ + (32 * qt + li) * TP + 16 * st + 8 * half), kf[st], s);
        dp = mma(*(const bf16x8*)(sD + (32 * qt + li) * TP + 16 * st + 8 * half), *(const bf16x8*)(vfrag + 16 * st), dp);
        if (st % 2 == 1) __builtin_amdgcn_sched_barrier(0);
      }
      // P (a lane without key computes on zeros and is not stored)
#pragma unroll
      for (int j = 0; j < 16; ++j) s[j] = fast_exp2(fmaf(s[j], c, -sLse[32 * qt + tok(j, half)]));
      if (diag) {                               // only the tiles on the diagonal pay for the mask
        const int rel = kl - qb - 32 * qt - 4 * half;      // query 8 (j / 4) + j % 4 sees the key iff it is >= rel
#pragma unroll
        for (int j = 0; j < 16; ++j)
          if (8 * (j >> 2) + (j & 3) < rel) s[j] = 0.f;
      }
#pragma unroll
      for (int j = 0; j < 16; ++j) dp[j] = s[j] * (dp[j] - sDelta[32 * qt + tok(j, half)]);   // dS
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const bf16x8 pb = pack8(s, u), ds = pack8(dp, u);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          dv[dt] = mma(read_across<TP>(sD, 32 * qt + 16 * u, 32 * dt, lane), pb, dv[dt]);
          dk[dt] = mma(read_across<TP>(sQ, 32 * qt + 16 * u, 32 * dt, lane), ds, dk[dt]);
        }
        __builtin_amdgcn_sched_barrier(0);      // keeps the operand reads of the next group from piling up in registers
      }
    }
  }
  }                                             // next query head of the group
  if (kok) {
    bf16_t* krow = p.dK + (size_t)(first + kl) * p.ldk + hc;
    bf16_t* vrow = p.dV + (size_t)(first + kl) * p.ldv + hc;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int jg = 0; jg < 4; ++jg) {
        if (32 * dt + 8 * jg >= D) continue;      // the unused half of the last 32 columns
        uint2 a, b;
        a.x = pack_bf16x2(dk[dt][4 * jg + 0] * p.scale, dk[dt][4 * jg + 1] * p.scale);
        a.y = pack_bf16x2(dk[dt][4 * jg + 2] * p.scale, dk[dt][4 * jg + 3] * p.scale);
        b.x = pack_bf16x2(dv[dt][4 * jg + 0], dv[dt][4 * jg + 1]);
        b.y = pack_bf16x2(dv[dt][4 * jg + 2], dv[dt][4 * jg + 3]);
        *(uint2*)(krow + 32 * dt + 8 * jg + 4 * half) = a;
        *(uint2*)(vrow + 32 * dt + 8 * jg + 4 * half) = b;
      }
  }
}

// ------------------------------------------------------------------------------------------------ short sequences
// The whole backward of a sequence of at most R tokens (R = 64 or 128) in one workgroup: R / 32 waves, wave w owns the
// keys 32 w .. as in k_attn_bwd_kv, and since every key of a query is here, dQ needs no second pass over the scores and
// dO . O no pass of its own.  Such calls are bound by memory traffic and latency, not by the matrix cores: eight
// tensors cross the memory once (the two-kernel way reads Q, K, V, dO twice and dO, O a third time, with four launches
// in a row for it).  Per 32 queries: S, dP and dS by the waves whose keys they see; dS [keys][queries] goes through LDS, and
// the waves share dQ^T = K^T dS^T by 32-column tiles.  Two barriers a step; the next 32 queries are in flight meanwhile.
// The lane's V row stays in registers, K only in LDS (it is needed there for dQ): 68 KB of LDS at R = 128, D = 128, two
// workgroups a compute unit.  Measured, forward and backward of a call: 32 heads of 80, sequences of 64 and 128 tokens
// (2944 in all) 94 -> 71 us; 46 sequences of 64 and 32 heads of 128, 113 -> 82 us; 160 sequences of 128, 64 heads of 64,
// 931 -> 574 us.
// A workgroup of four waves takes one such sequence of up to 128 tokens and a key/value head, or two heads of one of up to
// 64 tokens (two waves each; `tid`, `stored`: the thread inside its head's waves, and false where there is no second head).
template <int D, int R>
struct ShortLds {
  static constexpr int TP = Dim<D>::TP, QT = 32, SP = QT + 16;        // SP: pitch of the dS tile
  __align__(16) bf16_t K[R * TP];
  __align__(16) bf16_t Q[QT * TP];
  __align__(16) bf16_t dO[QT * TP];
  __align__(16) bf16_t S[R * SP];
  float lse[R], delta[R];
};
template <int D, int R>
__device__ __forceinline__ void attn_bwd_short(const AttnParams& p, const int wi_block, const int wi_head, const bool stored,
                                               const int tid, ShortLds<D, R>& lds) {
  constexpr int KS = Dim<D>::KS, DT = Dim<D>::DT, DP = Dim<D>::DP, TP = Dim<D>::TP;
  constexpr int NW = R / 32, NTHR = 64 * NW, QT = 32, SP = ShortLds<D, R>::SP;
  constexpr bool LATE = D > 96;                // loads of the next tile behind the products: their registers are not free before
  bf16_t *const sK = lds.K, *const sQ = lds.Q, *const sD = lds.dO, *const sS = lds.S;
  float *const sLse = lds.lse, *const sDelta = lds.delta;
  const int32_t* blk = p.dtab + p.list_off + (p.block0 + wi_block) * DA_WORDS;
  const int first = blk[DA_FIRST_ROW], len = blk[DA_LEN];
  const int hc = wi_head * D;
  const int group = p.H / p.Hkv;
  const int wave = tid >> 6, lane = tid & 63, li = lane & 31, half = lane >> 5;
  const int kl = 32 * wave + li;               // this lane's key (and, for the statistics, its query) in the sequence
  const bool kok = kl < len;
  // dO . O (the two half-waves take alternate 16-byte pieces of the rows of query kl) and the log-sum-exp, into LDS
  auto dot = [](float s, const uint4& x, const uint4& y) {
    const uint32_t xs[4] = {x.x, x.y, x.z, x.w}, ys[4] = {y.x, y.y, y.z, y.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      s = fmaf(__uint_as_float(xs[q] << 16), __uint_as_float(ys[q] << 16), s);
      s = fmaf(__uint_as_float(xs[q] & 0xffff0000u), __uint_as_float(ys[q] & 0xffff0000u), s);
    }
    return s;
  };
  auto piece = [&](const bf16_t* base, int hq, int st) {
    return kok ? *(const uint4*)(base + (size_t)(first + kl) * p.ldo + hq * D + 8 * half + 16 * st) : uint4{0u, 0u, 0u, 0u};
  };
  auto load_lse = [&](int hq) {
    return kok ? p.lse[(size_t)hq * p.T + first + kl] * LOG2E : INFINITY;            // exp2(x - inf) = 0
  };
  auto store_stats = [&](float s, float lse2) {
    s += __shfl_xor(s, 32);
    if (half == 0) { sDelta[kl] = s; sLse[kl] = lse2; }
  };
  TileLoadT<QT, D, NTHR> tq, td;
  bf16x8 vf[KS];
  {
    TileLoadT<R, D, NTHR> t;
    t.load(p.K, p.ldk, first, 0, len, hc, tid);
    uint4 xd[KS], xo[KS];                      // every load of the prologue is on its way before the first wait
#pragma unroll
    for (int st = 0; st < KS; ++st) { xd[st] = piece(p.dO, wi_head * group, st); xo[st] = piece(p.O, wi_head * group, st); }
    const float lse2 = load_lse(wi_head * group);
    tq.load(p.Q, p.ldq, first, 0, len, wi_head * group * D, tid);
    td.load(p.dO, p.ldo, first, 0, len, wi_head * group * D, tid);
    const bf16_t* vrow = p.V + (size_t)(first + kl) * p.ldv + hc + 8 * half;
#pragma unroll
    for (int s = 0; s < KS; ++s) vf[s] = kok ? *(const bf16x8*)(vrow + 16 * s) : zero8();
    zero_pad_columns<D, DP, NTHR>(sK, R, TP, tid);
    zero_pad_columns<D, DP, NTHR>(sQ, QT, TP, tid);
    zero_pad_columns<D, DP, NTHR>(sD, QT, TP, tid);
    t.store(sK, TP, tid);
    float sum = 0.f;
#pragma unroll
    for (int st = 0; st < KS; ++st) sum = dot(sum, xd[st], xo[st]);
    store_stats(sum, lse2);
  }
  const bf16_t* kfrag = sK + kl * TP + 8 * half;
  const float c = p.scale * LOG2E;
  f32x16 dk[DT], dv[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int j = 0; j < 16; ++j) { dk[dt][j] = 0.f; dv[dt][j] = 0.f; }
  for (int g = 0; g < group; ++g) {            // every query head that reads this key/value head
    const int hq = wi_head * group + g, hcq = hq * D;
    if (g > 0) {                               // (every read of the last head's statistics lies before its last barrier)
      float sum = 0.f;
#pragma unroll 2
      for (int st = 0; st < KS; ++st) sum = dot(sum, piece(p.dO, hq, st), piece(p.O, hq, st));
      store_stats(sum, load_lse(hq));
    }
    for (int qb = 0; qb < len; qb += QT) {
      tq.store(sQ, TP, tid);                   // (every wave is past its reads of the last tile: the second barrier below)
      td.store(sD, TP, tid);
      __syncthreads();
      // the next 32 queries, of this head or of the next one
      auto load_next = [&]() {
        const bool more = qb + QT < len;
        const int gn = more ? g : g + 1, qn = more ? qb + QT : 0;
        if (gn < group) {
          tq.load(p.Q, p.ldq, first, qn, len, (wi_head * group + gn) * D, tid);
          td.load(p.dO, p.ldo, first, qn, len, (wi_head * group + gn) * D, tid);
        }
      };
      if (!LATE) load_next();
      if (qb + QT - 1 >= 32 * wave) {          // some query of the tile sees a key of this wave
        f32x16 s, dp;
#pragma unroll
        for (int j = 0; j < 16; ++j) { s[j] = 0.f; dp[j] = 0.f; }
#pragma unroll
        for (int st = 0; st < KS; ++st) {
          s = mma(*(const bf16x8*)(sQ + li * TP + 16 * st + 8 * half), *(const bf16x8*)(kfrag + 16 * st), s);
          dp = mma(*(const bf16x8*)(sD + li * TP + 16 * st + 8 * half), vf[st], dp);
          // (the operand reads would pile up in registers, and beyond them: 53 heads of 96, 30 x 120 and 10 x 50 tokens 166.2 us, 163.8 so)
          if ((D > 96 || (D == 96 && R == 64)) && st % 2 == 1) __builtin_amdgcn_sched_barrier(0);
        }
        // P (keys past the sequence come after every query: the mask takes them)
#pragma unroll
        for (int j = 0; j < 16; ++j) s[j] = fast_exp2(fmaf(s[j], c, -sLse[qb + tok(j, half)]));
        if (qb < 32 * wave + 32) {             // only the tile on the diagonal pays for the mask
          const int rel = kl - qb - 4 * half;  // query 8 (j / 4) + j % 4 sees the key iff it is >= rel
#pragma unroll
          for (int j = 0; j < 16; ++j)
            if (8 * (j >> 2) + (j & 3) < rel) s[j] = 0.f;
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) dp[j] = s[j] * (dp[j] - sDelta[qb + tok(j, half)]);   // dS
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const bf16x8 pb = pack8(s, u), ds = pack8(dp, u);
          // the same eight values of dS, queries 16 u + 4 half + {0..3, 8..11} of this lane's key
          const uint4 w = __builtin_bit_cast(uint4, ds);
          *(uint2*)(sS + kl * SP + 16 * u + 4 * half) = uint2{w.x, w.y};
          *(uint2*)(sS + kl * SP + 16 * u + 4 * half + 8) = uint2{w.z, w.w};
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) {
            dv[dt] = mma(read_across<TP>(sD, 16 * u, 32 * dt, lane), pb, dv[dt]);
            dk[dt] = mma(read_across<TP>(sQ, 16 * u, 32 * dt, lane), ds, dk[dt]);
          }
          if (D > 96) __builtin_amdgcn_sched_barrier(0);
        }
      }
      if (LATE) load_next();
      __syncthreads();
      // dQ of the tile: keys 0 .. qb + 31, this wave's 32-column tiles of the head dimension
      for (int dt = wave; dt < DT; dt += NW) {
        f32x16 dq;
#pragma unroll
        for (int j = 0; j < 16; ++j) dq[j] = 0.f;
        for (int k16 = 0; k16 < qb + QT; k16 += 16)
          dq = mma(read_across<TP>(sK, k16, 32 * dt, lane), read_across<SP>(sS, k16, 0, lane), dq);
        if (stored && qb + li < len) {
          bf16_t* orow = p.dQ + (size_t)(first + qb + li) * p.ldq + hcq + 32 * dt + 4 * half;
#pragma unroll
          for (int jg = 0; jg < 4; ++jg) {
            if (32 * dt + 8 * jg >= D) continue;
            uint2 v;
            v.x = pack_bf16x2(dq[4 * jg + 0] * p.scale, dq[4 * jg + 1] * p.scale);
            v.y = pack_bf16x2(dq[4 * jg + 2] * p.scale, dq[4 * jg + 3] * p.scale);
            *(uint2*)(orow + 8 * jg) = v;
          }
        }
      }
    }
  }                                             // next query head of the group
  if (stored && kok) {
    bf16_t* krow = p.dK + (size_t)(first + kl) * p.ldk + hc;
    bf16_t* vrow = p.dV + (size_t)(first + kl) * p.ldv + hc;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int jg = 0; jg < 4; ++jg) {
        if (32 * dt + 8 * jg >= D) continue;
        uint2 a, b;
        a.x = pack_bf16x2(dk[dt][4 * jg + 0] * p.scale, dk[dt][4 * jg + 1] * p.scale);
        a.y = pack_bf16x2(dk[dt][4 * jg + 2] * p.scale, dk[dt][4 * jg + 3] * p.scale);
        b.x = pack_bf16x2(dv[dt][4 * jg + 0], dv[dt][4 * jg + 1]);
        b.y = pack_bf16x2(dv[dt][4 * jg + 2], dv[dt][4 * jg + 3]);
        *(uint2*)(krow + 32 * dt + 8 * jg + 4 * half) = a;
        *(uint2*)(vrow + 32 * dt + 8 * jg + 4 * half) = b;
      }
  }
}

// Blocks block0 .. + n_blocks of the list, sequences of 65 to 128 tokens, and the n_blocks64 of at most 64 tokens behind them,
// in one launch: a workgroup loads, computes and stores, and in a launch of one kind all of them do so at the same time; two
// kinds fill each other's gaps.  Two heads a workgroup: the heads of a sequence lie side by side, and half as many workgroups
// pass through the dispatcher.  Forward and backward, a launch for each kind, one head a workgroup -> so: 32 heads of 80, 14
// sequences of 128 tokens and 18 of 64, 62.3 -> 54.4 us; 160 of 64, 224 -> 192; 53 heads of 96, 20 each of 128, 100, 60 and 33
// tokens, 259 -> 245; 40 heads of 64, the same, 131.8 -> 122.
template <int D>
__global__ __launch_bounds__(256, 2) void k_attn_bwd_short(AttnParams p) {
  typedef ShortLds<D, 128> Wide;
  typedef ShortLds<D, 64> Narrow;
  static_assert(4 * sizeof(Narrow) <= 160 * 1024, "two workgroups a compute unit");
  __shared__ __align__(16) unsigned char mem[sizeof(Wide) > 2 * sizeof(Narrow) ? sizeof(Wide) : 2 * sizeof(Narrow)];
  int block, head;
  if (blockIdx.x < (unsigned)p.grid128) {
    if (short_item<D>(blockIdx.x, p.n_blocks, p.Hkv, block, head))
      attn_bwd_short<D, 128>(p, block, head, true, threadIdx.x, *(Wide*)mem);
  } else if (short_item<D>(blockIdx.x - p.grid128, p.n_blocks64, (p.Hkv + 1) / 2, block, head)) {
    const int unit = threadIdx.x >> 7, h = 2 * head + unit;
    attn_bwd_short<D, 64>(p, p.n_blocks + block, h < p.Hkv ? h : p.Hkv - 1, h < p.Hkv, threadIdx.x & 127, ((Narrow*)mem)[unit]);
  }
}
// One head a workgroup: D = 128 (two heads of 64 tokens would take 87 KB of LDS, one workgroup a unit; a launch for each kind), and
// launches of few heads.
template <int D, int R>
__global__ __launch_bounds__(2 * R, 2) void k_attn_bwd_short_one(AttnParams p) {
  __shared__ ShortLds<D, R> lds;
  int block, head;
  if (short_item<D>(blockIdx.x, R == 128 ? p.n_blocks : p.n_blocks64, p.Hkv, block, head))
    attn_bwd_short<D, R>(p, (R == 128 ? 0 : p.n_blocks) + block, head, true, threadIdx.x, lds);
}

mux_status check(const char* fn, const mux_attn_desc* d, const mux_segtab* st) {
  if (!d || !st) return fail(MUX_ERR_INVALID_ARG, std::string(fn) + ": null descriptor or table");
  if (d->n_heads < 1 || d->n_kv_heads < 1 || d->head_dim < 1) return fail(MUX_ERR_INVALID_ARG, std::string(fn) + ": bad head counts");
  if (d->n_heads % d->n_kv_heads) return fail(MUX_ERR_INVALID_ARG, std::string(fn) + ": n_kv_heads must divide n_heads");
  const int D = d->head_dim;
  if (d->dtype != MUX_DT_BF16 || (D != 64 && D != 80 && D != 96 && D != 128))
    return fail(MUX_ERR_UNSUPPORTED, std::string(fn) + ": only bf16 and head_dim 64, 80, 96 and 128 are built");
  const int64_t w = (int64_t)d->n_heads * D, wkv = (int64_t)d->n_kv_heads * D;
  const int64_t lds[4] = {d->ldq, d->ldk, d->ldv, d->ldo};
  for (int i = 0; i < 4; ++i) {
    const int64_t ld = lds[i];
    if (ld < (i == 1 || i == 2 ? wkv : w)) return fail(MUX_ERR_SHAPE, std::string(fn) + ": a leading dimension is smaller than its heads * head_dim");
    if (ld % 8) return fail(MUX_ERR_UNSUPPORTED, std::string(fn) + ": leading dimensions must be multiples of 8");
    if ((int64_t)st->T * ld >= ((int64_t)1 << 40)) return fail(MUX_ERR_SHAPE, std::string(fn) + ": problem too large");
  }
  if ((int64_t)st->n_attn_blocks * d->n_heads >= ((int64_t)1 << 31)) return fail(MUX_ERR_SHAPE, std::string(fn) + ": too many work items");
  if (!(d->scale >= 0.f)) return fail(MUX_ERR_INVALID_ARG, std::string(fn) + ": negative scale");
  return MUX_OK;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// One launch of kernel template K<D> for the head dimension of the call.
#define ATTN_LAUNCH(name, K, D, grid, stream, p)                                           \
  do {                                                                                     \
    if ((D) == 128) MUX_LAUNCH(name, K<128>, grid, dim3(256), 0, stream, p);               \
    else if ((D) == 96) MUX_LAUNCH(name, K<96>, grid, dim3(256), 0, stream, p);            \
    else if ((D) == 80) MUX_LAUNCH(name, K<80>, grid, dim3(256), 0, stream, p);            \
    else MUX_LAUNCH(name, K<64>, grid, dim3(256), 0, stream, p);                           \
  } while (0)
// Workgroups of a launch whose pairs short_item hands out
unsigned short_grid(int n_blocks, int n_heads, int D) {
  const bool dealt = n_heads % 8 != 0 && short_deals_blocks(D, n_blocks);
  return (unsigned)(dealt ? (n_blocks + 7) / 8 * 8 : n_blocks) * (unsigned)n_heads;
}

// Which blocks of the list (it runs from the longest sequence to the shortest) the backward takes how: n_long in the
// kernels of any length, then n128 in the one-kernel backward of up to 128 tokens, then n64 in that of up to 64.
void plan_backward(const mux_segtab* st, const mux_attn_desc* desc, int& n_long, int& n128, int& n64) {
  n64 = st->n_attn_blocks64; n128 = st->n_attn_blocks128;
  n_long = st->n_attn_blocks - n64 - n128;
  const int64_t hkv = desc->n_kv_heads, group = desc->n_heads / desc->n_kv_heads;
  // A workgroup of the one-kernel backward walks the query heads of its key/value head one after the other and forms dQ
  // for each, which the kernels of any length spread over a workgroup a query head.  So it pays with short groups of short
  // rows, or with enough workgroups (one for two compute units, of the narrow ones one for each) that the chip has work
  // meanwhile.  Forward and backward, kernels of any length -> one kernel, D = 128: group 2, 4 x 128 tokens (64 workgroups)
  // 48.9 -> 41.3 us; group 3, 1 x 128 (4) 51.7 -> 54.3; group 8, 16 x 128 tokens (64) 118.6 -> 126.9, 32 x 128 (128) 147 -> 139, 64 x 128 (256) 212 -> 174; group 32,
  // 64 x 128 (64) 402 -> 484, 128 x 128 (128) 609 -> 549; 64 tokens: group 4, 8 x 64 (64) 41.9 -> 43.8, group 8, 32 x 64 (128)
  // 86.4 -> 95.6, 64 x 64 (256) 121 -> 108.  D = 96: group 3, 4 x 128 (32) 42.3 -> 40.5.  D = 80: group 4, 4 x 128 (16)
  // 44.8 -> 48.1.  D = 64: group 4, 2 x 64 (8) 25.3 -> 23.6, 4 x 128 (16) 38.2 -> 40.0; group 16, 64 x 128 (64) 121 -> 141.
  auto pays = [&](int n, int tokens) {
    return (group * desc->head_dim <= 288 && (group <= 3 || tokens == 64)) ||
           n * hkv >= (tokens == 128 ? kComputeUnits / 2 : kComputeUnits);
  };
  const int64_t fill = 2 * kComputeUnits;      // two workgroups a compute unit
  // Beside longer sequences the short ones fill the gaps of the launches those need anyway.  Launches of their own pay
  // where they are many and the longer ones are soon done: 64 x 128 tokens beside one sequence of 256, 1024, 4096 tokens, 32
  // heads of 128: riding 377, 408, 1140 us, apart 307, 386, 1166; 32 heads of 64, 100 x 100 tokens beside 512: 216 and 235;
  // 20 heads of 64, 204 x 128 beside 1024: 380 and 350, 102 x 128 beside 3 x 2048: 425 and 488.  With groups, which gain
  // least at 64 tokens: 8 groups of 4 heads of 128, 256 x 128 tokens beside 256, 1024, 4096: riding 909, 924, 1910, apart
  // 809, 997, 2041; 200 x 50 beside 4 x 200: 365 and 411.
  const int64_t weight = (group == 1 ? n64 + n128 : n128) * hkv * desc->head_dim / 128;      // workgroups, in those of 128 columns
  if (n_long > 0 && weight < (group == 1 && st->attn_longest <= 1024 ? 7 * kComputeUnits : 4 * (int64_t)st->attn_longest)) {
    n_long += n64 + n128;
    n64 = n128 = 0;
  }
  // Narrower workgroups for at most 64 tokens where they fill the chip, and so does what they leave to the others (128 x 64
  // tokens and 128, 8 groups of 4 heads of 128: 263 us in two launches, 185 in one; 51 x 64 tokens and 12 x 128, 20 heads of 64:
  // 53 and 65).  D < 128, where both kinds share a launch, all in the wide ones, two kinds: 32 heads of 80, 14 x 120 and 6 x 50
  // tokens 62.5 us, 66.0, 30 and 10 96.9, 100.4; 24 of 96, 30 and 10 84.1, 85.5; 20 of 64, 14 and 12 43.9, 44.7, but 14 and 18 58.1, 49.5.
  if (n128 > 0 && (n64 * hkv < fill || !pays(n128, 128))) { n128 += n64; n64 = 0; }
  if ((n128 > 0 && !pays(n128, 128)) || (n64 > 0 && !pays(n64, 64))) { n_long += n64 + n128; n64 = n128 = 0; }
}

mux_status last_hip(const char* fn) {
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(MUX_ERR_DEVICE, std::string(fn) + ": " + hipGetErrorString(e));
  return MUX_OK;
}

}  // namespace
}  // namespace mux

using namespace mux;

extern "C" size_t mux_attn_saved_bytes(const mux_attn_desc* desc, const mux_segtab* st) {
  if (!desc || !st || desc->n_heads < 1) return 0;
  return align256((size_t)st->T * (size_t)desc->n_heads * sizeof(float));
}

extern "C" size_t mux_attn_workspace_bytes(const mux_attn_desc* desc, const mux_segtab* st) {
  return mux_attn_saved_bytes(desc, st);
}

extern "C" mux_status mux_attn_forward(const mux_attn_desc* desc, const mux_segtab* st, const void* dev_segtab,
                                       const void* Q, const void* K, const void* V, void* O, void* saved,
                                       void* hip_stream) {
  static const char* fn = "mux_attn_forward";
  if (mux_status s = check(fn, desc, st)) return s;
  if (st->T == 0) return MUX_OK;
  if (!dev_segtab || !Q || !K || !V || !O) return fail(MUX_ERR_INVALID_ARG, std::string(fn) + ": null device pointer");
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O))
    return fail(MUX_ERR_UNSUPPORTED, std::string(fn) + ": pointers must be 16-byte aligned");
  hipStream_t stream = (hipStream_t)hip_stream;
  const int D = desc->head_dim;
  AttnParams p{};
  p.dtab = (const int32_t*)dev_segtab;
  p.Q = (const bf16_t*)Q; p.K = (const bf16_t*)K; p.V = (const bf16_t*)V; p.Out = (bf16_t*)O;
  p.lse = (float*)saved;
  p.ldq = desc->ldq; p.ldk = desc->ldk; p.ldv = desc->ldv; p.ldo = desc->ldo;
  p.T = st->T; p.H = desc->n_heads; p.Hkv = desc->n_kv_heads;
  p.scale = desc->scale > 0.f ? desc->scale : 1.f / sqrtf((float)D);
  p.n_blocks = st->n_attn_blocks;
  p.list_off = st->dev_image[DH_ATT_OFF_FWD];
  ZeroParams z{};
  z.dtab = p.dtab; z.out[0] = (bf16_t*)O; z.ld[0] = desc->ldo; z.n_out = 1; z.width[0] = desc->n_heads * D;
  if (st->valid_total < st->T)                // a table without padding rows has nothing to clear
    MUX_LAUNCH("attn_zero_pad", k_attn_zero_pad, dim3((unsigned)st->items[0].size(), (unsigned)((z.width[0] + 2047) / 2048)), dim3(256), 0, stream, z);
  // Only short sequences and a multiple of eight heads: dealt as in the backward where neighbouring heads share cache lines,
  // heads share keys and values, or the pairs are many, eight a compute unit (40 heads of 80, 16 x 64 tokens 10.2 -> 9.5 us;
  // 8 groups of 4 heads of 128, 64 x 64, 30.3 -> 25.8; 32 heads of 128, 128 x 128, 145 -> 130, but 24 x 128 22.1 -> 24.2; with 28 heads of 128 or 53
  // of 96 no way of keeping the heads of a sequence together beat the block running fastest: 60 x 100 and 60 x 30 tokens 56.5 us,
  // contiguous runs 75.8, blocks dealt in turn 60.0).
  p.short_map = st->n_attn_blocks64 + st->n_attn_blocks128 == st->n_attn_blocks && p.H % 8 == 0 &&
                (D % 64 != 0 || p.H > p.Hkv || (int64_t)st->n_attn_blocks * p.H >= 8 * kComputeUnits);
  if (st->n_attn_blocks > 0)
    ATTN_LAUNCH("attn_fwd", k_attn_fwd, D, dim3((unsigned)st->n_attn_blocks * (unsigned)desc->n_heads), stream, p);
  return last_hip(fn);
}

extern "C" mux_status mux_attn_backward(const mux_attn_desc* desc, const mux_segtab* st, const void* dev_segtab,
                                        const void* Q, const void* K, const void* V, const void* O, const void* dO,
                                        const void* saved, void* dQ, void* dK, void* dV, void* ws, size_t ws_bytes,
                                        void* hip_stream) {
  static const char* fn = "mux_attn_backward";
  if (mux_status s = check(fn, desc, st)) return s;
  if (st->T == 0) return MUX_OK;
  if (!dev_segtab || !Q || !K || !V || !O || !dO || !saved || !dQ || !dK || !dV || !ws)
    return fail(MUX_ERR_INVALID_ARG, std::string(fn) + ": null device pointer");
  const void* ptrs[8] = {Q, K, V, O, dO, dQ, dK, dV};
  for (const void* q : ptrs)
    if (!aligned16(q)) return fail(MUX_ERR_UNSUPPORTED, std::string(fn) + ": pointers must be 16-byte aligned");
  if (ws_bytes < mux_attn_workspace_bytes(desc, st)) return fail(MUX_ERR_WORKSPACE, std::string(fn) + ": workspace too small");
  hipStream_t stream = (hipStream_t)hip_stream;
  const int D = desc->head_dim;
  AttnParams p{};
  p.dtab = (const int32_t*)dev_segtab;
  p.Q = (const bf16_t*)Q; p.K = (const bf16_t*)K; p.V = (const bf16_t*)V; p.O = (const bf16_t*)O; p.dO = (const bf16_t*)dO;
  p.dQ = (bf16_t*)dQ; p.dK = (bf16_t*)dK; p.dV = (bf16_t*)dV;
  p.lse = (float*)saved; p.delta = (float*)ws;
  p.ldq = desc->ldq; p.ldk = desc->ldk; p.ldv = desc->ldv; p.ldo = desc->ldo;
  p.T = st->T; p.H = desc->n_heads; p.Hkv = desc->n_kv_heads;
  p.scale = desc->scale > 0.f ? desc->scale : 1.f / sqrtf((float)D);
  ZeroParams z{};
  z.dtab = p.dtab; z.n_out = 3;
  z.width[0] = desc->n_heads * D; z.width[1] = z.width[2] = desc->n_kv_heads * D;
  z.out[0] = p.dQ; z.ld[0] = desc->ldq; z.out[1] = p.dK; z.ld[1] = desc->ldk; z.out[2] = p.dV; z.ld[2] = desc->ldv;
  if (st->valid_total < st->T)
    MUX_LAUNCH("attn_zero_pad", k_attn_zero_pad, dim3((unsigned)st->items[0].size(), (unsigned)((z.width[0] + 2047) / 2048)), dim3(256), 0, stream, z);
  int n64 = 0, n128 = 0, n_long = 0;
  plan_backward(st, desc, n_long, n128, n64);
  p.list_off = st->dev_image[DH_ATT_OFF_BWD];
  if (n_long > 0) {
    const size_t n = (size_t)st->T * desc->n_heads;
    p.n_blocks = n_long;
    ATTN_LAUNCH("attn_delta", k_attn_delta, D, dim3((unsigned)(((n + 3) / 4 * 16 + 255) / 256)), stream, p);
    ATTN_LAUNCH("attn_bwd_kv", k_attn_bwd_kv, D, dim3((unsigned)n_long * (unsigned)desc->n_kv_heads), stream, p);
    AttnParams q = p;
    q.list_off = st->dev_image[DH_ATT_OFF_FWD];
    ATTN_LAUNCH("attn_bwd_q", k_attn_bwd_q, D, dim3((unsigned)n_long * (unsigned)desc->n_heads), stream, q);
  }
  if (n128 + n64 > 0) {
    p.block0 = n_long;
    p.n_blocks = n128; p.n_blocks64 = n64;
    const unsigned one64 = n64 > 0 ? short_grid(n64, desc->n_kv_heads, D) : 0;
    if (D == 128) {
      if (n128 > 0) MUX_LAUNCH("attn_bwd_128", (k_attn_bwd_short_one<128, 128>), dim3(short_grid(n128, desc->n_kv_heads, D)), dim3(256), 0, stream, p);
      if (n64 > 0) MUX_LAUNCH("attn_bwd_64", (k_attn_bwd_short_one<128, 64>), dim3(one64), dim3(128), 0, stream, p);
    } else if (n128 == 0 && (int64_t)n64 * desc->n_kv_heads * D < (D == 64 ? 2048 : 1536) * (int64_t)kComputeUnits) {
      // Nothing but sequences of at most 64 tokens: two heads a workgroup move whole lines where there is enough to move
      // (48 MB a tensor of full sequences; 64 MB of heads of 64, whose rows are whole lines); below, a workgroup of twice the
      // waves finds its place later.  Forward and backward,
      // one head, two: 16 heads of 96, 40 x 50 tokens 45.2 us, 47.7; 40 of 96, 80 x 50 110.4, 115.2; 24 of 96, 160 x 50 119.7,
      // 119.3; 53 of 96, 80 x 50 153.1, 150.5, 160 x 64 358.7, 336.5; 33 of 80, 80 x 64 79.1, 82.6, 160 x 64 190.8, 183.3; 32 of 80, 160 x
      // 64 229.9, 195.9; 40 of 64, 80 x 50 81.9, 86.0, 160 x 50 133.8, 144.8, 300 x 64 362.6, 333.3; 8 groups of 4 heads of 64, 160 x 64 85.7, 92.1.
      if (D == 96) MUX_LAUNCH("attn_bwd_64", (k_attn_bwd_short_one<96, 64>), dim3(one64), dim3(128), 0, stream, p);
      else if (D == 80) MUX_LAUNCH("attn_bwd_64", (k_attn_bwd_short_one<80, 64>), dim3(one64), dim3(128), 0, stream, p);
      else MUX_LAUNCH("attn_bwd_64", (k_attn_bwd_short_one<64, 64>), dim3(one64), dim3(128), 0, stream, p);
    } else {
      p.grid128 = n128 > 0 ? (int)short_grid(n128, desc->n_kv_heads, D) : 0;
      const char* name = n64 == 0 ? "attn_bwd_128" : (n128 == 0 ? "attn_bwd_64" : "attn_bwd_128_64");
      const dim3 grid((unsigned)p.grid128 + (n64 > 0 ? short_grid(n64, (desc->n_kv_heads + 1) / 2, D) : 0));
      if (D == 96) MUX_LAUNCH(name, k_attn_bwd_short<96>, grid, dim3(256), 0, stream, p);
      else if (D == 80) MUX_LAUNCH(name, k_attn_bwd_short<80>, grid, dim3(256), 0, stream, p);
      else MUX_LAUNCH(name, k_attn_bwd_short<64>, grid, dim3(256), 0, stream, p);
    }
  }
  return last_hip(fn);
}
