// The consumer of X_b: GraphSAGE layers with the mean aggregator over the
// sampled blocks of a window (Algorithm 1 forward pass; Sec. VI-A model), all
// W batches of the window at once.
//
// Three launches prepare a call (four on graphs of more than 4.2M nodes): the
// rank prefixes of the N_b bit sets and the weights in matrix-core order
// (k_sage_prepare), each node's place in its own level (k_sage_places), and for
// every output node the input rows of itself and of its neighbours (k_sage_rows,
// every level in one launch).  Random lookups run there, with one thread each,
// and not in front of the row reads.  Then each layer,
// out_v = act(W_self^T h_v + W_neigh^T mean_{u in S(v)} h_u + bias), takes one
// of two forms (use_projection says which):
//  * k_sage_layer: a block gathers [h_v | mean h_u] of 32 or 64 output nodes
//    into LDS, up to 128 columns at a time, and multiplies them on the fp32
//    matrix cores (v_mfma_f32_16x16x4f32) by weights that come from L2 to
//    registers.  Nothing is projected that no output needs, and no projected row
//    goes through memory;
//  * k_sage_project and k_sage_mean: Z = H [W_self | W_neigh] for every input
//    row, then the mean of projected rows, which commutes with the linear
//    map: where rows are wide and outputs narrow, each input row is read once
//    and the random reads are of 128-byte rows.
//
// A node's row in level N_b is its rank in the batch's N_b bit set: the set bits
// before its chunk of 65,536 nodes, those of the chunk before its group of 128,
// and popcounts of the bits before it there.  In other levels it is its position
// in the ascending frontier, which k_sage_places notes at the node's N_b row.
#include <hip/hip_fp16.h>

#include "gg_host.hpp"

namespace gg {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));

constexpr int kSageBlock = 256;          // 4 waves
constexpr int kTileRows = 64;            // 16 rows per wave
constexpr int kGroup = 16;               // columns of the left operand per MFMA group
constexpr int kWLdsBytes = 65536;        // weights of k_sage_project in LDS at most
constexpr int kRankWords = 4;            // bit-set words per rank prefix
constexpr int kRankChunk = kSageBlock * 2 * kRankWords;   // words per rank chunk
constexpr int kMaxPitch = GG_MAX_FANOUT + 1;
static_assert(kRankChunk == kChunkWords, "rank chunks divide gg_bits_words");

// Packed weights of one layer: for MFMA group q, then W_self and W_neigh, then
// column tile t, lane l's four values W[k0 + e][16 t + l % 16], e = 0..3 (zero
// past the layer's sizes; k0 = 16 q + 4 (l / 16)): one 16-byte read feeds
// four MFMA steps.
struct PackArgs {
  const float* w[GG_MAX_LAYERS][2];
  int32_t d_in[GG_MAX_LAYERS], d_out[GG_MAX_LAYERS], nt[GG_MAX_LAYERS];
  int64_t first[GG_MAX_LAYERS + 1];   // first packed f32x4 of each layer
  int32_t L;
};

// Blocks below nch * W: the rank prefixes within chunk c of batch b (rank[w / 4]
// = set bits of the chunk before word w) and its bits (chunk[b * nch + c]).  The
// other blocks pack the weights.
__global__ void __launch_bounds__(kSageBlock) k_sage_prepare(const uint32_t* bits, int32_t nch,
                                                             int32_t W, int2* rank, int32_t* chunk,
                                                             PackArgs pk, f32x4* packed) {
  __shared__ int32_t lds[kSageBlock / kWave];
  const int64_t nrank = (int64_t)nch * W;
  if ((int64_t)blockIdx.x < nrank) {
    const int64_t bc = blockIdx.x;   // b * nch + c: the chunks of all sets back to back
    const u32x4* p = (const u32x4*)(bits + bc * kRankChunk) + threadIdx.x * 2;
    const u32x4 x = p[0], y = p[1];
    const int32_t sx = __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w);
    const int32_t sy = __popc(y.x) + __popc(y.y) + __popc(y.z) + __popc(y.w);
    int32_t tot;
    const int32_t before = block_excl_scan<kSageBlock>(sx + sy, lds, &tot);
    rank[bc * kSageBlock + threadIdx.x] = make_int2(before, before + sx);
    if (threadIdx.x == 0) chunk[bc] = tot;
    return;
  }
  const int64_t total = pk.first[pk.L];
  for (int64_t i = (blockIdx.x - nrank) * kSageBlock + threadIdx.x; i < total;
       i += (gridDim.x - nrank) * kSageBlock) {
    int j = 0;
    while (j + 1 < pk.L && i >= pk.first[j + 1]) ++j;
    const int32_t e = (int32_t)(i - pk.first[j]);
    const int nt = pk.nt[j], lane = e % kWave, r = e / kWave;
    const int t = r % nt, sn = r / nt % 2, q = r / nt / 2;
    const int col = t * 16 + (lane & 15), k0 = q * kGroup + 4 * (lane >> 4);
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (col < pk.d_out[j])
#pragma unroll
      for (int a = 0; a < 4; ++a)
        if (k0 + a < pk.d_in[j]) v[a] = pk.w[j][sn][(int64_t)(k0 + a) * pk.d_out[j] + col];
    packed[i] = v;
  }
}

// Exclusive scan of each batch's chunk bits, one block per batch: for
// more chunks than a wave scans at once.  Up to 64 (graphs of 4.2M nodes) the
// blocks of the first kernel that looks ranks up scan them into LDS themselves
// (chunk_starts), and one of them leaves the result for the next kernel: a launch
// for it took 4 of the 36 us of a pass over 68K rows of 12 columns.
constexpr int kChunkBlock = 1024;
__global__ void __launch_bounds__(kChunkBlock) k_sage_chunks(const int32_t* chunk, int32_t* first,
                                                             int32_t nch) {
  __shared__ int32_t lds[kChunkBlock / kWave];
  const int64_t at = (int64_t)blockIdx.x * nch;
  int32_t carry = 0;
  for (int32_t i0 = 0; i0 < nch; i0 += kChunkBlock) {
    const int32_t i = i0 + threadIdx.x;
    const int32_t v = i < nch ? chunk[at + i] : 0;
    int32_t tot;
    const int32_t before = block_excl_scan<kChunkBlock>(v, lds, &tot);
    if (i < nch) first[at + i] = carry + before;
    carry += tot;
  }
}

// ---------------------------------------------------------------------------
// Input rows of every output node.
// ---------------------------------------------------------------------------
struct RowsArgs {
  int32_t W, L;
  int32_t k[GG_MAX_LAYERS];            // by level
  uint32_t kmagic[GG_MAX_LAYERS];      // div_magic(k + 1)
  int32_t* table[GG_MAX_LAYERS];       // [rows of level l][k + 1]: self, then the slots
  int32_t* place[GG_MAX_LAYERS];       // level l >= 1: N_b row -> position in the batch's F_l
  const int32_t* fids;
  const int64_t* off;                  // frontier_off
  const int32_t* nbr;
  const int64_t* noff;
  const uint32_t* bits;
  const int32_t* rank;                 // set bits of the chunk before each 128-bit group
  const int32_t* chunk;                // bits of each chunk
  int32_t* before;                     // bits of the batch's set before each chunk
  int32_t nch;
  int64_t wpb;
  int64_t rows_cap;
};

// One batch's part of a level: where its entries, its slots, its N_b and its
// ranks lie.
struct Batch {
  int64_t out0, out1;      // entries of the output level, relative to the level's first
  int64_t in0, nin;        // entries of the input level: first (absolute), count
  int64_t nb0, nnb;        // N_b: first row, count
  int64_t slot0, nslot;    // the hop's neighbour slots: first (absolute), count
  const u32x4* bits;       // 128-bit groups of the batch's set
  const int32_t* rank;     // set bits of the chunk before each group
  int32_t chunk0;          // first chunk among all batches'
};

__device__ __forceinline__ Batch batch_at(const RowsArgs& a, int lvl, int b) {
  const int64_t s = (int64_t)lvl * a.W + b, sn = (int64_t)a.L * a.W;
  Batch t;
  const int64_t o0 = a.off[(int64_t)lvl * a.W];
  t.out0 = a.off[s] - o0;
  t.out1 = a.off[s + 1] - o0;
  t.in0 = a.off[s + a.W];
  t.nin = a.off[s + a.W + 1] - t.in0;
  t.nb0 = a.off[sn + b] - a.off[sn];
  t.nnb = a.off[sn + b + 1] - a.off[sn + b];
  t.slot0 = a.noff[s];
  t.nslot = a.noff[s + 1] - t.slot0;
  t.bits = (const u32x4*)(a.bits + (int64_t)b * a.wpb);
  t.rank = a.rank + (int64_t)b * (a.wpb / kRankWords);
  t.chunk0 = b * a.nch;
  return t;
}

// Batch of entry r of the level (off: the level's W + 1 offsets in LDS,
// relative, padded with INT64_MAX).
__device__ __forceinline__ int batch_of(const int64_t* off, int64_t r) {
  int b = 0;
#pragma unroll
  for (int step = 32; step >= 1; step >>= 1)
    if (off[b + step] <= r) b += step;
  return b;
}

// Rank of u among the set's n bits, from its 128-bit group and the bits before
// that group; -1 when its bit is clear.
__device__ __forceinline__ int64_t rank_in(u32x4 x, int32_t pre, int32_t u, int64_t n) {
  const uint32_t w[kRankWords] = {x.x, x.y, x.z, x.w};
  const uint32_t in = ((uint32_t)u >> 5) % kRankWords, bit = 1u << (u & 31);
  uint32_t mine = 0;
  int32_t before = 0;
#pragma unroll
  for (uint32_t j = 0; j < kRankWords; ++j) {
    before += j < in ? __popc(w[j]) : 0;
    mine = j == in ? w[j] : mine;
  }
  const int64_t r = (int64_t)pre + before + __popc(mine & (bit - 1u));
  return (mine & bit) && r < n ? r : -1;
}

// Set bits of the batch's set before its chunk c: in LDS (HERE) or in a.before.
template <bool HERE>
__device__ __forceinline__ int32_t chunk_first(const RowsArgs& a, const int32_t* s_chunk,
                                               const Batch& t, uint32_t c) {
  return HERE ? s_chunk[t.chunk0 + c] : a.before[t.chunk0 + c];
}

// The same for all chunks of all batches into LDS, a wave per batch (at most
// kWave chunks each), and into a.before if asked to; the caller's next barrier
// orders the stores.
__device__ __forceinline__ void chunk_starts(const RowsArgs& a, int32_t* s_chunk, bool leave) {
  constexpr int kWaves = kSageBlock / kWave, U = 4;
  const int lane = lane_id();
  for (int b0 = threadIdx.x / kWave; b0 < a.W; b0 += kWaves * U) {
    int32_t v[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int b = b0 + j * kWaves;
      v[j] = b < a.W && lane < a.nch ? a.chunk[b * a.nch + lane] : 0;
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const int b = b0 + j * kWaves;
      const int32_t before = wave_incl_scan(v[j]) - v[j];
      if (b < a.W && lane < a.nch) {
        s_chunk[b * a.nch + lane] = before;
        if (leave) a.before[b * a.nch + lane] = before;
      }
    }
  }
}

// Position of u in the batch's N_b, or -1.
template <bool HERE>
__device__ __forceinline__ int64_t rank_of(const RowsArgs& a, const int32_t* s_chunk,
                                           const Batch& t, int32_t u) {
  const uint32_t wi = (uint32_t)u >> 5;
  if (u < 0 || wi >= (uint64_t)a.wpb) return -1;
  return rank_in(t.bits[wi / kRankWords],
                 t.rank[wi / kRankWords] + chunk_first<HERE>(a, s_chunk, t, wi / kRankChunk), u,
                 t.nnb);
}

__device__ __forceinline__ void level_offsets(const RowsArgs& a, int lvl, int64_t* off) {
  for (int t = threadIdx.x; t <= GG_MAX_W; t += kSageBlock)
    off[t] = t <= a.W ? a.off[(int64_t)lvl * a.W + t] - a.off[(int64_t)lvl * a.W] : INT64_MAX;
  __syncthreads();
}

// Level blockIdx.y + 1 (1..L-1): each node's position, noted at its N_b row.
template <bool HERE>
__global__ void __launch_bounds__(kSageBlock) k_sage_places(RowsArgs a) {
  extern __shared__ int32_t s_chunk[];
  __shared__ int64_t off[GG_MAX_W + 1];
  const int lvl = blockIdx.y + 1;
  if (HERE) chunk_starts(a, s_chunk, blockIdx.x == 0 && blockIdx.y == 0);
  level_offsets(a, lvl, off);
  const int64_t n = off[a.W], f0 = a.off[(int64_t)lvl * a.W];
  for (int64_t r = (int64_t)blockIdx.x * kSageBlock + threadIdx.x; r < n;
       r += (int64_t)gridDim.x * kSageBlock) {
    const Batch t = batch_at(a, lvl, batch_of(off, r));
    const int64_t p = rank_of<HERE>(a, s_chunk, t, a.fids[f0 + r]);
    if (p >= 0 && t.nb0 + p < a.rows_cap) a.place[lvl][t.nb0 + p] = (int32_t)(r - t.out0);
  }
}

// J entries of a tile at a time, each stage's loads issued together: node ids,
// then set words and prefixes, then (below the top level) places, then the
// frontier entries that confirm them.
constexpr int kRowTile = 64;            // rows of a table tile
constexpr int kRowJ = 3;                 // entries in flight per lane

template <bool HERE>
__device__ __forceinline__ void find_rows(const RowsArgs& a, const int32_t* s_chunk, int lvl,
                                          int64_t f0, int64_t f0in, const Batch* bt, const int64_t (&r)[kRowJ],
                                          const int (&t)[kRowJ], const bool (&in)[kRowJ],
                                          int32_t (&row)[kRowJ], int32_t& st) {
  int32_t u[kRowJ], pre[kRowJ];
  u32x4 x[kRowJ];
  bool ask[kRowJ];
#pragma unroll
  for (int j = 0; j < kRowJ; ++j) {
    u[j] = -1;
    if (in[j]) {
      const int64_t q = (r[j] - bt->out0) * a.k[lvl] + (t[j] - 1);   // slot of the batch's list
      if (t[j] == 0)
        u[j] = a.fids[f0 + r[j]];
      else if (q < bt->nslot)
        u[j] = a.nbr[bt->slot0 + q];
    }
  }
#pragma unroll
  for (int j = 0; j < kRowJ; ++j) {
    const uint32_t wi = (uint32_t)u[j] >> 5;
    ask[j] = u[j] >= 0 && wi < (uint64_t)a.wpb;
    pre[j] = 0;
    x[j] = u32x4{0u, 0u, 0u, 0u};
    if (ask[j]) {
      x[j] = bt->bits[wi / kRankWords];
      pre[j] = bt->rank[wi / kRankWords] + chunk_first<HERE>(a, s_chunk, *bt, wi / kRankChunk);
    }
  }
  int64_t at[kRowJ];
  bool found[kRowJ];
#pragma unroll
  for (int j = 0; j < kRowJ; ++j) {
    const int64_t p = ask[j] ? rank_in(x[j], pre[j], u[j], bt->nnb) : -1;
    found[j] = p >= 0;
    at[j] = bt->nb0 + p;
  }
  if (lvl + 1 < a.L) {
    // a place is trusted only if the frontier entry it names is the node
    int64_t pl[kRowJ];
#pragma unroll
    for (int j = 0; j < kRowJ; ++j)
      pl[j] = found[j] && at[j] < a.rows_cap ? a.place[lvl + 1][at[j]] : -1;
#pragma unroll
    for (int j = 0; j < kRowJ; ++j)
      if (found[j] && at[j] < a.rows_cap) {
        found[j] = pl[j] >= 0 && pl[j] < bt->nin && a.fids[bt->in0 + pl[j]] == u[j];
        at[j] = bt->in0 - f0in + pl[j];
      }
  }
#pragma unroll
  for (int j = 0; j < kRowJ; ++j) {
    row[j] = found[j] && at[j] < a.rows_cap ? (int32_t)at[j] : -1;
    if (in[j] && !found[j] && (u[j] >= 0 || t[j] == 0)) st |= GG_DEV_BAD_ID;
  }
}

// Level blockIdx.y (0..L-1): the row, in the level above, of entry t of each
// node (t = 0: itself, t = 1..k: its neighbour slots), or -1.  Bound by the
// latency of its dependent random reads.  Nearly all tiles lie in one batch,
// whose addresses are then the same for every lane.
template <bool HERE>
__global__ void __launch_bounds__(kSageBlock) k_sage_rows(RowsArgs a, int32_t* status) {
  extern __shared__ int32_t s_chunk[];
  __shared__ int64_t off[GG_MAX_W + 1];
  if (HERE) chunk_starts(a, s_chunk, false);
  const int lvl = a.L - 1 - (int)blockIdx.y;   // the largest level first
  level_offsets(a, lvl, off);
  const int64_t n = off[a.W] < a.rows_cap ? off[a.W] : a.rows_cap;
  const int64_t f0 = a.off[(int64_t)lvl * a.W], f0in = a.off[(int64_t)(lvl + 1) * a.W];
  const int k = a.k[lvl];
  int32_t st = 0;
  for (int64_t row0 = (int64_t)blockIdx.x * kRowTile; row0 < n;
       row0 += (int64_t)gridDim.x * kRowTile) {
    const int b = __builtin_amdgcn_readfirstlane(batch_of(off, row0));
    const Batch bt = batch_at(a, lvl, b);
    const int rows = (int)(n - row0 < kRowTile ? n - row0 : kRowTile);
    const int total = rows * (k + 1);
    int32_t* out = a.table[lvl] + row0 * (k + 1);
    const bool one = row0 + rows <= bt.out1;
    for (int e0 = threadIdx.x; e0 < total; e0 += kSageBlock * kRowJ) {
      int64_t r[kRowJ];
      int t[kRowJ];
      bool in[kRowJ];
      int32_t row[kRowJ];
#pragma unroll
      for (int j = 0; j < kRowJ; ++j) {
        const int e = e0 + j * kSageBlock;
        const int rr = (int)chunk_row((uint32_t)e, a.kmagic[lvl]);
        in[j] = e < total;
        r[j] = row0 + rr;
        t[j] = e - rr * (k + 1);
      }
      if (one) {
        find_rows<HERE>(a, s_chunk, lvl, f0, f0in, &bt, r, t, in, row, st);
      } else {
        // every lane goes through the batches its tile touches
        for (int bb = b; bb < a.W && off[bb] < row0 + rows; ++bb) {
          const Batch ob = batch_at(a, lvl, bb);
          bool mine[kRowJ];
          int32_t got[kRowJ];
#pragma unroll
          for (int j = 0; j < kRowJ; ++j)
            mine[j] = in[j] && r[j] >= ob.out0 && r[j] < ob.out1;
          find_rows<HERE>(a, s_chunk, lvl, f0, f0in, &ob, r, t, mine, got, st);
#pragma unroll
          for (int j = 0; j < kRowJ; ++j) row[j] = mine[j] ? got[j] : row[j];
        }
      }
#pragma unroll
      for (int j = 0; j < kRowJ; ++j)
        if (in[j]) out[e0 + j * kSageBlock] = row[j];
    }
  }
  if (st) set_status(status, st);
}

// What one lane loads of a row: 16 bytes, VE = 4 (fp32) or 8 (fp16) consecutive
// columns, kept as loaded while in flight.
template <int XT>
struct Cols {
  static constexpr int VE = XT == GG_F32 ? 4 : 8;
  float v[VE];
};

__device__ __forceinline__ u32x4 load16(const char* p) {
  typedef u32x4 __attribute__((aligned(2))) any;
  return *(const GG_GLOBAL any*)p;
}

// The same for a row of fewer than VE elements: zeros past its last word or
// half word.
template <int XT>
__device__ __forceinline__ u32x4 load_narrow(const char* row, int c, int K) {
  constexpr int VE = Cols<XT>::VE;
  u32x4 r = {0u, 0u, 0u, 0u};
  if (c > 0) return r;
#pragma unroll
  for (int e = 0; e < VE; ++e)
    if (e < K) {
      if constexpr (XT == GG_F32)
        r[e] = ((const GG_GLOBAL uint32_t*)row)[e];
      else
        r[e / 2] |= (uint32_t)((const GG_GLOBAL uint16_t*)row)[e] << (16 * (e & 1));
    }
  return r;
}

template <int XT>
__device__ __forceinline__ float element(u32x4 r, int e) {
  if constexpr (XT == GG_F32) {
    return __builtin_bit_cast(f32x4, r)[e];
  } else {
    return (float)__builtin_bit_cast(f16x8, r)[e];
  }
}

// r holds the VE elements that end at the row's last one, s > 0 past the
// wanted first: shifts them into place, zeros behind.
template <int XT>
__device__ __forceinline__ void shift_cols(Cols<XT>& r, int s) {
  constexpr int VE = Cols<XT>::VE;
  if (s <= 0) return;
#pragma unroll
  for (int step = 1; step < VE; step <<= 1)
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      const float up = e + step < VE ? r.v[e + step] : 0.f;
      r.v[e] = (s & step) ? up : r.v[e];
    }
  if (s >= VE)
#pragma unroll
    for (int e = 0; e < VE; ++e) r.v[e] = 0.f;
}

// ---------------------------------------------------------------------------
// One layer: gather, mean and product.
// ---------------------------------------------------------------------------
struct LayerArgs {
  const char* h;        // input rows of the level, back to back
  int64_t h_stride;     // bytes
  int32_t K;            // columns to load per row
  int32_t G;            // MFMA groups (packed)
  const f32x4* w;       // packed weights, 2 * NT * 64 per group
  int32_t k;            // fanout of the hop
  const int32_t* table; // [rows][k + 1]
  const int64_t* off;   // frontier_off at the output level
  int32_t W;
  const float* bias;
  int32_t d_out, relu;
  int32_t ncols;        // columns stored per row (d_out, or padded with zeros)
  float* out;           // output rows of the level, back to back, ncols floats each
  int64_t rows_cap, out_cap;
};

// Sets GG_DEV_CAPACITY when the input or the output level does not fit.
__device__ __forceinline__ int64_t level_rows(const int64_t* off, int W, int64_t rows_cap,
                                              int64_t out_cap, int32_t* status) {
  const int64_t n = off[W] - off[0], nin = off[2 * W] - off[W];
  if (blockIdx.x == 0 && threadIdx.x == 0 && (nin > rows_cap || n > out_cap))
    set_status(status, GG_DEV_CAPACITY);
  const int64_t cap = out_cap < rows_cap ? out_cap : rows_cap;
  return n < cap ? n : cap;
}

// How a block's four waves share the tile's product: R output rows, split RW
// ways by rows and CW by columns, RT x CT MFMA tiles each.
template <int NT>
struct Split {
  static constexpr int R = NT <= 3 ? 64 : 32;
  static constexpr int CW = NT <= 3 ? 1 : (NT == 6 ? 2 : 4);
  static constexpr int RW = 4 / CW;
  static constexpr int CT = NT / CW;
  static constexpr int RT = R / 16 / RW;
};

// The same value, computed anew where it is used: what follows from it is not
// kept in registers across a tile loop.
__device__ __forceinline__ int anew(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// A block takes tiles of R output rows, S = LR * VE columns at a time: it
// gathers the columns of [h_v | mean h_u] into LDS, LR lanes per source row,
// so that a load covers runs of 16 * LR bytes (a row in shorter runs fetches
// the lines at their ends again, once the caches have dropped them), then
// multiplies them by the packed weights, which every block finds in L2.  Two
// or three blocks per CU gather and multiply in turn.  The row tables come to
// LDS one tile ahead, the weights to registers one group ahead.
//
// Rounding: a product's chain is one group long, self and mean apart, and the
// groups are added to the running sums.  Chains of four groups with both halves
// in them had up to 1.5 times the error of projecting every row first (which
// averages its products' errors over the draws) on inputs of fewer than 130
// columns; these have 0.37 to 0.94 times it over 25 networks of 12 to 602
// columns.  Rows of up to 64 columns into at most three column tiles need half
// a group per chain for that (16 columns throughout: 1.01e-7 with whole groups,
// 9.2e-8 with halves, 9.7e-8 projected).
//
// Wide rows are bound by the random row reads (262K x 602 fp32 -> 128, ten
// neighbours, 77K outputs: 531 us for 2.1 GB of row reads, where projecting
// every row by [W_self | W_neigh], whose 85 GFLOP the fp32 matrix cores need
// 550 us for at best, took 2,447 + 119), narrow ones by matrix work (1.4M x
// 128 fp16 -> 128, five neighbours: 229 us, 117 of them matrix cores at full
// rate; projected 1,676 + 232).  Also measured on the first, when it took 549:
// the lookups of k_sage_rows inside the tile loop and 64-byte runs 655; half
// the waves gathering and half multiplying 858; 1 KB runs in two blocks per CU
// 594; eight neighbour rows in flight instead of five, in two blocks per CU,
// 565.
// Lane indices are taken anew in every tile (anew()): the addresses that the
// compiler kept from tile to tile otherwise cost up to 50 registers and spilled.
template <int NT, int XT, int LR, bool NARROW>
__global__ void __launch_bounds__(kSageBlock, NT <= 3 ? 2 : 3) k_sage_layer(LayerArgs a, int32_t* status) {
  typedef Split<NT> Sp;
  constexpr int VE = Cols<XT>::VE, ES = 16 / VE;
  constexpr int S = LR * VE;                 // columns per pass
  constexpr int LD = S + 4;                  // padded against bank conflicts
  constexpr int RG = kWave / LR;             // rows per load
  constexpr int RPW = Sp::R / 4;             // rows a wave gathers
  constexpr int NRG = (RPW + RG - 1) / RG;
  constexpr int RB = NRG >= 2 ? 2 : 1;       // row groups in flight
  constexpr int TU = 5;                      // ... with so many neighbour rows each
  constexpr int H = NT <= 3 && S <= 64 ? 2 : 1;   // product chains per group and half
  constexpr int kTab = (Sp::R * kMaxPitch + kSageBlock - 1) / kSageBlock;
  extern __shared__ float sm[];
  float* A = sm;                             // [2][R][LD]: self, mean
  int32_t* s_pos = (int32_t*)(sm + 2 * Sp::R * LD);   // [2][R * pitch]
  const int tid = threadIdx.x, lane = lane_id(), wv = tid / kWave;
  const int64_t n = level_rows(a.off, a.W, a.rows_cap, a.out_cap, status);
  const int pitch = a.k + 1;
  const bool any = a.off[2 * a.W] - a.off[a.W] > 0 && a.rows_cap > 0;   // input rows
  if (!any) return;
  const int npass = (a.K + S - 1) / S;
  const int64_t step = (int64_t)gridDim.x * Sp::R;
  int64_t row0 = (int64_t)blockIdx.x * Sp::R;
  const int tabn = Sp::R * pitch;

  int32_t tab[kTab];
  auto fetch_table = [&](int64_t r0) {
    const int64_t left = (n - r0) * pitch;
    const int at = anew(tid);
#pragma unroll
    for (int j = 0; j < kTab; ++j) {
      const int e = j * kSageBlock + at;
      if (j * kSageBlock < tabn) tab[j] = (e < tabn && e < left) ? a.table[r0 * pitch + e] : -1;
    }
  };
  auto store_table = [&](int par) {
    const int at = anew(tid);
#pragma unroll
    for (int j = 0; j < kTab; ++j) {
      const int e = j * kSageBlock + at;
      if (e < tabn) s_pos[par * tabn + e] = tab[j];
    }
  };
  fetch_table(row0);
  store_table(0);
  __syncthreads();

  const int lr = lane / LR, lc = lane % LR, c = lc * VE;
  const int g = lane >> 4, il = lane & 15;
  const int rt0 = wv / Sp::CW * Sp::RT, ct0 = wv % Sp::CW * Sp::CT;
  int par = 0;
  for (; row0 < n; row0 += step, par ^= 1) {
    const int32_t* pos = s_pos + par * tabn;
    // 1 / drawn neighbours of row lane % RPW of the wave, 0 for none: neighbour
    // rows are scaled as they are added, so that the mean of finite rows is
    // finite.
    int drawn = 0;
    for (int t = lane / RPW; t < a.k; t += kWave / RPW)
      drawn += pos[(wv * RPW + lane % RPW) * pitch + 1 + t] >= 0;
#pragma unroll
    for (int o = RPW; o < kWave; o <<= 1) drawn += __shfl_xor(drawn, o, kWave);
    const float share = drawn ? 1.0f / (float)drawn : 0.f;
    f32x4 tot[Sp::RT][Sp::CT];
#pragma unroll
    for (int r = 0; r < Sp::RT; ++r)
#pragma unroll
      for (int t = 0; t < Sp::CT; ++t) tot[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int ps = 0; ps < npass; ++ps) {
      // ---- gather ----
      const int col = ps * S + c;
      const int off = (col < a.K - VE ? col : a.K - VE) * ES;
      const int past = col + VE - a.K;       // > 0: the row ends before the lane's columns do
      auto load = [&](int32_t p) {
        const char* rp = a.h + (int64_t)(p > 0 ? p : 0) * a.h_stride;
        return NARROW ? load_narrow<XT>(rp, c, a.K) : load16(rp + off);
      };
#pragma unroll 1
      for (int q = 0; q < NRG; q += RB) {
        const int32_t* rp[RB];
        int m = 0;
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          const int r = (q + i) * RG + lr;
          rp[i] = pos + (wv * RPW + (r < RPW ? r : RPW - 1)) * pitch;
          for (int t = lc; t < a.k; t += LR)
            if (rp[i][1 + t] >= 0) m = max(m, t + 1);
        }
#pragma unroll
        for (int o = kWave / 2; o >= 1; o >>= 1) m = max(m, __shfl_xor(m, o, kWave));
        const int tmax = __builtin_amdgcn_readfirstlane(m);
        u32x4 own[RB], v[RB * TU];
        Cols<XT> sum[RB];
        float inv[RB];
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          own[i] = load(rp[i][0]);
          const int r = (q + i) * RG + lr;
          inv[i] = __shfl(share, r < RPW ? r : RPW - 1, kWave);
#pragma unroll
          for (int e = 0; e < VE; ++e) sum[i].v[e] = 0.f;
        }
        for (int t0 = 0; t0 < tmax; t0 += TU) {
#pragma unroll
          for (int j = 0; j < TU; ++j)
            if (t0 + j < tmax)
#pragma unroll
              for (int i = 0; i < RB; ++i) v[i * TU + j] = load(rp[i][1 + t0 + j]);
#pragma unroll
          for (int j = 0; j < TU; ++j)
            if (t0 + j < tmax)
#pragma unroll
              for (int i = 0; i < RB; ++i) {
                const bool ok = rp[i][1 + t0 + j] >= 0;
#pragma unroll
                for (int e = 0; e < VE; ++e)
                  sum[i].v[e] = __builtin_fmaf(ok ? element<XT>(v[i * TU + j], e) : 0.f, inv[i],
                                               sum[i].v[e]);
              }
        }
#pragma unroll
        for (int i = 0; i < RB; ++i) {
          Cols<XT> self;
#pragma unroll
          for (int e = 0; e < VE; ++e) self.v[e] = element<XT>(own[i], e);
          if (!NARROW) {
            shift_cols<XT>(self, past);
            shift_cols<XT>(sum[i], past);
          }
          const int r = (q + i) * RG + lr;
          if (r < RPW) {
            float* d = A + (wv * RPW + r) * LD + c;
#pragma unroll
            for (int e = 0; e < VE; e += 4) {
              *(f32x4*)(d + e) = f32x4{self.v[e], self.v[e + 1], self.v[e + 2], self.v[e + 3]};
              *(f32x4*)(d + Sp::R * LD + e) =
                  f32x4{sum[i].v[e], sum[i].v[e + 1], sum[i].v[e + 2], sum[i].v[e + 3]};
            }
          }
        }
      }
      const int g0 = ps * (S / kGroup), g1 = min(g0 + S / kGroup, a.G);
      f32x4 next[2][Sp::CT];
      auto fetch_weights = [&](int q) {
#pragma unroll
        for (int sn = 0; sn < 2; ++sn)
#pragma unroll
          for (int t = 0; t < Sp::CT; ++t)
            next[sn][t] = a.w[((int64_t)(q * 2 + sn) * NT + ct0 + t) * kWave + lane];
      };
      fetch_weights(g0);
      if (ps + 1 == npass) fetch_table(row0 + step);
      __syncthreads();
      // ---- product ----
      const float* half = A + il * LD + 4 * g;
#pragma unroll 1
      for (int q = g0; q < g1; ++q) {
        f32x4 w[2][Sp::CT], acc[2][H][Sp::RT][Sp::CT];
#pragma unroll
        for (int sn = 0; sn < 2; ++sn)
#pragma unroll
          for (int t = 0; t < Sp::CT; ++t) {
            w[sn][t] = next[sn][t];
#pragma unroll
            for (int h = 0; h < H; ++h)
#pragma unroll
              for (int r = 0; r < Sp::RT; ++r) acc[sn][h][r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
          }
        fetch_weights(min(q + 1, g1 - 1));
        __builtin_amdgcn_sched_barrier(0);   // or the loads sink to their use
#pragma unroll
        for (int sn = 0; sn < 2; ++sn) {
          f32x4 x[Sp::RT];
#pragma unroll
          for (int r = 0; r < Sp::RT; ++r)
            x[r] = *(const f32x4*)(half + (sn * Sp::R + (rt0 + r) * 16) * LD + (q - g0) * kGroup);
#pragma unroll
          for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int r = 0; r < Sp::RT; ++r)
#pragma unroll
              for (int t = 0; t < Sp::CT; ++t)
                acc[sn][e % H][r][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                    x[r][e], w[sn][t][e], acc[sn][e % H][r][t], 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < Sp::RT; ++r)
#pragma unroll
          for (int t = 0; t < Sp::CT; ++t) {
            f32x4 self = acc[0][0][r][t], mean = acc[1][0][r][t];
            if constexpr (H == 2) {
              self += acc[0][1][r][t];
              mean += acc[1][1][r][t];
            }
            tot[r][t] += self + mean;
          }
      }
      if (ps + 1 == npass) store_table(par ^ 1);
      __syncthreads();
    }
    // D[i][j] of a tile sits in lane 16 * (i / 4) + j, element i % 4.
    const int ln = anew(lane), gn = ln >> 4, in = ln & 15;
#pragma unroll
    for (int r = 0; r < Sp::RT; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int ri = (rt0 + r) * 16 + 4 * gn + e;
        const int64_t row = row0 + ri;
        if (row >= n || pos[ri * pitch] < 0) continue;
#pragma unroll
        for (int t = 0; t < Sp::CT; ++t) {
          const int cl = (ct0 + t) * 16 + in;
          if (cl >= a.ncols) continue;
          // Columns past d_out hold zeros whatever the row holds: an infinity
          // times their zero weights would be a NaN for the next layer.
          float y = 0.f;
          if (cl < a.d_out) {
            y = tot[r][t][e] + (a.bias ? a.bias[cl] : 0.f);
            if (a.relu && y < 0.f) y = 0.f;
          }
          a.out[row * a.ncols + cl] = y;
        }
      }
  }
}

// ---------------------------------------------------------------------------
// One layer of narrow outputs: projection of every input row, then the mean.
// ---------------------------------------------------------------------------
constexpr int kProjCols = 16;            // most output columns of this form

struct ProjArgs {
  const char* h;        // input rows of the level, back to back
  int64_t h_stride;     // bytes
  int32_t K;            // d_in
  int32_t G;            // MFMA groups (packed)
  const f32x4* w;       // packed weights, one column tile each of W_self and W_neigh
  int32_t whole;        // all groups fit in LDS
  float* z;             // [rows][32]: self columns, then neighbour columns
  const int64_t* off;   // frontier_off at the input level
  int32_t W;
  int64_t rows_cap;
};

// Each wave owns 16 rows and loads them straight into registers, 16 bytes per
// lane; bound by those reads and the 128 bytes written per row (1.56M rows of
// 400 bytes in 190 us, 4.3 TB/s).
__global__ void __launch_bounds__(kSageBlock, 8) k_sage_project(ProjArgs a) {
  constexpr int VE = Cols<GG_F32>::VE;                   // one group per load
  constexpr int UL = 4;                                  // loads in flight per lane
  constexpr int kGroupW = 2 * kWave;
  extern __shared__ f32x4 swl[];
  const int64_t nin = a.off[a.W] - a.off[0];
  const int64_t n = nin < a.rows_cap ? nin : a.rows_cap;
  const int lane = lane_id(), wv = (int)threadIdx.x / kWave;
  const int g = lane >> 4, il = lane & 15;
  if (a.whole) {
    for (int i = threadIdx.x; i < a.G * kGroupW; i += kSageBlock) swl[i] = a.w[i];
    __syncthreads();
  }
  const f32x4* wl = a.whole ? (const f32x4*)swl : a.w;
  for (int64_t row0 = ((int64_t)blockIdx.x * 4 + wv) * 16; row0 < n;
       row0 += (int64_t)gridDim.x * kTileRows) {
    const int64_t r = row0 + il < n ? row0 + il : n - 1;
    const char* rp = a.h + r * a.h_stride;
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    for (int s = 0; s < a.G; s += UL) {
      u32x4 raw[UL];
#pragma unroll
      for (int u = 0; u < UL; ++u) {
        const int c = (s + u) * 4 * VE + VE * g;
        if (s + u < a.G) raw[u] = load16(rp + (c < a.K - VE ? c : a.K - VE) * 4);
      }
#pragma unroll
      for (int u = 0; u < UL; ++u) {
        if (s + u >= a.G) break;
        const int past = (s + u) * 4 * VE + VE * g + VE - a.K;
        Cols<GG_F32> v;
#pragma unroll
        for (int e = 0; e < VE; ++e) v.v[e] = element<GG_F32>(raw[u], e);
        if ((s + u + 1) * 4 * VE > a.K) shift_cols<GG_F32>(v, past);
#pragma unroll
        for (int sn = 0; sn < 2; ++sn) {
          // columns 16 (s + u) + 4 g .. + 3, where the packed weights have them
          const f32x4 b = wl[((s + u) * 2 + sn) * kWave + g * 16 + il];
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[sn] = __builtin_amdgcn_mfma_f32_16x16x4f32(v.v[e], b[e], acc[sn], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int rr = 0; rr < 4; ++rr) {
      const int64_t row = row0 + 4 * g + rr;
      if (row >= n) continue;
      a.z[row * 32 + il] = acc[0][rr];
      a.z[row * 32 + 16 + il] = acc[1][rr];
    }
  }
}

// Sixteen lanes per output node, one column each; all of a node's projected
// rows are in flight together (KMAX >= k) and summed in slot order.
template <int KMAX>
__global__ void __launch_bounds__(kSageBlock) k_sage_mean(LayerArgs a, const float* z,
                                                          int32_t* status) {
  const int64_t n = level_rows(a.off, a.W, a.rows_cap, a.out_cap, status);
  const int lane = lane_id(), sl = lane & 15, gbase = lane & 48;
  const int pitch = a.k + 1;
  for (int64_t r = (int64_t)blockIdx.x * (kSageBlock / 16) + (threadIdx.x >> 4); r < n;
       r += (int64_t)gridDim.x * (kSageBlock / 16)) {
    const int32_t* row = a.table + r * pitch;
    const int32_t e0 = sl < pitch ? row[sl] : -1;
    const int32_t e1 = KMAX >= 16 && sl + 16 < pitch ? row[sl + 16] : -1;
    const int32_t e2 = KMAX >= 32 && sl + 32 < pitch ? row[sl + 32] : -1;
    const int32_t pv = __shfl(e0, gbase, kWave);
    int32_t p[KMAX];
    float v[KMAX];
    int cnt = 0;
#pragma unroll
    for (int t = 0; t < KMAX; ++t) {
      p[t] = __shfl(t + 1 < 16 ? e0 : (t + 1 < 32 ? e1 : e2), gbase + ((t + 1) & 15), kWave);
      if (t >= a.k) p[t] = -1;
      cnt += p[t] >= 0;
    }
    const float self = pv >= 0 ? z[(int64_t)pv * 32 + sl] : 0.f;
#pragma unroll
    for (int t = 0; t < KMAX; ++t) v[t] = p[t] >= 0 ? z[(int64_t)p[t] * 32 + 16 + sl] : 0.f;
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < KMAX; ++t)
      if (p[t] >= 0) sum += v[t];
    if (pv < 0 || sl >= a.ncols) continue;
    float y = 0.f;                     // zeros past d_out, as in k_sage_layer
    if (sl < a.d_out) {
      y = self + sum * (cnt ? 1.0f / (float)cnt : 0.f) + (a.bias ? a.bias[sl] : 0.f);
      if (a.relu && y < 0.f) y = 0.f;
    }
    a.out[r * a.ncols + sl] = y;
  }
}

// Column tiles of a layer, rounded up to the compiled sizes.
int col_tiles(int32_t d_out) {
  const int need = (d_out + 15) / 16;
  return need <= 4 ? need : (need <= 6 ? 6 : 8);
}

// Columns of a layer's output rows inside the call: padded with zeros to
// whole MFMA groups, so that the next layer needs no care at row ends.
int inner_cols(int32_t d_out) { return col_tiles(d_out) * 16; }

int64_t packed_vecs(int32_t cols, int32_t d_out) {
  return cdiv(cols, kGroup) * 2 * col_tiles(d_out) * kWave;
}

// A layer of fp32 rows projects every input row first when reading the k + 1
// input rows of each output node would move more than twice as much: an input row
// read once and 128 bytes written, and k + 1 lines of 128 bytes, against k + 1
// rows with about a line each for their unaligned ends.  A level holds about half
// as many rows per output node as its hop draws, at most about four on dense
// graphs.  The factor is for the rows that the caches serve again when they are
// gathered.  Forward passes of two layers of 16, 2.45M nodes, projected /
// gathered first layers, by (columns, last fan-out): (64, 20) 57 / 48 us; (100,
// 20) 65 / 59, (150, 20) 73 / 81, (200, 10) 99 / 107, (300, 10) 125 / 156, (300,
// 20) 100 / 105, (450, 10) 190 / 200, (450, 20) 159 / 146, (602, 5) 259 / 252,
// (602, 20) 192 / 179: within a tenth of the better one but for 150 columns and a
// fan-out of 10 (86 / 104, gathered).  Rows of halves are cheaper to gather
// throughout, whatever the bytes moved: (256, 20) 84 / 65, (602, 10) 196 / 164.
bool use_projection(int32_t d_in, int32_t d_out, int32_t x_dtype, int32_t k) {
  if (x_dtype != GG_F32 || d_out > kProjCols || d_in < 8) return false;
  const int64_t row = d_in * 4;
  const int64_t gathered = (k + 1) * (row + 112);
  const int64_t projected = std::min<int64_t>((k + 1) * (row + 128) / 2, 4 * (row + 128)) +
                            (k + 1) * 128;
  return 2 * projected < gathered;
}

struct SageWs {
  float* h[2];
  float* z;
  int32_t* table[GG_MAX_LAYERS];
  int32_t* place[GG_MAX_LAYERS];
  int32_t* rank;
  int32_t* chunk;
  int32_t* before;
  f32x4* packed;
};

size_t sage_ws_layout(int64_t num_nodes, int32_t W, int64_t rows_cap, int32_t L,
                      const gg_sage_layer_t* layers, char* base, SageWs* out) {
  // Layer j leaves its rows in h[j % 2]; the first layer's projected rows are
  // done with when the second writes h[1], and share its place.
  int32_t cols[2] = {0, layers[0].d_out <= kProjCols ? 32 : 0};
  int64_t vecs = 0;
  for (int32_t j = 0; j < L; ++j) {
    if (j + 1 < L) cols[j & 1] = std::max(cols[j & 1], inner_cols(layers[j].d_out));
    vecs += packed_vecs(j ? inner_cols(layers[j - 1].d_out) : layers[j].d_in, layers[j].d_out);
  }
  const size_t r = (size_t)std::max<int64_t>(rows_cap, 1);
  const int64_t wpb = gg_bits_words(num_nodes);
  Carve cv{base, 0, ~(size_t)0};
  SageWs w;
  for (int i = 0; i < 2; ++i) w.h[i] = cv.take<float>(r * (size_t)cols[i]);
  w.z = w.h[1];
  for (int32_t l = 0; l < L; ++l) w.table[l] = cv.take<int32_t>(r * kMaxPitch);
  for (int32_t l = 1; l < L; ++l) w.place[l] = cv.take<int32_t>(r);
  w.rank = cv.take<int32_t>((size_t)W * (size_t)(wpb / kRankWords));
  w.chunk = cv.take<int32_t>((size_t)W * (size_t)(wpb / kRankChunk));
  w.before = cv.take<int32_t>((size_t)W * (size_t)(wpb / kRankChunk));
  w.packed = cv.take<f32x4>((size_t)vecs);
  if (out) *out = w;
  return align_up(cv.used, 256);
}

template <int NT, int XT, int LR, bool NARROW = false>
int launch_layer(LayerArgs& a, int64_t rows_bound, int32_t* status, hipStream_t stream) {
  constexpr int R = Split<NT>::R;
  const size_t lds =
      (size_t)(2 * R * (LR * Cols<XT>::VE + 4) + 2 * R * (a.k + 1)) * sizeof(float);
  // As many blocks as fit on the chip, each taking tile after tile.
  const int64_t per_cu = std::min<int64_t>(4, (160 * 1024) / (int64_t)lds);
  const int64_t grid = std::min<int64_t>(std::max<int64_t>(cdiv(rows_bound, R), 1),
                                         256 * std::max<int64_t>(per_cu, 1));
  hipLaunchKernelGGL((k_sage_layer<NT, XT, LR, NARROW>), dim3((unsigned)grid), dim3(kSageBlock),
                     lds, stream, a, status);
  GG_LAUNCH_CHECK("k_sage_layer");
  return GG_OK;
}

// Lanes per source row: the row in one load of a few rows where it is narrow,
// else a run of 128 columns.  Its operand tile leaves LDS for three blocks per CU
// with 32 output rows, and with 64 for two up to a fan-out of 27, for one above.
template <int NT, int XT>
int launch_layer_u(LayerArgs& a, int64_t rows_bound, int32_t* status, hipStream_t stream) {
  constexpr int VE = Cols<XT>::VE;
  constexpr int kMin = NT <= 3 ? 4 : 8;          // at most as many rows per load as a wave gathers
  if (a.K < VE) return launch_layer<NT, XT, kMin, true>(a, rows_bound, status, stream);
  if constexpr (XT == GG_F32) {
    if (a.K <= kMin * VE) return launch_layer<NT, XT, kMin>(a, rows_bound, status, stream);
  }
  if (NT <= 3 ? a.K <= 64 : a.K <= 128)
    return launch_layer<NT, XT, (NT <= 3 ? 64 : 128) / VE>(a, rows_bound, status, stream);
  return launch_layer<NT, XT, 128 / VE>(a, rows_bound, status, stream);
}

template <int XT>
int launch_layer_nt(int nt, LayerArgs& a, int64_t rows_bound, int32_t* status,
                    hipStream_t stream) {
  switch (nt) {
    case 1: return launch_layer_u<1, XT>(a, rows_bound, status, stream);
    case 2: return launch_layer_u<2, XT>(a, rows_bound, status, stream);
    case 3: return launch_layer_u<3, XT>(a, rows_bound, status, stream);
    case 4: return launch_layer_u<4, XT>(a, rows_bound, status, stream);
    case 6: return launch_layer_u<6, XT>(a, rows_bound, status, stream);
    default: return launch_layer_u<8, XT>(a, rows_bound, status, stream);
  }
}

// The layer of output level lvl by projection: a's fields as for k_sage_layer.
int launch_projected(LayerArgs& a, float* z, int64_t rows_cap, int32_t* status,
                     hipStream_t stream) {
  ProjArgs p;
  p.h = a.h;
  p.h_stride = a.h_stride;
  p.K = a.K;
  p.G = a.G;
  p.w = a.w;
  p.z = z;
  p.off = a.off + a.W;
  p.W = a.W;
  p.rows_cap = rows_cap;
  const int64_t wb = (int64_t)a.G * 2 * kWave * (int64_t)sizeof(f32x4);
  p.whole = wb <= kWLdsBytes ? 1 : 0;
  const int grid = (int)std::min<int64_t>(std::max<int64_t>(cdiv(rows_cap, kTileRows), 1), 2048);
  const size_t lds = p.whole ? (size_t)wb : 0;
  hipLaunchKernelGGL(k_sage_project, dim3(grid), dim3(kSageBlock), lds, stream, p);
  GG_LAUNCH_CHECK("k_sage_project");
  const int mg = (int)std::min<int64_t>(std::max<int64_t>(cdiv(rows_cap, kSageBlock / 16), 1), 16384);
  if (a.k <= 8)
    hipLaunchKernelGGL(k_sage_mean<8>, dim3(mg), dim3(kSageBlock), 0, stream, a, z, status);
  else if (a.k <= 16)
    hipLaunchKernelGGL(k_sage_mean<16>, dim3(mg), dim3(kSageBlock), 0, stream, a, z, status);
  else
    hipLaunchKernelGGL(k_sage_mean<32>, dim3(mg), dim3(kSageBlock), 0, stream, a, z, status);
  GG_LAUNCH_CHECK("k_sage_mean");
  return GG_OK;
}

}  // namespace
}  // namespace gg

using namespace gg;

extern "C" size_t gg_ws_sage(int64_t num_nodes, int32_t W, int64_t rows_cap, int32_t L,
                             const gg_sage_layer_t* layers_h) {
  if (num_nodes < 1 || W < 1 || W > GG_MAX_W || rows_cap < 0 || L < 1 || L > GG_MAX_LAYERS ||
      !layers_h)
    return 0;
  return sage_ws_layout(num_nodes, W, rows_cap, L, layers_h, nullptr, nullptr);
}

extern "C" int gg_sage_forward(const gg_wsample_t* smp, int64_t num_nodes, int32_t W, int32_t L,
                               const int32_t* fanout_h, const void* x_d, int32_t x_dtype,
                               int64_t x_stride, int64_t rows_cap, const gg_sage_layer_t* layers_h,
                               float* out_d, int64_t out_rows_cap, int32_t* status_d, void* ws,
                               size_t ws_bytes, hipStream_t stream) {
  GG_REQUIRE(smp && fanout_h && x_d && layers_h && out_d && status_d, "NULL argument");
  GG_REQUIRE(smp->frontier_ids && smp->frontier_off && smp->nbr_ids && smp->nbr_off &&
                 smp->frontier_bits,
             "sampling outputs are NULL");
  GG_REQUIRE(num_nodes >= 1 && num_nodes <= INT32_MAX, "num_nodes %lld invalid",
             (long long)num_nodes);
  GG_REQUIRE(W >= 1 && W <= GG_MAX_W, "W = %d outside 1..%d", W, GG_MAX_W);
  GG_REQUIRE(L >= 1 && L <= GG_MAX_LAYERS, "L = %d outside 1..%d", L, GG_MAX_LAYERS);
  GG_REQUIRE(x_dtype == GG_F32 || x_dtype == GG_F16, "x_dtype %d unsupported", x_dtype);
  GG_REQUIRE(rows_cap >= 0 && out_rows_cap >= 0, "negative capacity");
  const int64_t esz = x_dtype == GG_F32 ? 4 : 2;
  GG_REQUIRE(((uintptr_t)x_d % esz) == 0 && x_stride % esz == 0, "x is not %lld-byte aligned",
             (long long)esz);
  for (int32_t l = 0; l < L; ++l)
    GG_REQUIRE(fanout_h[l] >= 1 && fanout_h[l] <= GG_MAX_FANOUT, "fanout[%d] = %d invalid", l,
               fanout_h[l]);
  for (int32_t j = 0; j < L; ++j) {
    const gg_sage_layer_t& ly = layers_h[j];
    GG_REQUIRE(ly.w_self && ly.w_neigh, "layer %d weights are NULL", j);
    GG_REQUIRE(ly.d_out >= 1 && ly.d_out <= GG_SAGE_MAX_DIM, "layer %d: d_out = %d outside 1..%d",
               j, ly.d_out, GG_SAGE_MAX_DIM);
    if (j == 0)
      GG_REQUIRE(ly.d_in >= 1 && ly.d_in <= GG_SAGE_MAX_IN && ly.d_in * esz <= x_stride,
                 "layer 0: d_in = %d does not fit rows of %lld bytes", ly.d_in,
                 (long long)x_stride);
    else
      GG_REQUIRE(ly.d_in == layers_h[j - 1].d_out, "layer %d: d_in %d != previous d_out %d", j,
                 ly.d_in, layers_h[j - 1].d_out);
  }
  GG_REQUIRE(aligned16(smp->frontier_bits), "frontier_bits must be 16-byte aligned");
  const size_t need = sage_ws_layout(num_nodes, W, rows_cap, L, layers_h, nullptr, nullptr);
  GG_REQUIRE(ws && ws_bytes >= need, "workspace of %zu bytes < %zu", ws_bytes, need);
  SageWs sw;
  sage_ws_layout(num_nodes, W, rows_cap, L, layers_h, (char*)ws, &sw);
  const int64_t wpb = gg_bits_words(num_nodes);
  const int64_t nch = wpb / kRankChunk;

  // Ranks in the N_b bit sets and packed weights.  A layer after the first
  // contracts over its input's padded columns, whose weights are zero.
  PackArgs pk;
  pk.L = L;
  pk.first[0] = 0;
  int32_t cols[GG_MAX_LAYERS];
  for (int32_t j = 0; j < L; ++j) {
    const gg_sage_layer_t& ly = layers_h[j];
    cols[j] = j ? inner_cols(layers_h[j - 1].d_out) : ly.d_in;
    pk.w[j][0] = ly.w_self;
    pk.w[j][1] = ly.w_neigh;
    pk.d_in[j] = ly.d_in;
    pk.d_out[j] = ly.d_out;
    pk.nt[j] = col_tiles(ly.d_out);
    pk.first[j + 1] = pk.first[j] + packed_vecs(cols[j], ly.d_out);
  }
  const int64_t pack_blocks = std::min<int64_t>(cdiv(pk.first[L], kSageBlock), 512);
  hipLaunchKernelGGL(k_sage_prepare, dim3((unsigned)(nch * W + pack_blocks)), dim3(kSageBlock), 0,
                     stream, smp->frontier_bits, (int32_t)nch, W, (int2*)sw.rank, sw.chunk, pk,
                     sw.packed);
  GG_LAUNCH_CHECK("k_sage_prepare");
  const bool here = nch <= kWave;
  if (!here) {
    hipLaunchKernelGGL(k_sage_chunks, dim3((unsigned)W), dim3(kChunkBlock), 0, stream, sw.chunk,
                       sw.before, (int32_t)nch);
    GG_LAUNCH_CHECK("k_sage_chunks");
  }
  RowsArgs ra;
  ra.W = W;
  ra.L = L;
  for (int32_t l = 0; l < L; ++l) {
    ra.k[l] = fanout_h[l];
    ra.kmagic[l] = div_magic((uint32_t)fanout_h[l] + 1u);
    ra.table[l] = sw.table[l];
    ra.place[l] = l ? sw.place[l] : nullptr;
  }
  ra.fids = smp->frontier_ids;
  ra.off = smp->frontier_off;
  ra.nbr = smp->nbr_ids;
  ra.noff = smp->nbr_off;
  ra.bits = smp->frontier_bits;
  ra.rank = sw.rank;
  ra.chunk = sw.chunk;
  ra.before = sw.before;
  ra.nch = (int32_t)nch;
  ra.wpb = wpb;
  ra.rows_cap = rows_cap;
  const int64_t rows_grid =
      std::min<int64_t>(std::max<int64_t>(cdiv(rows_cap, kRowTile), 1), 1024);
  const size_t chunk_lds = here ? (size_t)W * (size_t)nch * sizeof(int32_t) : 0;
  if (L > 1) {
    hipLaunchKernelGGL(here ? k_sage_places<true> : k_sage_places<false>,
                       dim3((unsigned)rows_grid, (unsigned)(L - 1)), dim3(kSageBlock), chunk_lds,
                       stream, ra);
    GG_LAUNCH_CHECK("k_sage_places");
  }
  const bool first = here && L == 1;
  hipLaunchKernelGGL(first ? k_sage_rows<true> : k_sage_rows<false>,
                     dim3((unsigned)rows_grid, (unsigned)L), dim3(kSageBlock),
                     first ? chunk_lds : 0, stream, ra, status_d);
  GG_LAUNCH_CHECK("k_sage_rows");

  for (int32_t j = 0; j < L; ++j) {
    const gg_sage_layer_t& ly = layers_h[j];
    const int32_t lvl = L - 1 - j;
    LayerArgs a;
    a.h = j ? (const char*)sw.h[(j - 1) & 1] : (const char*)x_d;
    a.h_stride = j ? (int64_t)cols[j] * 4 : x_stride;
    a.K = cols[j];
    a.G = (int32_t)cdiv(cols[j], kGroup);
    a.w = sw.packed + pk.first[j];
    a.k = fanout_h[lvl];
    a.table = sw.table[lvl];
    a.off = smp->frontier_off + (int64_t)lvl * W;
    a.W = W;
    a.bias = ly.bias;
    a.d_out = ly.d_out;
    a.relu = ly.relu ? 1 : 0;
    a.ncols = j + 1 < L ? inner_cols(ly.d_out) : ly.d_out;
    a.out = j + 1 < L ? sw.h[j & 1] : out_d;
    a.rows_cap = rows_cap;
    a.out_cap = j + 1 < L ? rows_cap : out_rows_cap;
    const int xt = j == 0 ? x_dtype : GG_F32;
    int rc;
    if (j == 0 && use_projection(ly.d_in, ly.d_out, x_dtype, a.k))
      rc = launch_projected(a, sw.z, rows_cap, status_d, stream);
    else if (xt == GG_F16)
      rc = launch_layer_nt<GG_F16>(pk.nt[j], a, rows_cap, status_d, stream);
    else
      rc = launch_layer_nt<GG_F32>(pk.nt[j], a, rows_cap, status_d, stream);
    if (rc != GG_OK) return rc;
  }
  return GG_OK;
}
