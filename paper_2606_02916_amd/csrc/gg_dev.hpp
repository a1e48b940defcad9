// Device-side building blocks of libgg (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "copy_geom.hpp"
#include "gg.h"

namespace gg {

constexpr int kWave = 64;
constexpr int kBlock = 256;                  // 4 wavefronts
constexpr int kChunkWords = 2048;            // bit-set words per compaction block
constexpr int kWordsPerThread = kChunkWords / kBlock;

// ---------------------------------------------------------------------------
// Partition book, passed by value.  MOD uses a multiply-shift for u div P
// (exact for u < 2^34 and P <= 64); RANGE finds the last start <= u by a
// binary search over the P starts (the table is padded with N up to 64).
// ---------------------------------------------------------------------------
struct KPart {
  int32_t P;
  int32_t kind;
  int32_t local;
  int32_t step0;  // RANGE: largest power of two <= max(P - 1, 1)
  int64_t N;
  uint64_t div_magic;
  int64_t start[GG_MAX_PARTS + 1];  // entries past P hold N
};

__device__ __forceinline__ int32_t mod_div(const KPart& p, uint32_t u) {
  return (int32_t)(((uint64_t)u * p.div_magic) >> 40);
}

// start: the 65-entry table (kernarg or LDS copy).
__device__ __forceinline__ int32_t owner_of(const KPart& p, const int64_t* start, int32_t u) {
  if (p.kind == GG_PART_MOD) {
    const int32_t q = mod_div(p, (uint32_t)u);
    return u - q * p.P;
  }
  int32_t idx = 0;
  for (int step = p.step0; step >= 1; step >>= 1)
    if (start[idx + step] <= (int64_t)u) idx += step;
  return idx;
}

__device__ __forceinline__ int64_t row_of(const KPart& p, const int64_t* start, int32_t u,
                                          int32_t owner) {
  if (p.kind == GG_PART_MOD) return (int64_t)mod_div(p, (uint32_t)u);
  return (int64_t)u - start[owner];
}

// ---------------------------------------------------------------------------
// Feature shards, passed by value.
// ---------------------------------------------------------------------------
struct KFeat {
  int32_t row_bytes;
  int32_t P;
  const char* shard[GG_MAX_PARTS];
  int64_t stride[GG_MAX_PARTS];
  int64_t rows[GG_MAX_PARTS];
};

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon, Moraes, Dror and Shaw, SC'11): ten rounds of two
// 32x32->64 multiplies; the key advances by the Weyl increments each round.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
  const uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    const uint32_t lo0 = M0 * c.x, hi0 = __umulhi(M0, c.x);
    const uint32_t lo1 = M1 * c.z, hi1 = __umulhi(M1, c.z);
    c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
    k0 += W0;
    k1 += W1;
  }
  return c;
}

__device__ __forceinline__ void set_status(int32_t* status, int32_t bits) {
  atomicOr(status, bits);
}

// ---------------------------------------------------------------------------
// Wave and block primitives.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (kWave - 1)); }

// Number of set bits of `mask` in lanes below this one.
__device__ __forceinline__ int lanes_below(uint64_t mask) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                        __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Lane index of the (r+1)-th set bit of mask (r < popcount(mask)).
__device__ __forceinline__ int nth_set_lane(uint64_t mask, int r) {
  int lo = 0;
#pragma unroll
  for (int w = 32; w >= 1; w >>= 1) {
    // set bits below lane lo + w
    const uint64_t below = (lo + w >= 64) ? mask : (mask & ((1ull << (lo + w)) - 1ull));
    if (__popcll(below) <= r) lo += w;
  }
  return lo;
}

template <typename T>
__device__ __forceinline__ T wave_incl_scan(T v) {
  const int lane = lane_id();
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const T t = __shfl_up(v, o, kWave);
    if (lane >= o) v += t;
  }
  return v;
}

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int o = kWave / 2; o >= 1; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

// Exclusive scan over a block of NT threads; lds must hold NT/64 entries.
// Every thread of the block must call it.
template <int NT, typename T>
__device__ __forceinline__ T block_excl_scan(T v, T* lds, T* total) {
  constexpr int NW = NT / kWave;
  const int wid = (int)threadIdx.x / kWave;
  const T inc = wave_incl_scan(v);
  if (lane_id() == kWave - 1) lds[wid] = inc;
  __syncthreads();
  T base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    const T x = lds[w];
    base += (w < wid) ? x : (T)0;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return base + inc - v;
}

// hist[key] += number of active lanes with `valid` and that key: one LDS
// atomic per distinct key present in the wave.  Call from every active lane.
__device__ __forceinline__ void wave_hist_add(int32_t* hist, bool valid, int32_t key) {
  const int lane = lane_id();
  for (uint64_t act = __ballot(valid); act;) {
    const int leader = __ffsll((unsigned long long)act) - 1;
    const int32_t kl = __shfl(key, leader, kWave);
    const uint64_t sel = __ballot(valid && key == kl);
    if (lane == leader) atomicAdd(&hist[kl], (int32_t)__popcll(sel));
    act &= ~sel;
  }
}

// sum[j] += the entries j of the n rows of `cols` (at most kBlock) counters at
// p, by one block: the rows lie back to back, and a thread keeps to one
// column, so that all of its loads are in flight together.
__device__ __forceinline__ void sum_columns(const int32_t* p, int n, int cols, int32_t* sum) {
  const int rows = kBlock / cols;
  if ((int)threadIdx.x >= rows * cols) return;
  const int j = threadIdx.x % cols;
  int32_t v = 0;
#pragma unroll 8
  for (int x = threadIdx.x / cols; x < n; x += rows) v += p[(int64_t)x * cols + j];
  if (v) atomicAdd(&sum[j], v);
}

// ---------------------------------------------------------------------------
// Row copy engine.  A wavefront copies up to 64 rows: lane r supplies the
// source of row r (nullptr = skip that row) and the rows land at
// dst0 + r * dst_stride.  The row bytes are cut into VB-byte pieces that are
// spread over the wave, so consecutive lanes move consecutive pieces of one
// row and then of the next: every load and store instruction covers a
// contiguous run of up to 1 KB, and short rows do not leave lanes idle.
// Piece c belongs to row c / pieces (piece_at, copy_geom.hpp).
// VB is 16 for rows of 16 bytes and more, at whatever multiple of 4 the rows
// start (global_load/store_dwordx4 need dword alignment only), and 4 for
// narrower rows.  Bound by memory.  Moving unaligned rows in words held four
// times as many instructions per byte: windows of 211K unpadded 2,408-byte
// rows took 592 us and now take 322, of 8 launches of 23K 300-byte rows 578
// and now 323 (whole sequential windows).
// ---------------------------------------------------------------------------
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef u32x4 __attribute__((aligned(4))) u32x4_a4;   // at any multiple of 4

template <int VB>
struct Piece;
template <>
struct Piece<16> {
  typedef u32x4 val;
  typedef u32x4_a4 mem;
};
template <>
struct Piece<4> {
  typedef uint32_t val;
  typedef uint32_t mem;
};

// Row addresses come out of shuffles as integers, so the compiler can't tell
// that they are global memory and would issue flat accesses, whose results
// the wave counts together with its LDS operations: every shuffle's wait
// would then also wait for the loads in flight.
#define GG_GLOBAL __attribute__((address_space(1)))

template <int VB>
__device__ __forceinline__ typename Piece<VB>::val ld_piece(const char* p) {
  typedef typename Piece<VB>::mem mem;
  return *(const GG_GLOBAL mem*)p;
}

template <int VB, bool NT>
__device__ __forceinline__ void st_piece(char* p, typename Piece<VB>::val v) {
  typedef typename Piece<VB>::mem mem;
  if (NT)
    __builtin_nontemporal_store(v, (GG_GLOBAL mem*)p);
  else
    *(GG_GLOBAL mem*)p = v;
}

template <int VB, bool NT, int U = (VB == 16 ? 4 : 8)>
__device__ __forceinline__ void wave_copy_rows(const char* src, char* dst0, int64_t dst_stride,
                                               int nrows, const CopyGeom& g) {
  const int lane = lane_id();
  const uint32_t total = (uint32_t)nrows * g.pieces;
  const long long srcl = (long long)src;
  for (uint32_t base = 0; base < total; base += kWave * U) {
    // Destinations are recomputed at the stores: holding U 64-bit pointers
    // across the loads would cost 2U registers.
    typename Piece<VB>::val v[U];
    bool ok[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const uint32_t c = base + (uint32_t)(j * kWave + lane);
      uint32_t r;
      const uint32_t off = piece_at(g, c, VB, &r);
      const char* sp = (const char*)__shfl(srcl, (int)(r & 63u), kWave);
      ok[j] = (c < total) && (sp != nullptr);
      if (ok[j]) v[j] = ld_piece<VB>(sp + off);
    }
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const uint32_t c = base + (uint32_t)(j * kWave + lane);
      uint32_t r;
      const uint32_t off = piece_at(g, c, VB, &r);
      if (ok[j]) st_piece<VB, NT>(dst0 + (int64_t)r * dst_stride + off, v[j]);
    }
  }
}

// As wave_copy_rows, with a destination per row: lane r supplies both the
// source and the destination of row r (a nullptr source skips the row).
template <int VB, bool NT, int U = (VB == 16 ? 4 : 8)>
__device__ __forceinline__ void wave_copy_rows_to(const char* src, char* dst, int nrows,
                                                  const CopyGeom& g) {
  const int lane = lane_id();
  const uint32_t total = (uint32_t)nrows * g.pieces;
  const long long srcl = (long long)src, dstl = (long long)dst;
  for (uint32_t base = 0; base < total; base += kWave * U) {
    typename Piece<VB>::val v[U];
    char* dp[U];
    bool ok[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
      const uint32_t c = base + (uint32_t)(j * kWave + lane);
      uint32_t r;
      const uint32_t off = piece_at(g, c, VB, &r);
      const char* sp = (const char*)__shfl(srcl, (int)(r & 63u), kWave);
      dp[j] = (char*)__shfl(dstl, (int)(r & 63u), kWave) + off;
      ok[j] = (c < total) && (sp != nullptr);
      if (ok[j]) v[j] = ld_piece<VB>(sp + off);
    }
#pragma unroll
    for (int j = 0; j < U; ++j)
      if (ok[j]) st_piece<VB, NT>(dp[j], v[j]);
  }
}

}  // namespace gg
