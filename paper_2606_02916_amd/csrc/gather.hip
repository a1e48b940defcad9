// gg_gather_batch: feature assembly of one or more consecutive batches
// through the ID-to-slot remap, with the on-demand miss path.
//
// Grid (bx, nseg), bx blocks to a segment (batch), so that every block's
// statistics belong to one batch and reduce without atomics.  Each
// wavefront takes a tile of consecutive output rows at a time (up to 64
// rows and 8 KB); every lane of the tile resolves its row (local shard,
// cache slot, or the owner's shard for a miss) and the wave copies the
// resolved rows with the row copy engine.  Misses differ only in where the
// row comes from and in the counts per block and owner; a pass of their own
// over the same tiles would resolve every row again (a sequential window of
// 1.5M rows, two thirds of its remote ones misses: 480 us with two passes, 439
// with one).  A second launch of one block per segment sums the blocks'
// statistics.
#include <stdlib.h>
#include <string.h>

#include <mutex>

#include "gg_host.hpp"

// Scratch of gg_gather_batch_noalloc (see device_scratch below).
static __device__ __align__(256) int32_t scratch[GG_GATHER_SCRATCH_BYTES / sizeof(int32_t)];

namespace gg {
namespace {

constexpr int kTilesPerBlock = kBlock / kWave;  // 4 waves
// Blocks per launch, shared by the segments (tuning gather_blocks).  Alone,
// 1,024 (four per CU): whole sequential windows took 474 / 325 us (1.5M rows
// of 400 bytes with misses / 211K unaligned rows of 2,408) against 548 / 335
// with 512, 492 / 326 with 768 and 492 / 342 with 1,536.  Beside the next
// window's sampling and staging, 512: eight loads per lane keep enough bytes
// in flight with half the blocks, and the rest of the chip goes to the other
// chain (six look-ahead windows of 1.5M 400-byte rows / 295K 2,408-byte rows:
// 2,135 / 2,018 us, against 2,300 / 2,205 with 1,024, 2,205 / 2,117 with 768,
// 2,204 / 2,018 with 448 and 2,221 / 1,987 with 512 and four loads).  That is
// for windows that the gather bounds.  In smaller ones the build is the longer
// chain, and its small launches run slower on every CU that holds gather
// blocks, whatever these keep in flight (one batch of 4,096 seeds, 79 MB of
// rows, windows queued: 149 us with 512 blocks of eight loads or of two, 139
// with 128 of eight).  So below kSharedWhole bytes only one block per
// kSharedBytes works, 64 to 256 in all: the first of the grid, which the host
// sizes before it knows the rows, so that they lie on as many CUs as they can.
// Queued windows, 512 blocks / by bytes: 38 MB of rows 114 / 106 us, 79 MB 148 /
// 138, 152 MB 180 / 169, 154 MB 183 / 169, 292 MB 230 / 214, 313 MB 265 / 245,
// 351 MB of wide rows 222 / 200; six windows from start to end, 152 MB 1,210 /
// 1,180, 292 MB 1,547 / 1,450.  Fewer blocks still (one per 786,432 bytes) cost
// six windows of 154 MB 3%; from 370 MB on 256 blocks are no faster, and from
// 450 MB slower (264 / 278).
constexpr int64_t kSharedBytes = 5 << 17;
constexpr int64_t kSharedWhole = 340LL << 20;
constexpr int kSharedLeast = 64, kSharedMost = 256;

struct GatherArgs {
  int64_t n_cap;        // output rows available
  int64_t cache_stride;
  int64_t cache_rows;
  int64_t out_stride;
  int32_t nseg;
  int32_t nstat;        // 2 + P counters per block
  int32_t tile;         // rows per wave step (copy_tile)
  int32_t by_bytes;     // row bytes if the working blocks depend on them, else 0
  CopyGeom geom;
};

// Output rows [lo, hi) of segment s, relative to bounds[0], clamped to n_cap.
__device__ __forceinline__ void seg_range(const int64_t* bounds, int s, const GatherArgs& a,
                                          int64_t* lo, int64_t* hi) {
  const int64_t b0 = bounds[0];
  int64_t l = bounds[s] - b0, h = bounds[s + 1] - b0;
  l = l < 0 ? 0 : (l > a.n_cap ? a.n_cap : l);
  h = h < l ? l : (h > a.n_cap ? a.n_cap : h);
  *lo = l;
  *hi = h;
}

// Blocks of a segment that work, of the grid's bx.
__device__ __forceinline__ int working_blocks(const int64_t* bounds, const GatherArgs& a, int bx) {
  if (!a.by_bytes) return bx;
  int64_t rows = bounds[a.nseg] - bounds[0];
  rows = rows < a.n_cap ? rows : a.n_cap;
  const int64_t bytes = rows * a.by_bytes;
  if (bytes >= kSharedWhole) return bx;
  int blocks = (int)(bytes / kSharedBytes);
  blocks = blocks < kSharedLeast ? kSharedLeast : (blocks > kSharedMost ? kSharedMost : blocks);
  const int each = (blocks + a.nseg - 1) / a.nseg;
  return each < bx ? each : bx;
}

// Row ids and owners of one tile, loaded ahead of its copy.
struct TileIds {
  int32_t u;      // row id, or -1 for a lane past the tile or the segment
  int32_t m;      // owner of u (-1 when u is absent or out of range)
  int32_t s;      // slot of u for a remote owner, loaded one tile ahead
  bool in;        // the lane holds a row of the segment
};

__device__ __forceinline__ bool tile_lane(int64_t t, int64_t ntiles, int64_t lo, int64_t hi,
                                          int32_t tile, int lane) {
  return t < ntiles && lane < tile && lo + t * tile + lane < hi;
}

template <int VB, bool NT, int U>
__global__ void __launch_bounds__(kBlock) k_gather_rows(const int32_t* in_ids, const int64_t* bounds,
                                                        KPart part, KFeat feat, GatherArgs a,
                                                        const char* cache, const int32_t* slot_of,
                                                        char* out, int32_t* blk_stat,
                                                        int32_t* status) {
  const int bx = working_blocks(bounds, a, gridDim.x);
  const int block = blockIdx.y * gridDim.x + blockIdx.x;
  if (block >= bx * a.nseg) return;
  const int seg = block / bx, x = block - seg * bx;
  __shared__ int64_t s_start[GG_MAX_PARTS + 1];
  __shared__ int32_t s_cnt[2 + GG_MAX_PARTS];  // local, hits, misses per owner
  for (int t = threadIdx.x; t <= GG_MAX_PARTS; t += blockDim.x) s_start[t] = part.start[t];
  for (int t = threadIdx.x; t < 2 + GG_MAX_PARTS; t += blockDim.x) s_cnt[t] = 0;
  __syncthreads();
  int64_t lo, hi;
  seg_range(bounds, seg, a, &lo, &hi);
  const int64_t begin = bounds[0];
  const int lane = lane_id();
  const int64_t ntiles = (hi - lo + a.tile - 1) / a.tile;
  const int64_t step = (int64_t)bx * kTilesPerBlock;
  int32_t st = 0;
  int32_t c_local = 0, c_hit = 0;
  // Software pipeline over the wave's tiles: while tile t is copied, the
  // slots of tile t + step and the ids of tile t + 2 step are already in
  // flight, so neither lookup waits in front of a copy.
  auto load_ids = [&](int64_t t) -> TileIds {
    TileIds x{-1, -1, -1, tile_lane(t, ntiles, lo, hi, a.tile, lane)};
    if (x.in) x.u = in_ids[begin + lo + t * a.tile + lane];
    return x;
  };
  auto load_slot = [&](TileIds& x) {
    if (x.in && x.u >= 0 && (int64_t)x.u < part.N) {
      x.m = owner_of(part, s_start, x.u);
      if (x.m != part.local) x.s = slot_of[x.u];
    }
  };
  int64_t t = (int64_t)x * kTilesPerBlock + threadIdx.x / kWave;
  TileIds cur = load_ids(t);
  load_slot(cur);
  TileIds nxt = load_ids(t + step);
  for (; t < ntiles; t += step) {
    load_slot(nxt);
    const TileIds after = load_ids(t + 2 * step);
    const char* src = nullptr;
    bool miss = false, is_local = false, is_hit = false;
    if (cur.in) {
      if (cur.m < 0) {
        st |= GG_DEV_BAD_ID;
      } else if (cur.m == part.local) {
        const int64_t r = row_of(part, s_start, cur.u, cur.m);
        if (r < feat.rows[cur.m]) {
          src = feat.shard[cur.m] + r * feat.stride[cur.m];
          is_local = true;
        } else {
          st |= GG_DEV_BAD_ROW;
        }
      } else if (cur.s >= 0 && (int64_t)cur.s < a.cache_rows) {
        src = cache + (int64_t)cur.s * a.cache_stride;
        is_hit = true;
      } else {
        if (cur.s >= 0) st |= GG_DEV_BAD_ROW;
        miss = true;
        const int64_t r = row_of(part, s_start, cur.u, cur.m);
        if (r < feat.rows[cur.m])
          src = feat.shard[cur.m] + r * feat.stride[cur.m];   // on demand, from the owner
        else
          st |= GG_DEV_BAD_ROW;
      }
    }
    const uint64_t ml = __ballot(is_local), mh = __ballot(is_hit), mm = __ballot(miss);
    c_local += (int32_t)__popcll(ml);
    c_hit += (int32_t)__popcll(mh);
    // Per-owner miss counts: one ballot per owner present.
    for (uint64_t act = mm; act;) {
      const int leader = __ffsll((unsigned long long)act) - 1;
      const int32_t ol = __shfl(cur.m, leader, kWave);
      const uint64_t sel = __ballot(miss && cur.m == ol);
      if (lane == leader) atomicAdd(&s_cnt[2 + ol], (int32_t)__popcll(sel));
      act &= ~sel;
    }
    const int64_t r0 = lo + t * a.tile;
    const int64_t left = hi - r0;
    const int nrows = left < a.tile ? (int)left : a.tile;
    wave_copy_rows<VB, NT, U>(src, out + r0 * a.out_stride, a.out_stride, nrows, a.geom);
    cur = nxt;
    nxt = after;
  }
  if (lane == 0) {
    if (c_local) atomicAdd(&s_cnt[0], c_local);
    if (c_hit) atomicAdd(&s_cnt[1], c_hit);
  }
  if (st) set_status(status, st);
  __syncthreads();
  int32_t* dst = blk_stat + ((int64_t)seg * gridDim.x + x) * a.nstat;
  for (int t = threadIdx.x; t < a.nstat; t += blockDim.x) dst[t] = s_cnt[t];
}

// Block s: the statistics of batch s from its blocks' counts.
__global__ void __launch_bounds__(kBlock) k_gather_stats(const int64_t* bounds, int32_t P,
                                                         GatherArgs a, int32_t bx,
                                                         const int32_t* blk_stat,
                                                         gg_gather_stats_t* stats,
                                                         int32_t* status) {
  __shared__ int32_t s_sum[2 + GG_MAX_PARTS];
  const int s = blockIdx.x;
  for (int t = threadIdx.x; t < 2 + GG_MAX_PARTS; t += blockDim.x) s_sum[t] = 0;
  __syncthreads();
  sum_columns(blk_stat + (int64_t)s * bx * a.nstat, working_blocks(bounds, a, bx), a.nstat, s_sum);
  __syncthreads();
  gg_gather_stats_t* o = stats + s;
  if (threadIdx.x < GG_MAX_PARTS) {
    const int m = threadIdx.x;
    const int64_t rows = m < P ? (int64_t)s_sum[2 + m] : 0;
    o->miss_rows[m] = rows;
    o->miss_requests[m] = rows > 0 ? 1 : 0;
  }
  if (threadIdx.x == 0) {
    int64_t misses = 0;
    for (int m = 0; m < P; ++m) misses += s_sum[2 + m];
    int64_t lo, hi;
    seg_range(bounds, s, a, &lo, &hi);
    o->rows = hi - lo;
    o->local = s_sum[0];
    o->hits = s_sum[1];
    o->misses = misses;
    if (bounds[s + 1] - bounds[0] > a.n_cap) set_status(status, GG_DEV_CAPACITY);
  }
}

struct GatherWs {
  int32_t* blk_stat;   // per row block: local, hits, misses per owner
};

int32_t blocks_per_seg(int64_t n_cap, int32_t nseg, const Tune& tune, bool shared = false) {
  const int32_t blocks = tune.gather_blocks ? tune.gather_blocks
                         : shared           ? kGatherBlocksShared
                                            : kGatherBlocksAlone;
  int64_t bx = std::max<int64_t>(blocks / nseg, 8);
  bx = std::min<int64_t>(bx, std::max<int64_t>(1, cdiv(n_cap, kBlock)));
  return (int32_t)bx;
}

// Sized for a gather alone, which launches at least as many blocks as a shared one.
size_t gather_ws_layout(int64_t n_cap, int32_t nseg, int32_t P, const Tune& tune, char* base,
                        GatherWs* out) {
  const int64_t bx = blocks_per_seg(n_cap, nseg, tune);
  Carve cv{base, 0, ~(size_t)0};
  GatherWs g;
  g.blk_stat = cv.take<int32_t>((size_t)(nseg * bx * (2 + P)));
  if (out) *out = g;
  return align_up(cv.used, 256);
}

template <int VB, bool NT>
void launch_gather(hipStream_t stream, int unroll, int32_t bx, const int32_t* in_ids, const int64_t* bounds,
                   const KPart& kp, const KFeat& kf, const GatherArgs& a, const char* cache,
                   const int32_t* slot_of, char* out, const GatherWs& w, gg_gather_stats_t* stats,
                   int32_t* status) {
  if (VB == 16 && unroll == 8)
    hipLaunchKernelGGL((k_gather_rows<VB, NT, 8>), dim3(bx, a.nseg), dim3(kBlock), 0, stream, in_ids,
                       bounds, kp, kf, a, cache, slot_of, out, w.blk_stat, status);
  else if (VB == 16 && unroll == 4)
    hipLaunchKernelGGL((k_gather_rows<VB, NT, 4>), dim3(bx, a.nseg), dim3(kBlock), 0, stream, in_ids,
                       bounds, kp, kf, a, cache, slot_of, out, w.blk_stat, status);
  else if (VB == 16 && unroll == 2)
    hipLaunchKernelGGL((k_gather_rows<VB, NT, 2>), dim3(bx, a.nseg), dim3(kBlock), 0, stream, in_ids,
                       bounds, kp, kf, a, cache, slot_of, out, w.blk_stat, status);
  else
    hipLaunchKernelGGL((k_gather_rows<VB, NT, VB == 16 ? 4 : 8>), dim3(bx, a.nseg), dim3(kBlock), 0,
                       stream, in_ids, bounds, kp, kf, a, cache, slot_of, out, w.blk_stat, status);
  hipLaunchKernelGGL(k_gather_stats, dim3(a.nseg), dim3(kBlock), 0, stream, bounds, kp.P, a, bx,
                     w.blk_stat, stats, status);
}

}  // namespace
}  // namespace gg

using namespace gg;

extern "C" size_t gg_ws_gather(int64_t n_cap, int32_t nseg, int32_t num_parts,
                               const gg_tuning_t* tuning) {
  Tune tune;
  if (resolve_tuning(tuning, &tune) != GG_OK) return 0;
  // Every call with at most nseg segments and n_cap rows fits: the blocks
  // per segment divide the gather's block count, so fewer segments can
  // launch more blocks in all (1024 blocks: 3 x 341, but 1 x 1024).
  size_t need = 0;
  for (int32_t s = 1; s <= std::min(std::max(nseg, 1), GG_MAX_W); ++s)
    need = std::max(need, gather_ws_layout(n_cap, s, num_parts, tune, nullptr, nullptr));
  return need;
}

namespace gg {
namespace {

// The per-block statistics of gg_gather_batch_noalloc: a file-scope device
// array, one copy per GPU, held until the process ends.  Host code never
// hands the array's name to a kernel (in host code it is a stand-in, not a
// device address): it takes the array's address on each device from
// hipGetSymbolAddress, once, with that device current.
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

int device_scratch(hipStream_t stream, void** out) {
  int dev = 0;
  hipError_t e = stream ? hipStreamGetDevice(stream, &dev) : hipGetDevice(&dev);
  if (e != hipSuccess) {
    set_error("gg_gather_batch_noalloc: no device for the stream: %s", hipGetErrorString(e));
    return GG_ERR_HIP;
  }
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("gg_gather_batch_noalloc: device %d beyond the %d supported", dev, kMaxDevices);
    return GG_ERR_UNSUPPORTED;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    int cur = 0;
    e = hipGetDevice(&cur);
    if (e == hipSuccess && cur != dev) e = hipSetDevice(dev);
    void* p = nullptr;
    if (e == hipSuccess) e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (cur != dev) (void)hipSetDevice(cur);
    if (e != hipSuccess || !p) {
      set_error("gg_gather_batch_noalloc: address of the scratch array on device %d: %s", dev,
                hipGetErrorString(e));
      return GG_ERR_HIP;
    }
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return GG_OK;
}

// Both gather entry points: ws/ws_bytes is the caller's workspace, or with
// noalloc the device array (ws is then ignored).
int gather_impl(const int32_t* in_ids_d, const int64_t* bounds_d, int32_t nseg, int64_t n_cap,
                const gg_part_t* part, const gg_feat_t* feat, const void* cache_d,
                int64_t cache_stride, int64_t cache_rows, const int32_t* slot_of_d, void* out_d,
                int64_t out_stride, int32_t flags, gg_gather_stats_t* stats_d,
                const gg_tuning_t* tuning, int32_t* status_d, void* ws, size_t ws_bytes,
                bool noalloc, hipStream_t stream) {
  GG_REQUIRE(bounds_d && slot_of_d && stats_d && status_d, "NULL argument");
  Tune tune;
  if (resolve_tuning(tuning, &tune) != GG_OK) return GG_ERR_ARG;
  GG_REQUIRE((flags & ~GG_GATHER_SHARED) == 0, "unknown flags 0x%x", (unsigned)flags);
  GG_REQUIRE(nseg >= 1 && nseg <= GG_MAX_W, "nseg = %d outside 1..%d", nseg, GG_MAX_W);
  GG_REQUIRE(n_cap >= 0 && n_cap < (1LL << 31), "n_cap %lld unsupported", (long long)n_cap);
  GG_REQUIRE(n_cap == 0 || (in_ids_d && out_d), "NULL id or output buffer");
  GG_REQUIRE(cache_rows >= 0 && (cache_rows == 0 || cache_d), "cache is NULL");
  KPart kp;
  int rc = pack_part(part, &kp);
  if (rc != GG_OK) return rc;
  KFeat kf;
  rc = pack_feat(feat, part, &kf);
  if (rc != GG_OK) return rc;
  GG_REQUIRE(out_stride >= kf.row_bytes && out_stride % 4 == 0, "out_stride %lld invalid",
             (long long)out_stride);
  GG_REQUIRE(cache_rows == 0 || (cache_stride >= kf.row_bytes && cache_stride % 4 == 0),
             "cache_stride %lld invalid", (long long)cache_stride);
  GG_REQUIRE(((uintptr_t)out_d & 3u) == 0 && ((uintptr_t)cache_d & 3u) == 0,
             "output and cache must be 4-byte aligned");
  const size_t need_ws = gather_ws_layout(n_cap, nseg, kp.P, tune, nullptr, nullptr);
  if (noalloc) {
    if (need_ws > (size_t)GG_GATHER_SCRATCH_BYTES) {
      set_error("gg_gather_batch_noalloc: %d segments of %d blocks with %d owners need %zu bytes "
                "of scratch; the library's array holds %d",
                nseg, blocks_per_seg(n_cap, nseg, tune), kp.P, need_ws, GG_GATHER_SCRATCH_BYTES);
      return GG_ERR_CAPACITY;
    }
    rc = device_scratch(stream, &ws);
    if (rc != GG_OK) return rc;
    ws_bytes = GG_GATHER_SCRATCH_BYTES;
  }
  GG_REQUIRE(ws && ws_bytes >= need_ws, "workspace of %zu bytes < %zu", ws_bytes, need_ws);
  GatherWs gw;
  gather_ws_layout(n_cap, nseg, kp.P, tune, (char*)ws, &gw);
  const bool v16 = copy_by_16(kf.row_bytes);
  GatherArgs a;
  a.n_cap = n_cap;
  a.cache_stride = cache_stride;
  a.cache_rows = cache_rows;
  a.out_stride = out_stride;
  a.nseg = nseg;
  a.nstat = 2 + kp.P;
  // Tiles of up to 8 KB: more, smaller tiles leave a shorter tail of waves
  // still copying their last tile than 32 KB ones (400-byte rows 228 against
  // 237 us alone, 2,408-byte rows 246 against 261).  Shared, a tile holds as
  // many rows as fit, 20 of 400 bytes (500 pieces of a step's 512); alone it
  // stays a power of two, 16 rows and 2, which measured 1-3% faster there
  // than 20 and 3.
  const bool shared = (flags & GG_GATHER_SHARED) != 0;
  a.tile = copy_tile(tune, kf.row_bytes, 8192, !shared);
  a.by_bytes = shared && !tune.gather_blocks ? kf.row_bytes : 0;
  a.geom = copy_geom(kf.row_bytes);
  const int32_t bx = blocks_per_seg(n_cap, nseg, tune, shared);
  const char* cache = (const char*)cache_d;
  char* out = (char*)out_d;
  // Output rows are stored non-temporally: the gather never reads them back.
  if (v16)
    launch_gather<16, true>(stream, tune.gather_loads, bx, in_ids_d, bounds_d, kp, kf, a, cache, slot_of_d,
                            out, gw, stats_d, status_d);
  else
    launch_gather<4, true>(stream, tune.gather_loads, bx, in_ids_d, bounds_d, kp, kf, a, cache, slot_of_d,
                           out, gw, stats_d, status_d);
  GG_LAUNCH_CHECK("k_gather_rows/k_gather_stats");
  return GG_OK;
}

}  // namespace
}  // namespace gg

extern "C" int gg_gather_batch(const int32_t* in_ids_d, const int64_t* bounds_d, int32_t nseg,
                               int64_t n_cap, const gg_part_t* part, const gg_feat_t* feat,
                               const void* cache_d, int64_t cache_stride, int64_t cache_rows,
                               const int32_t* slot_of_d, void* out_d, int64_t out_stride,
                               int32_t flags, gg_gather_stats_t* stats_d,
                               const gg_tuning_t* tuning, int32_t* status_d, void* ws,
                               size_t ws_bytes, hipStream_t stream) {
  return gather_impl(in_ids_d, bounds_d, nseg, n_cap, part, feat, cache_d, cache_stride,
                     cache_rows, slot_of_d, out_d, out_stride, flags, stats_d, tuning, status_d,
                     ws, ws_bytes, false, stream);
}

extern "C" int gg_gather_batch_noalloc(const int32_t* in_ids_d, const int64_t* bounds_d,
                                       int32_t nseg, int64_t n_cap, const gg_part_t* part,
                                       const gg_feat_t* feat, const void* cache_d,
                                       int64_t cache_stride, int64_t cache_rows,
                                       const int32_t* slot_of_d, void* out_d, int64_t out_stride,
                                       int32_t flags, gg_gather_stats_t* stats_d,
                                       const gg_tuning_t* tuning, int32_t* status_d,
                                       hipStream_t stream) {
  return gather_impl(in_ids_d, bounds_d, nseg, n_cap, part, feat, cache_d, cache_stride,
                     cache_rows, slot_of_d, out_d, out_stride, flags, stats_d, tuning, status_d,
                     nullptr, 0, true, stream);
}
