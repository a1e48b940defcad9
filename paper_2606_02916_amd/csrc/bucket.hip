// gg_bucket_by_owner: stable partition of the hot set by partition owner.
//
// Two passes over the ids: per-block owner counts, and a scatter in which every
// block places itself from all blocks' counts and every wavefront ranks its
// ids among equal owners with ballots (one ballot per distinct owner present
// in the wave), so order is kept inside each owner.
//
// Range partitions first try the identity: when owners never decrease along
// the input (the ascending hot set always satisfies this), the input is
// already owner-major.  k_bucket_range copies it, writes owner_off from the
// owner changes and records per block whether its ids were in owner order;
// the general passes then run only if some block saw a decrease.  A caller
// that knows its input is in owner order (GG_BUCKET_OWNER_ORDERED) skips the
// general passes' launches altogether; a block that finds the order broken
// then raises GG_DEV_ORDER.
#include "gg_host.hpp"

namespace gg {
namespace {

// The general path cuts the n ids into at most max_blocks(P) equal spans of
// whole kSpanIds, one block each, sized on the device (the host knows the
// capacity only).  Its second launch places a block from all blocks' counts, so
// that they need no scan launch between the two.  More blocks share the ids but
// each reads more counts: up to kMaxCounts of them, 32 KB that stay in L2, and
// always as many as keep the chip busy, whose 256 KB at 64 owners cost less than
// the ids of fewer blocks one after the other (4M ids: 64 owners 711 us with
// 128 blocks, 378 with 256, 201 with 512, 130 with 1,024; 32 owners 265 with
// 256, 89 with 1,024; up to 300K ids no difference).
constexpr int kSpanIds = 1024;                 // four groups of 64 per wave
constexpr int kWaveGroups = kSpanIds / kBlock;
constexpr int kMaxCounts = 8192;
constexpr int kMinBlocks = 1024;

inline int max_blocks(int32_t P) { return std::max(kMaxCounts / P, kMinBlocks); }

// Ids per block for n ids and `blocks` blocks.
__device__ __forceinline__ int64_t span_of(int64_t n, int blocks) {
  const int64_t spans = (n + kSpanIds - 1) / kSpanIds;
  return (spans + blocks - 1) / blocks * kSpanIds;
}

__device__ __forceinline__ int64_t bucket_n(const int64_t* hot_count, int64_t cap) {
  const int64_t n = hot_count[0];
  return n < cap ? n : cap;
}

// Owner-order check and identity bucketing for range partitions.  A block
// takes every gridDim.x-th run of kRangeIds consecutive ids, four per thread,
// all loads issued before any store.  It copies them, writes the owner_off
// entries of every owner change it sees, and writes ok[blockIdx.x] = 1 when its
// ids were valid and in owner order.  The grid is capped: the capacity of a
// 111M-node graph's hot set asks for 17K runs, of which a thousand hold ids
// (34 us with a block each, 22 now, beside the window's other work).
constexpr int kRangePer = 4;
constexpr int kRangeIds = kBlock * kRangePer;
constexpr int kRangeBlocks = 2048;

__global__ void __launch_bounds__(kBlock) k_bucket_range(const int32_t* ids, const int64_t* hot_count,
                                                         int64_t cap, KPart part, int32_t* out,
                                                         int64_t* owner_off, int32_t* ok,
                                                         int32_t order_bit, int32_t* status) {
  __shared__ int64_t s_start[GG_MAX_PARTS + 1];
  __shared__ int32_t s_bad;
  for (int t = threadIdx.x; t <= GG_MAX_PARTS; t += blockDim.x) s_start[t] = part.start[t];
  if (threadIdx.x == 0) s_bad = 0;
  __syncthreads();
  const int64_t n = bucket_n(hot_count, cap);
  const int P = part.P;
  if (n == 0 && blockIdx.x == 0)
    for (int m = threadIdx.x; m <= P; m += blockDim.x) owner_off[m] = 0;
  int bad = 0, bad_id = 0;
  for (int64_t i0 = (int64_t)blockIdx.x * kRangeIds + (int64_t)threadIdx.x * kRangePer; i0 < n;
       i0 += (int64_t)gridDim.x * kRangeIds) {
    int32_t v[kRangePer + 1];  // v[0] = the id before this thread's first
#pragma unroll
    for (int j = 0; j <= kRangePer; ++j) {
      const int64_t i = i0 + j - 1;
      v[j] = (i >= 0 && i < n) ? ids[i] : -1;
    }
    int32_t op = -1;
    if (i0 > 0 && i0 <= n) {
      const int32_t up = v[0];
      op = (up < 0 || (int64_t)up >= part.N) ? P : owner_of(part, s_start, up);
    }
#pragma unroll
    for (int j = 1; j <= kRangePer; ++j) {
      const int64_t i = i0 + j - 1;
      if (i >= n) break;
      const int32_t u = v[j];
      if (u < 0 || (int64_t)u >= part.N) {
        bad = bad_id = 1;
        op = P;
        continue;
      }
      const int32_t o = owner_of(part, s_start, u);
      if (op > o) bad = 1;
      for (int32_t m = op + 1; m <= o; ++m) owner_off[m] = i;
      if (i == n - 1)
        for (int32_t m = o + 1; m <= P; ++m) owner_off[m] = n;
      out[i] = u;
      op = o;
    }
  }
  if (bad) atomicOr(&s_bad, bad_id ? 3 : 1);
  __syncthreads();
  if (threadIdx.x == 0) {
    if (ok) ok[blockIdx.x] = s_bad ? 0 : 1;
    // Trusted input: the general passes do not run, so report here.
    if (s_bad && order_bit) set_status(status, (s_bad & 2) ? (order_bit | GG_DEV_BAD_ID) : order_bit);
  }
}

// True when the identity pass of every block succeeded.
__device__ __forceinline__ bool range_done(const int32_t* ok, int32_t nok, int32_t* s_flag) {
  if (ok == nullptr) return false;
  if (threadIdx.x == 0) *s_flag = 1;
  __syncthreads();
  for (int x = threadIdx.x; x < nok; x += blockDim.x)
    if (ok[x] == 0) *s_flag = 0;
  __syncthreads();
  return *s_flag != 0;
}

// The block's ids per owner: cnt[block][owner].
__global__ void __launch_bounds__(kBlock) k_bucket_count(const int32_t* ids, const int64_t* hot_count,
                                                         int64_t cap, KPart part, int32_t* cnt,
                                                         const int32_t* ok, int32_t nok,
                                                         int32_t* status) {
  __shared__ int32_t s_flag;
  if (range_done(ok, nok, &s_flag)) return;
  __shared__ int32_t hist[GG_MAX_PARTS];
  __shared__ int64_t s_start[GG_MAX_PARTS + 1];
  for (int t = threadIdx.x; t < GG_MAX_PARTS; t += blockDim.x) hist[t] = 0;
  for (int t = threadIdx.x; t <= GG_MAX_PARTS; t += blockDim.x) s_start[t] = part.start[t];
  __syncthreads();
  const int64_t n = bucket_n(hot_count, cap);
  const int64_t span = span_of(n, gridDim.x);
  const int64_t lo = blockIdx.x * span, hi = lo + span < n ? lo + span : n;
  int32_t st = 0;
  for (int64_t i0 = lo + threadIdx.x; i0 < hi; i0 += kSpanIds) {
    int32_t u[kWaveGroups];
#pragma unroll
    for (int j = 0; j < kWaveGroups; ++j)
      u[j] = i0 + j * kBlock < hi ? ids[i0 + j * kBlock] : INT32_MIN;
#pragma unroll
    for (int j = 0; j < kWaveGroups; ++j) {
      if (u[j] >= 0 && (int64_t)u[j] < part.N)
        atomicAdd(&hist[owner_of(part, s_start, u[j])], 1);
      else if (i0 + j * kBlock < hi)
        st |= GG_DEV_BAD_ID;
    }
  }
  if (st) set_status(status, st);
  __syncthreads();
  for (int m = threadIdx.x; m < part.P; m += blockDim.x)
    cnt[(int64_t)blockIdx.x * part.P + m] = hist[m];
}

// Every block sums the counts of all blocks per owner (and of the blocks
// before it), which places its ids; block 0 writes owner_off.  Ids keep their
// order inside each owner: a wave takes 256 consecutive ids, ranks each group
// of 64 among equal owners by ballot (lane m keeps the wave's running count of
// owner m), and the waves' counts order the waves.  Bound by launch latency
// (105K ids, eight owners: 36 us with spans of 4,096 walked twice, and 19 + 5
// for the count and scan launches before it; now 10 + 4).
__global__ void __launch_bounds__(kBlock) k_bucket_scatter(const int32_t* ids, const int64_t* hot_count,
                                                           int64_t cap, KPart part,
                                                           const int32_t* cnt, int64_t* owner_off,
                                                           const int32_t* ok, int32_t nok,
                                                           int32_t* out) {
  __shared__ int32_t s_flag;
  if (range_done(ok, nok, &s_flag)) return;
  constexpr int kWaves = kBlock / kWave;
  __shared__ int32_t s_tot[GG_MAX_PARTS], s_before[GG_MAX_PARTS];
  __shared__ int32_t s_base[GG_MAX_PARTS];     // next output position of each owner
  __shared__ int32_t s_wave[kWaves][GG_MAX_PARTS];
  __shared__ int64_t s_start[GG_MAX_PARTS + 1];
  const int P = part.P, w = threadIdx.x / kWave, lane = lane_id();
  for (int t = threadIdx.x; t < GG_MAX_PARTS; t += blockDim.x) s_tot[t] = s_before[t] = 0;
  for (int t = threadIdx.x; t <= GG_MAX_PARTS; t += blockDim.x) s_start[t] = part.start[t];
  __syncthreads();
  const int64_t n = bucket_n(hot_count, cap);
  const int64_t span = span_of(n, gridDim.x);
  const int64_t lo = blockIdx.x * span, hi = lo + span < n ? lo + span : n;
  // threads in whole rows of P counts: each keeps to one owner
  const int rows = kBlock / P;
  if ((int)threadIdx.x < rows * P) {
    const int nb = span > 0 ? (int)((n + span - 1) / span) : 0;   // blocks with ids
    const int m = threadIdx.x % P;
    int32_t tot = 0, before = 0;
#pragma unroll 8
    for (int x = threadIdx.x / P; x < nb; x += rows) {
      const int32_t c = cnt[(int64_t)x * P + m];
      tot += c;
      before += x < (int)blockIdx.x ? c : 0;
    }
    if (tot) atomicAdd(&s_tot[m], tot);
    if (before) atomicAdd(&s_before[m], before);
  }
  __syncthreads();
  if (w == 0) {
    const int32_t t = lane < P ? s_tot[lane] : 0;
    const int32_t first = wave_incl_scan(t) - t;
    if (lane < P) {
      s_base[lane] = first + s_before[lane];
      if (blockIdx.x == 0) {
        owner_off[lane] = first;
        if (lane == P - 1) owner_off[P] = first + t;
      }
    }
  }
  __syncthreads();
  for (int64_t i0 = lo; i0 < hi; i0 += kSpanIds) {
    const int64_t iw = i0 + w * (kSpanIds / kWaves) + lane;
    int32_t u[kWaveGroups], o[kWaveGroups], rank[kWaveGroups];
    int32_t mine = 0;                          // lane m: the wave's ids of owner m so far
#pragma unroll
    for (int g = 0; g < kWaveGroups; ++g) u[g] = iw + g * kWave < hi ? ids[iw + g * kWave] : -1;
#pragma unroll
    for (int g = 0; g < kWaveGroups; ++g) {
      const bool valid = u[g] >= 0 && (int64_t)u[g] < part.N;
      o[g] = valid ? owner_of(part, s_start, u[g]) : -1;
      rank[g] = 0;
      for (uint64_t active = __ballot(valid); active;) {
        const int leader = __ffsll((unsigned long long)active) - 1;
        const int32_t ol = __shfl(o[g], leader, kWave);
        const uint64_t mm = __ballot(valid && o[g] == ol);
        const int32_t before = __shfl(mine, ol, kWave);
        if (o[g] == ol) rank[g] = before + lanes_below(mm);
        if (lane == ol) mine += (int32_t)__popcll(mm);
        active &= ~mm;
      }
    }
    if (lane < P) s_wave[w][lane] = mine;
    __syncthreads();
#pragma unroll
    for (int g = 0; g < kWaveGroups; ++g)
      if (o[g] >= 0) {
        int32_t at = s_base[o[g]] + rank[g];
        for (int v = 0; v < w; ++v) at += s_wave[v][o[g]];
        out[at] = u[g];
      }
    __syncthreads();
    if ((int)threadIdx.x < P)
      for (int v = 0; v < kWaves; ++v) s_base[threadIdx.x] += s_wave[v][threadIdx.x];
    __syncthreads();
  }
}

struct BucketWs {
  int32_t* cnt;
  int32_t* ok;
};

int bucket_blocks(int64_t cap, int32_t P) {
  return (int)std::min<int64_t>(std::max<int64_t>(1, cdiv(cap, kSpanIds)), max_blocks(P));
}

size_t bucket_ws_layout(int64_t cap, int32_t P, char* base, BucketWs* out) {
  Carve cv{base, 0, ~(size_t)0};
  BucketWs b;
  b.cnt = cv.take<int32_t>((size_t)bucket_blocks(cap, P) * (size_t)P);
  b.ok = cv.take<int32_t>((size_t)kRangeBlocks);
  if (out) *out = b;
  return align_up(cv.used, 256);
}

}  // namespace
}  // namespace gg

using namespace gg;

extern "C" size_t gg_ws_bucket(int64_t cap, int32_t num_parts) {
  return bucket_ws_layout(cap, num_parts, nullptr, nullptr);
}

extern "C" int gg_bucket_by_owner(const int32_t* hot_ids_d, const int64_t* hot_count_d, int64_t cap,
                                  const gg_part_t* part, int32_t flags, int32_t* bucket_ids_d,
                                  int64_t* owner_off_d, int32_t* status_d, void* ws,
                                  size_t ws_bytes, hipStream_t stream) {
  GG_REQUIRE(hot_count_d && owner_off_d && status_d, "NULL argument");
  GG_REQUIRE(cap >= 0 && cap < (1LL << 31), "capacity %lld unsupported", (long long)cap);
  GG_REQUIRE(cap == 0 || (hot_ids_d && bucket_ids_d), "NULL id buffer");
  GG_REQUIRE((flags & ~GG_BUCKET_OWNER_ORDERED) == 0, "unknown flags 0x%x", (unsigned)flags);
  KPart kp;
  int rc = pack_part(part, &kp);
  if (rc != GG_OK) return rc;
  BucketWs bw;
  const size_t need_ws = bucket_ws_layout(cap, kp.P, (char*)ws, &bw);
  GG_REQUIRE(ws && ws_bytes >= need_ws, "workspace of %zu bytes < %zu", ws_bytes, need_ws);
  const int32_t nrange = (int32_t)std::min<int64_t>(std::max<int64_t>(1, cdiv(cap, kRangeIds)), kRangeBlocks);
  const int32_t* ok = nullptr;
  if (kp.kind == GG_PART_RANGE) {
    // Owner-ordered input under ranges is its own bucketing.  When the
    // caller vouches for the order, this pass is the whole call and an
    // input out of order is reported instead of repaired.
    const bool trusted = (flags & GG_BUCKET_OWNER_ORDERED) != 0;
    hipLaunchKernelGGL(k_bucket_range, dim3(nrange), dim3(kBlock), 0, stream, hot_ids_d, hot_count_d,
                       cap, kp, bucket_ids_d, owner_off_d, trusted ? nullptr : bw.ok,
                       trusted ? (int32_t)GG_DEV_ORDER : 0, status_d);
    GG_LAUNCH_CHECK("k_bucket_range");
    if (trusted) return GG_OK;
    ok = bw.ok;
  }
  const int grid = bucket_blocks(cap, kp.P);
  hipLaunchKernelGGL(k_bucket_count, dim3(grid), dim3(kBlock), 0, stream, hot_ids_d, hot_count_d,
                     cap, kp, bw.cnt, ok, nrange, status_d);
  GG_LAUNCH_CHECK("k_bucket_count");
  hipLaunchKernelGGL(k_bucket_scatter, dim3(grid), dim3(kBlock), 0, stream, hot_ids_d, hot_count_d,
                     cap, kp, bw.cnt, owner_off_d, ok, nrange, bucket_ids_d);
  GG_LAUNCH_CHECK("k_bucket_scatter");
  return GG_OK;
}
