// Window-size simulator counts (Sec. IV-A simulation; Sec. IV-B, Eqs.
// (1)-(3)): one window's rebuild-delta and miss counters, taken from the
// staging and gather statistics the fetch path already writes, priced with
// the analytical energy model and added to a running total.
#include "gg_host.hpp"

namespace gg {
namespace {

// One transfer event: the energy (initiation for every owner with rows, plus
// the linear payload) and the duration (zero when no owner has rows) of owners'
// row counts x_m.
struct Event {
  double e, t;
  int64_t owners, rows;
};

__device__ Event price_event(const int64_t* x, int P, int local, const gg_sim_coeffs_t& c) {
#pragma clang fp contract(off)
  Event v = {0.0, 0.0, 0, 0};
  double tmax = 0.0;
  for (int m = 0; m < P; ++m) {
    if (m == local) continue;
    const int64_t xm = x[m];
    if (xm <= 0) continue;
    const double xd = (double)xm;
    v.e = v.e + (c.eps_init[m] + c.eps_row[m] * xd);
    const double tm = c.lam_init[m] + c.lam_row[m] * xd;
    tmax = tm > tmax ? tm : tmax;
    v.rows += xm;
    v.owners += 1;
  }
  if (v.rows > 0) {
    const double tbw = (double)v.rows * c.row_bytes / c.bw_bytes_per_s;
    v.t = tmax > tbw ? tmax : tbw;
  }
  return v;
}

// Bound by the chain of dependent steps, so all counts are read at once, a
// lane prices each event (the rebuild, then the batches), and a single lane
// adds the results in a fixed order (one lane with every read a round trip of
// its own: 17.9 us at 16 batches of 4 owners; now 4.1).
__global__ void __launch_bounds__(kBlock) k_sim_accumulate(const gg_stage_stats_t* st,
                                                           const gg_gather_stats_t* gs,
                                                           int32_t nseg, int32_t P, int32_t local,
                                                           gg_sim_coeffs_t c, gg_sim_acc_t* acc) {
#pragma clang fp contract(off)
  static_assert(GG_MAX_W + 1 <= kBlock, "a lane for every event");
  __shared__ int64_t s_rows[(GG_MAX_W + 1) * GG_MAX_PARTS];
  __shared__ int64_t s_hits[GG_MAX_W], s_misses[GG_MAX_W];
  __shared__ Event s_ev[GG_MAX_W + 1];
  const int tid = threadIdx.x;
  gg_sim_acc_t a;
  if (tid == 0) a = *acc;
  for (int i = tid; i < (nseg + 1) * P; i += kBlock) {
    const int ev = i / P, m = i - ev * P;
    s_rows[i] = ev == 0 ? st->delta_rows[m] : gs[ev - 1].miss_rows[m];
  }
  if (tid < nseg) {
    s_hits[tid] = gs[tid].hits;
    s_misses[tid] = gs[tid].misses;
  }
  __syncthreads();
  if (tid <= nseg) s_ev[tid] = price_event(s_rows + tid * P, P, local, c);
  __syncthreads();
  if (tid != 0) return;
  a.e_rebuild = a.e_rebuild + s_ev[0].e;
  a.rebuild_events += s_ev[0].owners;
  a.rebuild_rows += s_ev[0].rows;
  double t = a.t_stall + s_ev[0].t;
  for (int32_t b = 0; b < nseg; ++b) {
    const Event v = s_ev[b + 1];
    a.e_miss = a.e_miss + v.e;
    a.miss_events += v.owners;
    a.miss_rows += v.rows;
    t = t + v.t;
    a.hits += s_hits[b];
    a.remote_rows += s_hits[b] + s_misses[b];
  }
  a.t_stall = t;
  a.windows += 1;
  a.batches += nseg;
  a.e_stall = c.p_idle * a.t_stall;
  a.e_phy = (a.e_rebuild + a.e_miss) + a.e_stall;
  *acc = a;
}

}  // namespace
}  // namespace gg

using namespace gg;

extern "C" int gg_sim_accumulate(const gg_stage_stats_t* stage_d, const gg_gather_stats_t* gather_d,
                                 int32_t nseg, const gg_part_t* part, const gg_sim_coeffs_t* coeffs,
                                 gg_sim_acc_t* acc_d, hipStream_t stream) {
  GG_REQUIRE(stage_d && acc_d && coeffs && part, "NULL argument");
  GG_REQUIRE(nseg >= 0 && nseg <= GG_MAX_W, "nseg %d out of range [0, %d]", nseg, GG_MAX_W);
  GG_REQUIRE(nseg == 0 || gather_d, "gather statistics are NULL");
  GG_REQUIRE(part->num_parts >= 1 && part->num_parts <= GG_MAX_PARTS, "num_parts %d invalid",
             part->num_parts);
  GG_REQUIRE(coeffs->bw_bytes_per_s > 0.0, "bw_bytes_per_s must be positive");
  hipLaunchKernelGGL(k_sim_accumulate, dim3(1), dim3(kBlock), 0, stream, stage_d, gather_d, nseg,
                     part->num_parts, part->local_owner, *coeffs, acc_d);
  GG_LAUNCH_CHECK("k_sim_accumulate");
  return GG_OK;
}
