// Batched multi-cluster force evaluation: many independent systems of
// uneven size and uneven active blocks in one launch.
//
//   batch_plan_kernel  -- one workgroup turns the cluster descriptors into a
//                         per-cluster launch plan (i-particles per workgroup,
//                         j-splits) and a flat list of work items
//                         (cluster, i-block, j-split); the other workgroups
//                         clear the per-row counters of the calculation.
//   batch_kernel       -- persistent workgroups take items from work queues
//                         (a static first round, then eight atomic counters).
//                         An item predicts its j-tiles
//                         straight into LDS from the float64 j-memory (the
//                         predictor of Sec. 2.2 fused into the tile load),
//                         runs the interaction of Sec. 2.3 on them and stores
//                         its split partials.
//   batch_reduce       -- workgroups over parts of the i-blocks add the
//                         partials of all splits in a fixed order and write
//                         the results (the reduction of Sec. 2.3).
//   batch_nb_exact     -- exact neighbour lists for overflowed i-particles.
//
// Each cluster is what the paper's library evaluates per call; batching them
// fills the 256 compute units when every single cluster is far too small to
// do so, and removes the per-call launches.

#include "g6mi_batch_common.h"

namespace g6mi {

// -------------------------------------------------------------------- plan

// Threads of the plan kernel: one workgroup fills the work tables, whose time
// is the latency of its passes (cold instruction fetch, scans, divisions,
// binary searches), one cluster per thread and pass.  256 threads for up to
// kPlanFew clusters, 1024 for more: 24 clusters 6.9 us (9.3 before the wave
// scans below, the single scan per pass and the 32-bit divisions), 65 clusters
// 9.9 (9.9), 256 clusters 11.0 (12.4), 364 clusters 11.5 (21.8: every pass
// twice), 1000 clusters 12.9 (38.5).
constexpr int kPlanFew = 64;

// One step of a wave scan on the VALU's lane-shift paths (a cross-lane
// exchange through LDS has several times their latency): x plus the value of
// the lane the control names, zero where it names none.
template <int CTRL, int ROWS> __device__ __forceinline__ long long dpp_add(long long x) {
  const int lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(x), CTRL, ROWS, 0xf, false);
  const int hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(x >> 32), CTRL, ROWS, 0xf, false);
  return x + ((static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo));
}
// Inclusive sum over the 64 lanes of a wave: shifts by 1, 2, 4 and 8 inside
// rows of 16, then the last lane of a row added to the next (rows 1 and 3),
// and of lane 31 to the upper half.
__device__ __forceinline__ long long wave_scan(long long x) {
  x = dpp_add<0x111, 0xf>(x);
  x = dpp_add<0x112, 0xf>(x);
  x = dpp_add<0x114, 0xf>(x);
  x = dpp_add<0x118, 0xf>(x);
  x = dpp_add<0x142, 0xa>(x);
  return dpp_add<0x143, 0xc>(x);
}

// Inclusive sums of N values per thread over the workgroup (wave scans, then
// the wave totals through LDS, s_part[N * WG / 64]); all = the totals.
// Every thread must call it; it ends with a barrier, so s_part can be reused.
template <int WG, int N>
__device__ __forceinline__ void wg_scan(long long (&x)[N], long long *s_part, long long (&all)[N]) {
  constexpr int kWaves = WG / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < N; ++k) {
    x[k] = wave_scan(x[k]);
    if (lane == 63) s_part[k * kWaves + wave] = x[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < N; ++k) {
    // lane w of every wave holds the total of wave w
    const long long t = wave_scan(lane < kWaves ? s_part[k * kWaves + lane] : 0);
    auto at = [&](int w) {
      const int lo = __builtin_amdgcn_readlane(static_cast<int>(t), w);
      const int hi = __builtin_amdgcn_readlane(static_cast<int>(t >> 32), w);
      return (static_cast<long long>(hi) << 32) | static_cast<unsigned>(lo);
    };
    all[k] = at(63);
    const int w = __builtin_amdgcn_readfirstlane(wave);
    if (w > 0) x[k] += at(w - 1);
  }
  __syncthreads();
}

// Index of the first of WG non-decreasing counts above q (one exists).
template <int WG> __device__ __forceinline__ int first_above(const int *inc, int q) {
  int lo = 0, hi = WG - 1;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (inc[mid] > q) hi = mid;
    else lo = mid + 1;
  }
  return lo;
}

// Work items: for cluster c with ni i-particles in nib i-blocks of ipw and
// ntiles j-tiles in nsplit splits of `per` tiles, nib * nsplit items.  One
// tile costs a lane ipw pairs (narrow blocks) or 512 (wide blocks).  Items
// cost about the same: per = target / ipw tiles, where the target is
// item_work * 128 lane-pairs, lowered (down to one tile) until the whole
// batch makes at least about one item per persistent workgroup, so that a
// batch of few or small clusters still spreads over the GPU.  A narrow
// block holds at most the target's worth of i-particles (not below
// kBatchMinIpw), so that one tile of it stays within the target.
//
// Pass 1 checks the descriptors, picks the block shape of each cluster
// (kept in its plan entry) and adds up the batch's work; pass 1b cuts the
// blocks of clusters too small to fill their share of the GPU; pass 2 picks
// the splits, scans i-blocks, partial entries and the items of each queue
// class (plan_order) and fills the i-block -> cluster table; pass 3 puts the
// classes one after the other and fills the item -> cluster table.
// With at most WG clusters (one chunk) each thread keeps its cluster's entry in
// registers from pass to pass; with more, it reads back its own entry of each
// chunk.
template <int WG>
__global__ __launch_bounds__(WG) void batch_plan_kernel(BatchArgs b) {
  const int tid = threadIdx.x;
  if (blockIdx.x > 0) {
    // rows (blockIdx.x - 1) * chunk ...: neighbour counts
    const int base = (blockIdx.x - 1) * kPlanZeroChunk;
    if (b.nbl)
      for (int k = tid; k < kPlanZeroChunk; k += WG) {
        const int r = base + k;
        if (r < b.ni_total) b.fa.nb_count[r] = 0;
      }
    return;
  }
  __shared__ long long s_part[4 * WG / 64];
  __shared__ int s_inc[kItemOrders][WG], s_inc_ib[WG];
  __shared__ int s_flags;
  if (tid == 0) s_flags = 0;
  __syncthreads();

  BatchPlan pl_last{};
  const bool one_chunk = b.ncl <= WG;

  // pass 1: validity, block shape, work
  long long c_rows = 0, work = 0;
  for (int c0 = 0; c0 < b.ncl; c0 += WG) {
    const int c = c0 + tid;
    int ni = 0, nj = 0;
    bool ok = false;
    if (c < b.ncl) {
      const g6mi_cluster d = b.cl[c];
      ok = d.joff >= 0 && d.nj >= 0 && static_cast<long long>(d.joff) + d.nj <= b.nj_set && d.ioff >= 0 &&
           d.ni >= 0 && static_cast<long long>(d.ioff) + d.ni <= b.ni_total && isfinite(d.ti) &&
           isfinite(d.eps2) && d.eps2 >= 0.0;
      ni = ok ? d.ni : 0;
      nj = ok ? d.nj : 0;
    }
    BatchPlan pl = plan_shape(ni, nj, b.tune); // splits in pass 2
    long long sum[2] = {ni, plan_work(pl)}, all[2];
    wg_scan<WG>(sum, s_part, all);
    // Clusters sharing i-rows could add up to more rows than ni_total, and
    // the i-block counters and partial sums are sized by ni_total: every
    // cluster past that many rows in total is skipped.
    if (c_rows + all[0] > b.ni_total) {
      if (ok && c_rows + sum[0] > b.ni_total) {
        ok = false;
        pl = plan_shape(0, 0, b.tune);
      }
      long long kept[1] = {plan_work(pl)}, kept_all[1];
      wg_scan<WG>(kept, s_part, kept_all);
      all[1] = kept_all[0];
    }
    if (c < b.ncl && !ok) atomicOr(&s_flags, kFlagBadCluster);
    if (c < b.ncl && !one_chunk) b.plan[c] = pl;
    pl_last = pl;
    work += all[1];
    c_rows += all[0];
  }
  // pass 1b: clusters too small for their share of the persistent
  // workgroups (plan_share); the share is the grid times the cluster's
  // fraction of the batch's work
  const long long work0 = max(1LL, work);
  work = 0;
  for (int c0 = 0; c0 < b.ncl; c0 += WG) {
    const int c = c0 + tid;
    long long w[1] = {0}, all[1];
    if (c < b.ncl) {
      BatchPlan pl = one_chunk ? pl_last : b.plan[c];
      if (pl.nib > 0) {
        const long long share = plan_div(static_cast<long long>(b.grid) * plan_work(pl) + work0 - 1, work0);
        if (plan_share(pl, share, b.tune) && !one_chunk) b.plan[c] = pl;
        w[0] = plan_work(pl);
      }
      pl_last = pl;
    }
    wg_scan<WG>(w, s_part, all);
    work += all[0];
  }
  const long long target = plan_target(work, b.grid, b.tune);

  // pass 2: splits, the scans of i-blocks and partial entries in cluster order
  // and of the items of each queue class (plan_order), and the i-block ->
  // cluster table, filled by all threads: i-block q of the chunk belongs to
  // the first cluster whose inclusive i-block count exceeds q.  item0 is
  // counted inside the class until the classes' totals are known.  Classes 0
  // and 1 share a scanned word (fewer than 2^31 items each).
  int c_nib = 0, c_class[kItemOrders] = {0, 0, 0};
  long long c_pent = 0;
  static_assert(kItemOrders == 3, "three classes in two scanned words");
  for (int c0 = 0; c0 < b.ncl; c0 += WG) {
    const int c = c0 + tid;
    BatchPlan pl{};
    int n[kItemOrders] = {0, 0, 0}, order = 0;
    if (c < b.ncl) {
      pl = one_chunk ? pl_last : b.plan[c];
      plan_splits(pl, target, b.tune);
      order = plan_order(pl);
#pragma unroll
      for (int k = 0; k < kItemOrders; ++k) n[k] = order == k ? pl.nib * pl.nsplit : 0;
    }
    const long long pent = static_cast<long long>(pl.ni) * pl.nsplit;
    long long sum[4] = {pl.nib, pent, n[0] + (static_cast<long long>(n[1]) << 32), n[2]}, all[4];
    wg_scan<WG>(sum, s_part, all);
    const int inc[kItemOrders] = {static_cast<int>(sum[2]), static_cast<int>(sum[2] >> 32), static_cast<int>(sum[3])};
    const int tot[kItemOrders] = {static_cast<int>(all[2]), static_cast<int>(all[2] >> 32), static_cast<int>(all[3])};
    if (c < b.ncl) {
      pl.ib0 = c_nib + static_cast<int>(sum[0]) - pl.nib;
      pl.pbase = c_pent + sum[1] - pent;
#pragma unroll
      for (int k = 0; k < kItemOrders; ++k)
        if (order == k) pl.item0 = c_class[k] + inc[k] - n[k];
      if (!one_chunk) b.plan[c] = pl;
    }
    pl_last = pl;
    s_inc_ib[tid] = static_cast<int>(sum[0]);
    if (one_chunk)
#pragma unroll
      for (int k = 0; k < kItemOrders; ++k) s_inc[k][tid] = inc[k];
    __syncthreads();
    for (int q = tid; q < static_cast<int>(all[0]); q += WG) b.ib_cl[c_nib + q] = c0 + first_above<WG>(s_inc_ib, q);
    __syncthreads(); // s_inc_ib is rewritten by the next chunk
    c_nib += static_cast<int>(all[0]);
    c_pent += all[1];
#pragma unroll
    for (int k = 0; k < kItemOrders; ++k) c_class[k] += tot[k];
  }
  // pass 3: each cluster's items put after the classes before its own, and the
  // item -> cluster table, one class after the other, in cluster order within
  // a class
  const int base[kItemOrders] = {0, c_class[0], c_class[0] + c_class[1]};
  const int c_items = base[2] + c_class[2];
  if (one_chunk) {
    if (tid < b.ncl) {
#pragma unroll
      for (int k = 0; k < kItemOrders; ++k)
        if (plan_order(pl_last) == k) pl_last.item0 += base[k];
      b.plan[tid] = pl_last;
    }
    for (int q = tid; q < min(c_items, b.item_cap); q += WG) {
      const int k = q >= base[2] ? 2 : (q >= base[1] ? 1 : 0);
      b.item_cl[q] = first_above<WG>(s_inc[k], q - (k == 2 ? base[2] : (k == 1 ? base[1] : 0)));
    }
  } else {
    int done[kItemOrders] = {0, 0, 0}; // items of each class in the chunks before
    for (int c0 = 0; c0 < b.ncl; c0 += WG) {
      const int c = c0 + tid;
      BatchPlan pl{};
      int order = -1;
      if (c < b.ncl) {
        pl = b.plan[c];
        order = plan_order(pl);
      }
      const int n = pl.nib * pl.nsplit;
      // inclusive counts inside the chunk, by class: a thread of another class
      // repeats the count before it
      long long sum[2] = {order == 0 ? n : (order == 1 ? static_cast<long long>(n) << 32 : 0), order == 2 ? n : 0};
      long long all[2];
      wg_scan<WG>(sum, s_part, all);
      s_inc[0][tid] = static_cast<int>(sum[0]);
      s_inc[1][tid] = static_cast<int>(sum[0] >> 32);
      s_inc[2][tid] = static_cast<int>(sum[1]);
      const int tot[kItemOrders] = {static_cast<int>(all[0]), static_cast<int>(all[0] >> 32), static_cast<int>(all[1])};
      __syncthreads();
#pragma unroll
      for (int k = 0; k < kItemOrders; ++k) {
        if (order == k) b.plan[c].item0 = base[k] + pl.item0;
        for (int q = tid; q < tot[k]; q += WG)
          if (base[k] + done[k] + q < b.item_cap) b.item_cl[base[k] + done[k] + q] = c0 + first_above<WG>(s_inc[k], q);
        done[k] += tot[k];
      }
      __syncthreads(); // s_inc is rewritten by the next chunk
    }
  }
  if (tid == 0) {
    for (int x = 0; x < kQueues; ++x) b.work->head[x] = 0;
    b.work->nitems = min(c_items, b.item_cap);
    b.work->nib = c_nib;
    // more items than the table holds cannot happen with the host's bound;
    // it would drop work, so it is reported like a bad descriptor
    b.status[kStatusFlags] = s_flags | (c_items > b.item_cap ? kFlagBadCluster : 0);
    b.status[kStatusOverflowCount] = 0;
  }
}

// ------------------------------------------------------ persistent kernel

// Persistent workgroups: workgroup g starts with item g, then takes the
// next item from its queue until the items run out (every wave reaches the
// exit: items are finite and each workgroup takes one item per round).  The
// items after the first grid's worth are dealt round-robin to kQueues
// queues, one counter each, and workgroup g takes from queue g mod kQueues:
// workgroups go to the 8 XCDs round-robin, so each XCD's workgroups share
// one counter, and no counter serves the whole grid.  The first round needs
// no atomic at all: hundreds of workgroups incrementing one counter at once
// queue up behind each other.
// Partial entry of i-particle il (cluster row) in split s: pbase + s * ni +
// il.
// WIDE = false: the narrow-only kernel, for batches whose plan cannot make a
// wide block (the host launches it only when tune.wide_min > ni_total); its
// registers fit four waves per SIMD.
template <int PREC, bool NBL, bool WIDE>
__global__ __launch_bounds__(kWG, WIDE ? wide_waves<PREC>() : kNarrowWaves) void batch_kernel(BatchArgs b) {
  using R = real_t<PREC>;
  constexpr int REC = rec4<PREC>();
  __shared__ __attribute__((aligned(16))) unsigned char lds[narrow_lds_bytes<PREC>()];
  __shared__ int s_item;
  float4 *tile = reinterpret_cast<float4 *>(lds);
  const int tid = threadIdx.x;
  const int nitems = b.work->nitems;

  for (int q = blockIdx.x; q < nitems;) {
    // q is uniform across the workgroup: the item's cluster, descriptor and
    // plan are then scalar loads held in scalar registers
    const int c = b.item_cl[q];
    const g6mi_cluster d = b.cl[c];
    const BatchPlan p = b.plan[c];
    const int r = q - p.item0;
    const int ib = r / p.nsplit;
    const int sp = r - ib * p.nsplit;
    const int ntiles = (d.nj + kTile - 1) / kTile;
    const int tb = sp * p.per;
    const int te = min(ntiles, tb + p.per);
    const int jend = d.joff + d.nj;
    const R eps2 = static_cast<R>(d.eps2);
    const size_t e0 = static_cast<size_t>(p.pbase) + static_cast<size_t>(sp) * d.ni;

    if (!WIDE && p.ipw > kWG) {
      // not reached (see above); the item is dropped and the batch flagged
      if (tid == 0) atomicOr(b.status + kStatusFlags, kFlagBadCluster);
    } else if (WIDE && p.ipw == 2 * kWG) {
      const int il0 = ib * (2 * kWG) + tid, il1 = il0 + kWG;
      WideLanes<PREC, NBL> w;
      w.init(b.fa, d.ioff + il0, d.ioff + il1, il0 < d.ni, il1 < d.ni);
      for (int tt = tb; tt < te; ++tt) {
        const int jbase = d.joff + tt * kTile;
        const int cnt = min(kTile, jend - jbase);
        __syncthreads();
        if (tid < cnt) predict_record<PREC>(b.jm, static_cast<size_t>(jbase + tid), d.ti, tile + tid * REC);
        __syncthreads();
        // DS: every group goes straight to the float64 totals (see WideLanes::tile)
        w.template tile<PREC == G6MI_PREC_DS, true>(tile, jbase, cnt, eps2, b.fa.nb_count, b.fa.nb_slot);
        w.resolve(tile, jbase); // while the tile is still in LDS
      }
      if (w.v0) store_part(b.part, b.nn_slot, e0 + il0, w.t0, static_cast<double>(w.ebest0), w.eslot0);
      if (w.v1) store_part(b.part, b.nn_slot, e0 + il1, w.t1, static_cast<double>(w.ebest1), w.eslot1);
    } else {
      const int ipw = p.ipw;
      const int lil = tid & (ipw - 1);
      const int il = ib * ipw + lil;
      NarrowLane<PREC, NBL> n;
      n.init(b.fa, d.ioff + il, il < d.ni, tid >> p.log2ipw, 8 - p.log2ipw);
      for (int tt = tb; tt < te; ++tt) {
        const int jbase = d.joff + tt * kTile;
        const int cnt = min(kTile, jend - jbase);
        __syncthreads();
        if (tid < cnt) predict_record<PREC>(b.jm, static_cast<size_t>(jbase + tid), d.ti, tile + tid * REC);
        __syncthreads();
        n.tile(tile, jbase, cnt, eps2, b.fa.nb_count, b.fa.nb_slot);
        n.resolve(tile, jbase);
      }
      double bestd;
      int bslot;
      n.lane_sum(reinterpret_cast<double *>(lds), tid, lil, ipw, bestd, bslot);
      if (n.sub == 0 && n.valid) store_part(b.part, b.nn_slot, e0 + il, n.t, bestd, bslot);
    }
    if (static_cast<int>(gridDim.x) >= nitems) break; // no second round
    __syncthreads(); // the item is done with the LDS and s_item
    if (tid == 0) {
      // every queue needs a workgroup: one queue for a grid smaller than kQueues
      const int nq = static_cast<int>(gridDim.x) >= kQueues ? kQueues : 1;
      const int x = static_cast<int>(blockIdx.x) % nq;
      s_item = static_cast<int>(gridDim.x) + x + nq * atomicAdd(&b.work->head[x], 1);
    }
    __syncthreads();
    q = __builtin_amdgcn_readfirstlane(s_item);
  }
}

// One workgroup per part of an i-block (reduce_parts; grid-strided over the
// work->nib i-blocks of the batch when they outnumber the grid, ib_cl giving
// each one's cluster): the float64 sum of the rows' split partials
// (split_sum) and their results (finish_out).  A launch of its own: the kernel boundary
// makes every item's partials visible, where a release fence per item would
// write back the XCD's whole L2 (buffer_wbl2) and an acquire invalidate it,
// once per item.
__global__ __launch_bounds__(kWG) void batch_reduce_kernel(BatchArgs b) {
  __shared__ SplitShared sh;
  const int nib_total = b.work->nib;
  const int P = reduce_parts(nib_total, static_cast<int>(gridDim.x), 64);
  int fl = 0;
  for (int u = blockIdx.x; u < nib_total * P; u += gridDim.x)
    fl |= reduce_iblock(b, u / P, u % P, P, sh, [](int, bool) {}, [](int, bool, double2) {});
  if (fl) atomicOr(b.status + kStatusFlags, fl);
}

// ------------------------------------------------- neighbour-list overflow

// One workgroup per queued i-particle: its list rebuilt from the slots of
// its own cluster, each record predicted again exactly as in batch_kernel.
template <int PREC>
__global__ __launch_bounds__(kWG) void batch_nb_exact_kernel(BatchArgs b) {
  __shared__ unsigned s_cnt;
  __shared__ int s_keep[kNbMax];
  const int novf = b.status[kStatusOverflowCount];
  for (int q = blockIdx.x; q < novf; q += gridDim.x) {
    const int row = b.ovf_list[q];
    const g6mi_cluster d = b.cl[b.ovf_tag[q]];
    IState<PREC> st;
    int slot;
    real_t<PREC> h2;
    load_i<PREC>(st, b.fa, row, true, slot, h2);
    const JMem jm = b.jm;
    const double ti = d.ti;
    auto rec_of = [jm, ti](int js, float4 *buf) -> const float4 * {
      predict_record<PREC>(jm, static_cast<size_t>(js), ti, buf);
      return buf;
    };
    exact_list<PREC>(st, slot, h2, d.joff, d.joff + d.nj, jm.index, rec_of,
                     b.fa.nb_slot + static_cast<size_t>(row) * kNbMax, b.fa.nb_count + row, s_cnt, s_keep);
  }
}

// ---------------------------------------------------------------- launchers

hipError_t launch_batch_plan(const BatchArgs &b, hipStream_t s) {
  const unsigned zero_blocks = static_cast<unsigned>((b.ni_total + kPlanZeroChunk - 1) / kPlanZeroChunk);
  if (b.ncl <= kPlanFew)
    hipLaunchKernelGGL(batch_plan_kernel<256>, dim3(1 + zero_blocks), dim3(256), 0, s, b);
  else
    hipLaunchKernelGGL(batch_plan_kernel<1024>, dim3(1 + zero_blocks), dim3(1024), 0, s, b);
  return hipGetLastError();
}

template <int PREC>
static void launch_batch_prec(const BatchArgs &b, int grid, hipStream_t s) {
  if (b.wide) {
    if (b.nbl)
      hipLaunchKernelGGL((batch_kernel<PREC, true, true>), dim3(grid), dim3(kWG), 0, s, b);
    else
      hipLaunchKernelGGL((batch_kernel<PREC, false, true>), dim3(grid), dim3(kWG), 0, s, b);
  } else {
    if (b.nbl)
      hipLaunchKernelGGL((batch_kernel<PREC, true, false>), dim3(grid), dim3(kWG), 0, s, b);
    else
      hipLaunchKernelGGL((batch_kernel<PREC, false, false>), dim3(grid), dim3(kWG), 0, s, b);
  }
}

static hipError_t launch_batch_items(int prec, const BatchArgs &b, int grid, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  switch (prec) {
  case G6MI_PREC_FP32: launch_batch_prec<G6MI_PREC_FP32>(b, grid, s); break;
  case G6MI_PREC_DS: launch_batch_prec<G6MI_PREC_DS>(b, grid, s); break;
  default: launch_batch_prec<G6MI_PREC_FP64>(b, grid, s);
  }
  return hipGetLastError();
}

hipError_t launch_batch_force(int prec, const BatchArgs &b, int grid, hipStream_t s) {
  if (grid <= 0) return hipSuccess;
  const hipError_t e = launch_batch_items(prec, b, grid, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(batch_reduce_kernel, dim3(reduce_grid(grid, b.ni_total)), dim3(kWG), 0, s, b);
  return hipGetLastError();
}

hipError_t launch_batch_nb_exact(int prec, const BatchArgs &b, int novf, hipStream_t s) {
  if (novf <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(novf < 1024 ? novf : 1024));
  switch (prec) {
  case G6MI_PREC_FP32: hipLaunchKernelGGL(batch_nb_exact_kernel<G6MI_PREC_FP32>, grid, dim3(kWG), 0, s, b); break;
  case G6MI_PREC_DS: hipLaunchKernelGGL(batch_nb_exact_kernel<G6MI_PREC_DS>, grid, dim3(kWG), 0, s, b); break;
  default: hipLaunchKernelGGL(batch_nb_exact_kernel<G6MI_PREC_FP64>, grid, dim3(kWG), 0, s, b);
  }
  return hipGetLastError();
}

} // namespace g6mi
