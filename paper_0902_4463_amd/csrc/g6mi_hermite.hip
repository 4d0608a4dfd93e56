// Device-resident block steps of the 4th-order Hermite integrator (the
// client side of the paper's CPU/GPU split, Sec. 2 and 2.1, moved onto the
// GPU): one block step is
//
//   hs_select_kernel   the particles with t_k + dt_k = t_b, predicted to t_b
//                      in float64 (Eq. (1)-(2) with the particle's own
//                      a and jerk); t_b = min_k (t_k + dt_k) was gathered by
//                      the previous step: the others' times here, the
//                      corrected ones' in hs_correct_kernel
//   hs_force_kernel    forces on the block: each workgroup makes the launch
//                      plan of the block as a one-cluster batch and takes its
//                      share of the items of batch_kernel (g6mi_batch.hip)
//   hs_correct_kernel  the split partials added (the batch reduction), then
//                      the Hermite corrector, Aarseth time step, power-of-two
//                      block quantisation; the corrected particle is written
//                      back into the j-memory (its a/2 and jerk/6 too)
//
// (The first force evaluation, of all particles, goes through
// hs_publish_kernel and the batched kernels themselves.)
//
// Every launch has a fixed grid and reads the block size from device
// memory, so a whole step is one captured graph, replayed without the host.
// The integrator's formulas follow the host driver (hermite/driver.py) term
// by term, with float contraction switched off so that both round alike.

#include "g6mi_batch_common.h"

namespace g6mi {

// Order-preserving map of doubles onto unsigned 64-bit keys, so that the
// minimum over a grid is one atomicMin.
__device__ __forceinline__ unsigned long long order_key(double x) {
  const unsigned long long b = static_cast<unsigned long long>(__double_as_longlong(x));
  return (b >> 63) ? ~b : (b | 0x8000000000000000ull);
}
__device__ __forceinline__ double key_value(unsigned long long k) {
  const unsigned long long b = (k >> 63) ? (k & 0x7fffffffffffffffull) : ~k;
  return __longlong_as_double(static_cast<long long>(b));
}
constexpr unsigned long long kKeyInf = 0xfff0000000000000ull; // order_key(+inf)

// One step of a wave minimum on the VALU's lane-shift paths (the steps of
// wave_scan in the batch plan): a lane that the control names none for keeps
// its own key.  The minimum is the last serial step of the selection and of the
// corrector (5.06 -> 4.88 us and 7.99 -> 7.79 against exchanges through LDS).
template <int CTRL, int ROWS> __device__ __forceinline__ unsigned long long dpp_min(unsigned long long x) {
  const int l = static_cast<int>(x), h = static_cast<int>(x >> 32);
  const unsigned lo = static_cast<unsigned>(__builtin_amdgcn_update_dpp(l, l, CTRL, ROWS, 0xf, false));
  const unsigned hi = static_cast<unsigned>(__builtin_amdgcn_update_dpp(h, h, CTRL, ROWS, 0xf, false));
  const unsigned long long o = (static_cast<unsigned long long>(hi) << 32) | lo;
  return o < x ? o : x;
}

// Workgroup minimum of one key per thread, folded into *dst with one
// atomic (none when every key is +inf).  Every thread must call it, at most
// once per launch (its LDS words are read after the barrier without a second
// one).
__device__ __forceinline__ void key_min(unsigned long long key, unsigned long long *dst) {
  __shared__ unsigned long long s_key[4];
  key = dpp_min<0x111, 0xf>(key);
  key = dpp_min<0x112, 0xf>(key);
  key = dpp_min<0x114, 0xf>(key);
  key = dpp_min<0x118, 0xf>(key);
  key = dpp_min<0x142, 0xa>(key);
  key = dpp_min<0x143, 0xc>(key);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 63) s_key[wave] = key;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long m = s_key[0];
    for (int w = 1; w < static_cast<int>(blockDim.x >> 6); ++w) m = s_key[w] < m ? s_key[w] : m;
    if (m != kKeyInf) atomicMin(dst, m);
  }
}

// Taylor prediction of particle k to time tb from its own a and jerk, the
// host driver's expression: x + tau (v + tau (a/2 + tau j/6)).
__device__ __forceinline__ void predict_particle(const HermiteArgs &h, int k, double tb, double *xp,
                                                 double *vp) {
#pragma clang fp contract(off)
  const double tau = tb - h.jm.t[k];
  for (int d = 0; d < 3; ++d) {
    const size_t e = d * h.jm.cap + k;
    const double a2 = 0.5 * h.acc[e];
    const double j6 = h.jrk[e] / 6.0;
    xp[d] = h.jm.x[e] + tau * (h.jm.v[e] + tau * (a2 + tau * j6));
    vp[d] = h.jm.v[e] + tau * (2.0 * a2 + tau * (3.0 * j6));
  }
}

__global__ __launch_bounds__(256) void hs_select_kernel(HermiteArgs h) {
  __shared__ int s_wave[4], s_base;
  const int tid = threadIdx.x;
  const int k = blockIdx.x * 256 + tid;
  HermiteCtl *ctl = h.ctl;
  // both keys read with the phase, not after it (one dependent load fewer)
  const int ph = ctl->phase;
  const unsigned long long k0 = ctl->key[0], k1 = ctl->key[1];
  const double tb = key_value(ph ? k1 : k0);
  const bool go = tb <= ctl->t_end;
  const double tn = k < h.n ? h.jm.t[k] + h.dt[k] : INFINITY;
  const bool act = go && k < h.n && tn == tb;
  // the active particles' loads go out before the block-wide steps below
  double xp[3], vp[3];
  if (act) predict_particle(h, k, tb, xp, vp);
  // the next block time, first part: the particles this step leaves alone
  key_min(act ? kKeyInf : order_key(tn), &ctl->key[ph ^ 1]);
  // slots of this block's active particles: wave counts, one atomic per block
  const unsigned long long m = __ballot(act);
  const int lane = tid & 63, wave = tid >> 6;
  if (lane == 0) s_wave[wave] = __popcll(m);
  __syncthreads();
  if (tid == 0) {
    const int tot = s_wave[0] + s_wave[1] + s_wave[2] + s_wave[3];
    s_base = tot ? atomicAdd(&ctl->ni_count, tot) : 0;
  }
  __syncthreads();
  if (act) {
    int q = s_base + __popcll(m & ((1ull << lane) - 1ull));
    for (int w = 0; w < wave; ++w) q += s_wave[w];
    h.active[q] = k;
    for (int d = 0; d < 3; ++d) {
      h.xi[3 * static_cast<size_t>(q) + d] = xp[d];
      h.vi[3 * static_cast<size_t>(q) + d] = vp[d];
    }
  }
}

// The block selected as a one-cluster descriptor, or an empty block once
// t_b > t_end, so that replays past the end change nothing.
__device__ __forceinline__ g6mi_cluster current_block(const HermiteArgs &h) {
  const HermiteCtl *ctl = h.ctl;
  const unsigned long long k0 = ctl->key[0], k1 = ctl->key[1];
  const int count = ctl->ni_count;
  const double t_end = ctl->t_end, time = ctl->time;
  const double tb = key_value(ctl->phase ? k1 : k0);
  const bool go = tb <= t_end;
  g6mi_cluster d;
  d.joff = 0;
  d.nj = h.n;
  d.ioff = 0;
  d.ni = go ? count : 0;
  d.ti = go ? tb : time;
  d.eps2 = h.eps2;
  return d;
}

// The batch's launch plan for that one cluster (the plan kernel's decisions
// for a batch of one: plan_shape, plan_share with the whole grid as its
// share, plan_target, plan_splits).
__device__ __forceinline__ BatchPlan plan_block(const g6mi_cluster &d, const BatchArgs &b) {
  BatchPlan pl = plan_shape(d.ni, d.nj, b.tune);
  if (pl.nib > 0) plan_share(pl, b.grid, b.tune);
  plan_splits(pl, plan_target(plan_work(pl), b.grid, b.tune), b.tune);
  pl.ib0 = pl.item0 = 0;
  pl.pbase = 0;
  return pl;
}

// First force evaluation: the block's descriptor, plan and work tables for
// the batched kernels; then the block-time keys turn over (see HermiteCtl).
__global__ __launch_bounds__(256) void hs_publish_kernel(HermiteArgs h, BatchArgs b) {
  __shared__ int s_items, s_nib;
  if (threadIdx.x == 0) {
    HermiteCtl *ctl = h.ctl;
    const int ph = ctl->phase;
    const g6mi_cluster d = current_block(h);
    ctl->desc = d;
    const BatchPlan pl = plan_block(d, b);
    b.plan[0] = pl;
    const int items = pl.nib * pl.nsplit;
    for (int x = 0; x < kQueues; ++x) b.work->head[x] = 0;
    b.work->nitems = min(items, b.item_cap);
    b.work->nib = pl.nib;
    b.status[kStatusFlags] = items > b.item_cap ? kFlagBadCluster : 0;
    b.status[kStatusOverflowCount] = 0;
    s_items = min(items, b.item_cap);
    s_nib = pl.nib;
    // the corrector adds the block's new times to key[ph ^ 1]; the next
    // selection reads it and fills key[ph] afresh
    ctl->ni_count = 0;
    ctl->key[ph] = kKeyInf;
    ctl->phase = ph ^ 1;
  }
  __syncthreads();
  for (int q = threadIdx.x; q < s_items; q += 256) b.item_cl[q] = 0;
  for (int q = threadIdx.x; q < s_nib; q += 256) b.ib_cl[q] = 0;
}

// Forces on the block of a step: the items of batch_kernel for a batch of one
// cluster, dealt to the workgroups in turn.  Every workgroup reads the block
// from the control block and makes the plan itself, so that the step needs no
// launch for it, and workgroup 0 writes the descriptor and plan for
// hs_correct_kernel.  Items are short (a block of 341 against 32768 makes 704
// items of two tiles against 32 particles): bound by the latency of their
// dependent loads, so the next tile's j-memory entries are loaded while a
// tile is evaluated, and nothing is computed that the integrator does not
// use: no neighbour lists, and the nearest neighbour only as far as it
// decides the float32 sums (fold_or_add; the exact r^2 on splits that end in
// a ragged tile).  The sums are those of batch_kernel.  Per step of the
// 32768-particle run 21.0-21.6 us, against 24.6 us of batch_kernel and 3.3 us of a
// launch for the plan before it.
template <int PREC>
__global__ __launch_bounds__(kWG, wide_waves<PREC>()) void hs_force_kernel(HermiteArgs h, BatchArgs b) {
  using R = real_t<PREC>;
  constexpr int REC = rec4<PREC>();
  __shared__ __attribute__((aligned(16))) unsigned char lds[narrow_lds_bytes<PREC>()];
  float4 *tile = reinterpret_cast<float4 *>(lds);
  const int tid = threadIdx.x;
  const g6mi_cluster d = current_block(h);
  const BatchPlan p = plan_block(d, b);
  const int nitems = p.nib * p.nsplit;
  if (blockIdx.x == 0 && tid == 0) {
    HermiteCtl *ctl = h.ctl;
    ctl->desc = d;
    ctl->done = d.ni > 0 ? 0 : 1;
    ctl->gather = ctl->phase ^ 1;
    b.plan[0] = p;
    b.work->nib = p.nib;
    b.status[kStatusFlags] = 0;
    b.status[kStatusOverflowCount] = 0;
  }
  const int ntiles = (d.nj + kTile - 1) / kTile;
  const bool ragged = d.nj % kTile != 0;
  const R eps2 = static_cast<R>(d.eps2);
  for (int q = blockIdx.x; q < nitems; q += gridDim.x) {
    const int ib = q / p.nsplit;
    const int sp = q - ib * p.nsplit;
    const int tb = sp * p.per;
    const int te = min(ntiles, tb + p.per);
    const size_t e0 = static_cast<size_t>(sp) * d.ni;
    JRaw nxt;
    if (tb < te) nxt.load(b.jm, static_cast<size_t>(min(tb * kTile + tid, d.nj - 1)));
    // one tile into LDS; past the last record nothing is stored
    auto stage = [&](int tt, int cnt) {
      __syncthreads();
      if (tid < cnt) predict_raw<PREC>(nxt, d.ti, tile + tid * REC);
      if (tt + 1 < te) nxt.load(b.jm, static_cast<size_t>(min((tt + 1) * kTile + tid, d.nj - 1)));
      __syncthreads();
    };
    if (p.ipw == 2 * kWG) {
      const int il0 = ib * (2 * kWG) + tid, il1 = il0 + kWG;
      WideLanes<PREC, false> w;
      w.init(b.fa, il0, il1, il0 < d.ni, il1 < d.ni);
      for (int tt = tb; tt < te; ++tt) {
        const int cnt = min(kTile, d.nj - tt * kTile);
        stage(tt, cnt);
        // whole waves without an i-particle have no work
        if (__any(w.v0)) w.template tile<PREC == G6MI_PREC_DS, true>(tile, tt * kTile, cnt, eps2, nullptr, nullptr);
      }
      if (w.v0) store_part(b.part, b.nn_slot, e0 + il0, w.t0, INFINITY, -1);
      if (w.v1) store_part(b.part, b.nn_slot, e0 + il1, w.t1, INFINITY, -1);
    } else {
      const int lil = tid & (p.ipw - 1);
      const int il = ib * p.ipw + lil;
      NarrowLane<PREC, false> n;
      n.init(b.fa, il, il < d.ni, tid >> p.log2ipw, 8 - p.log2ipw);
      const bool resolve = ragged && te == ntiles;
      for (int tt = tb; tt < te; ++tt) {
        const int cnt = min(kTile, d.nj - tt * kTile);
        stage(tt, cnt);
        n.tile(tile, tt * kTile, cnt, eps2, nullptr, nullptr);
        if (resolve) n.resolve(tile, tt * kTile);
      }
      double bestd;
      int bslot;
      n.template lane_sum<false>(reinterpret_cast<double *>(lds), tid, lil, p.ipw, bestd, bslot);
      if (n.sub == 0 && n.valid) store_part(b.part, b.nn_slot, e0 + il, n.t, INFINITY, -1);
    }
    __syncthreads(); // the item is done with the LDS
  }
}

__device__ __forceinline__ double norm3(const double *a) {
#pragma clang fp contract(off)
  return sqrt(a[0] * a[0] + a[1] * a[1] + a[2] * a[2]);
}

// Power-of-two step at or below dt, within [dt_min, dt_max]: 2^floor(log2)
// taken exactly from the binary exponent.
__device__ __forceinline__ double quantise(double dt, double dt_min, double dt_max) {
  dt = fmin(fmax(dt, dt_min), dt_max);
  int e;
  (void)frexp(dt, &e); // dt = f 2^e, f in [0.5, 1)
  return ldexp(1.0, e - 1);
}

// What the corrector needs of the particle at block position q besides its
// new force: loaded before the split sums, by the four lanes of its team (lane
// c takes component c of the vectors; the last lane repeats component 2).
struct CorrectState {
  int k = 0;
  double t = 0, dt = 0, a0 = 0, j0 = 0, xp = 0, vp = 0;
  __device__ __forceinline__ void load(const HermiteArgs &h, int q, int c) {
    k = h.active[q];
    const size_t e = static_cast<size_t>(c) * h.jm.cap + k, r = 3 * static_cast<size_t>(q) + c;
    xp = h.xi[r];
    vp = h.vi[r];
    t = h.jm.t[k];
    dt = h.dt[k];
    a0 = h.acc[e];
    j0 = h.jrk[e];
  }
};

// Corrector (Makino & Aarseth 1992) of a particle (s) at block time tb, given
// its new force sums f (acc xyz, jerk xyz, sum m/r), then the Aarseth
// criterion with the second derivative at the end of the step, and the block
// rule: halve while too long, double only when the time is a multiple of the
// doubled step.  The team's four lanes call it: lane c corrects component c,
// the norms collect the components by lane exchange, and all lanes return the
// new step.
__device__ __forceinline__ double correct_particle(const HermiteArgs &h, const CorrectState &s, int c, double tb,
                                                   const double *f) {
#pragma clang fp contract(off)
  HermiteCtl *ctl = h.ctl;
  const size_t cap = h.jm.cap;
  const double dt = tb - s.t;
  const int d = min(c, 2);
  const double a1[3] = {f[0], f[1], f[2]}, j1[3] = {f[3], f[4], f[5]};
  bool finite = true;
  for (int u = 0; u < 3; ++u) finite = finite && isfinite(a1[u]) && isfinite(j1[u]);
  const double a1d = d == 0 ? a1[0] : (d == 1 ? a1[1] : a1[2]);
  const double j1d = d == 0 ? j1[0] : (d == 1 ? j1[1] : j1[2]);
  const double dt2 = dt * dt, dt3 = dt2 * dt, dt4 = dt3 * dt, dt5 = dt4 * dt;
  const double a2d = (-6.0 * (s.a0 - a1d) - dt * (4.0 * s.j0 + 2.0 * j1d)) / dt2;
  const double a3d = (12.0 * (s.a0 - a1d) + 6.0 * dt * (s.j0 + j1d)) / dt3;
  const double a2ed = a2d + dt * a3d;
  const int base = threadIdx.x & 60;
  double a3[3], a2e[3];
  for (int u = 0; u < 3; ++u) {
    a3[u] = __shfl(a3d, base + u);
    a2e[u] = __shfl(a2ed, base + u);
  }
  const double na1 = norm3(a1), nj1 = norm3(j1), na3 = norm3(a3), na2e = norm3(a2e);
  const double num = na1 * na2e + nj1 * nj1;
  const double den = nj1 * na3 + na2e * na2e;
  const double dt_new = sqrt(h.eta * num / fmax(den, 1e-300));
  const double old = s.dt;
  double nw = old;
  while (dt_new < nw && nw > h.dt_min) nw *= 0.5; // never below dt_min
  if (dt_new >= 2.0 * old && fmod(tb, 2.0 * old) == 0.0 && 2.0 * old <= h.dt_max) nw = 2.0 * old;
  if (c < 3) {
    const size_t e = static_cast<size_t>(c) * cap + s.k;
    h.jm.x[e] = s.xp + a2d * dt4 / 24.0 + a3d * dt5 / 120.0;
    h.jm.v[e] = s.vp + a2d * dt3 / 6.0 + a3d * dt4 / 24.0;
    h.acc[e] = a1d;
    h.jrk[e] = j1d;
    h.jm.a2[e] = a1d / 2.0;
    h.jm.j6[e] = j1d / 6.0;
  } else {
    h.jm.t[s.k] = tb;
    h.dt[s.k] = nw;
    h.pot[s.k] = -f[6];
    if (!finite) atomicOr(&ctl->flags, 1);
  }
  return nw;
}

// The block's forces finished from the split partials (reduce_iblock, one
// workgroup per part of an i-block, at most kHsReduceWgs workgroups with
// rows) and each particle corrected by the lanes that finished it
// (correct_particle); the minimum of their new t + dt is folded into the
// next block time, one atomic per workgroup with rows.
__global__ __launch_bounds__(256) void hs_correct_kernel(HermiteArgs h, BatchArgs b) {
  HermiteCtl *ctl = h.ctl;
  const int ni = ctl->desc.ni;
  const double tb = ctl->desc.ti;
  const int gather = ctl->gather;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (ni > 0) {
      ctl->block_steps += 1;
      ctl->particle_steps += ni;
      ctl->time = tb;
    }
    // this step's key and count are read by no one any more
    ctl->key[gather ^ 1] = kKeyInf;
    ctl->ni_count = 0;
    ctl->phase = gather;
  }
  unsigned long long next = kKeyInf;
  int fl = 0;
  __shared__ SplitShared sh;
  const int c = threadIdx.x & 3;
  CorrectState st;
  const int nib_total = b.work->nib;
  const int P = reduce_parts(nib_total, min(static_cast<int>(gridDim.x), kHsReduceWgs), 64);
  for (int u = blockIdx.x; u < nib_total * P; u += gridDim.x)
    fl |= reduce_iblock<true>(
        b, u / P, u % P, P, sh,
        [&](int q, bool valid) {
          if (valid) st.load(h, q, min(c, 2));
        },
        [&](int q, bool valid, double2 v) {
          const int base = threadIdx.x & 60;
          const double sum[7] = {__shfl(v.x, base),     __shfl(v.y, base),     __shfl(v.x, base + 1),
                                 __shfl(v.y, base + 1), __shfl(v.x, base + 2), __shfl(v.y, base + 2),
                                 __shfl(v.x, base + 3)};
          if (valid) {
            const unsigned long long key = order_key(tb + correct_particle(h, st, c, tb, sum));
            next = key < next ? key : next;
          }
        });
  if (fl) atomicOr(b.status + kStatusFlags, fl);
  // the next block time, second part: this block's particles
  key_min(next, &ctl->key[gather]);
}

// First step of block position q: a, jerk and potential stored, the step
// eta_s |a| / |jerk| quantised.  Returns the step.
__device__ __forceinline__ double start_particle(const HermiteArgs &h, int q) {
#pragma clang fp contract(off)
  HermiteCtl *ctl = h.ctl;
  const int k = h.active[q];
  const size_t cap = h.jm.cap;
  double a1[3], j1[3];
  bool finite = true;
  for (int d = 0; d < 3; ++d) {
    a1[d] = h.acc1[3 * static_cast<size_t>(q) + d];
    j1[d] = h.jrk1[3 * static_cast<size_t>(q) + d];
    finite = finite && isfinite(a1[d]) && isfinite(j1[d]);
    h.acc[d * cap + k] = a1[d];
    h.jrk[d * cap + k] = j1[d];
    h.jm.a2[d * cap + k] = a1[d] / 2.0;
    h.jm.j6[d * cap + k] = j1[d] / 6.0;
  }
  const double dt = h.eta_s * norm3(a1) / fmax(norm3(j1), 1e-300);
  const double step = quantise(dt, h.dt_min, h.dt_max);
  h.dt[k] = step;
  h.pot[k] = h.pot1[q];
  if (!finite) atomicOr(&ctl->flags, 1);
  return step;
}

// First force evaluation of every particle at the common start time
// (start_particle, one thread each) and the first next block time.
__global__ __launch_bounds__(256) void hs_start_kernel(HermiteArgs h) {
  HermiteCtl *ctl = h.ctl;
  const int ni = ctl->desc.ni;
  const int q = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.x == 0 && threadIdx.x == 0) ctl->time = ctl->desc.ti;
  if (blockIdx.x * 256 >= ni) return; // whole workgroups past the block
  const double dt = q < ni ? start_particle(h, q) : INFINITY;
  key_min(q < ni ? order_key(ctl->desc.ti + dt) : kKeyInf, &ctl->key[ctl->phase]);
}

// Clear the step state before the first force evaluation: every particle
// due at its own (common) time, a and jerk zero as in the host driver.
__global__ __launch_bounds__(256) void hs_reset_kernel(HermiteArgs h) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    h.ctl->flags = 0;
    h.ctl->done = 0;
    h.ctl->block_steps = 0;
    h.ctl->particle_steps = 0;
  }
  if (k >= h.n) return;
  const size_t cap = h.jm.cap;
  h.dt[k] = 0.0;
  h.h2i[k] = h.h2; // rows 0 .. n-1, for every block
  for (int d = 0; d < 3; ++d) {
    h.acc[d * cap + k] = 0.0;
    h.jrk[d * cap + k] = 0.0;
    h.jm.a2[d * cap + k] = 0.0;
    h.jm.j6[d * cap + k] = 0.0;
  }
}

// 64 particles per workgroup: read component by component (64 consecutive
// slots each), written row by row, so that both sides are contiguous.
__global__ __launch_bounds__(256) void hs_export_kernel(HermiteArgs h, int k0, int n, double *__restrict__ rows) {
  __shared__ double s_row[64][kHsRowDoubles + 1];
  const int tid = threadIdx.x, lane = tid & 63, r0 = blockIdx.x * 64;
  const size_t cap = h.jm.cap, k = static_cast<size_t>(k0) + r0 + lane;
  for (int c = tid >> 6; c < kHsRowDoubles && r0 + lane < n; c += 4) {
    const double *src = c == 0 ? h.jm.t
                        : c < 4  ? h.jm.x + (c - 1) * cap
                        : c < 7  ? h.jm.v + (c - 4) * cap
                        : c < 10 ? h.acc + (c - 7) * cap
                        : c < 13 ? h.jrk + (c - 10) * cap
                        : c == 13 ? h.pot
                                  : h.dt;
    s_row[lane][c] = c < 15 ? src[k] : 0.0;
  }
  __syncthreads();
  for (int q = tid; q < 64 * kHsRowDoubles; q += 256) {
    const int r = q / kHsRowDoubles;
    if (r0 + r < n) rows[static_cast<size_t>(r0) * kHsRowDoubles + q] = s_row[r][q % kHsRowDoubles];
  }
}

// ---------------------------------------------------------------- launchers

static inline dim3 grid_n(int n) { return dim3(static_cast<unsigned>((n > 0 ? n : 1) + 255) / 256); }

hipError_t launch_hs_reset(const HermiteArgs &h, hipStream_t s) {
  hipLaunchKernelGGL(hs_reset_kernel, grid_n(h.n), dim3(256), 0, s, h);
  return hipGetLastError();
}
hipError_t launch_hs_export(const HermiteArgs &h, int k0, int n, double *rows, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(hs_export_kernel, dim3(static_cast<unsigned>((n + 63) / 64)), dim3(256), 0, s, h, k0, n, rows);
  return hipGetLastError();
}
hipError_t launch_hs_first(const HermiteArgs &h, const BatchArgs &b, hipStream_t s) {
  hipLaunchKernelGGL(hs_select_kernel, grid_n(h.n), dim3(256), 0, s, h);
  hipLaunchKernelGGL(hs_publish_kernel, dim3(1), dim3(256), 0, s, h, b);
  return hipGetLastError();
}
hipError_t launch_hs_force(int prec, const HermiteArgs &h, const BatchArgs &b, int grid, hipStream_t s) {
  if (grid <= 0) return hipErrorInvalidValue;
  hipLaunchKernelGGL(hs_select_kernel, grid_n(h.n), dim3(256), 0, s, h);
  const dim3 g(static_cast<unsigned>(grid));
  switch (prec) {
  case G6MI_PREC_FP32: hipLaunchKernelGGL(hs_force_kernel<G6MI_PREC_FP32>, g, dim3(kWG), 0, s, h, b); break;
  case G6MI_PREC_DS: hipLaunchKernelGGL(hs_force_kernel<G6MI_PREC_DS>, g, dim3(kWG), 0, s, h, b); break;
  default: hipLaunchKernelGGL(hs_force_kernel<G6MI_PREC_FP64>, g, dim3(kWG), 0, s, h, b);
  }
  return hipGetLastError();
}
hipError_t launch_hs_start(const HermiteArgs &h, hipStream_t s) {
  hipLaunchKernelGGL(hs_start_kernel, grid_n(h.n), dim3(256), 0, s, h);
  return hipGetLastError();
}
hipError_t launch_hs_correct(const HermiteArgs &h, const BatchArgs &b, int grid, hipStream_t s) {
  hipLaunchKernelGGL(hs_correct_kernel, dim3(static_cast<unsigned>(grid > 0 ? grid : 1)), dim3(256), 0, s, h, b);
  return hipGetLastError();
}

} // namespace g6mi
