// gfx950 kernels of the direct-summation force evaluation.
//
//   predict_kernel  -- j-particle predictor, Eq. (1)-(2) of Sec. 2.2, in
//                      float64, writing the predicted j-records in the layout
//                      of the selected precision variant (HBM-bound).
//   force_wide, force_one, force_kernel
//                   -- the i x j interaction (Sec. 2.3) with two, one or part
//                      of a lane per i-particle: LDS-staged j-tiles, j-split
//                      across workgroups, nearest neighbour and neighbour
//                      lists fused in the same loop (VALU-bound).
//   piece_min_kernel, force_piece
//                   -- blocks whose j-splits are too few for the device, in
//                      pieces of a split (PieceArgs).
//   force_fused, force_fused_one
//                   -- one i-block, the predictor fused in.
//   reduce_kernel   -- fixed-order float64 sum of the j-split partials, the
//                      nearest-neighbour minimum and the neighbour-list
//                      finalisation (slot -> particle index, ascending).
//
// The pair interaction is elementwise per (i, j) pair, not a contraction,
// so it runs on the vector ALUs; no matrix-core instructions are used.

#include "g6mi_device.h"

#include <mutex>

namespace g6mi {

size_t pred_record_bytes(int prec) {
  switch (prec) {
  case G6MI_PREC_FP32: return 32;
  case G6MI_PREC_DS: return 48;
  default: return 64;
  }
}

// ---------------------------------------------------------------- predictor

// One thread per j-slot: the record of slot k predicted to ti (Sec. 2.2,
// Eq. (1)-(2)) in the layout of the precision variant.  The same launch
// clears the neighbour counters and status words of the calculation.
template <int PREC>
__global__ __launch_bounds__(256) void predict_kernel(int nj, double ti, JMem jm,
                                                      void *__restrict__ out,
                                                      int *__restrict__ nb_count, int ni,
                                                      int *__restrict__ status) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < ni) nb_count[k] = 0; // fresh neighbour counters for this call
  if (k < kStatusWords) status[k] = 0;
  if (k >= nj) return;
  predict_record<PREC>(jm, static_cast<size_t>(k), ti,
                       static_cast<float4 *>(out) + rec4<PREC>() * static_cast<size_t>(k));
}

// ------------------------------------------------- interaction, wide blocks

// Wide blocks (WideLanes): lane tid owns i-particles base + tid and
// base + 256 + tid, 512 per workgroup.  Grid: x = i-blocks of 512,
// y = j-splits; the partials of split y go to part[y][7][ni].
template <int PREC, bool NBL>
__global__ __launch_bounds__(kWG, wide_waves<PREC>()) void force_wide(ForceArgs a) {
  constexpr int REC = rec4<PREC>();
  constexpr int kLoads = kTile * REC / kWG; // 16-byte loads per lane per tile
  static_assert(kTile * REC % kWG == 0, "whole loads per lane");
  __shared__ __attribute__((aligned(16))) float4 tile[kTile * REC];

  const int tid = threadIdx.x;
  const int i0 = blockIdx.x * (2 * kWG) + tid;
  const int i1 = i0 + kWG;
  WideLanes<PREC, NBL> w;
  w.init(a, i0, i1, i0 < a.ni, i1 < a.ni);
  const real_t<PREC> eps2 = static_cast<real_t<PREC>>(a.eps2);

  const int ntiles = (a.nj + kTile - 1) / kTile;
  const int per = (ntiles + gridDim.y - 1) / gridDim.y;
  const int tb = blockIdx.y * per;
  const int te = min(ntiles, tb + per);
  const float4 *jp = static_cast<const float4 *>(a.jpred);

  for (int tt = tb; tt < te; ++tt) {
    const int jbase = tt * kTile;
    const int cnt = min(kTile, a.nj - jbase);
    __syncthreads();
    {
      // coalesced 16-byte loads of the tile into LDS (records < nj only)
      const float4 *src = jp + static_cast<size_t>(jbase) * REC;
      const int n4 = cnt * REC;
#pragma unroll
      for (int q = 0; q < kLoads; ++q) {
        const int idx = q * kWG + tid;
        if (idx < n4) tile[idx] = src[idx];
      }
    }
    __syncthreads();
    // DS: every group goes straight to the float64 totals (see WideLanes::tile)
    w.template tile<PREC == G6MI_PREC_DS, true>(tile, jbase, cnt, eps2, a.nb_count, a.nb_slot);
  }
  // exact slot of the fast-path nearest neighbours: their groups are
  // re-read from global memory (every slot is < nj)
  w.resolve(jp, 0);

  const size_t e0 = static_cast<size_t>(blockIdx.y) * a.ni;
  if (w.v0) store_part(a.part, a.nn_slot, e0 + i0, w.t0, static_cast<double>(w.ebest0), w.eslot0);
  if (w.v1) store_part(a.part, a.nn_slot, e0 + i1, w.t1, static_cast<double>(w.ebest1), w.eslot1);
}

// K float4 per lane of a tile of n4 float4 (lane tid holds elements tid,
// tid + 256, ...), in named registers of a plain vector type (an aggregate
// float4 copy would go through the stack).  Loads are clamped to the last
// element so that every lane loads unconditionally; the store writes only
// the elements below n4.
template <int K> struct TileRegs {
  static_assert(K >= 1 && K <= 4, "one to four float4 per lane");
  typedef float v4 __attribute__((ext_vector_type(4)));
  v4 v0, v1, v2, v3;
  __device__ __forceinline__ void load(const float4 *__restrict__ src4, int tid, int n4) {
    const v4 *src = reinterpret_cast<const v4 *>(src4);
    v0 = src[min(tid, n4 - 1)];
    if constexpr (K > 1) v1 = src[min(kWG + tid, n4 - 1)];
    if constexpr (K > 2) v2 = src[min(2 * kWG + tid, n4 - 1)];
    if constexpr (K > 3) v3 = src[min(3 * kWG + tid, n4 - 1)];
  }
  __device__ __forceinline__ void store(float4 *__restrict__ dst4, int tid, int n4) const {
    v4 *dst = reinterpret_cast<v4 *>(dst4);
    if (tid < n4) dst[tid] = v0;
    if constexpr (K > 1)
      if (kWG + tid < n4) dst[kWG + tid] = v1;
    if constexpr (K > 2)
      if (2 * kWG + tid < n4) dst[2 * kWG + tid] = v2;
    if constexpr (K > 3)
      if (3 * kWG + tid < n4) dst[3 * kWG + tid] = v3;
  }
};

// Small blocks (NarrowLane): ipw i-particles per workgroup (a power of two,
// at most 256) and L = 256 / ipw lanes per i-particle; lane tid handles
// i-particle (tid mod ipw) and the records sub, sub + L, ... of every tile,
// sub = tid / ipw.  For ipw >= 64 every lane of a wave reads the same record
// (an LDS broadcast).  The L lane totals of an i-particle are added in a
// fixed order.  Grid: x = i-blocks, y = j-splits, or (PIECES) the pieces of
// the j-splits one split after the other, each starting from the minima of
// its split's earlier tiles that piece_min_kernel found.
template <int PREC, bool NBL, bool PIECES = false>
__global__ __launch_bounds__(kWG) void force_kernel(ForceArgs a, PieceArgs pc) {
  constexpr int REC = rec4<PREC>();
  constexpr int kLoads = kTile * REC / kWG;
  __shared__ __attribute__((aligned(16))) unsigned char lds[narrow_lds_bytes<PREC>()];
  float4 *tile = reinterpret_cast<float4 *>(lds);

  const int tid = threadIdx.x;
  const int ipw = a.ipw;
  const int il = tid & (ipw - 1);
  const BlockRows rows(a);
  const int i = rows.first + il;
  NarrowLane<PREC, NBL> n;
  n.init(a, i, i < rows.end, tid >> a.log2ipw, 8 - a.log2ipw);
  const real_t<PREC> eps2 = static_cast<real_t<PREC>>(a.eps2);

  const bool busy = __any(n.valid); // whole waves without an i-particle have no work
  const int ntiles = (a.nj + kTile - 1) / kTile;
  const float4 *jp = static_cast<const float4 *>(a.jpred);
  int tb, te;
  if constexpr (PIECES) {
    const PieceRange r = piece_range(pc, ntiles, blockIdx.y);
    tb = r.begin;
    te = r.end;
    for (int tt = r.split; busy && tt < tb; ++tt) {
      const size_t e = (static_cast<size_t>(tt) * gridDim.x + blockIdx.x) * kWG + tid;
      const float m = pc.least[e];
      if (m < n.gbest) {
        n.gbest = m;
        if (pc.exact && r.split == pc.vlast) n.ebest = fminf(n.ebest, pc.exact[e]);
      }
    }
  } else {
    const int per = (ntiles + gridDim.y - 1) / gridDim.y;
    tb = blockIdx.y * per;
    te = min(ntiles, tb + per);
  }

  // The next tile's records are loaded into registers while the current
  // one is evaluated: a block of few i-particles spends little time per
  // tile, too little to cover the load on its own.
  TileRegs<kLoads> nxt;
  if (tb < te) nxt.load(jp + static_cast<size_t>(tb) * kTile * REC, tid, min(kTile, a.nj - tb * kTile) * REC);
  for (int tt = tb; tt < te; ++tt) {
    const int jbase = tt * kTile;
    const int cnt = min(kTile, a.nj - jbase);
    __syncthreads();
    nxt.store(tile, tid, cnt * REC);
    {
      const int tn = min(tt + 1, te - 1); // the last tile loads itself again
      nxt.load(jp + static_cast<size_t>(tn) * kTile * REC, tid, min(kTile, a.nj - tn * kTile) * REC);
    }
    __syncthreads();
    if (busy) {
      n.tile(tile, jbase, cnt, eps2, a.nb_count, a.nb_slot);
      // while the tile is still in LDS: the exact nearest neighbour so far
      // decides which groups of a ragged tile fold into float64 (fold_or_add),
      // as in force_fused and the batched kernel
      n.resolve(tile, jbase);
    }
  }

  double bestd;
  int bslot;
  n.lane_sum(reinterpret_cast<double *>(lds), tid, il, ipw, bestd, bslot);
  if (n.sub == 0 && n.valid)
    store_part(a.part, a.nn_slot, static_cast<size_t>(blockIdx.y) * a.ni + i, n.t, bestd, bslot);
}

// First launch of a calculation in pieces (PieceArgs): the predictor, and
// each lane's least softened r^2 in each tile.  Where a group is folded into
// the float64 totals depends on the least r^2 that the lane met before it in
// its split (fold_or_add), so a split of eight or more tiles is one serial
// chain; with the minima of its earlier tiles known, every piece of a split
// can start on its own and make the same decisions.  The minima take a third
// of the operations of the full pair.
// Workgroup (x, y): i-block x, tile y, S sets of 256 lanes, set k taking every
// S-th group (see force_piece).  i-block 0 writes the predicted records; the
// tiles of a split's last piece need no minima.  For the split that holds the
// ragged tile, whose lanes go by the exact r^2 found so far (MaskedRun), the
// exact r^2 of the group holding the minimum is kept too: the group that
// NarrowLane would resolve after the tile if it lies below the minima before.
// The same launch clears the neighbour counters and status words.
template <int PREC, int S>
__global__ __launch_bounds__(S * kWG) void piece_min_kernel(ForceArgs a, JMem jm, double ti, PieceArgs pc,
                                                            float4 *__restrict__ jpred, int *__restrict__ status) {
  static_assert(PREC != G6MI_PREC_FP64, "float64 sums do not depend on the splits");
  constexpr int REC = rec4<PREC>();
  __shared__ __attribute__((aligned(16))) float4 tile[kTile * REC];
  __shared__ float s_min[S][kWG];
  __shared__ int s_grp[S][kWG];
  const int set = S > 1 ? threadIdx.x / kWG : 0, lid = turned_lane(threadIdx.x, set), tt = blockIdx.y;
  const BlockRows rows(a);
  const int il = lid & (a.ipw - 1), i = rows.first + il;
  const bool valid = i < rows.end;
  if (tt == 0 && set == 0) {
    if (blockIdx.x == 0 && lid < kStatusWords) status[lid] = 0;
    if (lid < a.ipw && valid) a.nb_count[i] = 0;
  }
  const int jbase = tt * kTile, cnt = min(kTile, a.nj - jbase);
  const bool need = piece_follows(pc, (a.nj + kTile - 1) / kTile, tt);
  if (blockIdx.x > 0 && !need) return;
  if (set == 0 && lid < cnt) {
    predict_record<PREC>(jm, static_cast<size_t>(jbase + lid), ti, tile + lid * REC);
    if (blockIdx.x == 0)
#pragma unroll
      for (int q = 0; q < REC; ++q) jpred[static_cast<size_t>(jbase + lid) * REC + q] = tile[lid * REC + q];
  }
  if (!need) return;
  IState<PREC> st;
  int slot;
  float h2;
  load_i<PREC>(st, a, i, valid, slot, h2);
  __syncthreads();
  if (S == 1 && !__any(valid)) return;
  // a tile with a later piece is full
  const int log2L = 8 - a.log2ipw, sub = lid >> a.log2ipw, own = slot - jbase;
  const float eps2 = static_cast<float>(a.eps2);
  float best = INFINITY;
  int grp = -1;
  const int kend = S == 1 || __any(valid) ? kTile >> log2L : 0;
  for (int k0 = set * kGroup; k0 < kend; k0 += S * kGroup) {
    float m = INFINITY;
#pragma unroll
    for (int u = 0; u < kGroup; ++u) {
      const int jj = sub + ((k0 + u) << log2L);
      float d[3], w[3], mj;
      separation<PREC>(st, tile + jj * REC, d, w, mj);
      const float s = fma(d[2], d[2], fma(d[1], d[1], fma(d[0], d[0], eps2))); // as in pair_core
      m = fmin(m, jj == own ? INFINITY : s);
    }
    if (m < best) {
      best = m;
      grp = jbase + sub + (k0 << log2L);
    }
  }
  if constexpr (S > 1) {
    s_min[set][lid] = best;
    s_grp[set][lid] = grp;
    __syncthreads();
    if (set > 0) return;
    // the least minimum, of equal ones the first group's
#pragma unroll
    for (int k = 1; k < S; ++k) {
      const float m = s_min[k][lid];
      const int g = s_grp[k][lid];
      if (g >= 0 && (m < best || (m == best && g < grp))) {
        best = m;
        grp = g;
      }
    }
  }
  const size_t e = (static_cast<size_t>(tt) * gridDim.x + blockIdx.x) * kWG + lid;
  pc.least[e] = best;
  if (pc.exact && tt >= pc.vlast) {
    float r2 = INFINITY;
    int bs = -1;
    resolve_group<PREC>(st, grp, 1 << log2L, tile, jbase, r2, bs, slot);
    pc.exact[e] = r2;
  }
}

// The pieces of a calculation in pieces, after piece_min_kernel: i-blocks of
// 32 to 256 i-particles as in force_kernel, S sets of 256 lanes per workgroup.
// The lanes of one set are those of force_kernel; set k evaluates every S-th
// group of kGroup records of their chains (k, k + S, ...), and set 0 adds the
// group sums of a round in order, through LDS, by the rule of fold_or_add.  A
// block of a few hundred i-particles against 2^15 records is one workgroup
// per compute unit: with one set the chains' latency is exposed (341 against
// 2^15 in double-single: this kernel 38.5 us with one set, 23.9 with four,
// piece_min_kernel 18.8 and 12.9; 21.6 and 12.1 since the waves are dealt
// evenly over the i-blocks, first_row).
// Grid: x = i-blocks, y = pieces, one split after the other; each starts from
// the minima of its split's earlier tiles.  The double buffer lets the other
// sets go on to the next round while set 0 adds.  Which sums a group goes to
// follows NarrowLane::grouped for full tiles and MaskedRun for ragged ones: a
// change to either rule has to be made here too, or the bits part.
template <int PREC, bool NBL, int S>
__global__ __launch_bounds__(S * kWG, 4) void force_piece(ForceArgs a, PieceArgs pc) {
  constexpr int REC = rec4<PREC>();
  constexpr int kTileBytes = kTile * REC * 16;
  constexpr int kXBytes = 2 * (S - 1) * kWG * 48;
  static_assert(kXBytes >= kWG * 9 * 8, "the lane sums reuse the exchange area");
  __shared__ __attribute__((aligned(16))) unsigned char lds[kTileBytes + kXBytes];
  float4 *tile = reinterpret_cast<float4 *>(lds);
  // group sums of sets 1 .. S - 1: [buffer][set - 1][lane][3]: a, min; j1, p; j2, slot
  float4 *xch = reinterpret_cast<float4 *>(lds + kTileBytes);

  const int tid = threadIdx.x, set = __builtin_amdgcn_readfirstlane(tid / kWG), lid = turned_lane(tid, set);
  const BlockRows rows(a);
  const int ipw = a.ipw, il = lid & (ipw - 1), i = rows.first + il;
  NarrowLane<PREC, NBL> n;
  n.init(a, i, i < rows.end, lid >> a.log2ipw, 8 - a.log2ipw);
  const float eps2 = static_cast<float>(a.eps2);
  const bool busy = __any(n.valid); // whole waves without an i-particle have no work

  const int ntiles = (a.nj + kTile - 1) / kTile;
  const float4 *jp = static_cast<const float4 *>(a.jpred);
  const PieceRange range = piece_range(pc, ntiles, blockIdx.y);
  if (set == 0 && busy)
    for (int tt = range.split; tt < range.begin; ++tt) {
      const size_t e = (static_cast<size_t>(tt) * gridDim.x + blockIdx.x) * kWG + lid;
      const float m = pc.least[e];
      if (m < n.gbest) {
        n.gbest = m;
        if (pc.exact && range.split == pc.vlast) n.ebest = fminf(n.ebest, pc.exact[e]);
      }
    }

  for (int tt = range.begin; tt < range.end; ++tt) {
    const int jbase = tt * kTile;
    const int cnt = min(kTile, a.nj - jbase);
    __syncthreads();
    for (int q = tid; q < cnt * REC; q += S * kWG) tile[q] = jp[static_cast<size_t>(jbase) * REC + q];
    __syncthreads();
    const bool ragged = cnt < kTile;
    const int L = n.L, rounds = (n.K / kGroup + S - 1) / S;
    const int own = n.slot - jbase; // own slot relative to the tile
    const bool self = __any(own >= 0 && own < cnt);
    const float fb = nb_flag_bound(n.h2, eps2);
    unsigned nbm = 0u;
    for (int r = 0; r < rounds; ++r) {
      const int k0 = (r * S + set) * kGroup; // first record of this set's group in the lane's chain
      Sums<float> gs;
      float m = INFINITY;
      int bs = -1, got = 0; // a ragged tile: the slot at the minimum, records in the group
      if (busy && !ragged) {
        auto group = [&](auto masked) {
          constexpr bool SELF = decltype(masked)::value;
          int jj = n.sub + (k0 << n.log2L);
          m = pair_core<PREC, true, SELF>(n.st, gs, tile + jj * REC, eps2, jj == own);
#pragma unroll
          for (int u = 1; u < kGroup; ++u) {
            jj = n.sub + ((k0 + u) << n.log2L);
            m = fmin(m, pair_core<PREC, false, SELF>(n.st, gs, tile + jj * REC, eps2, jj == own));
          }
        };
        if (self) group(std::true_type{});
        else group(std::false_type{});
        got = kGroup;
      } else if (busy) {
        // per pair, with the exact r^2, as in MaskedRun
        gs.zero();
        int *cp = a.nb_count + (n.valid ? n.row : 0);
        int *lp = a.nb_slot + static_cast<size_t>(n.valid ? n.row : 0) * kNbMax;
        for (int u = 0; u < kGroup; ++u) {
          const int jj = n.sub + ((k0 + u) << n.log2L);
          if (jj < cnt) {
            pair<PREC, true, NBL>(n.st, gs, tile + jj * REC, jbase + jj, n.slot, eps2, n.h2, m, bs, cp, lp);
            ++got;
          }
        }
      }
      float4 *x = xch + static_cast<size_t>(r & 1) * (S - 1) * kWG * 3;
      if (set > 0 && busy) {
        float4 *o = x + ((set - 1) * kWG + lid) * 3;
        o[0] = make_float4(gs.a[0], gs.a[1], gs.a[2], m);
        o[1] = make_float4(gs.j1[0], gs.j1[1], gs.j1[2], gs.p);
        o[2] = make_float4(gs.j2[0], gs.j2[1], gs.j2[2], __int_as_float(bs));
      }
      __syncthreads();
      if (set == 0 && busy) {
        // the round's groups in the order of the records
        auto take = [&](Sums<float> &g, float mg, int slot, int k, int records) {
          if (!ragged) {
            fold_or_add(g, n.ts, n.t, mg < n.gbest);
            if (mg < n.gbest) {
              n.gbest = mg;
              n.grp = jbase + n.sub + (k << n.log2L);
            }
            if constexpr (NBL) nbm |= (mg < fb ? 1u : 0u) << (k / kGroup);
          } else if (records > 0) {
            if (records == kGroup) fold_or_add(g, n.ts, n.t, mg < n.ebest);
            else n.ts.add(g);
            if (mg < n.ebest) {
              n.ebest = mg;
              n.eslot = slot;
            }
          }
        };
        take(gs, m, bs, k0, got);
#pragma unroll
        for (int k = 1; k < S; ++k) {
          const int kk = (r * S + k) * kGroup;
          if (kk < n.K) {
            const float4 *o = x + ((k - 1) * kWG + lid) * 3;
            const float4 q0 = o[0], q1 = o[1], q2 = o[2];
            Sums<float> g;
            g.a[0] = q0.x; g.a[1] = q0.y; g.a[2] = q0.z;
            g.j1[0] = q1.x; g.j1[1] = q1.y; g.j1[2] = q1.z;
            g.p = q1.w;
            g.j2[0] = q2.x; g.j2[1] = q2.y; g.j2[2] = q2.z;
            // records of that group in this lane's chain
            const int rest = (cnt - n.sub + L - 1) / L - kk;
            take(g, q0.w, __float_as_int(q2.w), kk, min(rest, kGroup));
          }
        }
      }
    }
    if (set == 0 && busy) {
      fold(n.ts, n.t);
      if constexpr (NBL) n.append_flagged(tile, jbase, nbm, own, a.nb_count, a.nb_slot);
      n.resolve(tile, jbase); // while the tile is still in LDS
    }
  }

  double bestd;
  int bslot;
  n.lane_sum(reinterpret_cast<double *>(xch), lid, il, ipw, bestd, bslot, set == 0);
  if (set == 0 && n.sub == 0 && n.valid)
    store_part(a.part, a.nn_slot, static_cast<size_t>(blockIdx.y) * a.ni + i, n.t, bestd, bslot);
}

// The blocks of force_wide with one i-particle per lane, 256 per workgroup
// (NarrowLane with WIDE sums): half the i-particles and half the work per
// workgroup and tile, and waves without an i-particle skip the tiles, so
// blocks of a few hundred to a few thousand i-particles, whose tiles would
// not fill the compute units evenly in workgroups of 512, spread better; four
// workgroups fit a compute unit (three of force_wide).  The float32 sums are
// those of force_wide.  785 i-particles against 2^17 in float32: 102 us with
// one to four tiles per split, 300 us as force_wide in 128 workgroups of
// eight tiles; 2048 against 2^18, same splits: 366 against 407 us (double-
// single 438 against 476).
template <int PREC, bool NBL>
__global__ __launch_bounds__(kWG, 4) void force_one(ForceArgs a) {
  constexpr int REC = rec4<PREC>();
  constexpr int kLoads = kTile * REC / kWG;
  __shared__ __attribute__((aligned(16))) float4 tile[kTile * REC];

  const int tid = threadIdx.x;
  const BlockRows rows(a);
  const int i = rows.first + tid;
  NarrowLane<PREC, NBL, true> n;
  n.init(a, i, i < rows.end, 0, 0);
  const real_t<PREC> eps2 = static_cast<real_t<PREC>>(a.eps2);

  const int ntiles = (a.nj + kTile - 1) / kTile;
  const int per = (ntiles + gridDim.y - 1) / gridDim.y;
  const int tb = blockIdx.y * per;
  const int te = min(ntiles, tb + per);
  const float4 *jp = static_cast<const float4 *>(a.jpred);
  const bool busy = __any(n.valid);

  TileRegs<kLoads> nxt;
  if (tb < te) nxt.load(jp + static_cast<size_t>(tb) * kTile * REC, tid, min(kTile, a.nj - tb * kTile) * REC);
  for (int tt = tb; tt < te; ++tt) {
    const int jbase = tt * kTile;
    const int cnt = min(kTile, a.nj - jbase);
    __syncthreads();
    nxt.store(tile, tid, cnt * REC);
    {
      const int tn = min(tt + 1, te - 1); // the last tile loads itself again
      nxt.load(jp + static_cast<size_t>(tn) * kTile * REC, tid, min(kTile, a.nj - tn * kTile) * REC);
    }
    __syncthreads();
    if (busy) n.tile(tile, jbase, cnt, eps2, a.nb_count, a.nb_slot);
  }
  n.resolve(jp, 0); // exact slots from the records in global memory, as in force_wide
  if (n.valid)
    store_part(a.part, a.nn_slot, static_cast<size_t>(blockIdx.y) * a.ni + i, n.t, static_cast<double>(n.ebest),
               n.eslot);
}

// ------------------------------------ small blocks, predictor fused in

// A block of at most 256 i-particles (one i-block, NarrowLane as in
// force_kernel) reads the float64 j-memory and predicts every tile into LDS
// itself (Sec. 2.2 fused into the tile load, as in the batched kernel), so
// the predicted records are never written to HBM and read back: for a block
// of a few particles the step is the predictor's HBM traffic, 112 B per
// j-particle instead of 112 + 48 + 48.  The next tile's j-memory entries are
// loaded into registers while the current tile is evaluated.  The
// neighbours are counted in nb_work, which the reduction clears again, so no
// launch before this one has to clear counters; workgroup (0, 0) clears the
// status words, which only the reduction after this launch writes.
template <int PREC, bool NBL>
__global__ __launch_bounds__(kWG) void force_fused(ForceArgs a, JMem jm, double ti, int *__restrict__ nb_work,
                                                   int *__restrict__ status) {
  constexpr int REC = rec4<PREC>();
  __shared__ __attribute__((aligned(16))) unsigned char lds[narrow_lds_bytes<PREC>()];
  float4 *tile = reinterpret_cast<float4 *>(lds);

  const int tid = threadIdx.x;
  if (blockIdx.x == 0 && blockIdx.y == 0 && tid < kStatusWords) status[tid] = 0;
  const int ipw = a.ipw;
  const int il = tid & (ipw - 1);
  const int i = blockIdx.x * ipw + il;
  NarrowLane<PREC, NBL> n;
  n.init(a, i, i < a.ni, tid >> a.log2ipw, 8 - a.log2ipw);
  const real_t<PREC> eps2 = static_cast<real_t<PREC>>(a.eps2);

  const int ntiles = (a.nj + kTile - 1) / kTile;
  const int per = (ntiles + gridDim.y - 1) / gridDim.y;
  const int tb = blockIdx.y * per;
  const int te = min(ntiles, tb + per);

  // whole waves without an i-particle have no work (160 against 2^18 in
  // float64 106 -> 99 us, 150 against 2^20 in double-single 307 -> 300)
  const bool busy = __any(n.valid);

  // lane tid predicts record tid of each tile; past nj it loads slot nj - 1
  // (in bounds) and stores nothing
  JRaw nxt;
  if (tb < te) nxt.load(jm, static_cast<size_t>(min(tb * kTile + tid, a.nj - 1)));
  for (int tt = tb; tt < te; ++tt) {
    const int jbase = tt * kTile;
    const int cnt = min(kTile, a.nj - jbase);
    __syncthreads();
    if (tid < cnt) predict_raw<PREC>(nxt, ti, tile + tid * REC);
    if (tt + 1 < te) nxt.load(jm, static_cast<size_t>(min((tt + 1) * kTile + tid, a.nj - 1)));
    __syncthreads();
    if (busy) {
      n.tile(tile, jbase, cnt, eps2, nb_work, a.nb_slot);
      n.resolve(tile, jbase); // while the tile is still in LDS
    }
  }

  double bestd;
  int bslot;
  n.lane_sum(reinterpret_cast<double *>(lds), tid, il, ipw, bestd, bslot);
  if (n.sub == 0 && n.valid)
    store_part(a.part, a.nn_slot, static_cast<size_t>(blockIdx.y) * a.ni + i, n.t, bestd, bslot);
}

// One i-particle (ipw = 1, all 256 lanes on it): lane tid takes records
// tid, tid + 256, ... of the split, predicts each one itself and uses it at
// once, so no record goes through LDS and no barrier is needed; the next
// record's j-memory entries are loaded while the current one is evaluated.
// The arithmetic and the order of the sums are those of force_fused (and of
// force_kernel on predicted records) for one i-particle: each record is a
// group of one pair, added to the float64 totals.
template <int PREC, bool NBL>
__global__ __launch_bounds__(kWG) void force_fused_one(ForceArgs a, JMem jm, double ti, int *__restrict__ nb_work,
                                                       int *__restrict__ status) {
  constexpr int REC = rec4<PREC>();
  __shared__ __attribute__((aligned(16))) double red[9 * kWG]; // lane_sum
  const int tid = threadIdx.x;
  if (blockIdx.y == 0 && tid < kStatusWords) status[tid] = 0;
  NarrowLane<PREC, NBL> n;
  n.init(a, 0, true, tid, 8);
  const real_t<PREC> eps2 = static_cast<real_t<PREC>>(a.eps2);

  const int ntiles = (a.nj + kTile - 1) / kTile;
  const int per = (ntiles + gridDim.y - 1) / gridDim.y;
  const int tb = blockIdx.y * per;
  const int te = min(ntiles, tb + per);
  const int je = min(a.nj, te * kTile);
  // kFusedDepth records per lane in flight: record js + u * kWG sits in q[u]
  // and is replaced, once used, by the one kFusedDepth records further on
  constexpr int D = kFusedDepth;
  JRaw q[D];
  const int j0 = tb * kTile + tid;
#pragma unroll
  for (int u = 0; u < D; ++u)
    if (j0 + u * kWG < je) q[u].load(jm, static_cast<size_t>(j0 + u * kWG));
  for (int js = j0; js < je; js += D * kWG) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      const int jj = js + u * kWG;
      if (jj < je) {
        float4 rec[REC];
        predict_raw<PREC>(q[u], ti, rec);
        if (jj + D * kWG < je) q[u].load(jm, static_cast<size_t>(jj + D * kWG));
        MaskedRun<PREC, NBL, false, true> run;
        run.start();
        run.step(n.st, n.ts, n.t, rec, jj, n.slot, eps2, n.h2, n.ebest, n.eslot, nb_work, a.nb_slot);
        run.finish(n.ts);
        fold(n.ts, n.t);
      }
    }
  }

  double bestd;
  int bslot;
  n.lane_sum(red, tid, 0, 1, bestd, bslot);
  if (tid == 0) store_part(a.part, a.nn_slot, static_cast<size_t>(blockIdx.y) * a.ni, n.t, bestd, bslot);
}

// Clear n counters (a new or regrown nb_work buffer).
__global__ __launch_bounds__(256) void zero_kernel(int n, int *__restrict__ p) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k < n) p[k] = 0;
}

// --------------------------------------------------------------- reduction

// 2^log2I i-particles per workgroup (split_sum, then finish_out): the float64
// sum over the j-splits in a fixed order, nearest-neighbour minimum,
// neighbour-list finalisation.  Bound by the latency of its loads for small
// blocks and by HBM for large ones: against one or 64 lanes per i-particle
// over component arrays, 512 splits of 100 i-particles take 7.1 us (15.3),
// of 3000 27 us (51), 8 splits of 2^20 226 us (260).  The partials of
// position i belong to row iperm[i] when iperm is given (the spatially
// ordered kernel writes them in sorted order), else to row i.
// status[kStatusFlags] bit 0: a non-finite output; bit 1: a neighbour list
// overflowed (those i-particles are queued in ovf_list for nb_exact_kernel).
__global__ __launch_bounds__(256) void reduce_kernel(
    int nsplit, int ni, int log2I, const int *__restrict__ iperm, const double *__restrict__ part,
    const int *__restrict__ nn_slot, const int *__restrict__ jindex, int *__restrict__ nb_count,
    int *__restrict__ nb_slot, int nbl, double *__restrict__ acc,
    double *__restrict__ jerk, double *__restrict__ pot, int *__restrict__ nnb,
    double *__restrict__ r2nn, int *__restrict__ status, int *__restrict__ ovf_list,
    int *__restrict__ nb_work) {
  __shared__ SplitShared sh;
  const int tid = threadIdx.x;
  const int i0 = static_cast<int>(blockIdx.x) << log2I;
  double2 v;
  int bslot;
  split_sum(nsplit, log2I, ni - i0, part, nn_slot, static_cast<size_t>(i0), static_cast<size_t>(ni), sh, v, bslot);
  if ((tid & ~63) >= (4 << log2I)) return; // whole waves without a row
  const int i = i0 + (tid >> 2);
  const bool valid = tid < (4 << log2I) && i < ni;
  const int row = valid ? (iperm ? iperm[i] : i) : 0;
  const int fl = finish_out(v, bslot, valid, row, jindex, nb_count, nb_slot, nbl != 0, acc, jerk, pot, nnb, r2nn,
                            status, ovf_list, nullptr, 0, nb_work);
  if (fl) atomicOr(status + kStatusFlags, fl);
}

// --------------------------------------------- neighbour-list overflow

// One workgroup per queued i-particle (grid-strided over the queue): its
// list rebuilt by exact_list over slots 0 .. nj - 1 of the predicted records.
template <int PREC>
__global__ __launch_bounds__(kWG) void nb_exact_kernel(ForceArgs a, const int *__restrict__ jindex,
                                                        const int *__restrict__ status,
                                                        const int *__restrict__ ovf_list) {
  constexpr int REC = rec4<PREC>();
  __shared__ unsigned s_cnt;
  __shared__ int s_keep[kNbMax];
  const float4 *jp = static_cast<const float4 *>(a.jpred);
  auto rec_of = [jp](int js, float4 *) { return jp + static_cast<size_t>(js) * REC; };
  const int novf = status[kStatusOverflowCount];
  for (int q = blockIdx.x; q < novf; q += gridDim.x) {
    const int i = ovf_list[q];
    IState<PREC> st;
    int slot;
    real_t<PREC> h2;
    load_i<PREC>(st, a, i, true, slot, h2);
    exact_list<PREC>(st, slot, h2, 0, a.nj, jindex, rec_of, a.nb_slot + static_cast<size_t>(i) * kNbMax,
                     a.nb_count + i, s_cnt, s_keep);
  }
}

// The same for a calculation of force_fused, which kept no predicted
// records: each record is predicted again from the j-memory exactly as in
// force_fused.
template <int PREC>
__global__ __launch_bounds__(kWG) void nb_exact_fused_kernel(ForceArgs a, JMem jm, double ti,
                                                              const int *__restrict__ status,
                                                              const int *__restrict__ ovf_list) {
  __shared__ unsigned s_cnt;
  __shared__ int s_keep[kNbMax];
  auto rec_of = [jm, ti](int js, float4 *buf) -> const float4 * {
    predict_record<PREC>(jm, static_cast<size_t>(js), ti, buf);
    return buf;
  };
  const int novf = status[kStatusOverflowCount];
  for (int q = blockIdx.x; q < novf; q += gridDim.x) {
    const int i = ovf_list[q];
    IState<PREC> st;
    int slot;
    real_t<PREC> h2;
    load_i<PREC>(st, a, i, true, slot, h2);
    exact_list<PREC>(st, slot, h2, 0, a.nj, jm.index, rec_of, a.nb_slot + static_cast<size_t>(i) * kNbMax,
                     a.nb_count + i, s_cnt, s_keep);
  }
}

// ------------------------------------------------------------ j-memory I/O

// Component c of a staged record (kRecDoubles = 16 doubles: t, m, x, v, a2,
// j6, index, pad) to slot k of the j-memory.
__device__ __forceinline__ void scatter_component(const JMem &jm, size_t k, int c, double v) {
  if (c == 0) jm.t[k] = v;
  else if (c == 1) jm.m[k] = v;
  else if (c < 5) jm.x[(c - 2) * jm.cap + k] = v;
  else if (c < 8) jm.v[(c - 5) * jm.cap + k] = v;
  else if (c < 11) jm.a2[(c - 8) * jm.cap + k] = v;
  else if (c < 14) jm.j6[(c - 11) * jm.cap + k] = v;
  else if (c == 14) jm.index[k] = static_cast<int>(v);
}

// Sixteen lanes per record, so that a record is one contiguous read: bound
// by the latency of that read and the scattered stores.
__device__ __forceinline__ void scatter_records(int block, int nd, const int *__restrict__ slots,
                                                const double *__restrict__ rec, const JMem &jm) {
  const int q = block * 16 + (threadIdx.x >> 4), c = threadIdx.x & 15;
  if (q >= nd) return;
  const size_t k = static_cast<size_t>(slots[q]);
  if (k < jm.cap) scatter_component(jm, k, c, rec[16 * static_cast<size_t>(q) + c]);
}

__global__ __launch_bounds__(256) void scatter_kernel(int nd, const int *__restrict__ slots,
                                                      const double *__restrict__ rec, JMem jm) {
  scatter_records(blockIdx.x, nd, slots, rec, jm);
}

// Inputs of a small host call from pinned host memory: the first workgroups
// scatter the nd staged records (their slots follow them), the others copy
// the i-block.
__global__ __launch_bounds__(256) void stage_in_kernel(int nd, const double *__restrict__ rec, JMem jm,
                                                       int rec_blocks, int n16, const double2 *__restrict__ src,
                                                       double2 *__restrict__ dst) {
  if (static_cast<int>(blockIdx.x) < rec_blocks) {
    scatter_records(blockIdx.x, nd, reinterpret_cast<const int *>(rec + 16 * static_cast<size_t>(nd)), rec, jm);
    return;
  }
  const int k = (static_cast<int>(blockIdx.x) - rec_blocks) * 256 + threadIdx.x;
  if (k < n16) dst[k] = src[k];
}

// One wave per row (see launch_export_lists).
__global__ __launch_bounds__(64) void export_lists_kernel(int n, const int *__restrict__ status,
                                                          const int *__restrict__ nb_count,
                                                          const int *__restrict__ nb_slot, int *__restrict__ out) {
  const int i = blockIdx.x, lane = threadIdx.x;
  if (i == 0 && lane < kStatusWords) out[lane] = status[lane];
  const int cnt = nb_count[i];
  if (lane == 0) out[kStatusWords + i] = cnt;
  int *lst = out + kStatusWords + n + static_cast<size_t>(i) * kNbMax;
  for (int k = lane; k < min(cnt, kNbMax); k += 64) lst[k] = nb_slot[static_cast<size_t>(i) * kNbMax + k];
}

__global__ __launch_bounds__(256) void load_kernel(int nj, const double *__restrict__ t,
                                                   const double *__restrict__ m,
                                                   const int *__restrict__ index,
                                                   const double *__restrict__ x,
                                                   const double *__restrict__ v,
                                                   const double *__restrict__ a2,
                                                   const double *__restrict__ j6, JMem jm) {
  const int k = blockIdx.x * 256 + threadIdx.x;
  if (k >= nj) return;
  jm.t[k] = t[k];
  jm.m[k] = m[k];
  jm.index[k] = index[k];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    jm.x[d * jm.cap + k] = x[3 * static_cast<size_t>(k) + d];
    jm.v[d * jm.cap + k] = v[3 * static_cast<size_t>(k) + d];
    jm.a2[d * jm.cap + k] = a2[3 * static_cast<size_t>(k) + d];
    jm.j6[d * jm.cap + k] = j6[3 * static_cast<size_t>(k) + d];
  }
}

// ------------------------------------------------------ static scratch

// Work buffers of g6mi_calc_device_noalloc (callers that cannot allocate):
// one array of G6MI_NOALLOC_SCRATCH_BYTES in each GPU's memory, held from
// the library's load on that GPU until the process ends.  In host code the
// name stands for no device address: only the address that
// hipGetSymbolAddress returns for the current device is used.
static __device__ __align__(256) unsigned char scratch[G6MI_NOALLOC_SCRATCH_BYTES];

hipError_t scratch_region(int device, void **ptr, size_t *bytes) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void *addr[kMaxDevices] = {};
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[device]) {
    // once per device, with that device current
    int cur = -1;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return e;
    if (cur != device) return hipErrorInvalidDevice;
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[device] = p;
  }
  *ptr = addr[device];
  *bytes = sizeof(scratch);
  return hipSuccess;
}

// ---------------------------------------------------------------- launchers

// Workgroups of the reduction from which on more lanes per i-particle gain
// nothing (about four per compute unit).
constexpr int kReduceFill = 1024;

static inline unsigned blocks_for(long n) { return static_cast<unsigned>((n + 255) / 256); }

hipError_t launch_predict(int prec, int nj, double ti, const JMem &jm, void *out,
                          int *nb_count, int ni, int *status, hipStream_t s) {
  long n = nj > ni ? nj : ni;
  if (n < kStatusWords) n = kStatusWords;
  if (n <= 0) return hipSuccess;
  const dim3 grid(blocks_for(n)), block(256);
  switch (prec) {
  case G6MI_PREC_FP32:
    hipLaunchKernelGGL(predict_kernel<G6MI_PREC_FP32>, grid, block, 0, s, nj, ti, jm, out, nb_count,
                       ni, status);
    break;
  case G6MI_PREC_DS:
    hipLaunchKernelGGL(predict_kernel<G6MI_PREC_DS>, grid, block, 0, s, nj, ti, jm, out, nb_count,
                       ni, status);
    break;
  default:
    hipLaunchKernelGGL(predict_kernel<G6MI_PREC_FP64>, grid, block, 0, s, nj, ti, jm, out, nb_count,
                       ni, status);
  }
  return hipGetLastError();
}

template <int PREC>
static void launch_force_prec(bool nbl, const ForceArgs &a, dim3 grid, hipStream_t s) {
  if (a.one) {
    if (nbl)
      hipLaunchKernelGGL((force_one<PREC, true>), grid, dim3(kWG), 0, s, a);
    else
      hipLaunchKernelGGL((force_one<PREC, false>), grid, dim3(kWG), 0, s, a);
  } else if (a.ipw == 2 * kWG) {
    if (nbl)
      hipLaunchKernelGGL((force_wide<PREC, true>), grid, dim3(kWG), 0, s, a);
    else
      hipLaunchKernelGGL((force_wide<PREC, false>), grid, dim3(kWG), 0, s, a);
  } else if (nbl)
    hipLaunchKernelGGL((force_kernel<PREC, true>), grid, dim3(kWG), 0, s, a, PieceArgs{});
  else
    hipLaunchKernelGGL((force_kernel<PREC, false>), grid, dim3(kWG), 0, s, a, PieceArgs{});
}

hipError_t launch_force(int prec, bool nbl, const ForceArgs &a, int nsplit, hipStream_t s) {
  if (a.ni <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>((a.ni + a.ipw - 1) / a.ipw), static_cast<unsigned>(nsplit));
  switch (prec) {
  case G6MI_PREC_FP32: launch_force_prec<G6MI_PREC_FP32>(nbl, a, grid, s); break;
  case G6MI_PREC_DS: launch_force_prec<G6MI_PREC_DS>(nbl, a, grid, s); break;
  default: launch_force_prec<G6MI_PREC_FP64>(nbl, a, grid, s);
  }
  return hipGetLastError();
}

template <int PREC, int S>
static void launch_pieces_sets(bool nbl, const ForceArgs &a, const JMem &jm, double ti, const PieceArgs &pc,
                               void *jpred, int *status, int npieces, hipStream_t s) {
  const unsigned nib = static_cast<unsigned>((a.ni + a.ipw - 1) / a.ipw);
  const unsigned ntiles = static_cast<unsigned>((a.nj + kTile - 1) / kTile);
  hipLaunchKernelGGL((piece_min_kernel<PREC, S>), dim3(nib, ntiles), dim3(S * kWG), 0, s, a, jm, ti, pc,
                     static_cast<float4 *>(jpred), status);
  const dim3 grid(nib, static_cast<unsigned>(npieces));
  if constexpr (S == 1) {
    if (nbl)
      hipLaunchKernelGGL((force_kernel<PREC, true, true>), grid, dim3(kWG), 0, s, a, pc);
    else
      hipLaunchKernelGGL((force_kernel<PREC, false, true>), grid, dim3(kWG), 0, s, a, pc);
  } else if (nbl)
    hipLaunchKernelGGL((force_piece<PREC, true, S>), grid, dim3(S * kWG), 0, s, a, pc);
  else
    hipLaunchKernelGGL((force_piece<PREC, false, S>), grid, dim3(S * kWG), 0, s, a, pc);
}

// pc.sets: one, two, or four where a lane's chain has four groups in a tile
// (64 i-particles per workgroup and more).
template <int PREC>
static void launch_pieces_prec(bool nbl, const ForceArgs &a, const JMem &jm, double ti, const PieceArgs &pc,
                               void *jpred, int *status, int npieces, hipStream_t s) {
  if (pc.sets == 4 && a.ipw * 4 >= kWG)
    launch_pieces_sets<PREC, 4>(nbl, a, jm, ti, pc, jpred, status, npieces, s);
  else if (pc.sets > 1)
    launch_pieces_sets<PREC, 2>(nbl, a, jm, ti, pc, jpred, status, npieces, s);
  else
    launch_pieces_sets<PREC, 1>(nbl, a, jm, ti, pc, jpred, status, npieces, s);
}

hipError_t launch_force_pieces(int prec, bool nbl, const ForceArgs &a, const JMem &jm, double ti,
                               const PieceArgs &pc, void *jpred, int *status, int npieces, hipStream_t s) {
  if (a.ni <= 0 || a.nj <= 0 || a.ipw > kWG || a.ipw < 32 || pc.per < 1 || pc.vper < pc.per || !pc.least)
    return hipErrorInvalidValue;
  if (prec == G6MI_PREC_DS) launch_pieces_prec<G6MI_PREC_DS>(nbl, a, jm, ti, pc, jpred, status, npieces, s);
  else if (prec == G6MI_PREC_FP32) launch_pieces_prec<G6MI_PREC_FP32>(nbl, a, jm, ti, pc, jpred, status, npieces, s);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

template <int PREC>
static void launch_fused_prec(bool nbl, const ForceArgs &a, const JMem &jm, double ti, int *nb_work, int *status,
                              dim3 grid, hipStream_t s) {
  if (a.ipw == 1) {
    if (nbl)
      hipLaunchKernelGGL((force_fused_one<PREC, true>), grid, dim3(kWG), 0, s, a, jm, ti, nb_work, status);
    else
      hipLaunchKernelGGL((force_fused_one<PREC, false>), grid, dim3(kWG), 0, s, a, jm, ti, nb_work, status);
    return;
  }
  if (nbl)
    hipLaunchKernelGGL((force_fused<PREC, true>), grid, dim3(kWG), 0, s, a, jm, ti, nb_work, status);
  else
    hipLaunchKernelGGL((force_fused<PREC, false>), grid, dim3(kWG), 0, s, a, jm, ti, nb_work, status);
}

hipError_t launch_force_fused(int prec, bool nbl, const ForceArgs &a, const JMem &jm, double ti, int *nb_work,
                              int *status, int nsplit, hipStream_t s) {
  if (a.ni <= 0 || a.ipw > kWG) return hipErrorInvalidValue;
  const dim3 grid(static_cast<unsigned>((a.ni + a.ipw - 1) / a.ipw), static_cast<unsigned>(nsplit));
  switch (prec) {
  case G6MI_PREC_FP32: launch_fused_prec<G6MI_PREC_FP32>(nbl, a, jm, ti, nb_work, status, grid, s); break;
  case G6MI_PREC_DS: launch_fused_prec<G6MI_PREC_DS>(nbl, a, jm, ti, nb_work, status, grid, s); break;
  default: launch_fused_prec<G6MI_PREC_FP64>(nbl, a, jm, ti, nb_work, status, grid, s);
  }
  return hipGetLastError();
}

hipError_t launch_zero(int n, int *p, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(zero_kernel, dim3(blocks_for(n)), dim3(256), 0, s, n, p);
  return hipGetLastError();
}

hipError_t launch_reduce(int nsplit, int ni, const int *iperm, const double *part,
                         const int *nn_slot, const int *jindex, int *nb_count, int *nb_slot,
                         bool nbl, double *acc, double *jerk, double *pot, int *nnb,
                         double *r2nn, int *status, int *ovf_list, hipStream_t s, int *nb_work) {
  if (ni <= 0) return hipSuccess;
  const int l = split_log2rows(nsplit, ni, kReduceFill);
  hipLaunchKernelGGL(reduce_kernel, dim3(static_cast<unsigned>((ni + (1LL << l) - 1) >> l)), dim3(256), 0, s, nsplit,
                     ni, l, iperm, part, nn_slot, jindex, nb_count, nb_slot, nbl ? 1 : 0, acc, jerk, pot, nnb, r2nn,
                     status, ovf_list, nb_work);
  return hipGetLastError();
}

template <int PREC>
static void launch_exact_prec(const ForceArgs &a, const int *jindex, const int *status,
                              const int *ovf_list, int ngroups, hipStream_t s) {
  hipLaunchKernelGGL(nb_exact_kernel<PREC>, dim3(ngroups), dim3(kWG), 0, s, a, jindex,
                     status, ovf_list);
}

hipError_t launch_nb_exact(int prec, const ForceArgs &a, const int *jindex, const int *status,
                           const int *ovf_list, int novf, hipStream_t s) {
  if (novf <= 0) return hipSuccess;
  const int ngroups = novf < 1024 ? novf : 1024;
  switch (prec) {
  case G6MI_PREC_FP32: launch_exact_prec<G6MI_PREC_FP32>(a, jindex, status, ovf_list, ngroups, s); break;
  case G6MI_PREC_DS: launch_exact_prec<G6MI_PREC_DS>(a, jindex, status, ovf_list, ngroups, s); break;
  default: launch_exact_prec<G6MI_PREC_FP64>(a, jindex, status, ovf_list, ngroups, s);
  }
  return hipGetLastError();
}

hipError_t launch_nb_exact_fused(int prec, const ForceArgs &a, const JMem &jm, double ti, const int *status,
                                 const int *ovf_list, int novf, hipStream_t s) {
  if (novf <= 0) return hipSuccess;
  const dim3 grid(static_cast<unsigned>(novf < 1024 ? novf : 1024));
  switch (prec) {
  case G6MI_PREC_FP32:
    hipLaunchKernelGGL(nb_exact_fused_kernel<G6MI_PREC_FP32>, grid, dim3(kWG), 0, s, a, jm, ti, status, ovf_list);
    break;
  case G6MI_PREC_DS:
    hipLaunchKernelGGL(nb_exact_fused_kernel<G6MI_PREC_DS>, grid, dim3(kWG), 0, s, a, jm, ti, status, ovf_list);
    break;
  default:
    hipLaunchKernelGGL(nb_exact_fused_kernel<G6MI_PREC_FP64>, grid, dim3(kWG), 0, s, a, jm, ti, status, ovf_list);
  }
  return hipGetLastError();
}

hipError_t launch_scatter(int nd, const int *slots, const double *rec, const JMem &jm,
                          hipStream_t s) {
  if (nd <= 0) return hipSuccess;
  hipLaunchKernelGGL(scatter_kernel, dim3(blocks_for(16L * nd)), dim3(256), 0, s, nd, slots, rec, jm);
  return hipGetLastError();
}

hipError_t launch_stage_in(int nd, const double *rec, const JMem &jm, size_t ibytes, const void *i_src,
                           void *i_dst, hipStream_t s) {
  const int rec_blocks = static_cast<int>(blocks_for(16L * nd)), n16 = static_cast<int>(ibytes / 16);
  hipLaunchKernelGGL(stage_in_kernel, dim3(static_cast<unsigned>(rec_blocks) + blocks_for(n16)), dim3(256), 0, s,
                     nd, rec, jm, rec_blocks, n16, static_cast<const double2 *>(i_src),
                     static_cast<double2 *>(i_dst));
  return hipGetLastError();
}

hipError_t launch_export_lists(int n, const int *status, const int *nb_count, const int *nb_slot, int *out,
                               hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(export_lists_kernel, dim3(static_cast<unsigned>(n)), dim3(64), 0, s, n, status, nb_count,
                     nb_slot, out);
  return hipGetLastError();
}

hipError_t launch_load(int nj, const double *t, const double *m, const int *index,
                       const double *x, const double *v, const double *a2, const double *j6,
                       const JMem &jm, hipStream_t s) {
  if (nj <= 0) return hipSuccess;
  hipLaunchKernelGGL(load_kernel, dim3(blocks_for(nj)), dim3(256), 0, s, nj, t, m, index, x, v,
                     a2, j6, jm);
  return hipGetLastError();
}

} // namespace g6mi
