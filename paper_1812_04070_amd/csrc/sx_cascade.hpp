// Windowed relaxation with workgroup-local cascades: the light phases of BFS
// and SSSP on sparse graphs of high diameter, one step over a (virtual) grid;
// k_cascade (sx_cascade.hip) runs a step per launch, k_batch (sx_traverse.hip)
// a step per team barrier.
//
// One launch per level pays a fixed cost (launch, run-state line, record
// prefix, appends: ~12 us) for a frontier of a thousand vertices, thousands of
// times over.  Here a step advances the run by a window of distances [lo, B)
// instead: each workgroup takes a stretch of the listed vertices, and a vertex
// it improves to a distance below B is expanded by the same workgroup from a
// queue in LDS, round after round, until its queue is empty.  Vertices
// improved to B or beyond go to the next step's list.  Within a step
// workgroups do not wait for each other, so a vertex near the border of two
// stretches may first get a distance that is too long; whoever lowers it
// later expands it again (a BFS depth is lowered by the same atomic minimum
// as an SSSP distance, with arcs of length 1; unvisited is 0xFFFFFFFF).  A
// step ends with every arc out of a vertex below B relaxed with that
// vertex's current value, so the distances below B are final, as after a
// bucket of delta-stepping (Section 3.3 of the paper), and the run ends when
// the list is empty: the result does not depend on the window.
//
// Bound: a round's chain of an LDS queue read, the neighbour's row offsets
// beside the atomic minimum, its first four ids (read for every neighbour, so
// that the queue entry carries them, in one load without a branch per id, which
// the compiler would put behind the minimum), and
// the append; and the instructions around it.  So an entry has four lanes, an
// arc each: with four arcs to a lane, whose appends follow one another, a
// round took 3.5 us against 1.2.  2048^2 grid BFS: 49.7 ms in levels, 5.1 here
// (ids read when the entry is expanded 5.2; workgroups of 64 / 128 / 512 threads 6.0 / 5.3 /
// 6.0; 16 or 32 listed vertices a workgroup 5.5 / 5.9; 16, 32, 128 levels a
// step 7.1 / 5.9 / 5.3); 4096^2 grid SSSP 167 -> 21.6 (ids read when the entry is
// expanded 24.3; window 4 / 6 / 20 mean weights: 32 / 27 / 34).  Reading an entry's
// distance again before expanding it saved a quarter of the arcs and no time.
// In a batch (a step per team barrier), 48 queries over 8 R-MAT graphs of
// scale 12-17 and grids of side 128 and 512: 20.0 -> 3.8 ms.
//
// An improved vertex that finds its workgroup's queue full goes to the next
// list too, and so does a vertex of kCasHub arcs or more, whose
// row the next step spreads over all workgroups.  A vertex enters a list
// once per step (stamp), so a list holds at most n entries; a listed vertex
// is expanded from its current value when that lies below B, whatever put it
// there.
//
// A list that outgrows the cascade (cas_outgrown) goes back to the level phases
// (cas_way_back): it has met a part of the graph of low diameter, where a
// window of unsynchronised relaxations does most of its work many times over.
// Random graph of 3 M vertices and 6 arcs each behind a path of 20: BFS in
// phases alone 0.92 ms, in the cascade to its end 4.9, with the way back 0.86;
// SSSP of 8 mean weights a bucket 3.0 / 10.8 / 2.7.  Behind a path of 600: BFS 13.6 /
// 9.4 / 2.0, SSSP 21.1 / 16.2 / 6.0.
#pragma once

#include "sx_frontier.hpp"

namespace sx {

constexpr int kCasBlock = 256;         // threads per workgroup of k_cascade
constexpr int kCasPer = 8;             // listed vertices that are worth a workgroup
constexpr int kCasQ = 256;             // LDS queue entries (two queues)
constexpr int kCasFar = 512;           // listed vertices gathered in LDS
constexpr int kCasLane = 16;           // arcs up to which four lanes walk a row
constexpr int kCasHub = 4096;          // and from which the grid does
constexpr unsigned kCasMaxList = 1u << 16;  // longer lists go back to the phases
constexpr int kCasJump = 2048;         // and lists that jump beyond 4 times the last by this
constexpr int kCasHold = 16;           // ... for this many iterations at least

typedef int Arcs4 __attribute__((ext_vector_type(4), aligned(4)));

template <bool kWeighted>
struct LdsCas {
  uint4 q[2][kCasQ];                   // vertex, distance, row begin, row end
  int4 qi[2][kCasQ];                   // its first four neighbours
  uint4 qw[2][kWeighted ? kCasQ : 1];  // and their arcs' weights
  int far[kCasFar];
  unsigned in[64];                     // run state and control words
  unsigned qn[3], fn, base, low, err;
  unsigned long long edges;
};

// One LDS counter position per lane with `on` (the lanes that call agree on
// the counter).
SX_DEV unsigned cas_append(bool on, unsigned *count) {
  const uint64_t mk = ballot(on);
  const int lead = mk ? __ffsll((long long)mk) - 1 : 0;
  unsigned base = 0;
  if (lane_id() == lead) base = atomicAdd(count, (unsigned)__popcll(mk));
  return (unsigned)__builtin_amdgcn_readlane((int)base, lead) + lane_prefix(mk);
}

// Empty queues (all threads; a barrier follows in the caller).
template <bool kWeighted>
SX_DEV void cas_begin(LdsCas<kWeighted> &S) {
  if (threadIdx.x == 64) {
    S.qn[0] = S.qn[1] = S.qn[2] = S.fn = S.err = 0u;
    S.low = 0xFFFFFFFFu;
    S.edges = 0ull;
  }
}

// Levels of a finished BFS (the deepest depth + 1) into the iteration count.
template <int kThreads>
SX_DEV void cas_levels(const VGrid &vg, const TravArgs &a) {
  const unsigned *dist = (const unsigned *)a.state_i;
  unsigned top = 0;
  for (long long v = (long long)vg.bid * kThreads + threadIdx.x; v < a.g.n; v += (long long)vg.nb * kThreads) {
    const unsigned d = dist[v] + 1u;   // unvisited: 0
    top = d > top ? d : top;
  }
  top = ~wave_min_u(~top);
  unsigned *levels = &a.w.ctrl->stats.v[6];
  if (lane_id() == 0 && top > load_relaxed(levels)) __hip_atomic_fetch_max(levels, top, __ATOMIC_RELAXED, SX_AG);
}

// BFS: levels of the next step, fewer while the lists grow, more while they
// do not.
SX_DEV unsigned cas_window(unsigned window, unsigned cnt, unsigned before, unsigned most) {
  if (cnt > before + before / 2 + 64u) return window > 1 ? window / 2 : 1u;
  return window * 2 < most ? window * 2 : most;
}

// Eight times the mean weight, of 512 arcs spread over the graph: an SSSP
// step's window (a whole wavefront; the same in all).
SX_DEV unsigned cas_mean8(const TravArgs &a) {
  long long sum = 0;
  for (int k = 0; k < 8; ++k) sum += a.g.w[a.g.m * (lane_id() * 8 + k) / 512];
  const unsigned long long mean8 = (unsigned long long)wave_sum_ll(sum) / 64;
  return mean8 < 1 ? 1u : mean8 > 0x7FFFFFFFull ? 0x7FFFFFFFu : (unsigned)mean8;
}

// Whether a list is the phases' business: long, or many times the one before
// (meshes' lists grow by half a step at most; a blob's first vertices overflow
// one workgroup's queue, and the next step would walk all of it unsynchronised).
SX_DEV bool cas_outgrown(unsigned cnt, unsigned before) {
  return cnt > kCasMaxList || cnt > 4u * before + (unsigned)kCasJump;
}

// One step: the `cnt` vertices listed in reg_s[par] and the `hubs` in
// reg_m[par], up to distance B.  Ctrl::aux, by step number s % 3 (`nxt`: of
// s + 1): words 8.. the list's length, 12.. its smallest distance, 24.. hubs
// listed.  `tag`: a
// stamp no other step and no iteration of the run uses.  The graph has at least
// four arcs.
template <bool kWeighted, int kThreads>
SX_DEV void cascade_step(const VGrid &vg, const TravArgs &a, LdsCas<kWeighted> &S, unsigned cnt, unsigned hubs,
                         unsigned B, unsigned par, unsigned nxt, int tag) {
  const unsigned want = (cnt + kCasPer - 1) / kCasPer;
  const unsigned act = want < vg.nb ? want : vg.nb;
  if (vg.bid >= act && hubs == 0) return;
  const int t = threadIdx.x, n = a.g.n;
  Ctrl *C = a.w.ctrl;
  unsigned *dist = (unsigned *)a.state_i;
  const unsigned per = act ? (cnt + act - 1) / act : 0u;
  const unsigned lo = vg.bid * per < cnt ? vg.bid * per : cnt, hi = lo + per < cnt ? lo + per : cnt;
  const int *list = a.w.reg_s[par];
  int *olist = a.w.reg_s[par ^ 1u];
  const int *off = a.g.off, *idx = a.g.idx;
  const unsigned *wt = a.g.w;
  unsigned low = 0xFFFFFFFFu, err = 0, edges = 0, ents = 0;
  // u (a row of `len` arcs) into the next launch's list; whole wavefront
  auto list_append = [&](bool on, int u, unsigned d, int len) {
    if (!ballot(on)) return;
    low = on && d < low ? d : low;   // also of a vertex that is listed already
    on = on && atomic_exch_i32(&a.w.stamp[u], tag) != tag;
    const bool hub = on && len >= kCasHub;
    if (hub) a.w.reg_m[par ^ 1u][atomic_add_u32(&C->aux.v[24 + nxt], 1u)] = u;
    on = on && !hub;
    const unsigned pos = cas_append(on, &S.fn);
    if (on) {
      if (pos < (unsigned)kCasFar) S.far[pos] = u;
      else olist[atomic_add_u32(&C->aux.v[8 + nxt], 1u)] = u;
    }
  };
  // four ids from a row's first arc on, in one load; the arrays' last rows
  // read the last four (an arc j of such a row sits at j + tail(row))
  const int last4 = (int)a.g.m - 4;
  auto tail = [&](int rb) { return rb > last4 ? rb - last4 : 0; };
  auto first_arcs = [&](int rb, int4 &ids, uint4 &w) {
    const int e = rb > last4 ? last4 : rb;
    const Arcs4 x = *(const Arcs4 *)(idx + e);
    ids = make_int4(x[0], x[1], x[2], x[3]);
    if constexpr (kWeighted) {
      const Arcs4 y = *(const Arcs4 *)(wt + e);
      w = make_uint4((unsigned)y[0], (unsigned)y[1], (unsigned)y[2], (unsigned)y[3]);
    }
  };
  // a vertex to expand from d into queue `buf`; what does not fit, and hubs,
  // to the next list; whole wavefront
  auto enqueue = [&](bool near, bool far, int u, unsigned d, int rb, int re, const int4 &ids, const uint4 &w,
                     int buf, unsigned *count) {
    const bool hub = near && re - rb >= kCasHub;
    near = near && !hub;
    bool full = false;
    if (ballot(near)) {
      const unsigned pos = cas_append(near, count);
      if (near && pos < (unsigned)kCasQ) {
        S.q[buf][pos] = make_uint4((unsigned)u, d, (unsigned)rb, (unsigned)re);
        S.qi[buf][pos] = ids;
        if constexpr (kWeighted) S.qw[buf][pos] = w;
      }
      full = near && pos >= (unsigned)kCasQ;
    }
    list_append(far || hub || full, u, d, re - rb);
  };
  // one arc per lane, to u at distance d + w: the offsets of u's row and the
  // minimum are in flight together, then the row's first arcs
  auto relax = [&](bool ok, int u, unsigned d, unsigned w, int buf, unsigned *count) {
    const unsigned nd = d + w;
    const bool bad = kWeighted && (nd < d || nd == 0xFFFFFFFFu);
    bool on = ok && (unsigned)u < (unsigned)n;
    if (on && bad) err = SX_ERR_OVERFLOW;
    on = on && !bad;
    bool better = false;
    int rb = 0, re = 0;
    int4 ids;
    uint4 ws;
    if (on) {
      edges += 1u;
      rb = off[u];
      re = off[u + 1];
      const unsigned old = atomic_min_u32(&dist[u], nd);
      first_arcs(rb, ids, ws);
      better = nd < old;
    }
    if (ballot(better)) enqueue(better && nd < B, better && nd >= B, u, nd, rb, re, ids, ws, buf, count);
  };
  unsigned round = 0;
  // rounds until the queue is empty: queue round & 1 is read, the other one
  // filled; its counter is round % 3.  A grid of workgroups stops at a round that
  // overflows the queue: of its 64 listed vertices at most no mesh makes so many,
  // and the workgroup would walk a blob alone until the window's end (the step
  // that meets one of 3 M vertices 387 us; with it the BFS above 1.24 ms).  A
  // team's lists are longer.
  constexpr bool kStopFull = kThreads == kCasBlock;
  auto drain = [&]() {
    // (0 and too many in one comparison; the first round may be any number)
    unsigned most = 0xFFFFFFFFu;
    for (;; ++round, most = kStopFull ? (unsigned)kCasQ : most) {
      const int cur = (int)(round & 1u), nx = cur ^ 1;
      const unsigned filled = S.qn[round % 3];
      if (filled - 1u >= most) break;
      const unsigned have = filled < (unsigned)kCasQ ? filled : (unsigned)kCasQ;
      unsigned *count = &S.qn[(round + 1) % 3];
      ents += have;
      if (t == 0) S.qn[(round + 2) % 3] = 0u;
      // four lanes an entry, an arc each
      const int part = t & 3;
      for (unsigned i0 = (unsigned)wave_in_wg() * 16u; i0 < have; i0 += kThreads / 4) {
        const unsigned i = i0 + (unsigned)lane_id() / 4u;
        uint4 x = make_uint4(0u, 0u, 0u, 0u);
        int u = 0;
        unsigned w = 1u;
        if (i < have) {
          x = S.q[cur][i];
          const int at = (part + tail((int)x.z)) & 3;
          u = ((const int *)&S.qi[cur][i])[at];
          if constexpr (kWeighted) w = ((const unsigned *)&S.qw[cur][i])[at];
        }
        const int len = (int)(x.w - x.z);
        relax(len <= kCasLane && part < len, u, x.y, w, nx, count);
        if (ballot(len > 4) == 0) continue;
        for (int j = 4; ballot(len <= kCasLane && j < len); j += 4) {
          const bool ok = len <= kCasLane && j + part < len;
          const int e = ok ? (int)x.z + j + part : 0;
          relax(ok, ok ? idx[e] : 0, x.y, kWeighted && ok ? wt[e] : 1u, nx, count);
        }
        for (uint64_t rows = ballot(part == 0 && len > kCasLane); rows; rows &= rows - 1) {
          const int src = __ffsll((long long)rows) - 1;
          const int rb = __shfl((int)x.z, src), re = __shfl((int)x.w, src);
          const unsigned d = __shfl(x.y, src);
          for (unsigned e0 = (unsigned)rb; e0 < (unsigned)re; e0 += 64u) {
            const unsigned e = e0 + (unsigned)lane_id();
            const bool ok = e < (unsigned)re;
            relax(ok, ok ? idx[e] : 0, d, kWeighted && ok ? wt[e] : 1u, nx, count);
          }
        }
      }
      __syncthreads();
    }
  };
  // hubs: every workgroup takes its part of the row.  Read at B or beyond: the
  // first workgroup carries it; a smaller value read by some workgroups only
  // was set in this launch, and whoever set it listed the hub again.
  for (unsigned h = 0; h < hubs; ++h) {
    const int v = a.w.reg_m[par][h];
    if ((unsigned)v >= (unsigned)n) continue;
    const unsigned d = load_relaxed(&dist[v]);
    const int rb = off[v], re = off[v + 1];
    if (d >= B) {
      if (vg.bid == 0) list_append(t == 0, v, d, re - rb);
      continue;
    }
    for (long long e0 = rb + (long long)vg.bid * kThreads; e0 < re; e0 += (long long)vg.nb * kThreads) {
      const long long e = e0 + t;
      const bool ok = e < re;
      relax(ok, ok ? idx[e] : 0, d, kWeighted && ok ? wt[e] : 1u, (int)(round & 1u), &S.qn[round % 3]);
    }
  }
  // the stretch of the list: below B into the queue, the others carried
  // (at least once: hubs may have filled the queue)
  for (unsigned b0 = lo; b0 < hi || b0 == lo; b0 += kThreads) {
    const unsigned i = b0 + (unsigned)t;
    const int v = i < hi ? list[i] : -1;
    const bool ok = (unsigned)v < (unsigned)n;
    if (ballot(ok)) {
      const unsigned d = ok ? dist[v] : 0u;
      const int rb = ok ? off[v] : 0, re = ok ? off[v + 1] : 0;
      int4 ids;
      uint4 ws;
      first_arcs(rb, ids, ws);
      enqueue(ok && d < B, ok && d >= B, v, d, rb, re, ids, ws, (int)(round & 1u), &S.qn[round % 3]);
    }
    __syncthreads();
    drain();
    if (kStopFull && S.qn[round % 3] != 0u) {
      // stopped: what the queue holds is listed like what it had no room for
      __syncthreads();
      for (unsigned i = (unsigned)t; i < (unsigned)kCasQ; i += kThreads) {
        const uint4 x = S.q[round & 1u][i];
        list_append(true, (int)x.x, x.y, (int)(x.w - x.z));
      }
      if (t == 0) S.qn[round % 3] = 0u;
    }
    __syncthreads();
  }
  // this workgroup's part of the next list
  low = wave_min_u(low);
  const unsigned ew = (unsigned)wave_sum_i((int)edges);
  const bool any_err = ballot(err != 0) != 0;
  if (lane_id() == 0) {
    if (low != 0xFFFFFFFFu) atomicMin(&S.low, low);
    if (any_err) S.err = 1u;
    atomicAdd(&S.edges, (unsigned long long)ew);
  }
  __syncthreads();
  const unsigned fn = S.fn < (unsigned)kCasFar ? S.fn : (unsigned)kCasFar;
  if (t == 0) {
    if (fn) S.base = atomic_add_u32(&C->aux.v[8 + nxt], fn);
    if (S.low != 0xFFFFFFFFu) atomic_min_u32(&C->aux.v[12 + nxt], S.low);
    if (S.err) store_relaxed(&C->error.v[0], (unsigned)SX_ERR_OVERFLOW);
    Line &l = C->statw[vg.bid % kStatLines];
    atomic_add_u64((unsigned long long *)&l.v[0], S.edges);
    atomic_add_u64((unsigned long long *)&l.v[2], (unsigned long long)ents);
  }
  __syncthreads();
  for (unsigned i = t; i < fn; i += kThreads) olist[S.base + i] = S.far[i];
}

// Words of step s + 2 (read by step s - 1, written by step s + 1), cleared
// during step s by lanes of one workgroup.
SX_DEV void cas_clear(Ctrl *C, unsigned step, int t) {
  const unsigned clr = (step + 2) % 3;
  if (t == 0) store_relaxed(&C->aux.v[8 + clr], 0u);
  if (t == 1) store_relaxed(&C->aux.v[12 + clr], 0xFFFFFFFFu);
  if (t == 2) store_relaxed(&C->aux.v[24 + clr], 0u);
}

// The run as the phases know it, in place of a step: `cnt` vertices listed in
// reg_s[par], `hubs` in reg_m[par], the smallest value `lowest` (the phases'
// next iteration is `it`, which the caller chose: BFS `lowest`).  What lies at
// `lowest` or below is final, and every pending vertex is listed.
//   BFS   Deeper vertices are unvisited again (their depths may be too long,
//         and the phases take a depth for final), the vertices at `lowest` are
//         the frontier.  Ctrl::aux words 28, 29 add up the arcs of the visited
//         ones: the rest is unexplored, which the direction rule goes by.
//   SSSP  The listed vertices are the frontier (stamp `it`).
// The lists then come from a ballot scan.
template <bool kWeighted, int kThreads>
SX_DEV void cas_way_back(const VGrid &vg, const TravArgs &a, unsigned cnt, unsigned hubs, unsigned par,
                         unsigned lowest, int it) {
  const long long tid = (long long)vg.bid * kThreads + threadIdx.x, nt = (long long)vg.nb * kThreads;
  if constexpr (kWeighted) {
    for (long long i = tid; i < cnt; i += nt) {
      const int v = a.w.reg_s[par][i];
      if ((unsigned)v < (unsigned)a.g.n) store_relaxed(&a.w.stamp[v], it);
    }
    for (long long i = tid; i < hubs; i += nt) store_relaxed(&a.w.stamp[a.w.reg_m[par][i]], it);
  } else {
    unsigned *dist = (unsigned *)a.state_i;
    long long arcs = 0;
    for (long long v = tid; v < a.g.n; v += nt) {
      const unsigned d = dist[v];
      if (d <= lowest) arcs += a.g.off[v + 1] - a.g.off[v];
      else if (d != 0xFFFFFFFFu) store_relaxed(&dist[v], 0xFFFFFFFFu);
    }
    arcs = wave_sum_ll(arcs);
    if (lane_id() == 0 && arcs) atomic_add_u64((unsigned long long *)&a.w.ctrl->aux.v[28], (unsigned long long)arcs);
  }
}
// Arcs of the vertices that a run come back has not reached.
SX_DEV unsigned long long cas_unexplored(const TravArgs &a) {
  return (unsigned long long)a.g.m - load_relaxed((const unsigned long long *)&a.w.ctrl->aux.v[28]);
}

}  // namespace sx
