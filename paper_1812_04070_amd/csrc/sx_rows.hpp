// Rows of a pull over all vertices (PageRank, belief propagation): every
// vertex once per iteration, its arcs shared by as many lanes as the row is
// worth.
//
// The rows are classed by length once per run (a ballot pass over the
// vertices, as Section 4 has it for programs whose vertices are all active)
// and written out as records (vertex, first arc, arcs, out-degree), class by
// class in vertex order, so that an iteration reads them in one coalesced load
// instead of a list entry, its region's prefix and two offsets in turn.
//
// What bounds an iteration once the gathers hit: the chain of record, neighbour
// ids, gathers and the lanes' sums, which a wavefront walks once per row it
// takes.  So a wavefront takes several rows at a time (64, 16, 4 or 1, by
// class), loads the next records while it works on these ones, and on small
// graphs walks one class where another wavefront walks the next.  PageRank, 20
// iterations, directed R-MAT: s24 34.4 ms with binned lists and a wavefront
// per row from 64 arcs on (14 of it without any gather), 29.6 now; s20 2.53 ->
// 1.66 ms; s16 0.84 -> 0.59.  Classes from 16 / 64 / 512 or 8 / 32 / 512 arcs:
// 31.2 and 30.9 at s24 against 30.3 before the classes shared wavefronts.
#pragma once

#include "sx_frontier.hpp"

namespace sx {

// classes: no arcs, a lane, 4 lanes, 16 lanes, a wavefront, a workgroup
constexpr int kRowClasses = 6;
constexpr int kRow4 = 8, kRow16 = 32, kRowWave = 256;   // arcs from which a class starts

// A pull kernel's workgroup: 16 wavefronts, one workgroup per CU, so that the
// whole LDS holds one copy of the sources most arcs lead to.
constexpr int kPullBlock = 1024;
constexpr int kPullWaves = kPullBlock / 64;

struct LdsRows {
  unsigned cnt[kPullWaves][kRowClasses];
  unsigned total[kRowClasses], before[kRowClasses];
};

// The records, in the worklist arrays (2 n + 1024 kMaxGrid entries each).
struct Rows {
  int *v, *beg, *len, *od;
  unsigned at[kRowClasses + 1];   // class k: [at[k], at[k + 1])
};

SX_DEV int row_class(int d, const Params &P) {
  // a caller's thresholds know lanes, wavefronts and workgroups only
  const int t4 = P.bins_fixed ? P.t1 : kRow4, t16 = P.bins_fixed ? P.t1 : kRow16;
  const int tw = P.bins_fixed ? P.t1 : kRowWave, tg = P.t2 > tw ? P.t2 : tw;
  return (d > 0) + (d > 0 && d >= t4) + (d > 0 && d >= t16) + (d > 0 && d >= tw) + (d > 0 && d >= tg);
}

// How many of the first `most` vertices' values a workgroup copies into its LDS
// in each iteration: none where their arcs (the gathers that the copies serve)
// are few for the words copied, all workgroups together.  A copied word is a
// sixteenth of a coalesced request, a gather one of its own.  Without the rule
// graphs that have no hubs in front paid for the copy: random graph of 100,000
// vertices and 8 arcs each, PageRank to 1e-5 669 us, with it 561; 512^2 grid, 20
// iterations 466 -> 295, belief propagation 305 -> 203; R-MAT as before.
SX_DEV int hot_sources(const DevGraph &g, int most) {
  const int h = g.n < most ? g.n : most;
  return 16ll * g.off[h] >= (long long)h * gridDim.x ? h : 0;
}

// Workgroup `bid`'s stretch of the vertices, wavefront by wavefront.
struct RowRange {
  long long lo, hi;
};
SX_DEV RowRange row_range(const VGrid &vg, int n) {
  const long long unit = 64 * kPullWaves;
  const long long per = (((long long)n + vg.nb - 1) / vg.nb + unit - 1) / unit * unit;
  const long long lo = (long long)vg.bid * per + per / kPullWaves * wave_in_wg();
  const long long hi = lo + per / kPullWaves;
  return RowRange{lo, hi < n ? hi : (long long)n};
}

// First pass: this workgroup's rows per class (published for the grid; a
// global barrier follows).
SX_DEV void rows_count(const VGrid &vg, const Work &w, int n, const int *off, const Params &P, LdsRows &S) {
  const RowRange R = row_range(vg, n);
  unsigned c[kRowClasses] = {0, 0, 0, 0, 0, 0};
  for (long long s = R.lo; s < R.hi; s += 64) {
    const long long v = s + lane_id();
    const int k = v < R.hi ? row_class(off[v + 1] - off[v], P) : -1;
#pragma unroll
    for (int i = 0; i < kRowClasses; ++i) c[i] += (unsigned)__popcll(ballot(k == i));
  }
  if (lane_id() == 0)
    for (int i = 0; i < kRowClasses; ++i) S.cnt[wave_in_wg()][i] = c[i];
  __syncthreads();
  if (threadIdx.x < kRowClasses) {
    const int i = threadIdx.x;
    unsigned t = 0;
    for (int x = 0; x < kPullWaves; ++x) t += S.cnt[x][i];
    w.rec[i / NBINS].cnt[i % NBINS][vg.bid] = t;
  }
}

// Second pass: the records (a global barrier follows).  od: the out-degree
// from `out_off`.
SX_DEV Rows rows_place(const VGrid &vg, const Work &w, int n, const int *off, const int *out_off,
                       const Params &P, LdsRows &S) {
  if (wave_in_wg() < kRowClasses) {
    const int i = wave_in_wg();
    const unsigned *cnt = w.rec[i / NBINS].cnt[i % NBINS];
    int all = 0, mine = 0;
    for (unsigned b = lane_id(); b < vg.nb; b += 64) {
      const int x = (int)cnt[b];
      all += x;
      mine += b < vg.bid ? x : 0;
    }
    all = wave_sum_i(all);
    mine = wave_sum_i(mine);
    if (lane_id() == 0) {
      S.total[i] = (unsigned)all;
      S.before[i] = (unsigned)mine;
    }
  }
  __syncthreads();
  Rows r{w.reg_s[0], w.reg_s[1], w.reg_m[0], w.reg_m[1], {}};
  unsigned pos[kRowClasses];
  r.at[0] = 0;
#pragma unroll
  for (int i = 0; i < kRowClasses; ++i) {
    r.at[i + 1] = r.at[i] + (unsigned)__builtin_amdgcn_readfirstlane((int)S.total[i]);
    pos[i] = r.at[i] + S.before[i];
    for (int x = 0; x < wave_in_wg(); ++x) pos[i] += S.cnt[x][i];
  }
  const RowRange R = row_range(vg, n);
  for (long long s = R.lo; s < R.hi; s += 64) {
    const long long v = s + lane_id();
    const int beg = v < R.hi ? off[v] : 0, end = v < R.hi ? off[v + 1] : 0;
    const int k = v < R.hi ? row_class(end - beg, P) : -1;
    unsigned at = 0;
#pragma unroll
    for (int i = 0; i < kRowClasses; ++i) {
      const uint64_t mk = ballot(k == i);
      if (k == i) at = pos[i] + lane_prefix(mk);
      pos[i] += (unsigned)__popcll(mk);
    }
    if (k >= 0) {
      r.v[at] = (int)v;
      r.beg[at] = beg;
      r.len[at] = end - beg;
      r.od[at] = out_off == off ? end - beg : out_off[v + 1] - out_off[v];
    }
  }
  return r;
}

struct Row {
  int v, beg, len, od;            // v = -1: none
};
SX_DEV Row row_load(const Rows &r, unsigned i, unsigned end) {
  Row x{-1, 0, 0, 0};
  if (i < end) x = Row{r.v[i], r.beg[i], r.len[i], r.od[i]};
  return x;
}

// Rows of one class, kLanes lanes each: body(r, sub) with the row and the
// lane's place in it, convergent.  Wavefront gw of nw; `turn` counts the tasks
// (64 / kLanes rows) of the classes walked before, so that each class goes on
// with the wavefronts the last one left idle: on a small graph most
// wavefronts walk one chain and not one per class.
template <int kLanes, class Body>
SX_DEV void rows_walk(const Rows &r, int cls, unsigned gw, unsigned nw, unsigned &turn, Body body) {
  constexpr unsigned per = 64 / kLanes;
  const unsigned end = r.at[cls + 1], step = nw * per;
  const int sub = lane_id() % kLanes;
  const unsigned w = gw >= turn ? gw - turn : gw + nw - turn;
  turn = (turn + (end - r.at[cls] + per - 1) / per) % nw;
  unsigned base = r.at[cls] + w * per;
  Row next = row_load(r, base + lane_id() / kLanes, end);
  for (; base < end; base += step) {
    const Row x = next;
    next = row_load(r, base + step + lane_id() / kLanes, end);
    body(x, sub);
  }
}

// The compensated sum over the kLanes lanes of a row.
template <int kLanes>
SX_DEV CSum lanes_merge(CSum a) {
#pragma unroll
  for (int o = kLanes / 2; o >= 1; o >>= 1) {
    CSum b{__shfl_xor(a.s, o), __shfl_xor(a.c, o)};
    a = cmerge(a, b);
  }
  return a;
}

// K sums over a workgroup of kPullBlock threads at once (fixed order; valid in
// every thread).
template <int K>
SX_DEV void pull_merge(CSum (&a)[K], float *lds /* 2 * kPullWaves * K */) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      CSum b{__shfl_xor(a[k].s, o), __shfl_xor(a[k].c, o)};
      a[k] = cmerge(a[k], b);
    }
  }
  __syncthreads();
  if (lane_id() == 0) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      lds[2 * (wave_in_wg() * K + k)] = a[k].s;
      lds[2 * (wave_in_wg() * K + k) + 1] = a[k].c;
    }
  }
  __syncthreads();
  // every wavefront adds the wavefronts' sums up the same way
  const int w = lane_id() % kPullWaves;
#pragma unroll
  for (int k = 0; k < K; ++k) a[k] = CSum{lds[2 * (w * K + k)], lds[2 * (w * K + k) + 1]};
#pragma unroll
  for (int o = kPullWaves / 2; o >= 1; o >>= 1) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      CSum b{__shfl_xor(a[k].s, o), __shfl_xor(a[k].c, o)};
      a[k] = cmerge(a[k], b);
    }
  }
  __syncthreads();
}
SX_DEV CSum pull_merge1(CSum a, float *lds) {
  CSum x[1] = {a};
  pull_merge(x, lds);
  return x[0];
}

}  // namespace sx
