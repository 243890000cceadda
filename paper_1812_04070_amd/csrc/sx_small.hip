// BFS and SSSP on small graphs: the whole run in one workgroup, the vertex
// state in its LDS.
//
// On a graph of a few thousand vertices a run of phase launches is their fixed
// cost: the launches, the record prefix, the read-back of the state line
// (R-MAT s10 BFS: 4 iterations, 117 us).  Here one workgroup of 1,024 threads
// keeps every distance in LDS, so that a relaxation is an LDS atomic and only
// rows are read from memory; an iteration ends with a workgroup barrier.
//
// An iteration expands the listed vertices from the distances they had when
// the list was made, so the iterations are the synchronous rounds of the
// frontier form (Active, Compute and Combine as in sx_traverse.hip), whatever
// the order of the updates within one.  Rows go to 2 or 8 lanes, a wavefront or
// the workgroup by length.  Two lanes hold the short rows of graphs of at most 4
// arcs per vertex: with 8, a list of most of 20,000 vertices took 160 passes of
// the workgroup (star of 20,000 SSSP 196 -> 101 us, the phases 103; a
// random graph of 24,000 and 3.3 447 -> 228, the phases 364).
//
// Bound by one CU's rate of row reads and LDS atomics once the graph is large:
// the limits (sx_host.cpp) lie where the grid's phases catch up.
#include "sx_frontier.hpp"
#include "sx_kernels.hpp"

namespace sx {

constexpr int kSmIlp = 4;                // arcs of a lane in flight
constexpr int kSmBlock = 1024, kSmWaves = kSmBlock / 64;
constexpr int kSmWaveRow = 64;           // arcs from which a wavefront takes a row
constexpr int kSmGroupRow = 2048;        // and the workgroup
constexpr int kSmLong = 1024, kSmHuge = 64;   // such rows listed per iteration (the others stay)

struct LdsSmall {
  unsigned dist[kSmallN];
  unsigned short list[kSmallN];          // BFS: every vertex reached, in order
  unsigned next[kSmallN / 32];           // SSSP: vertices improved in this iteration
  unsigned short wrow[kSmLong], grow[kSmHuge];
  unsigned wn, gn, tail, err;
  unsigned sum[kSmWaves];
  unsigned long long edges;
};

template <bool kWeighted, int kLanes>
__global__ void __launch_bounds__(kSmBlock) k_small(TravArgs a, int *out, const int *inv) {
  __shared__ LdsSmall S;
  const int n = a.g.n, t = threadIdx.x, lane = lane_id(), wv = wave_in_wg();
  const int *off = a.g.off, *idx = a.g.idx;
  const unsigned *wt = a.g.w;
  unsigned *at_list = (unsigned *)a.state_i;   // SSSP: distances the list was made with
  Ctrl *C = a.w.ctrl;
  for (int v = t; v < n; v += kSmBlock) S.dist[v] = v == a.src ? 0u : 0xFFFFFFFFu;
  if (kWeighted)
    for (int i = t; i < kSmallN / 32; i += kSmBlock) S.next[i] = 0u;
  if (t == 0) {
    S.list[0] = (unsigned short)a.src;
    S.wn = S.gn = S.err = 0u;
    S.tail = 1u;
    S.edges = 0ull;
    if (kWeighted) at_list[a.src] = 0u;
  }
  if (t < 32) {
    C->state.v[t] = 0u;
    C->stats.v[t] = 0u;
  }
  if (t == 32) C->error.v[0] = 0u;
  reset_stat_lines(C);
  __syncthreads();
  unsigned lo = 0, hi = 1, it = 0, edges = 0, ents = 0;
  bool bad = false;
  // kSmIlp arcs per lane of a row at distance d
  auto relax = [&](const int *e, const bool *ok, unsigned d) {
    int u[kSmIlp];
    unsigned w[kSmIlp];
#pragma unroll
    for (int r = 0; r < kSmIlp; ++r) {
      u[r] = ok[r] ? idx[e[r]] : -1;
      w[r] = kWeighted && ok[r] ? wt[e[r]] : 1u;
    }
    // all distances, then only the arcs that lower one: most find their end
    // reached, and a chain of read, branch and atomic per arc cost more than
    // the reads together
    bool less[kSmIlp], any = false;
#pragma unroll
    for (int r = 0; r < kSmIlp; ++r) {
      const bool in = (unsigned)u[r] < (unsigned)n;
      const unsigned cur = S.dist[in ? u[r] : 0], nd = d + w[r];
      const bool over = kWeighted && (nd < d || nd == 0xFFFFFFFFu);
      edges += in ? 1u : 0u;
      bad = bad || (in && over);
      less[r] = in && !over && nd < cur;
      any = any || less[r];
    }
    if (!any) return;
#pragma unroll
    for (int r = 0; r < kSmIlp; ++r) {
      if (!less[r]) continue;
      const unsigned nd = d + w[r], old = atomicMin(&S.dist[u[r]], nd);
      if constexpr (kWeighted) {
        if (nd < old) atomicOr(&S.next[u[r] >> 5], 1u << (u[r] & 31));
      } else {
        if (old == 0xFFFFFFFFu) S.list[atomicAdd(&S.tail, 1u)] = (unsigned short)u[r];
      }
    }
  };
  // a row by `lanes` lanes, this one the k-th
  auto walk = [&](int beg, int end, unsigned d, int k, int lanes) {
    for (int b = beg + k; b < end; b += lanes * kSmIlp) {
      int e[kSmIlp];
      bool ok[kSmIlp];
#pragma unroll
      for (int r = 0; r < kSmIlp; ++r) {
        e[r] = b + r * lanes;
        ok[r] = e[r] < end;
      }
      relax(e, ok, d);
    }
  };
  while (lo < hi) {
    ++it;
    if (t == 0) ents += hi - lo;
    for (unsigned i = lo + (unsigned)t / kLanes; i < hi; i += kSmBlock / kLanes) {
      const int v = S.list[i];
      const int beg = off[v], end = off[v + 1];
      const unsigned d = kWeighted ? at_list[v] : it - 1;
      bool own = true;
      if (end - beg >= kSmWaveRow) {
        // the first of the lanes lists it; all follow
        unsigned p = 0;
        const bool huge = end - beg >= kSmGroupRow;
        if (lane % kLanes == 0) p = atomicAdd(huge ? &S.gn : &S.wn, 1u);
        p = __shfl(p, lane & ~(kLanes - 1));
        own = p >= (unsigned)(huge ? kSmHuge : kSmLong);
        if (!own && lane % kLanes == 0) (huge ? S.grow : S.wrow)[p] = (unsigned short)v;
      }
      if (own) walk(beg, end, d, lane % kLanes, kLanes);
    }
    __syncthreads();
    const unsigned wn = S.wn < (unsigned)kSmLong ? S.wn : (unsigned)kSmLong;
    const unsigned gn = S.gn < (unsigned)kSmHuge ? S.gn : (unsigned)kSmHuge;
    for (unsigned i = wv; i < wn; i += kSmWaves) {
      const int v = S.wrow[i];
      walk(off[v], off[v + 1], kWeighted ? at_list[v] : it - 1, lane, 64);
    }
    for (unsigned i = 0; i < gn; ++i) {
      const int v = S.grow[i];
      walk(off[v], off[v + 1], kWeighted ? at_list[v] : it - 1, t, kSmBlock);
    }
    __syncthreads();
    if constexpr (kWeighted) {
      // the next list: a word of the improved vertices per thread
      const int word = t < kSmallN / 32 ? t : kSmallN / 32 - 1;
      const unsigned bits = t < kSmallN / 32 ? S.next[word] : 0u;
      const int incl = wave_incl_scan(__popc(bits));
      if (lane == 63) S.sum[wv] = (unsigned)incl;
      if (t == 0) S.wn = S.gn = 0u;
      __syncthreads();
      unsigned pos = (unsigned)(incl - __popc(bits)), total = 0;
      for (int w = 0; w < kSmWaves; ++w) {
        if (w < wv) pos += S.sum[w];
        total += S.sum[w];
      }
      for (unsigned b = bits; b; b &= b - 1) {
        const int v = word * 32 + __ffs((int)b) - 1;
        S.list[pos++] = (unsigned short)v;
        at_list[v] = S.dist[v];
      }
      if (bits) S.next[word] = 0u;
      lo = 0;
      hi = total;
    } else {
      lo = hi;
      hi = S.tail;
      if (t == 0) S.wn = S.gn = 0u;
    }
    __syncthreads();
  }
  static_assert(kSmallN / 32 <= kSmBlock, "a word per thread");
  if (bad) S.err = 1u;
  const unsigned ew = (unsigned)wave_sum_i((int)edges);
  if (lane == 0) atomicAdd(&S.edges, (unsigned long long)ew);
  __syncthreads();
  // (a failed run leaves the caller's array)
  if (!S.err)
    for (int v = t; v < n; v += kSmBlock) out[v] = (int)S.dist[inv ? inv[v] : v];
  if (t == 0) {
    C->state.v[0] = EXIT_DONE;
    C->stats.v[6] = it;
    *(unsigned long long *)&C->statw[0].v[0] = S.edges;
    *(unsigned long long *)&C->statw[0].v[2] = ents;
    if (S.err) C->error.v[0] = SX_ERR_OVERFLOW;
  }
}

hipError_t small_launch(const TravArgs &a, bool weighted, int *out, const int *inv, hipStream_t s) {
  const bool sparse = a.g.m <= 4ll * a.g.n;
  const auto k = weighted ? (sparse ? k_small<true, 2> : k_small<true, 8>)
                          : (sparse ? k_small<false, 2> : k_small<false, 8>);
  hipLaunchKernelGGL(k, dim3(1), dim3(kSmBlock), 0, s, a, out, inv);
  return hipGetLastError();
}

}  // namespace sx
