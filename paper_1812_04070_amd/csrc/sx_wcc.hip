// Connected components by hooking and pointer jumping, for runs whose policy
// leaves every choice to the engine.  The result is the one of SX_WCC's
// minimum-label propagation (sx_traverse.hip, which runs whenever the policy
// fixes a direction, filter, bin, grid or arrangement): the smallest vertex
// id of each vertex's component.
//
// Propagation moves a label one hop per iteration, so its work grows with the
// diameter (1024^2 grid: 3,300 iterations).  Here every vertex keeps a parent
// of smaller id in the same component (itself: a root), an arc hooks the
// larger of its ends' roots under the smaller with one compare-and-swap, and
// finds halve the paths they walk.  A root is the smallest id of its tree, so
// at the end the root is the label.  The scheme is the sampled form of
// Sutton, Ben-Nun and Barak ("Optimizing Parallel Graph Connectivity
// Computation via Subgraph Sampling", IPDPS 2018): link the first two arcs of
// every vertex, take the component most vertices are then in, and walk the
// remaining arcs only of vertices outside it (an arc between it and another
// component is seen from the other end, the graph being symmetric).
//
// Reads of parents are plain loads and may be stale: a parent only ever moves
// to a smaller id of the same component, so a stale value is still an
// ancestor, and the compare-and-swap on a root decides at the coherence
// point (one that fails returns the parent to go on from).  Ids fall along
// every path, so all walks end.
//
// Bound by the gather of each row's first cache line and of the parents.
// MI355X, against propagation: see the figures at run_wcc (sx_host.cpp).
#include "sx_frontier.hpp"
#include "sx_kernels.hpp"

namespace sx {

constexpr int kWccSamples = kBlock;   // vertices sampled for the largest component
constexpr int kWccWaveRow = 32;       // arcs from which a wavefront shares a row
constexpr int kWccGroupRow = 1024;    // and a workgroup

SX_DEV int par_load(const int *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}
SX_DEV void par_store(int *p, int v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
}

SX_DEV int find_root(int *par, int x) {
  for (;;) {
    const int c = par_load(&par[x]);
    if (c == x) return x;
    const int g = par_load(&par[c]);
    if (g == c) return c;
    par_store(&par[x], g);
    x = g;
  }
}

// The trees of roots a and b become one.  A root read from this XCD's L2 may
// have been hooked long ago by a workgroup elsewhere, so it is read again at
// the coherence point before the compare-and-swap: most attempts on a mesh
// find it hooked, and failed swaps on one address serialise (1024^2 grid
// 424 -> 170 us, 4096^2 2,887 -> 1,570 us).
SX_DEV void hook(int *par, int a, int b) {
  while (a != b) {
    const int hi = a > b ? a : b, lo = a > b ? b : a;
    int up = load_relaxed(&par[hi]);
    if (up == hi) {
      up = atomic_cas_old_i32(&par[hi], hi, lo);
      if (up == hi) return;
    }
    a = find_root(par, up);
    b = find_root(par, lo);
  }
}

// x and y end in one tree
SX_DEV void link(int *par, int x, int y) { hook(par, find_root(par, x), find_root(par, y)); }

// Which of its first two arcs gives vertex v its first parent: the second
// when it leads to a smaller vertex of the same wavefront's tile, else the
// first when it leads to a smaller vertex (rows are sorted, so it is the
// smallest neighbour: hubs, on a degree-ordered graph; an unsorted row only
// starts from another vertex).  On a mesh numbered by rows the second arc
// makes each stretch of a row one tree, and the arcs to the row above, left to
// k_wcc_second_arcs, then repeat the same pairs of roots lane after lane
// (4096^2 grid 1,570 -> 950 us).
SX_DEV bool second_first(int v, int u1) { return u1 < v && v - u1 < 64; }

// First parents, the run's control block and, for a renumbered graph, the
// components' smallest original ids.
__global__ void __launch_bounds__(kBlock) k_wcc_init(WccArgs a) {
  const int n = a.g.n;
  Ctrl *C = a.ctrl;
  if (blockIdx.x == 0) {
    if (threadIdx.x < 32) {
      C->state.v[threadIdx.x] = 0u;
      C->stats.v[threadIdx.x] = threadIdx.x == 6 ? 3u : 0u;   // link phases
    }
    if (threadIdx.x == 0) C->error.v[0] = 0u;
    reset_stat_lines(C);
  }
  for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < n;
       i += (long long)gridDim.x * kBlock) {
    const int v = (int)i;
    const int beg = a.g.off[v], end = a.g.off[v + 1];
    const int u0 = beg < end ? a.g.idx[beg] : v, u1 = beg + 1 < end ? a.g.idx[beg + 1] : v;
    a.par[v] = second_first(v, u1) ? u1 : (u0 < v ? u0 : v);
    if (a.inv) a.low[v] = 0xFFFFFFFFu;
  }
}

// What k_wcc_init left of the first two arcs of every row.  Whole wavefronts;
// a lane whose two roots are those of the lane below leaves the hooking to it.
__global__ void __launch_bounds__(kBlock) k_wcc_second_arcs(WccArgs a) {
  __shared__ long long red[kWaves];
  const int n = a.g.n;
  long long edges = 0;
  for (long long base = (long long)blockIdx.x * kBlock; base < n; base += (long long)gridDim.x * kBlock) {
    const long long i = base + threadIdx.x;
    const int v = i < n ? (int)i : n - 1;
    const int beg = a.g.off[v], end = a.g.off[v + 1];
    const int u0 = i < n && beg < end ? a.g.idx[beg] : v, u1 = i < n && beg + 1 < end ? a.g.idx[beg + 1] : v;
    const int u = second_first(v, u1) ? u0 : u1;
    const int x = find_root(a.par, v), y = find_root(a.par, u);
    const int xb = __shfl_up(x, 1), yb = __shfl_up(y, 1);
    if (lane_id() == 0 || xb != x || yb != y) hook(a.par, x, y);
    if (u0 > v) link(a.par, v, u0);
    if (i < n) edges += end - beg < 2 ? end - beg : 2;
  }
  add_stats(a.ctrl, blockIdx.x, edges, blockIdx.x == 0 ? 2ull * n : 0ull, red);
}

// Every vertex's parent becomes its root.  Walks without halving: a halving
// store that lands after the other vertex's own would put an ancestor in the
// place of its root.
__global__ void __launch_bounds__(kBlock) k_wcc_compress(WccArgs a) {
  for (long long v = (long long)blockIdx.x * kBlock + threadIdx.x; v < a.g.n;
       v += (long long)gridDim.x * kBlock) {
    int r = par_load(&a.par[v]);
    for (int c = par_load(&a.par[r]); c != r; c = par_load(&a.par[r])) r = c;
    par_store(&a.par[v], r);
  }
}

// The root most of the sampled vertices have (one workgroup): the component
// whose vertices k_wcc_link skips.
__global__ void __launch_bounds__(kBlock) k_wcc_sample(WccArgs a) {
  __shared__ int root[kWccSamples];
  __shared__ unsigned best;
  const int t = threadIdx.x;
  root[t] = a.par[(long long)a.g.n * t / kWccSamples];
  if (t == 0) best = 0u;
  __syncthreads();
  unsigned same = 0;
  for (int i = 0; i < kWccSamples; ++i) same += root[i] == root[t] ? 1u : 0u;
  atomicMax(&best, same << 16 | (unsigned)t);
  __syncthreads();
  if (t == 0) a.ctrl->aux.v[0] = (unsigned)root[best & 0xffffu];
}

// Every arc from the third on of the vertices
// outside the skipped component: a lane per short row, the wavefront together
// on each longer one, the workgroup on each hub.  A vertex whose parent is
// the skipped root is in that component for certain, whatever other lanes
// hook meanwhile; one that lost this parent to path halving is only walked
// for nothing.
__global__ void __launch_bounds__(kBlock) k_wcc_link(WccArgs a) {
  __shared__ int hub[kBlock];
  __shared__ int hubs;
  __shared__ long long red[kWaves];
  const int n = a.g.n;
  const int skip = (int)a.ctrl->aux.v[0];
  constexpr int from = 2;   // arcs linked by the kernels before
  const int *idx = a.g.idx;
  const int lane = lane_id();
  long long edges = 0, walked = 0;
  for (long long base = (long long)blockIdx.x * kBlock; base < n; base += (long long)gridDim.x * kBlock) {
    if (threadIdx.x == 0) hubs = 0;
    __syncthreads();
    const long long v = base + threadIdx.x;
    int beg = 0, end = 0;
    if (v < n && par_load(&a.par[v]) != skip) {
      end = a.g.off[v + 1];
      beg = a.g.off[v];
      beg = end - beg > from ? beg + from : end;
    }
    const int len = end - beg;
    edges += len;
    walked += len > 0 ? 1 : 0;
    if (len >= kWccGroupRow) hub[atomicAdd(&hubs, 1)] = (int)v;
    if (len < kWccWaveRow)
      for (int e = beg; e < end; ++e) link(a.par, (int)v, idx[e]);
    for (uint64_t rows = ballot(len >= kWccWaveRow && len < kWccGroupRow); rows; rows &= rows - 1) {
      const int r = __ffsll((long long)rows) - 1;
      const int x = __shfl((int)v, r), b = __shfl(beg, r), f = __shfl(end, r);
      for (unsigned e = (unsigned)(b + lane); e < (unsigned)f; e += 64u) link(a.par, x, idx[e]);
    }
    __syncthreads();
    for (int h = 0; h < hubs; ++h) {
      const int x = hub[h], f = a.g.off[x + 1];
      for (long long e = (long long)a.g.off[x] + from + threadIdx.x; e < f; e += kBlock) link(a.par, x, idx[e]);
    }
    __syncthreads();
  }
  const long long w = wg_sum_ll<kBlock>(walked, red);
  add_stats(a.ctrl, blockIdx.x, edges, (unsigned long long)w, red);
}

// A renumbered graph: out[v] = root of v (v an original id), and the smallest
// original id of each component.  Most vertices share one root, and atomics
// on one address serialise (~11 ns each): lanes whose root is that of the
// workgroup's first vertex take the minimum in LDS, one atomic per workgroup,
// the others only where the value read is larger than theirs.
__global__ void __launch_bounds__(kBlock) k_wcc_lowest(WccArgs a) {
  __shared__ int common;
  __shared__ unsigned low;
  const int n = a.g.n;
  const long long per = (((long long)n + gridDim.x - 1) / gridDim.x + kBlock - 1) / kBlock * kBlock;
  const long long lo = (long long)blockIdx.x * per, hi = lo + per < n ? lo + per : n;
  if (lo >= hi) return;
  if (threadIdx.x == 0) {
    common = find_root(a.par, a.inv[lo]);
    low = 0xFFFFFFFFu;
  }
  __syncthreads();
  const int c = common;
  for (long long v = lo + threadIdx.x; v < hi; v += kBlock) {
    const int r = find_root(a.par, a.inv[v]);
    a.out[v] = r;
    if (r == c) {
      if ((unsigned)v < low) atomicMin(&low, (unsigned)v);
    } else if ((unsigned)v < a.low[r]) {
      atomic_min_u32(&a.low[r], (unsigned)v);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0 && low < load_relaxed(&a.low[c])) atomic_min_u32(&a.low[c], low);
}

__global__ void __launch_bounds__(kBlock) k_wcc_relabel(WccArgs a) {
  for (long long v = (long long)blockIdx.x * kBlock + threadIdx.x; v < a.g.n;
       v += (long long)gridDim.x * kBlock)
    a.out[v] = (int)a.low[a.out[v]];
}

hipError_t wcc_launch(const WccArgs &a, int cus, hipStream_t s, int *launches) {
  const dim3 b(kBlock);
  long long g = ((long long)a.g.n + kBlock - 1) / kBlock;
  const dim3 wide((unsigned)(g < 16ll * cus ? (g > 1 ? g : 1) : 16ll * cus));
  const dim3 grid((unsigned)(g < 4ll * cus ? (g > 1 ? g : 1) : 4ll * cus));
  hipLaunchKernelGGL(k_wcc_init, wide, b, 0, s, a);
  hipLaunchKernelGGL(k_wcc_second_arcs, wide, b, 0, s, a);
  hipLaunchKernelGGL(k_wcc_compress, wide, b, 0, s, a);
  hipLaunchKernelGGL(k_wcc_sample, dim3(1), b, 0, s, a);
  hipLaunchKernelGGL(k_wcc_link, grid, b, 0, s, a);
  *launches = a.inv ? 7 : 6;
  if (a.inv) {
    hipLaunchKernelGGL(k_wcc_lowest, grid, b, 0, s, a);
    hipLaunchKernelGGL(k_wcc_relabel, wide, b, 0, s, a);
  } else {
    hipLaunchKernelGGL(k_wcc_compress, wide, b, 0, s, a);
  }
  return hipGetLastError();
}

}  // namespace sx
