// Belief propagation as an ACC program (Section 6, "Belief propagation":
// sum-product message passing on a Markov random field, with the vertex's
// probability as its metadata; Section 3.2: every vertex active in every
// iteration, the updates of its neighbours summed), in FP32 for a fixed
// number of synchronous iterations over a binary pairwise MRF.
//
// The model: vertex v has the prior phi_v(1) = p_v; the edge {u, v} has the
// potential psi(x, y) = s_uv if x == y else 1 - s_uv with
//   s_uv = (1 + c_uv) / 2,   c_uv = kappa * theta_uv / max(deg u, deg v),
//   theta_uv = (((w_uv - 1) mod 64) - 31.5) / 31.5  (1 on an unweighted graph).
// With q = 2 b - 1, the message of u to v has the ratio
//   m_{u->v}(1) / m_{u->v}(0) = (1 + c_uv q_u) / (1 - c_uv q_u) = exp(2 atanh(c_uv q_u)),
// so one sum-product iteration is, in the logit / 2 of the belief,
//   x_v = atanh(2 p_v - 1) + sum_{u in N(v)} atanh(c_uv q_u),   q_v' = tanh(x_v),
// and the belief is b_v = 1 / (1 + exp(-2 x_v)).
//
//   Active   every vertex, every iteration.
//   Compute  atanh(c_uv q_u) from the neighbour's q_u, stored per vertex once
//            per iteration, and the arc's coupling (the first iteration's
//            gathers bring the neighbour's degree too).
//   Combine  sum over the neighbours (aggregation), single writer per
//            vertex, compensated FP32 in a fixed order.
//
// Task management as for PageRank: every vertex's row, classed by length once
// before the first iteration (Section 4: BP needs the ballot filter exactly
// once) and reused; one persistent launch runs all iterations, with one global
// barrier each (Section 5).
#include <type_traits>

#include "sx_kernels.hpp"
#include "sx_rows.hpp"

namespace sx {

// Coupling sign and strength of an arc from its weight (weights 1..64 span
// -1..1; an unweighted graph couples every edge with theta = 1).
SX_DEV float bp_theta(const unsigned *w, long long e) {
  return w ? ((float)((w[e] - 1u) & 63u) - 31.5f) / 31.5f : 1.f;
}

// atanh: the odd series up to x^7 for |x| <= 1/16, where the next term is
// below 3e-11 of x and the leading x carries the only rounding that counts
// (the couplings of all but low-degree pairs); the library's function beyond.
SX_DEV float bp_atanh(float x) {
  const float x2 = x * x;
  const float t = x2 * fmaf(x2, fmaf(x2, 1.f / 7.f, 0.2f), 1.f / 3.f);
  return fabsf(x) <= 0.0625f ? fmaf(x, t, x) : atanhf(x);
}

// The hottest neighbours' state in LDS, as for PageRank (sx_pagerank.hip):
// q alone, or (q, deg) pairs for half as many.
constexpr int kHotBp = 39936;

// How an iteration gets an arc's coupling c_uv = kappa theta / max(deg, deg):
// from the weight and the gathered degree (kBpWeigh); the same, and stores it
// (kBpStore: the first of several iterations); or from the store (kBpStored),
// so that the others gather 4 bytes an arc and divide nothing.
enum { kBpWeigh, kBpStore, kBpStored };

// s += atanh(c_uv q_u) over the arcs beg + e, e = e0, e0 + stride, ... < len of
// a vertex of degree len, kIlp arcs of a lane in flight, added in order.
// Whole wavefronts; a place past the row's end adds zero (as in sx_pagerank.hip).
template <int kMode>
SX_DEV void bp_gather(CSum &s, const BpArgs &a, const float2 *src2, const float *src, int beg, unsigned e0, unsigned len,
                      unsigned stride, const float *hot, int nhot) {
  const int *ii = a.g.idx;
  const float dv = (float)len;
  for (unsigned e = e0; ballot(e < len); e += kIlp * stride) {
    int u[kIlp];
    float c[kIlp], q[kIlp];
#pragma unroll
    for (unsigned r = 0; r < kIlp; ++r) {
      const int at = beg + (int)(e + r * stride < len ? e + r * stride : 0u);
      u[r] = ii[at];
      c[r] = kMode == kBpStored ? a.couple[at] : bp_theta(a.g.w, at);
    }
#pragma unroll
    for (unsigned r = 0; r < kIlp; ++r) {
      const bool ok = e + r * stride < len;
      const int i = ok ? u[r] : 0;
      if constexpr (kMode == kBpStored) {
        q[r] = i < nhot ? hot[i] : src[i];
      } else {
        const float2 x = i < nhot ? ((const float2 *)hot)[i] : src2[i];
        q[r] = x.x;
        c[r] = a.kappa * c[r] / fmaxf(x.y, dv);
        if (kMode == kBpStore && ok) a.couple[beg + (int)(e + r * stride)] = c[r];
      }
      q[r] = ok ? c[r] * q[r] : 0.f;
    }
#pragma unroll
    for (int r = 0; r < kIlp; ++r) cadd(s, bp_atanh(q[r]));
  }
}

// One iteration; `last` writes beliefs, else the next state (q alone from a
// run that stores its couplings, else (q, deg)).
template <int kMode>
SX_DEV void bp_iteration(const BpArgs &a, int t, const Rows &rows, float *lf, float *hot, int nhot) {
  const float2 *src2 = a.w.bpq[t & 1];
  const float *src = a.w.contrib[t & 1];
  constexpr int words = kMode == kBpStored ? 1 : 2;
  const float *from = kMode == kBpStored ? src : (const float *)src2;
  for (int i = threadIdx.x; i < nhot * words; i += kPullBlock) hot[i] = from[i];
  __syncthreads();
  const bool last = t == a.iters - 1;
  auto finish = [&](const Row &x, CSum s) {
    const float f = a.w.bph[x.v] + (s.s + s.c);
    if (last) a.belief[x.v] = 1.f / (1.f + expf(-2.f * f));
    else if (kMode == kBpWeigh) a.w.bpq[(t + 1) & 1][x.v] = make_float2(tanhf(f), (float)x.len);
    else a.w.contrib[(t + 1) & 1][x.v] = tanhf(f);
  };
  // one workgroup per long row
  for (unsigned i = rows.at[5] + blockIdx.x; i < rows.at[6]; i += gridDim.x) {
    const Row x = row_load(rows, i, rows.at[6]);
    CSum s{0.f, 0.f};
    bp_gather<kMode>(s, a, src2, src, x.beg, threadIdx.x, (unsigned)x.len, kPullBlock, hot, nhot);
    s = pull_merge1(s, lf);
    if (threadIdx.x == 0) finish(x, s);
  }
  const unsigned gw = blockIdx.x * kPullWaves + wave_in_wg();
  const unsigned nw = gridDim.x * kPullWaves;
  unsigned turn = 0;
  auto some = [&](auto lanes, int cls) {
    constexpr int kLanes = decltype(lanes)::value;
    rows_walk<kLanes>(rows, cls, gw, nw, turn, [&](const Row &x, int sub) {
      CSum s{0.f, 0.f};
      bp_gather<kMode>(s, a, src2, src, x.beg, (unsigned)sub, (unsigned)x.len, kLanes, hot, nhot);
      s = lanes_merge<kLanes>(s);
      if (sub == 0 && x.v >= 0) finish(x, s);
    });
  };
  some(std::integral_constant<int, 64>(), 4);
  some(std::integral_constant<int, 16>(), 3);
  some(std::integral_constant<int, 4>(), 2);
  some(std::integral_constant<int, 1>(), 1);
  rows_walk<1>(rows, 0, gw, nw, turn, [&](const Row &x, int) {
    if (x.v >= 0) finish(x, CSum{0.f, 0.f});
  });
}

// Bounds: the gathers, as for PageRank, and the arithmetic of an arc: with two
// divisions and the library's atanh it took 12.5 ms for 10 iterations of R-MAT
// s22; with the couplings stored by the first iteration, the short series and
// the row classes 7.5 (s20 3.75 -> 1.82, s16 1.03 -> 0.41).
__global__ void __launch_bounds__(kPullBlock) k_bp_fused(BpArgs a) {
  __shared__ LdsRows lds;
  __shared__ float lf[2 * kPullWaves];
  __shared__ alignas(8) float hot[kHotBp];
  Ctrl *C = a.w.ctrl;
  const VGrid vg = hw_grid();
  GridBarrier bar(C, load_relaxed(&C->bar_gen.v[0]), a.P.watchdog);
  rows_count(vg, a.w, a.g.n, a.g.off, a.P, lds);
  if (!bar.sync()) return;
  const Rows rows = rows_place(vg, a.w, a.g.n, a.g.off, a.g.off, a.P, lds);
  if (!bar.sync()) return;
  const int pairs = hot_sources(a.g, kHotBp / 2), single = hot_sources(a.g, kHotBp);
  for (int t = 0; t < a.iters; ++t) {
    if (!a.couple) bp_iteration<kBpWeigh>(a, t, rows, lf, hot, pairs);
    else if (t == 0) bp_iteration<kBpStore>(a, t, rows, lf, hot, pairs);
    else bp_iteration<kBpStored>(a, t, rows, lf, hot, single);
    if (!bar.sync()) return;
  }
  if (vg.bid == 0 && threadIdx.x == 0) {
    store_relaxed(&C->state.v[0], (unsigned)EXIT_DONE);
    store_relaxed(&C->stats.v[6], (unsigned)a.iters);
    store_relaxed(&C->stats.v[4], 1u);
    atomic_add_u64((unsigned long long *)&C->statw[0].v[0], (unsigned long long)a.iters * (unsigned long long)a.g.m);
    atomic_add_u64((unsigned long long *)&C->statw[0].v[2], (unsigned long long)a.iters * (unsigned long long)a.g.n);
  }
}

// Set-up: the prior field atanh(2 p - 1) and iteration 0's (q, degree) from
// the priors; a prior outside (0, 1) (or NaN) raises SX_ERR_INPUT.
__global__ void __launch_bounds__(kBlock) k_bp_init(BpArgs a) {
  Ctrl *C = a.w.ctrl;
  if (blockIdx.x == 0) reset_barrier(C);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    for (int i = 0; i < 32; ++i) { C->state.v[i] = 0; C->stats.v[i] = 0; }
    C->error.v[0] = 0;
  }
  if (blockIdx.x == 1 || gridDim.x == 1) reset_stat_lines(C);
  bool bad = false;
  for (long long v = (long long)blockIdx.x * kBlock + threadIdx.x; v < a.g.n;
       v += (long long)gridDim.x * kBlock) {
    const float p = a.belief[v];
    if (!(p > 0.f && p < 1.f)) bad = true;
    const float q = 2.f * p - 1.f;
    a.w.bph[v] = atanhf(q);
    a.w.bpq[0][v] = make_float2(q, (float)(a.g.off[v + 1] - a.g.off[v]));
  }
  // a flag of its own (cleared by the launch before), turned into the error
  // word by the launch after, so that it cannot race with the reset above
  if (ballot(bad) && lane_id() == 0) atomic_or_u64((unsigned long long *)&C->aux.v[0], 1ull);
}

// Turns the input flag into the error word once the set-up is complete.
__global__ void k_bp_check(Ctrl *C) {
  if (threadIdx.x == 0 && C->aux.v[0]) C->error.v[0] = SX_ERR_INPUT;
}

__global__ void k_bp_clear_flag(Ctrl *C) {
  if (threadIdx.x == 0) {
    C->aux.v[0] = 0u;
    C->aux.v[1] = 0u;
  }
}

hipError_t bp_launch(const BpArgs &a, int grid, hipStream_t s) {
  hipLaunchKernelGGL(k_bp_clear_flag, dim3(1), dim3(64), 0, s, a.w.ctrl);
  hipLaunchKernelGGL(k_bp_init, dim3(grid), dim3(kBlock), 0, s, a);
  hipLaunchKernelGGL(k_bp_check, dim3(1), dim3(64), 0, s, a.w.ctrl);
  hipLaunchKernelGGL(k_bp_fused, dim3(grid), dim3(kPullBlock), 0, s, a);
  return hipGetLastError();
}

static_assert(kBpBlock == kPullBlock, "host and kernel agree on the workgroup");
const void *bp_kernel() { return (const void *)k_bp_fused; }

}  // namespace sx
