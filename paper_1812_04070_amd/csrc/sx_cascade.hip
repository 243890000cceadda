// The cascade of sx_cascade.hpp, a step per launch.
#include "sx_cascade.hpp"
#include "sx_kernels.hpp"

namespace sx {

// One launch of the window loop.  Run state as in the sequenced arrangement
// (launch L reads Ctrl::seq[L & 1] and writes the other line); the cascade's
// own words: [16] window, [17] vertices listed before the last step, [18] step
// number s, [19] the list's buffer.
template <bool kWeighted>
__global__ void __launch_bounds__(kCasBlock) k_cascade(TravArgs a, unsigned L) {
  __shared__ LdsCas<kWeighted> S;
  Ctrl *C = a.w.ctrl;
  const int t = threadIdx.x;
  if (t < 64)
    S.in[t] = t < 32 ? load_relaxed(&C->seq[L & 1].v[t])
                     : (t == 32 ? load_relaxed(&C->error.v[0]) : load_relaxed(&C->aux.v[t - 32]));
  cas_begin(S);
  __syncthreads();
  const unsigned *in = S.in, *aux = S.in + 32;
  Line &out = C->seq[(L + 1) & 1];
  const unsigned step = in[18];
  // the run is not in the cascade (any more): hand the state on
  if (in[0] != PH_CASCADE || in[32]) {
    if (blockIdx.x == 0 && t < 32)
      store_relaxed(&out.v[t], t == 0 && in[32] && in[0] < SEQ_DONE ? (unsigned)SEQ_ERROR : in[t]);
    return;
  }
  const unsigned now = step % 3, nxt = (step + 1) % 3;
  const unsigned cnt = aux[8 + now], lowest = aux[12 + now], hubs = aux[24 + now];
  if (cnt + hubs == 0) {
    // the run is over; BFS counts its levels (the depths reached)
    if (!kWeighted) cas_levels<kCasBlock>(hw_grid(), a);
    if (blockIdx.x == 0 && t < 32) store_relaxed(&out.v[t], t == 0 ? (unsigned)SEQ_DONE : in[t]);
    if (blockIdx.x == 0 && t == 32) store_relaxed(&C->stats.v[12], L + 1u);
    return;
  }
  // back to the phases: a ballot scan after iteration it - 1, then iteration `it`
  if (cas_outgrown(cnt, in[17])) {
    const unsigned it = kWeighted ? in[1] + 2u : lowest;
    cas_way_back<kWeighted, kCasBlock>(hw_grid(), a, cnt, hubs, in[19] & 1u, lowest, (int)it);
    if (blockIdx.x == 0 && t < 32) {
      // [13] buckets go on at the one that holds the smallest distance
      const unsigned long long nb = kWeighted && a.P.delta ? ((unsigned long long)lowest / a.P.delta + 1ull) * a.P.delta : 0ull;
      const unsigned bound = in[13] == 0xFFFFFFFFu || nb >= 0xFFFFFFFFull ? 0xFFFFFFFFu : (unsigned)nb;
      const unsigned x = t == 0 ? (unsigned)PH_BALLOT : t == 1 ? it - 1u : t == 11 ? 3u : t == 12 ? 0u
                       : t == 13 && kWeighted ? bound : t == 15 ? it + (unsigned)kCasHold : in[t];
      store_relaxed(&out.v[t], x);
      if (!kWeighted && t == 6) store_relaxed(&C->stats.v[6], lowest);   // levels done
      if (kWeighted && t < 3) store_relaxed(&C->aux.v[t], 0xFFFFFFFFu);  // smallest distances of the steps to come
    }
    return;
  }
  const unsigned window = kWeighted ? in[16] : cas_window(in[16], cnt, in[17], a.cascade_window);
  const unsigned B = lowest + window < lowest ? 0xFFFFFFFFu : lowest + window;
  if (blockIdx.x == 0) {
    if (t < 32) {
      const unsigned x = t == 16 ? window : t == 17 ? cnt : t == 18 ? step + 1 : t == 19 ? in[19] ^ 1u : in[t];
      store_relaxed(&out.v[t], x);
    }
    cas_clear(C, step, t - 32);
    if (kWeighted && t == 36) atomic_add_u32(&C->stats.v[6], 1u);
  }
  cascade_step<kWeighted, kCasBlock>(hw_grid(), a, S, cnt, hubs, B, in[19] & 1u, nxt, (int)(0x40000000u | L));
}

hipError_t cascade_launch(const TravArgs &a, bool weighted, unsigned L, int grid, hipStream_t s) {
  if (weighted) hipLaunchKernelGGL(k_cascade<true>, dim3(grid), dim3(kCasBlock), 0, s, a, L);
  else hipLaunchKernelGGL(k_cascade<false>, dim3(grid), dim3(kCasBlock), 0, s, a, L);
  return hipGetLastError();
}

}  // namespace sx
