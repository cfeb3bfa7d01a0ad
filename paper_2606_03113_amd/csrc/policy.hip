// The paper's exit policy on the device (gfx950): the state of a candidate
// exit layer (Section 3.1.1) from that layer's next-token logits, the
// 2-action Q-network (Section 3.2), and the window of committed confidences.
#include "rowops.h"

namespace lede {

// Keep the POLICY_TOPK largest values seen, in descending order: x bubbles
// down the list (static indices, no branches).
__device__ __forceinline__ void top_insert(float (&t)[POLICY_TOPK], float x) {
#pragma unroll
  for (int j = 0; j < POLICY_TOPK; ++j) {
    const float hi = fmaxf(t[j], x), lo = fminf(t[j], x);
    t[j] = hi;
    x = lo;
  }
}

// One block: features (top-k confidence, entropy, trace) of softmax(logits)
// at temperature 1, Q-values and the greedy action (ties: continue).
//   C_k = log S - mean_{top k} (z - m),  H = log S - sum e (z - m) / S,
// with m the max logit, e = exp(z - m), S = sum e.
// Latency-bound: the host waits for the answer between draft tokens.  One pass,
// since the head's argmax key already holds m; the row comes in shared 64-byte
// pieces through LDS, and the Q-network's weights load before it.  15.3 us over
// 32000 logits, 19.5 with a pass for m first and serial weight loads.
__global__ __launch_bounds__(SB) void k_exit_policy(ExitPolicyArgs a) {
  __shared__ float red[SW];
  __shared__ float tops[SW][POLICY_TOPK];
  __shared__ float hid[SB];
  __shared__ float w2s[2][SB], trs[POLICY_TRACE];
  static_assert(SB >= 1024, "a thread per hidden unit (at most 1024)");
  // what the decision reads after the pass, requested before it: a load per
  // step of a serial sum is a memory round trip each
  const int tid = threadIdx.x, hc = min(tid, a.hidden - 1);
  const float w10 = a.w1[hc * 3], w11 = a.w1[hc * 3 + 1], w12 = a.w1[hc * 3 + 2], b1 = a.b1[hc];
  const float w20 = a.w2[hc], w21 = a.w2[a.hidden + hc];
  const float b20 = a.b2[0], b21 = a.b2[1];
  const float trv = a.trace[min(tid, POLICY_TRACE - 1)];
  const int n_trace = min(a.trace_state[0], POLICY_TRACE);
  const float* z = a.logits;
  const int V = a.vocab;
  const int C = chunk_len(V);
  // one pass over this thread's chunk: the top k, S = sum e and W = sum e (z - m),
  // each in index order.  The head's argmax key holds m.
  const float m = key_logit(key_value(a.keys, a.key));
  float s_e = 0.f, s_w = 0.f;
  float t[POLICY_TOPK];
#pragma unroll
  for (int j = 0; j < POLICY_TOPK; ++j) t[j] = -INFINITY;
  for (int j0 = 0; j0 < C; j0 += CB) {
    float r[CB];
    load_chunks(z, V, C, j0, r);
    const int n = chunk_count(V, C, j0);
#pragma unroll
    for (int j = 0; j < CB; ++j) {
      top_insert(t, j < n ? r[j] : -INFINITY);
      if (j < n) {
        const float d = r[j] - m, e = expf(d);
        s_e += e;
        s_w += e * d;
      }
    }
  }
  // the top-k lists of a wavefront merged pairwise through shuffles, then
  // the waves' lists by one thread below
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    float u[POLICY_TOPK];
#pragma unroll
    for (int j = 0; j < POLICY_TOPK; ++j) u[j] = __shfl_xor(t[j], o);
#pragma unroll
    for (int j = 0; j < POLICY_TOPK; ++j) top_insert(t, u[j]);
  }
  if ((threadIdx.x & 63) == 0)
#pragma unroll
    for (int j = 0; j < POLICY_TOPK; ++j) tops[threadIdx.x >> 6][j] = t[j];
  float S, wtot;
  (void)block_excl_scan(s_e, red, S);
  __syncthreads();
  (void)block_excl_scan(s_w, red, wtot);
  __syncthreads();
  __shared__ float state[3];
  w2s[0][tid] = w20;
  w2s[1][tid] = w21;
  if (tid < POLICY_TRACE) trs[tid] = trv;
  if (tid < 64) {  // the wavefronts' lists, one per lane, merged like those of the lanes
#pragma unroll
    for (int j = 0; j < POLICY_TOPK; ++j) t[j] = tid < SW ? tops[tid][j] : -INFINITY;
#pragma unroll
    for (int o = 1; o < SW; o <<= 1) {
      float u[POLICY_TOPK];
#pragma unroll
      for (int j = 0; j < POLICY_TOPK; ++j) u[j] = __shfl_xor(t[j], o);
#pragma unroll
      for (int j = 0; j < POLICY_TOPK; ++j) top_insert(t, u[j]);
    }
  }
  __syncthreads();
  if (tid == 0) {
    const int kk = min(POLICY_TOPK, V);
    float ts = 0.f;
#pragma unroll
    for (int j = 0; j < POLICY_TOPK; ++j)
      if (j < kk) ts += t[j] - m;
    const float logS = logf(S);
    const int n = n_trace;
    float tr = 0.f;
#pragma unroll
    for (int i = 0; i < POLICY_TRACE; ++i)
      if (i < n) tr += trs[i];
    state[0] = logS - ts / (float)kk;
    state[1] = logS - wtot / S;
    state[2] = n ? tr / (float)n : 0.f;
  }
  __syncthreads();
  hid[tid] = fmaxf(fmaf(w12, state[2], fmaf(w11, state[1], fmaf(w10, state[0], b1))), 0.f);
  __syncthreads();
  if (tid < 64) {  // lane o sums output o in order
    const int o = tid & 1;
    float x = o ? b21 : b20;
#pragma unroll 8
    for (int h = 0; h < a.hidden; ++h) x = fmaf(w2s[o][h], hid[h], x);
    const float q[2] = {__shfl(x, 0), __shfl(x, 1)};
    if (tid != 0) return;
    a.out[0] = a.kind;
    a.out[1] = a.index;
    a.out[2] = state[0];
    a.out[3] = state[1];
    a.out[4] = state[2];
    a.out[5] = q[0];
    a.out[6] = q[1];
    a.out[7] = q[1] > q[0] ? 1.f : 0.f;
  }
}

// Push -log max p (= log S at temperature 1) of each committed row into the
// window, oldest first (k_row_stats takes the rows side by side; one block that
// took them in turn needed 10 us for each).
__global__ __launch_bounds__(64) void k_trace_push(TracePushArgs a) {
  const int n = a.record ? a.record[0] + 1 : a.n_rows;
  // the window as it was, kept so that a failed call can be rolled back
  static_assert(64 >= POLICY_TRACE, "one thread per slot");
  if (threadIdx.x < POLICY_TRACE) a.backup[threadIdx.x] = a.trace[threadIdx.x];
  if (threadIdx.x < 2) ((int32_t*)(a.backup + POLICY_TRACE))[threadIdx.x] = a.trace_state[threadIdx.x];
  __syncthreads();
  // row j's value goes to slot next + j (at most 16 rows, one lane each)
  const int slot = a.trace_state[1], count = a.trace_state[0];
  __syncthreads();
  if ((int)threadIdx.x < n) a.trace[(slot + threadIdx.x) % POLICY_TRACE] = logf(a.stats[2 * threadIdx.x + 1]);
  if (threadIdx.x == 0) {
    a.trace_state[1] = (slot + n) % POLICY_TRACE;
    a.trace_state[0] = min(count + n, POLICY_TRACE);
  }
}

hipError_t launch_exit_policy(const ExitPolicyArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_exit_policy, dim3(1), dim3(SB), ROW_LDS, s, a);
  return hipGetLastError();
}

hipError_t launch_trace_push(const TracePushArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(k_trace_push, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace lede
