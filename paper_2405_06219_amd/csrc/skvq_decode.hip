// Merge of the split partials of skvq_decode_attention (Eq. 1; Algorithm 1 with l = 1) for
// gfx950, and the launcher of one decode call.
//
// The packed region of every (sequence, kv head) is cut into n_splits chunks of whole 64-token
// tiles; the chunk kernel (skvq_decode_mfma.hip) keeps a running (max, sum, weighted value sum)
// per query head (online softmax) and writes one partial per chunk, in original channel order.
// A kv head read as one chunk has its output written by the chunk kernel, which also combines the
// partials of a few chunks; many chunks' partials are combined by the merge kernel below.
#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>

#include <math.h>

#include "skvq_internal.h"

namespace skvq {

namespace {

// Cross-lane moves inside a row of 16 lanes (data-parallel moves: no round trip through LDS) ...
template <int CTRL>
__device__ __forceinline__ float row_move(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}
__device__ __forceinline__ float lane_value(float x, int lane) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), lane));
}
// ... and the maximum and the sum over the 64 lanes, in every lane.
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, row_move<0xB1>(v));   // quad_perm [1,0,3,2]
  v = fmaxf(v, row_move<0x4E>(v));   // quad_perm [2,3,0,1]
  v = fmaxf(v, row_move<0x141>(v));  // row_half_mirror
  v = fmaxf(v, row_move<0x140>(v));  // row_mirror
  return fmaxf(fmaxf(lane_value(v, 0), lane_value(v, 16)), fmaxf(lane_value(v, 32), lane_value(v, 48)));
}
__device__ __forceinline__ float wave_sum(float v) {
  v += row_move<0xB1>(v);
  v += row_move<0x4E>(v);
  v += row_move<0x141>(v);
  v += row_move<0x140>(v);
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Combines the chunk partials of one (sequence, query head): out = sum_i acc_i 2^(m_i - m*) /
// sum_i l_i 2^(m_i - m*).  Partials hold base-2 exponents.  grid (Hq, B), 256 threads: thread (slice,
// four channels) adds every eighth partial.
// Bound by latency (17 KB per workgroup): what counts is the chain from the launch to the store.  So
// every wavefront works out all weights itself, lane i holding those of partials i and 64 + i, while the
// partials' values are on their way: one memory round trip and one barrier.  A pass over eight layers against
// 1024 threads, wavefront 0's weights through LDS and shuffles: 32 q / 8 kv heads, 131072 tokens, 177 -> 174 us
// (32 partials a row), 100003 tokens in two groups 167 -> 160, four query tokens 218 -> 214.  Traced alone the kernel
// takes as long as before (3.9 us, four query tokens 5.2): what is shorter is the way from the chunks' end to it.
// Behind the chunks it costs 1.5 - 2.4 us a call (against calls without it).
constexpr int kMergeThreads = 256, kMergeSlices = 8;
static_assert(kMergeThreads == kMergeSlices * kD / 4, "one thread per slice and four channels");
__global__ __launch_bounds__(kMergeThreads) void merge_kernel(Layout L, float *__restrict__ out_f32,
                                                              __half *__restrict__ out_f16, int n_all, int n_heads) {
  typedef float float4_t __attribute__((ext_vector_type(4)));
  __shared__ __align__(16) float red[kMergeSlices][kD];
  const int hq = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // n_heads = query tokens x query heads per sequence; hq counts (token, head) pairs
  const float *base = L.workspace + ((long long)b * n_heads + hq) * (SKVQ_MAX_SPLITS + 1) * kPartialStride;
  constexpr int kLaneSets = SKVQ_MAX_SPLITS / 64, kBatch = 32, kSteps = kBatch / kMergeSlices;
  static_assert(SKVQ_MAX_SPLITS % 64 == 0 && 64 % kBatch == 0, "whole sets of lanes, whole batches in them");
  float mi[kLaneSets], li[kLaneSets];
#pragma unroll
  for (int j = 0; j < kLaneSets; ++j) {
    const int i = lane + 64 * j;
    mi[j] = -INFINITY, li[j] = 0.f;
    if (i < n_all) {
      const float2 ml = *reinterpret_cast<const float2 *>(base + i * kPartialStride);
      mi[j] = ml.x, li[j] = ml.y;
    }
  }
  const int x = tid & 31, sl = tid >> 5;  // (a wavefront has the slices 2 wave and 2 wave + 1)
  auto value = [&](int i) {               // (past the end: the last partial again, with weight 0)
    const unsigned at = (unsigned)min(i + sl, n_all - 1) * (unsigned)(kPartialStride * sizeof(float)) + 16u * x + 16u;
    return *reinterpret_cast<const float4_t *>(reinterpret_cast<const char *>(base) + at);
  };
  float4_t part[SKVQ_MAX_SPLITS / kBatch][kSteps];  // every value is requested before the first weight is known
#pragma unroll
  for (int t = 0; t < SKVQ_MAX_SPLITS; t += kBatch)
    if (t < n_all) {  // (uniform)
#pragma unroll
      for (int k = 0; k < kSteps; ++k) part[t / kBatch][k] = value(t + kMergeSlices * k);
    }
  float mstar = -INFINITY;
#pragma unroll
  for (int j = 0; j < kLaneSets; ++j)
    if (li[j] > 0.f) mstar = fmaxf(mstar, mi[j]);
  mstar = wave_max(mstar);
  float w[kLaneSets], den = 0.f;  // (partials without tokens weigh nothing)
#pragma unroll
  for (int j = 0; j < kLaneSets; ++j) {
    w[j] = li[j] > 0.f ? exp2f(mi[j] - mstar) : 0.f;
    den += w[j] * li[j];
  }
  den = wave_sum(den);
  float4_t num = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int t = 0; t < SKVQ_MAX_SPLITS; t += kBatch)
    if (t < n_all) {
#pragma unroll
      for (int k = 0; k < kSteps; ++k) {
        const int i = t % 64 + kMergeSlices * k + 2 * wave;
        const float even = lane_value(w[t / 64], i), odd = lane_value(w[t / 64], i + 1), f = sl & 1 ? odd : even;
#pragma unroll
        for (int c = 0; c < 4; ++c) num[c] = f > 0.f ? fmaf(f, part[t / kBatch][k][c], num[c]) : num[c];
      }
    }
  *reinterpret_cast<float4_t *>(&red[sl][4 * x]) = num;
  __syncthreads();
  if (tid < kD) {
    float tot = 0.f;
#pragma unroll
    for (int k = 0; k < kMergeSlices; ++k) tot += red[k][tid];
    const float o = tot / den;
    const long long idx = ((long long)b * n_heads + hq) * kD + tid;
    out_f32[idx] = o;
    if (out_f16) out_f16[idx] = __float2half_rn(o);
  }
}

}  // namespace

hipError_t launch_decode(const Layout &L, const __half *q, float *out_f32, __half *out_f16, long long T,
                         long long n_kept, DecodePlan plan, int n_new, hipStream_t s, const __half *k_new,
                         const __half *v_new) {
  const Counts n = counts_with(T, L.W, n_kept);
  if (n_kept < 0 || n_kept > L.S || n.n_quant < 0 || n.n_quant > L.Tcap) return hipErrorInvalidValue;
  if (L.Hk > 65535 || L.B > 65535 || (long long)L.Hq * n_new > 65535) return hipErrorInvalidValue;
  if (n_new < 1 || n_new > n.n_win) return hipErrorInvalidValue;  // the new tokens are all in the window
  if (plan.n_splits > SKVQ_MAX_SPLITS || (n.n_quant > 0 && plan.n_splits < 1)) return hipErrorInvalidValue;
  if (plan.n_splits < 1) plan.n_splits = 1;  // nothing packed yet: one chunk, fp16 tokens only
  const int n_splits = plan.n_splits;
  if (k_new && (n_new != 1 || !append_fusable(L, plan, T, false))) return hipErrorInvalidValue;
  // (with the new token taken along: the leaving token's packed row is the last one)
  const long long te = k_new && T - 1 >= L.W ? n.n_quant - 1 : -1;
  MergeOut mo;
  mo.out_f32 = out_f32;
  mo.out_f16 = out_f16;
  mo.mode = n_splits == 1 ? kMergeDirect : plan.merge_last && can_merge_last(L, n_splits, n_new) ? kMergeLast : kMergeSeparate;
  mo.tickets = L.tickets;
  hipError_t e = launch_decode_mfma(L, q, T, n.n_quant, (int)n.n_sink, plan, n_new, k_new, v_new, te, mo, s);
  if (e != hipSuccess || mo.mode != kMergeSeparate) return e;
  // the fp16 tokens are folded into the chunks' partials
  hipLaunchKernelGGL(merge_kernel, dim3(L.Hq * n_new, L.B), dim3(kMergeThreads), 0, s, L, out_f32, out_f16, n_splits,
                     L.Hq * n_new);
  return hipGetLastError();
}

}  // namespace skvq
