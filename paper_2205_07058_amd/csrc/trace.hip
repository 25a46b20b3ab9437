// Hit-list kernels: the first K occupied leaves along each ray (SVLF
// sections 4.2-4.3), one ray per lane.
#include <hip/hip_runtime.h>

#include "svlf_internal.hpp"
#include "traverse.hpp"

namespace svlf {
namespace {

// One wave per block (kTraceThreads): a block's LDS and slots are free as soon
// as its own longest ray is done, and few rays spread over more CUs (4,096
// rays at depth 8: 55 us with 256-thread blocks, 50 us with 64).

__device__ __forceinline__ Ray load_ray(const float* __restrict__ o, const float* __restrict__ d,
                                        int64_t r) {
  return make_ray(o[3 * r], o[3 * r + 1], o[3 * r + 2], d[3 * r], d[3 * r + 1], d[3 * r + 2]);
}

// Public layout: separate leaf / t_in / t_out arrays [n][K], padded.
__global__ __launch_bounds__(kTraceThreads) void k_trace_public(
    const svlf_node* __restrict__ nodes, int depth, int64_t n_leaves,
    const float* __restrict__ o, const float* __restrict__ d, int64_t n, int K,
    int32_t* leaf_out, float* tin_out, float* tout_out,
    int32_t* __restrict__ cnt_out) {
  extern __shared__ uint2 stk[];
  const int64_t r = static_cast<int64_t>(blockIdx.x) * kTraceThreads + threadIdx.x;
  if (r >= n) return;
  int count = 0;
  const int64_t base = r * K;
  if (n_leaves > 0) {
    const Ray ray = load_ray(o, d, r);
    count = traverse(ray, nodes, depth, K, stk + threadIdx.x, kTraceThreads,
                     [&](int g, int32_t x, uint32_t y, uint32_t z) {
                       leaf_out[base + g] = x;
                       tin_out[base + g] = __uint_as_float(y);
                       tout_out[base + g] = __uint_as_float(z);
                     },
                     [&](int g, int32_t& x, uint32_t& y, uint32_t& z) {
                       x = leaf_out[base + g];
                       y = __float_as_uint(tin_out[base + g]);
                       z = __float_as_uint(tout_out[base + g]);
                     },
                     [&](int slot, int32_t leaf, float t0, float t1, uint32_t) {
                       leaf_out[base + slot] = leaf;
                       tin_out[base + slot] = t0;
                       tout_out[base + slot] = t1;
                     });
  }
  for (int s = count; s < K; ++s) {
    leaf_out[base + s] = -1;
    tin_out[base + s] = 0.0f;
    tout_out[base + s] = 0.0f;
  }
  cnt_out[r] = count;
}

// Internal layout for the shading kernels: one 16-byte record per hit slot
// (unused slots are left unwritten), rays grouped by scene.  The first block
// also clears the shading kernels' work-item counters (a launch of its own
// costs about 5 us; a 4,096-ray render takes 24).
__global__ __launch_bounds__(kTraceThreads) void k_trace_internal(
    SceneTable tab, const float* __restrict__ o, const float* __restrict__ d, int K,
    HitRec* hits, int32_t* __restrict__ cnt_out, int32_t* __restrict__ zero, int n_zero) {
  extern __shared__ uint2 stk[];
  const int b = blockIdx.x;
  if (b == 0 && static_cast<int>(threadIdx.x) < n_zero) zero[threadIdx.x] = 0;
  int s = 0;
  while (s + 1 < tab.n && b >= tab.s[s + 1].trace_begin) ++s;
  const DevScene& sc = tab.s[s];
  const int64_t r = sc.ray_begin + static_cast<int64_t>(b - sc.trace_begin) * kTraceThreads +
                    threadIdx.x;
  if (r >= sc.ray_end) return;
  int count = 0;
  if (sc.nodes != nullptr) {
    const Ray ray = load_ray(o, d, r);
    HitRec* out = hits + r * K;
    count = traverse(ray, sc.nodes, sc.depth, K, stk + threadIdx.x, kTraceThreads,
                     [&](int g, int32_t x, uint32_t y, uint32_t z) {
                       out[g] = HitRec{x, __uint_as_float(y), __uint_as_float(z), 0u};
                     },
                     [&](int g, int32_t& x, uint32_t& y, uint32_t& z) {
                       const HitRec q = out[g];
                       x = q.leaf;
                       y = __float_as_uint(q.tin);
                       z = __float_as_uint(q.tout);
                     },
                     [&](int slot, int32_t leaf, float t0, float t1, uint32_t ijk) {
                       HitRec h;
                       h.leaf = leaf;
                       h.tin = t0;
                       h.tout = t1;
                       h.ijk = ijk;
                       out[slot] = h;
                     });
  }
  cnt_out[r] = count;
  if (tab.live_n != nullptr) {
    const uint64_t m = __ballot(count > 0);
    if (threadIdx.x == 0) {
      tab.live_n[b] = static_cast<uint8_t>(__popcll(m));
      tab.live_mask[b] = m;
    }
  }
}

// The live-ray arrays of a call that reuses hits, from their counts: one wave per
// traversal block.  It also clears the work-item counters, in place of a launch of
// its own.
__global__ __launch_bounds__(4 * kTraceThreads) void k_live(SceneTable tab, const int32_t* __restrict__ cnt,
                                                            int32_t* __restrict__ zero, int n_zero) {
  const int lane = threadIdx.x % kTraceThreads;
  const int b = blockIdx.x * 4 + threadIdx.x / kTraceThreads;
  if (blockIdx.x == 0 && static_cast<int>(threadIdx.x) < n_zero) zero[threadIdx.x] = 0;
  if (b >= tab.n_trace) return;
  const int64_t r = tab.s[0].ray_begin + static_cast<int64_t>(b) * kTraceThreads + lane;
  const uint64_t m = __ballot(r < tab.s[0].ray_end && cnt[r] > 0);
  if (lane == 0) {
    tab.live_n[b] = static_cast<uint8_t>(__popcll(m));
    tab.live_mask[b] = m;
  }
}

size_t stack_bytes(int depth) {
  const int levels = depth > 1 ? depth - 1 : 1;
  return static_cast<size_t>(levels) * kTraceThreads * sizeof(uint2);
}

}  // namespace

hipError_t launch_trace_public(const svlf_octree& oct, const float* o, const float* d, int64_t n,
                               int K, int32_t* leaf, float* tin, float* tout, int32_t* cnt,
                               hipStream_t s) {
  if (n == 0) return hipSuccess;
  const int64_t blocks = (n + kTraceThreads - 1) / kTraceThreads;
  hipLaunchKernelGGL(k_trace_public, dim3(static_cast<unsigned>(blocks)), dim3(kTraceThreads),
                     stack_bytes(oct.depth), s, oct.nodes, oct.depth, oct.n_leaves, o, d, n, K,
                     leaf, tin, tout, cnt);
  return hipGetLastError();
}

hipError_t launch_trace_internal(const SceneTable& tab, const float* o, const float* d, int K,
                                 HitRec* hits, int32_t* cnt, int32_t* zero, int n_zero,
                                 hipStream_t s) {
  if (tab.n_trace == 0) return hipSuccess;
  int max_depth = 1;
  for (int i = 0; i < tab.n; ++i) max_depth = tab.s[i].depth > max_depth ? tab.s[i].depth : max_depth;
  hipLaunchKernelGGL(k_trace_internal, dim3(static_cast<unsigned>(tab.n_trace)),
                     dim3(kTraceThreads), stack_bytes(max_depth), s, tab, o, d, K, hits, cnt,
                     zero, n_zero);
  return hipGetLastError();
}

hipError_t launch_live(const SceneTable& tab, const int32_t* cnt, int32_t* zero, int n_zero, hipStream_t s) {
  hipLaunchKernelGGL(k_live, dim3(static_cast<unsigned>((tab.n_trace + 3) / 4)), dim3(4 * kTraceThreads), 0, s, tab,
                     cnt, zero, n_zero);
  return hipGetLastError();
}

}  // namespace svlf
