// Building blocks of the kernels that split a decoder's layers over the waves
// of a block (light field, single-decoder backward): work items and hit
// windows, operand fragments, and LDS tiles that are MFMA operands as stored.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "mfma_common.hpp"
#include "svlf_internal.hpp"

namespace svlf {
namespace detail {

constexpr int kThreads = 256;
static_assert(kThreads == kRaysPerBlock, "one ray per thread in a work item");
constexpr int kWaves = 4;

// Dynamic LDS.  Every LDS address is derived from this array directly, so the
// compiler keeps LDS accesses as ds_* operations (an LDS pointer stored in an
// object would be accessed as a generic address, and each generic access
// waits for all outstanding global memory traffic).
extern __shared__ __attribute__((aligned(16))) char g_lds[];

// Work items of a persistent kernel: dealt round-robin over the grid, except
// the last of them (dealt_items), which `counter` hands out in order to whichever
// block asks first (null: none).  The logical block index groups the blocks of one
// XCD (hardware places block b on XCD b % 8), so that each XCD works on
// neighbouring rays in every round and shares their features in its L2.
// Uniform over the block; scr[10] carries the counter's value.
struct ItemDeal {
  int G, lb, nb, n_static;
  int32_t* counter;
  __device__ __forceinline__ ItemDeal(int n_items, int32_t* item_counter)
      : G(gridDim.x), nb(n_items), counter(item_counter) {
    const int b = blockIdx.x;
    lb = (G % 8 == 0) ? (b % 8) * (G / 8) + b / 8 : b;
    n_static = counter != nullptr ? dealt_items(nb, G) : nb;
  }
  __device__ int first(int* scr) { return lb < n_static ? lb : tail(scr); }
  __device__ int next(int item, int* scr) { return item + G < n_static ? item + G : tail(scr); }
  __device__ int tail(int* scr) {
    if (n_static == nb) return nb;
    if (threadIdx.x == 0) scr[10] = n_static + atomicAdd(counter, 1);
    __syncthreads();
    const int it = scr[10];
    __syncthreads();
    return it;
  }
};
// Work items over the live rays of a call (SceneTable::live_n): item i takes
// live rays [i rays, (i + 1) rays) in ray order, rays = what gives every
// block the same number of items of at most kLiveItemRays.  Every ray of an
// item has hits, so items carry nearly the same number of hits and fill their
// windows, where items over all rays carry what their rays happen to hit
// (random rays, a fifth of them live with seven hits each: 1.4 times the mean
// in the fullest of 255 items, windows two thirds full).
// Each block counts the live rays itself, from one byte per traversal block
// (16 KB for 2^20 rays), and finds an item's rays by their rank: the thread's
// stretch of bytes by bisection over the stretches' prefix sums, the traversal
// block by its bytes, the ray by its bit.
struct LiveRays {
  int items, rays;        // work items, rays of an item
  int total;              // live rays
  int pre, stretch;       // live rays before this thread's traversal blocks; blocks per thread
};

__device__ __forceinline__ uint32_t byte_sum(const uint4& v) {
  uint32_t s = __builtin_amdgcn_sad_u8(v.x, 0u, 0u);
  s = __builtin_amdgcn_sad_u8(v.y, 0u, s);
  s = __builtin_amdgcn_sad_u8(v.z, 0u, s);
  return __builtin_amdgcn_sad_u8(v.w, 0u, s);
}

// Called by all threads; ends with a barrier.
__device__ __forceinline__ LiveRays live_rays(const SceneTable& tab, int* scr) {
  LiveRays lr;
  const int n = tab.n_trace, G = gridDim.x;
  lr.stretch = (n + 4095) / 4096 * 16;
  const int w0 = static_cast<int>(threadIdx.x) * lr.stretch;
  uint32_t s = 0;
  for (int w = w0; w < w0 + lr.stretch && w < n; w += 16) {
    uint4 v = *reinterpret_cast<const uint4*>(tab.live_n + w);
    auto keep = [&](int k) {           // bytes of the 4 from w + 4 k that are below n
      const int left = n - w - 4 * k;
      return left >= 4 ? ~0u : left <= 0 ? 0u : (1u << (8 * left)) - 1u;
    };
    v.x &= keep(0);
    v.y &= keep(1);
    v.z &= keep(2);
    v.w &= keep(3);
    s += byte_sum(v);
  }
  lr.pre = block_excl_scan<kWaves>(static_cast<int>(s), scr, lr.total);
  const int round = G * kLiveItemRays;
  const int rounds = lr.total > 0 ? (lr.total + round - 1) / round : 1;
  lr.rays = lr.total > 0 ? (lr.total + G * rounds - 1) / (G * rounds) : 1;
  lr.items = (lr.total + lr.rays - 1) / lr.rays;
  return lr;
}

// The rays of an item, relative to the scene's first: thread t gets the
// item's ray t, or -1, and ids[t] holds it for the block after its next
// barrier.  Called by all threads; `prefix` (1 KB) is free again after the
// block's next barrier.
__device__ __forceinline__ int find_rays(const SceneTable& tab, const LiveRays& lr, int item, int* prefix,
                                         int* ids) {
  const int tid = threadIdx.x, rank = item * lr.rays + tid;
  prefix[tid] = lr.pre;
  __syncthreads();
  int r = -1;
  if (tid < lr.rays && rank < lr.total) {
    int t = 0;                         // last stretch that starts at or before the rank
#pragma unroll
    for (int step = kThreads / 2; step > 0; step >>= 1)
      if (prefix[t + step] <= rank) t += step;
    int i = rank - prefix[t], w = t * lr.stretch;
    const int end = w + lr.stretch;
    uint4 v = *reinterpret_cast<const uint4*>(tab.live_n + w);
    for (int s = byte_sum(v); i >= s && w + 16 < end; s = byte_sum(v)) {
      i -= s;
      w += 16;
      v = *reinterpret_cast<const uint4*>(tab.live_n + w);
    }
    const uint32_t q[4] = {v.x, v.y, v.z, v.w};
    uint32_t x = q[0];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int s = __builtin_amdgcn_sad_u8(q[k], 0u, 0u);
      if (w % 16 == 4 * k && i >= s) {
        i -= s;
        w += 4;
        x = q[k + 1];
      }
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int s = static_cast<int>(x & 0xFFu);
      if (w % 4 == k && i >= s) {
        i -= s;
        ++w;
        x >>= 8;
      }
    }
    // bit i (from 0) of the mask's set bits
    const uint64_t m = tab.live_mask[w];
    uint32_t b = static_cast<uint32_t>(m);
    int bit = 0;
    const int lo = __popc(b);
    if (i >= lo) {
      i -= lo;
      bit = 32;
      b = static_cast<uint32_t>(m >> 32);
    }
#pragma unroll
    for (int step = 16; step > 0; step >>= 1) {
      const int c = __popc(b & ((1u << step) - 1u));
      if (i >= c) {
        i -= c;
        bit += step;
        b >>= step;
      }
    }
    r = 64 * w + bit;
  }
  if (tid < kLiveItemRays) ids[tid] = r;
  return r;
}

// Hit window [s0, s1): the rays whose hits all fit in [s0, s0 + WIN), from the
// map of the item's hits (hit -> lane | slot << 8, written once per item): the
// window ends at the start of the ray that holds hit s0 + WIN (no ray is longer
// than a window).  No barrier.
template <int WIN>
__device__ __forceinline__ int open_window(int s0, int total, int off, int count,
                                           const uint16_t* imap, bool& in_win) {
  const int p = s0 + WIN;
  const int s1 = p < total ? p - (imap[p] >> 8) : total;
  in_win = count > 0 && off >= s0 && off + count <= s1;
  return s1;
}

__device__ __forceinline__ int scene_of(const SceneTable& tab, int item) {
  int si = 0;
  while (si + 1 < tab.n && item >= tab.s[si + 1].item_begin) ++si;
  return si;
}

__device__ __forceinline__ void trilinear(float ux, float uy, float uz, float (&w)[8]) {
  const float wx[2] = {1.0f - ux, ux}, wy[2] = {1.0f - uy, uy}, wz[2] = {1.0f - uz, uz};
#pragma unroll
  for (int j = 0; j < 8; ++j) w[j] = wx[j & 1] * wy[(j >> 1) & 1] * wz[j >> 2];
}

__device__ __forceinline__ float clamp01(float x) { return fminf(fmaxf(x, 0.0f), 1.0f); }

// ------------------------------------------------------------ operands

template <bool BF>
struct Types {
  using Elem = typename std::conditional<BF, uint16_t, float>::type;
  using El = Elem;
  static constexpr int EB = BF ? 2 : 4;
};

template <bool BF>
__device__ __forceinline__ typename Types<BF>::Elem to_el(float v) {
  if constexpr (BF) return static_cast<uint16_t>(bf16_rne(v));
  else return v;
}

// Operands come in fragments of 16 bytes per lane: one K step of the BF16 MFMA
// or four of the FP32 one.  K index of fragment i, lane group g, element j:
// kfrag_d for operands made of result tiles (drow), kfrag_x for natural rows.
typedef int frag_t __attribute__((ext_vector_type(4)));
template <bool BF>
constexpr int kFragK = BF ? 16 : 8;
template <bool BF>
__device__ __forceinline__ int kfrag_d(int i, int g, int j) {
  return BF ? 16 * i + 8 * (j >> 2) + 4 * g + (j & 3) : 8 * i + 4 * g + j;
}
template <bool BF>
__device__ __forceinline__ int kfrag_x(int i, int g, int j) {
  return BF ? 16 * i + 8 * g + j : 8 * i + 4 * g + j;
}

template <bool BF>
__device__ __forceinline__ f32x16 mma_frag(frag_t a, frag_t b, f32x16 c) {
  if constexpr (BF) {
    return mma(__builtin_bit_cast(s16x8, a), __builtin_bit_cast(s16x8, b), c);
  } else {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int j = 0; j < 4; ++j) c = mma(x[j], y[j], c);
    return c;
  }
}

// ------------------------------------------------------------ LDS tiles

// The compiler would hoist every tile address (a register per chunk and tile)
// out of the window loop; recomputing them where they are used costs a few
// instructions instead of some two hundred registers.
__device__ __forceinline__ int here(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// LDS tile [hit][column], ROWB bytes a row, addressed in 16-byte chunks.  The
// chunk index is swizzled by the hit so that neither of the two access
// patterns conflicts: 16 lanes reading the same chunk of 16 hits (operands
// with the features along K), and the transpose read's 4 hits x 64 bytes
// (operands with the hits along K).  A 256- or 512-byte row covers all banks,
// so hit bits 0-1 choose the 64-byte quarter and bits 2-3 the chunk in it;
// the other widths start neighbouring rows in different banks already and
// need fewer bits or none.
template <int ROWB>
__device__ __forceinline__ int tile_swz(int hit) {
  if constexpr (ROWB == 256 || ROWB == 512) return ((hit & 3) << 2) | ((hit >> 2) & 3);
  else if constexpr (ROWB == 640) return (hit >> 1) & 7;
  else if constexpr (ROWB == 64 || ROWB == 192) return (hit >> 2) & 3;
  else if constexpr (ROWB == 304 || ROWB == 96 || ROWB == 32) return 0;
  else {
    static_assert(ROWB == 128, "tile width");
    return ((hit & 2) << 1) | ((hit >> 2) & 3);
  }
}
template <int ROWB>
__device__ __forceinline__ char* tile_at(int base, int hit, int chunk) {
  return g_lds + base + hit * ROWB + ((chunk ^ tile_swz<ROWB>(hit)) << 4);
}
template <int ROWB>
__device__ __forceinline__ frag_t frag_at(int base, int hit, int chunk) {
  return *reinterpret_cast<const frag_t*>(tile_at<ROWB>(base, hit, chunk));
}

// Chunks of a 32-feature result tile: chunk q of tile t holds result registers
// [16 / NCH q, 16 / NCH (q + 1)) of one lane, at chunk 2 (NCH t + q) + g of its
// hit's row, which makes it fragment NCH t + q of the next layer's operand.
template <bool BF>
constexpr int kTileChunks = BF ? 2 : 4;

template <bool BF>
__device__ __forceinline__ frag_t pack_chunk(const f32x16& v, int q) {
  if constexpr (BF)
    return __builtin_bit_cast(frag_t, bf16_rne8(v[8 * q], v[8 * q + 1], v[8 * q + 2], v[8 * q + 3],
                                                v[8 * q + 4], v[8 * q + 5], v[8 * q + 6], v[8 * q + 7]));
  else
    return __builtin_bit_cast(frag_t, f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]});
}

template <bool BF, int ROWB>
__device__ __forceinline__ void store_tile(int base, int t, int hit, int g, const f32x16& v) {
  hit = here(hit);
#pragma unroll
  for (int q = 0; q < kTileChunks<BF>; ++q)
    *reinterpret_cast<frag_t*>(tile_at<ROWB>(base, hit, 2 * (kTileChunks<BF> * t + q) + g)) = pack_chunk<BF>(v, q);
}

// dL/dz of a hidden layer's tile from dL/da (v): masked by the activations
// that the tile holds and stored in their place.
template <bool BF, int ROWB>
__device__ __forceinline__ void mask_store_tile(int base, int t, int hit, int g, const f32x16& v) {
  hit = here(hit);
#pragma unroll
  for (int q = 0; q < kTileChunks<BF>; ++q) {
    frag_t* at = reinterpret_cast<frag_t*>(tile_at<ROWB>(base, hit, 2 * (kTileChunks<BF> * t + q) + g));
    if constexpr (BF) {
      const s16x8 act = __builtin_bit_cast(s16x8, *at);
      float z[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) z[j] = act[j] > 0 ? v[8 * q + j] : 0.0f;
      *at = __builtin_bit_cast(frag_t, bf16_rne8(z[0], z[1], z[2], z[3], z[4], z[5], z[6], z[7]));
    } else {
      const f32x4 act = __builtin_bit_cast(f32x4, *at);
      f32x4 r;
#pragma unroll
      for (int j = 0; j < 4; ++j) r[j] = act[j] > 0.0f ? v[4 * q + j] : 0.0f;
      *at = __builtin_bit_cast(frag_t, r);
    }
  }
}

// Feature (within its 32-tile) at column position p of a tile row: BF16 chunks
// hold result registers in pairs of row quads (drow).
template <bool BF>
__device__ __forceinline__ int tile_feature(int p) {
  return BF ? (p & 16) | ((p & 4) << 1) | ((p & 8) >> 1) | (p & 3) : p;
}

// Operand with the hits along K: row / column p = lane & 31 of tile t, K = hits.
// BF16: step k covers hits [16 k, 16 k + 16).  The transpose read gives lane i
// of a 16-lane group column i of the 4 x 16 block whose row r lanes 4 r .. 4 r + 3
// address, 4 columns each; two reads make the lane's 8 hits 16 k + 8 g + j.
typedef short s16x4 __attribute__((ext_vector_type(4)));
template <int ROWB>
__device__ __forceinline__ s16x8 hits_operand_bf16(int base, int t, int k, int lane) {
  typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
  const int i = lane & 15, g = lane >> 5;
  const int col = (lane & 16) + 4 * (i & 3);
  s16x8 r;
#pragma unroll
  for (int half = 0; half < 2; ++half) {
    const int hit = 16 * k + 8 * g + 4 * half + (i >> 2);
    const s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        (lds_s16x4*)(tile_at<ROWB>(base, hit, 4 * t + (col >> 3)) + (col & 7) * 2));
#pragma unroll
    for (int j = 0; j < 4; ++j) r[4 * half + j] = v[j];
  }
  return r;
}
// FP32: step k covers hits 2 k and 2 k + 1.
template <int ROWB>
__device__ __forceinline__ float hits_operand_fp32(int base, int t, int k, int lane) {
  const int col = lane & 31;
  return *reinterpret_cast<const float*>(tile_at<ROWB>(base, 2 * k + (lane >> 5), 8 * t + (col >> 2)) + (col & 3) * 4);
}

// ------------------------------------------------------------ gradient scatter

// The feature-gradient atomics are bound by the memory side, one transaction
// per row of each corner, so a row that two consecutive hits of a ray have in
// common (leaves that touch share 1 to 4 corners; on a batch over surfaces at
// depth 9, 31.6% of all rows) is sent once.
//
// shared_corners: bit j of the result = corner j of this thread's hit is also a
// corner of the next thread's hit, if that is the same ray's next hit in a
// touching leaf; 0 otherwise.  mp = the hit's map entry (lane | slot << 8, -1:
// none), ijk = its packed leaf coordinates.  All lanes of the wave call it.
__device__ __forceinline__ uint32_t shared_corners(int mp, uint32_t ijk) {
  const int mp1 = __shfl_down(mp, 1, 64);
  const uint32_t ijk1 = static_cast<uint32_t>(__shfl_down(static_cast<int>(ijk), 1, 64));
  uint32_t m = mp >= 0 && mp1 == mp + 256 ? 0xFFu : 0u;
  constexpr uint32_t hi[3] = {0xAAu, 0xCCu, 0xF0u};     // corners on the high side of each axis
#pragma unroll
  for (int x = 0; x < 3; ++x) {
    const int d = static_cast<int>((ijk1 >> (10 * x)) & 1023u) - static_cast<int>((ijk >> (10 * x)) & 1023u);
    m &= d == 0 ? 0xFFu : d == 1 ? hi[x] : d == -1 ? 0xFFu ^ hi[x] : 0u;
  }
  return m;
}

// One channel's gradient of a hit's 8 corners on its way through the ray's
// hits: flush(m, add) calls add(j, value) for the corners that are not shared
// (m = shared_corners) and renumbers the others to the next hit's corners.  A
// shared set lies on one side of every axis on which the leaves differ (its
// mask is then confined to that side), and crossing the axis swaps the sides.
struct CornerCarry {
  float v[8] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
  template <class Add>
  __device__ __forceinline__ void flush(uint32_t m, Add&& add) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (((m >> j) & 1u) == 0u) {
        add(j, v[j]);
        v[j] = 0.0f;
      }
    }
    constexpr uint32_t hi[3] = {0xAAu, 0xCCu, 0xF0u};
#pragma unroll
    for (int x = 0; x < 3; ++x) {
      const bool cross = (m & hi[x]) == 0u || (m & ~hi[x]) == 0u;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if ((j >> x) & 1) continue;
        const int k = j | (1 << x);
        const float lo = v[j], up = v[k];
        v[j] = cross ? up : lo;
        v[k] = cross ? lo : up;
      }
    }
  }
};

// 16 bytes of a feature row as floats, and 16 bytes of a tile row from floats.
template <bool BF>
constexpr int kRowVals = BF ? 8 : 4;
template <bool BF>
__device__ __forceinline__ void unpack_row(uint4 raw, float (&f)[kRowVals<BF>]) {
  const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (BF) {
      f[2 * i] = bf16_f32(static_cast<uint16_t>(w[i] & 0xFFFFu));
      f[2 * i + 1] = bf16_f32(static_cast<uint16_t>(w[i] >> 16));
    } else {
      f[i] = __uint_as_float(w[i]);
    }
  }
}
template <bool BF>
__device__ __forceinline__ frag_t pack_row(const float* f) {
  if constexpr (BF) return __builtin_bit_cast(frag_t, bf16_rne8(f[0], f[1], f[2], f[3], f[4], f[5], f[6], f[7]));
  else return __builtin_bit_cast(frag_t, f32x4{f[0], f[1], f[2], f[3]});
}
template <bool BF>
__device__ __forceinline__ uint4 load_row(const DevScene& sc, int64_t block, int64_t elem) {
  if constexpr (BF) return *reinterpret_cast<const uint4*>(sc.feat16 + block + elem);
  else return *reinterpret_cast<const uint4*>(sc.feat32 + block + elem);
}

}  // namespace detail
}  // namespace svlf
