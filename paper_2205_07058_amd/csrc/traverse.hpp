// Front-to-back sparse-octree traversal of one ray per lane.
//
// SVLF lists, for every ray, the occupied voxels it crosses in order along the
// ray with their entry/exit distances (section 4.3), using a ray-AABB slab
// test (section 4.2).  The paper runs a level-synchronous traversal with
// device-wide scans between levels; on gfx950 this is a per-lane depth-first
// walk instead: children are visited in the order of their entry distances,
// so the walk can stop after K leaves and needs no global synchronisation.
// The per-level stack lives in LDS, laid out [level][lane] so that lanes
// never conflict.
//
// Every plane distance is RN(RN(b - o) * inv) in binary32 with no
// contraction; as each value depends only on the plane b, a child is hit only
// if its parent is, sibling order equals t_in order, and the produced t_in /
// t_out equal those of testing each leaf directly (the library's documented
// predicate).
//
// The walk runs in a frame mirrored on every axis where d < 0 (x -> -x):
// there every finite reciprocal is positive, so the half of a cell that a ray
// enters first is always the low half and the visiting order of the children
// is their index in that frame.  Mirroring changes no distance: the mirrored
// cell planes are the negated true planes (exact, as all planes are dyadic
// with at most 11 significant bits), RN(-a) = -RN(a), and the product of two
// negated factors is the original product; only the sign of an exact zero
// distance can differ, which no comparison sees and the t_in clamp removes.
// The child index in the octree's own frame is (mirrored index) ^ oct.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "svlf.h"

namespace svlf {

struct Ray {
  float ox, oy, oz;   // origin, negated on the axes where d < 0
  float ix, iy, iz;   // RN(1 / d), negated likewise
  uint32_t oct;       // bit a set iff d_a < 0
  uint32_t nonfin;    // bit a set iff RN(1 / d_a) is not finite
  bool valid;
};

__device__ __forceinline__ bool finite32(float x) { return __builtin_isfinite(x); }

__device__ __forceinline__ Ray make_ray(float ox, float oy, float oz, float dx, float dy,
                                        float dz) {
  Ray r;
  r.valid = finite32(ox) && finite32(oy) && finite32(oz) && finite32(dx) && finite32(dy) &&
            finite32(dz) && (dx != 0.0f || dy != 0.0f || dz != 0.0f);
  // correctly rounded division (the library is built without fast-math)
  const float ix = 1.0f / dx, iy = 1.0f / dy, iz = 1.0f / dz;
  r.oct = (dx < 0.0f ? 1u : 0u) | (dy < 0.0f ? 2u : 0u) | (dz < 0.0f ? 4u : 0u);
  r.nonfin = (finite32(ix) ? 0u : 1u) | (finite32(iy) ? 0u : 2u) | (finite32(iz) ? 0u : 4u);
  r.ox = (r.oct & 1u) ? -ox : ox;
  r.oy = (r.oct & 2u) ? -oy : oy;
  r.oz = (r.oct & 4u) ? -oz : oz;
  r.ix = (r.oct & 1u) ? -ix : ix;
  r.iy = (r.oct & 2u) ? -iy : iy;
  r.iz = (r.oct & 4u) ? -iz : iz;
  return r;
}

// Distances to the three planes lo < mid < hi of a cell along one axis (in
// the mirrored frame): the low child spans [p0, p1], the high child [p1, p2].
struct Axis {
  float p0, p1, p2;
};

__device__ __forceinline__ Axis axis_planes(float o, float inv, float lo, float mid, float hi) {
#pragma clang fp contract(off)
  Axis a;
  a.p0 = (lo - o) * inv;
  a.p1 = (mid - o) * inv;
  a.p2 = (hi - o) * inv;
  return a;
}

// A ray parallel to the axis (non-finite reciprocal) is constrained on it only
// through where the origin lies; the true-frame half-open interval [a, b)
// becomes (-b, -a] after mirroring.  A cell that the walk expands contains
// the origin on such an axis, so the origin is in exactly one half: the middle
// plane counts as crossed before the cell (high half) or never (low half).
__device__ __forceinline__ bool inside(float o, float lo, float hi, bool mirrored) {
  return mirrored ? (lo < o && o <= hi) : (lo <= o && o < hi);
}

__device__ __forceinline__ Axis axis_parallel(float o, bool mirrored, float lo, float mid) {
  const float inf = __builtin_inff();
  return {-inf, inside(o, lo, mid, mirrored) ? inf : -inf, inf};
}

struct Kids {
  Axis x, y, z;
};

// Cell side at level l: 2^(1-l), exact.
__device__ __forceinline__ float cell_size(int level) {
  return __int_as_float((128 - level) << 23);
}

// Plane distances of the node at `level` with mirrored cell coordinates
// (ci, cj, ck).  PAR: the ray has an axis with a non-finite reciprocal.
template <bool PAR>
__device__ __forceinline__ Kids node_kids(const Ray& r, int level, uint32_t ci, uint32_t cj,
                                          uint32_t ck) {
  const float h = cell_size(level);
  const float hh = cell_size(level + 1);
  const float lx = -1.0f + static_cast<float>(ci) * h;
  const float ly = -1.0f + static_cast<float>(cj) * h;
  const float lz = -1.0f + static_cast<float>(ck) * h;
  Kids k;
  k.x = axis_planes(r.ox, r.ix, lx, lx + hh, lx + h);
  k.y = axis_planes(r.oy, r.iy, ly, ly + hh, ly + h);
  k.z = axis_planes(r.oz, r.iz, lz, lz + hh, lz + h);
  if (PAR) {
    if (r.nonfin & 1u) k.x = axis_parallel(r.ox, r.oct & 1u, lx, lx + hh);
    if (r.nonfin & 2u) k.y = axis_parallel(r.oy, r.oct & 2u, ly, ly + hh);
    if (r.nonfin & 4u) k.z = axis_parallel(r.oz, r.oct & 4u, lz, lz + hh);
  }
  return k;
}

// The children that a ray meets in a node that it meets (t0 < t1, the node's
// own interval).  A line crosses the three middle planes in some order, so
// there are at most four, in visiting order: mirrored child 0 until the first
// crossing, the child with the first crossed axis' bit, the one lacking only
// the last crossed axis' bit, and child 7; each is hit iff its stretch of
// [t0, t1] is not empty.  With q_a = the middle-plane distance p1_a clamped to
// [t0, t1] this is the test max(t_n, 0) < t_out of every child: the planes are
// ordered (p0 <= p1 <= p2 on each axis, rounding is monotone), so the child
// with high-half set S has max(t_n, 0) = max(t0, p1_a for a in S) and t_out =
// min(t1, p1_a for a not in S).
// Returns the mirrored children hit, bit i = child i (visiting order).
__device__ __forceinline__ uint32_t kid_hits(const Kids& k) {
  const float t0 = __builtin_fmaxf(__builtin_fmaxf(__builtin_fmaxf(k.x.p0, k.y.p0), k.z.p0), 0.0f);
  const float t1 = __builtin_fminf(__builtin_fminf(k.x.p2, k.y.p2), k.z.p2);
  const float qx = __builtin_amdgcn_fmed3f(k.x.p1, t0, t1), qy = __builtin_amdgcn_fmed3f(k.y.p1, t0, t1),
              qz = __builtin_amdgcn_fmed3f(k.z.p1, t0, t1);
  const float mn = __builtin_fminf(__builtin_fminf(qx, qy), qz);
  const float mx = __builtin_fmaxf(__builtin_fmaxf(qx, qy), qz);
  const float md = __builtin_amdgcn_fmed3f(qx, qy, qz);
  uint32_t first = qy == mn ? 1u << 2 : 1u << 4;
  first = qx == mn ? 1u << 1 : first;
  uint32_t last = qy == mx ? 1u << 5 : 1u << 3;
  last = qx == mx ? 1u << 6 : last;
  return (t0 < mn ? 1u : 0u) | (mn < md ? first : 0u) | (md < mx ? last : 0u) | (mx < t1 ? 1u << 7 : 0u);
}

// Child mask in the octree's own frame -> mirrored frame: bit i <- bit
// (i ^ oct).  One butterfly stage per axis, a stage being a no-op where the
// axis is not mirrored (shift 0, mask all ones): constants of the ray.
struct Mirror {
  uint32_t m0, s0, m1, s1, s2;
  __device__ __forceinline__ explicit Mirror(uint32_t oct)
      : m0(oct & 1u ? 0x55u : 0xFFu), s0(oct & 1u), m1(oct & 2u ? 0x33u : 0xFFu), s1(oct & 2u), s2(oct & 4u) {}
  __device__ __forceinline__ uint32_t operator()(uint32_t m) const {
    m = ((m & m0) << s0) | ((m >> s0) & m0);
    m = ((m & m1) << s1) | ((m >> s1) & m1);
    return (m | (m << 8)) >> s2;     // bits above 7 are for the caller to drop
  }
};

// Root cell [-1, 1]^3 test (the cell is its own mirror image).
__device__ __forceinline__ bool root_hit(const Ray& r) {
#pragma clang fp contract(off)
  const float inf = __builtin_inff();
  float n[3], f[3];
  const float o[3] = {r.ox, r.oy, r.oz};
  const float v[3] = {r.ix, r.iy, r.iz};
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    if (r.nonfin & (1u << a)) {
      const bool in = inside(o[a], -1.0f, 1.0f, r.oct & (1u << a));
      n[a] = in ? -inf : inf;
      f[a] = in ? inf : -inf;
    } else {
      n[a] = (-1.0f - o[a]) * v[a];
      f[a] = (1.0f - o[a]) * v[a];
    }
  }
  const float tn = __builtin_fmaxf(__builtin_fmaxf(n[0], n[1]), n[2]);
  const float tin = tn > 0.0f ? tn : 0.0f;
  const float tout = __builtin_fminf(__builtin_fminf(f[0], f[1]), f[2]);
  return tin < tout;
}

// One node as a single 64-bit buffer load.  A plain load lets the compiler
// merge it with the stack pop into one flat load through a selected pointer
// (LDS or global) behind a full wait at the loop head.
__device__ __forceinline__ svlf_node load_node(__amdgpu_buffer_rsrc_t rs, int32_t idx) {
  typedef unsigned int v2u_t __attribute__((ext_vector_type(2)));
  const v2u_t v = __builtin_bit_cast(
      v2u_t, __builtin_amdgcn_raw_buffer_load_b64(rs, static_cast<uint32_t>(idx) * 8u, 0, 0));
  svlf_node n;
  n.child = static_cast<int32_t>(v.x);
  n.mask = v.y;
  return n;
}

// [t_in, t_out] of the leaf with mirrored cell coordinates (mi, mj, mk) of
// side h: the planes are those of its parent's children, so the values are
// the ones the walk compared.
template <bool PAR>
__device__ __forceinline__ void leaf_interval(const Ray& r, float h, uint32_t mi, uint32_t mj,
                                              uint32_t mk, float& tin, float& tout) {
#pragma clang fp contract(off)
  const float inf = __builtin_inff();
  const float o[3] = {r.ox, r.oy, r.oz}, inv[3] = {r.ix, r.iy, r.iz};
  const uint32_t m[3] = {mi, mj, mk};
  float n[3], f[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) {
    const float lo = -1.0f + static_cast<float>(m[a]) * h;
    n[a] = (lo - o[a]) * inv[a];
    f[a] = (lo + h - o[a]) * inv[a];
    if (PAR && (r.nonfin & (1u << a))) {
      n[a] = -inf;                     // the leaf was hit, so the axis does not constrain it
      f[a] = inf;
    }
  }
  const float tn = __builtin_fmaxf(__builtin_fmaxf(n[0], n[1]), n[2]);
  tin = tn > 0.0f ? tn : 0.0f;
  tout = __builtin_fminf(__builtin_fminf(f[0], f[1]), f[2]);
}

// The walk is bound by instruction issue under divergence (at eight waves per
// SIMD; by latency when the rays do not fill the chip), so its loop holds only
// what every node needs: one node is expanded per iteration, backing up goes
// straight to the deepest level with a child left (a bit mask of such levels,
// no loop over the levels between), and a leaf parent leaves its hit children
// as ONE group (put) instead of computing them there, where the lanes at a
// leaf parent differ in every iteration.  After the walk the groups are
// expanded into hits, last first (get, emit): group e starts at hit slot
// >= e, so the groups may live in the storage of the hit slots themselves.
// Measured against the loop that tested all eight children, popped level by
// level and emitted hits in place: 2^20 random rays at depth 9 261 -> 171 us,
// a 1600^2 view of the same scene 255 -> 154 us, 4,096 rays at depth 8 (one
// wave's longest chain of nodes) 91 -> 50 us.  Testing the child mask in the
// octree's frame instead (four bit extracts, no Mirror) took 187 and 173 us.
//
// A node in progress is its first child and one word: child mask | mirrored
// hit children left to visit << 8.
template <bool PAR, class Put, class Get, class Emit>
__device__ __forceinline__ int walk(const Ray& r, const svlf_node* __restrict__ nodes, int depth,
                                    int K, uint2* stk, int stride, Put put, Get get, Emit emit) {
  // node indices are < 2^28, so byte offsets fit the 32-bit buffer range
  const __amdgpu_buffer_rsrc_t nrs =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<svlf_node*>(nodes), 0, 0x7FFFFFFF, 0x00020000);
  int count = 0, groups = 0;
  int level = 0;
  uint32_t pend = 0;                 // levels whose stack entry holds children left to visit
  uint32_t ci = 0, cj = 0, ck = 0;   // mirrored cell coordinates
  const Mirror mirror(r.oct);
  svlf_node nd = load_node(nrs, 0);
  bool more = true;
  while (more) {
    const uint32_t kh = kid_hits(node_kids<PAR>(r, level, ci, cj, ck));
    int32_t child = nd.child;
    uint32_t mask = nd.mask & 0xFFu;
    uint32_t rem = kh & mirror(mask);
    if (level == depth - 1) {
      // the children are leaves
      if (rem) put(groups, child, ci | (cj << 10) | (ck << 20), mask | (rem << 8));
      groups += rem ? 1 : 0;
      count += __builtin_popcount(rem);
      rem = 0;
      if (count >= K) pend = 0;
    }
    if (rem == 0) {
      // back to the deepest level with a child left
      more = pend != 0;
      const int up = more ? 31 - __builtin_clz(pend) : 0;
      const int dl = level - up;
      level = up;
      ci >>= dl;
      cj >>= dl;
      ck >>= dl;
      const uint2 e = stk[level * stride];
      child = static_cast<int32_t>(e.x);
      mask = e.y & 0xFFu;
      rem = e.y >> 8;
    }
    if (more) {
      const uint32_t i = __builtin_ctz(rem), c = i ^ r.oct;
      rem &= rem - 1;
      stk[level * stride] = make_uint2(static_cast<uint32_t>(child), mask | (rem << 8));
      pend = (pend & ~(1u << level)) | ((rem ? 1u : 0u) << level);
      ++level;
      ci = 2 * ci + (i & 1);
      cj = 2 * cj + ((i >> 1) & 1);
      ck = 2 * ck + (i >> 2);
      nd = load_node(nrs, child + __builtin_popcount(mask & ((1u << c) - 1u)));
    }
  }
  // expand the groups; leaf coordinates flip back to the octree's frame
  const uint32_t full = (1u << depth) - 1u;
  const uint32_t fx = (r.oct & 1u) ? full : 0u, fy = (r.oct & 2u) ? full : 0u,
                 fz = (r.oct & 4u) ? full : 0u;
  const float h = cell_size(depth);
  uint32_t rem = 0, mask = 0;
  int32_t child = 0;
  uint32_t gi = 0, gj = 0, gk = 0;
  for (int s = count - 1; s >= 0; --s) {
    if (rem == 0) {
      uint32_t cell, bits;
      get(--groups, child, cell, bits);
      mask = bits & 0xFFu;
      rem = bits >> 8;
      gi = 2 * (cell & 1023u);
      gj = 2 * ((cell >> 10) & 1023u);
      gk = 2 * (cell >> 20);
    }
    const uint32_t i = 31 - __builtin_clz(rem), c = i ^ r.oct;
    rem ^= 1u << i;
    if (s >= K) continue;              // the last group may hold more hits than fit
    const int32_t leaf = child + __builtin_popcount(mask & ((1u << c) - 1u));
    const uint32_t mi = gi + (i & 1), mj = gj + ((i >> 1) & 1), mk = gk + (i >> 2);
    float tin, tout;
    leaf_interval<PAR>(r, h, mi, mj, mk, tin, tout);
    emit(s, leaf, tin, tout, (mi ^ fx) | ((mj ^ fy) << 10) | ((mk ^ fz) << 20));
  }
  return count < K ? count : K;
}

// Walks the octree front to back; calls emit(slot, leaf, t_in, t_out, ijk)
// for the first K hit leaves (ijk = i | j << 10 | k << 20 in the octree's own
// frame), in descending slot order.  put(g, a, b, c) keeps three words of
// group g (g < the number of hits so far) and get(g, a, b, c) reads them back;
// emit(slot) may overwrite groups >= slot.  `stk` points at this lane's entry
// of level 0 of an LDS array laid out [level][stride].  Returns the number of
// hits.  Rays parallel to an axis take a separate instance of the walk, so
// that the common one carries no code for them.
template <class Put, class Get, class Emit>
__device__ __forceinline__ int traverse(const Ray& r, const svlf_node* __restrict__ nodes,
                                        int depth, int K, uint2* stk, int stride,
                                        Put put, Get get, Emit emit) {
  if (!r.valid || !root_hit(r)) return 0;
  if (r.nonfin) return walk<true>(r, nodes, depth, K, stk, stride, put, get, emit);
  return walk<false>(r, nodes, depth, K, stk, stride, put, get, emit);
}

}  // namespace svlf
