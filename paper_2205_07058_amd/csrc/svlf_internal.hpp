// Internal declarations shared by the host API and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>
#include <vector>

#include "svlf.h"

namespace svlf {

// Per-thread error string behind svlf_last_error().
void set_error(const std::string& msg);
void clear_error();
const char* error_cstr();

// One scene as the kernels see it (passed by value in kernel arguments).
struct DevScene {
  const svlf_node* nodes;
  const int32_t* leaf_corners;
  const float* feat32;
  const uint16_t* feat16;
  float* grad;            // backward only
  int64_t n_vertices;
  int64_t ray_begin;      // first ray of this scene
  int64_t ray_end;
  int32_t depth;
  int32_t item_begin;     // first work item of this scene (plan_items)
  int32_t items;          // work items of this scene (plan_items)
  int32_t trace_begin;    // first traversal block of this scene
};

struct SceneTable {
  DevScene s[SVLF_MAX_SCENES];
  int32_t n;
  int32_t item_rays;      // rays per work item (plan_items)
  int32_t spread;         // items take rays over the whole scene (plan_items)
  int32_t n_items;        // work items over all scenes (plan_items)
  int32_t n_trace;        // traversal blocks over all scenes
  // Live rays (rays with hits) of every traversal block, written by the
  // traversal (reused hits: launch_live): their number and their bit mask.  Null: work items are planned
  // over all rays (plan_items), otherwise over the live ones (LiveRays).
  uint8_t* live_n;        // [n_trace], readable up to live_bytes()
  uint64_t* live_mask;    // [n_trace]
};

// Calls of one scene with kMinLiveRays to kMaxLiveRays rays are planned over live
// rays (one scene: ranks run over the whole call).  Measured, all rays -> live
// rays: 640,000-ray FP32 view 172 -> 155 us, 2,560,000-ray BF16 view 484 -> 457,
// FP32 train step of 262,144 rays 361 -> 262, BF16 of 2^20 1226 -> 1167; renders on
// reused hits, whose arrays are made from the counts (launch_live): 10^6 rays, C =
// 8, FP32 86 -> 64, C = 16, BF16 94 -> 68.
// Below the range a render loses the 2 us that counting takes (4,096 rays 33 -> 34
// us, 32,000 36 -> 38), while backward kernels of one block per CU would gain
// (light field, FP32: 8,192 rays 310 -> 229 us, 32,000 632 -> 547; C = 32, FP32, K =
// 16: 12,000 rays 129 -> 95): one limit serves both families.  Above it the arrays
// outgrow the smallest decoder's rows (756 KB) and the search for a ray in a
// thread's stretch 16 reads, though larger views would gain too (2200^2: C = 8,
// BF16 499 -> 457 us, C = 32 774 -> 710).
// Deterministic calls keep items over all rays (100,003 rays: 384 us, 377 over
// live rays).
constexpr int64_t kMinLiveRays = 1 << 15, kMaxLiveRays = 1 << 22;
constexpr bool live_planned(int64_t n) { return n >= kMinLiveRays && n <= kMaxLiveRays; }
constexpr int kLiveItemRays = 128;   // most live rays of a work item
// Room for them: live_n padded to 16 bytes per thread of a block, then live_mask.
// Calls past the range keep the largest size, so that a workspace sized for some
// rays serves every call with fewer.
constexpr size_t live_bytes(int64_t n) {
  const int64_t waves = ((n < kMaxLiveRays ? n : kMaxLiveRays) + 63) / 64;
  return n < kMinLiveRays ? 0 : static_cast<size_t>((waves + 4095) / 4096 * 4096 + waves * 8);
}
inline void set_live(SceneTable* tab, int64_t n, void* p) {
  tab->live_n = static_cast<uint8_t*>(p);
  tab->live_mask = reinterpret_cast<uint64_t*>(tab->live_n + ((n + 63) / 64 + 4095) / 4096 * 4096);
}

// Internal hit record, one per (ray, slot): leaf id, t_in, t_out and the
// leaf's cell coordinates packed as i | j << 10 | k << 20.
struct HitRec {
  int32_t leaf;
  float tin;
  float tout;
  uint32_t ijk;
};

constexpr int kRaysPerBlock = 256;   // most rays of a work item (one per thread)
constexpr int kTraceThreads = 64;    // rays (threads) of a traversal block

// Work items of the shading kernels: up to kRaysPerBlock rays of one scene.
// Where the rays fill a few rounds of the persistent grid at most, an item
// takes the share of the rays that gives every block the same number of
// items, in as few rounds as 256-ray items would need: 4,096 rays in 256-ray
// items keep 16 of 256 blocks busy, and 100,003 rays give 391 items, two
// rounds with the second half empty.  Such items are spread over the scene's
// rays (item j takes rays j, j + items, j + 2 items, ...): consecutive rays hit
// or miss together, and the launch would wait for the items with the most
// hits (40,009 rays in 255 items: 2.9 times the mean; spread, within a few
// percent).  Beyond that many rounds, full items are interleaved (below) and
// the last rounds are handed out on demand, which balances as well and keeps
// neighbouring rays together.  The limit is higher in the backward kernels,
// whose items are long (400,009 rays over three scenes, 3.1 rounds: 470 us
// with on-demand rounds, 374 us spread; at 8 rounds no difference).  Forward, the
// light field sets it: its kernels gain from neighbours sharing rows in L2 (800^2
// view, 5 rounds: BF16 337 us, spread 354; FP32 1,388 and 1,466; 500^2, 2 rounds:
// BF16 203, spread 186).  Renders of several scenes by the single decoder would
// gain further up (three scenes, 640,000 rays, 4 and 5 rounds: FP32, C = 32, 254
// us, 150 spread; BF16, C = 32, 129 and 95).
constexpr int kBalancedRounds = 3, kBalancedRoundsBwd = 6;
constexpr int kMinItemRays = 16;

inline void plan_items(SceneTable* tab, int blocks, bool backward) {
  const int balanced = backward ? kBalancedRoundsBwd : kBalancedRounds;
  const int64_t n = tab->s[tab->n - 1].ray_end - tab->s[0].ray_begin;
  const int64_t round = static_cast<int64_t>(blocks) * kRaysPerBlock;
  const int64_t rounds = (n + round - 1) / round;
  int64_t rays = kRaysPerBlock;
  if (rounds >= 1 && rounds <= balanced) {
    rays = (n + rounds * blocks - 1) / (rounds * blocks);
    if (rays < kMinItemRays) rays = kMinItemRays;
  }
  tab->item_rays = static_cast<int32_t>(rays);
  tab->spread = rounds <= balanced ? 1 : 0;
  int64_t items = 0;
  for (int s = 0; s < tab->n; ++s) {
    tab->s[s].item_begin = static_cast<int32_t>(items);
    tab->s[s].items = static_cast<int32_t>((tab->s[s].ray_end - tab->s[s].ray_begin + rays - 1) / rays);
    items += tab->s[s].items;
  }
  tab->n_items = static_cast<int32_t>(items);
}

// Work items that are dealt to fixed blocks of a grid; the rest, up to two rounds,
// are handed out on demand, as blocks become free.  The first round never is: all
// blocks ask at once, and the one counter serves them one after the other before
// any has an item (a 65,536-ray C = 8 BF16 render on reused hits: 33 us, 27 so,
// where the same items on a quarter of the blocks took 28).
__host__ __device__ constexpr int dealt_items(int n_items, int blocks) {
  const int first = n_items < blocks ? n_items : blocks, all_but_two = n_items - 2 * blocks;
  return all_but_two > first ? all_but_two : first;
}

// Rays of one work item.  The rays of kIlvItems consecutive full
// kRaysPerBlock-ray items of a scene are interleaved: item j of such a group
// takes rays j, j + kIlvItems, j + 2 kIlvItems, ... of the group, so that one
// item's rays lie far apart in the caller's order while the group, whose
// items run at about the same time, covers one contiguous range.  Spread items
// (plan_items) are interleaved over the whole scene; other items take
// consecutive rays.  Lane t < n of the item handles ray base + t * stride
// (which may be past the scene's last ray).
constexpr int kIlvItems = 256;

struct ItemRays {
  int64_t base;
  int stride, n;
  __device__ __forceinline__ int64_t ray(int lane) const {
    return base + static_cast<int64_t>(lane) * stride;
  }
};

__device__ __forceinline__ ItemRays item_rays(const SceneTable& tab, const DevScene& sc, int item) {
  const int n = tab.item_rays;
  const int64_t li = item - sc.item_begin, g0 = li / kIlvItems * kIlvItems;
  if (tab.spread) return {sc.ray_begin + li, sc.items, n};
  if (n == kRaysPerBlock && (g0 + kIlvItems) * kRaysPerBlock <= sc.ray_end - sc.ray_begin)
    return {sc.ray_begin + g0 * kRaysPerBlock + (li - g0), kIlvItems, n};
  return {sc.ray_begin + li * n, 1, n};
}

// Launchers (defined in the .hip files).
hipError_t launch_trace_public(const svlf_octree& oct, const float* o, const float* d,
                               int64_t n, int K, int32_t* leaf, float* tin, float* tout,
                               int32_t* cnt, hipStream_t s);
hipError_t launch_trace_internal(const SceneTable& tab, const float* o, const float* d,
                                 int K, HitRec* hits, int32_t* cnt, int32_t* zero, int n_zero,
                                 hipStream_t s);
hipError_t launch_live(const SceneTable& tab, const int32_t* cnt, int32_t* zero, int n_zero, hipStream_t s);

struct ShadeArgs {
  SceneTable tab;
  const float* o;
  const float* d;
  const HitRec* hits;
  const int32_t* cnt;
  int32_t K;
  int32_t tau_mode;
  int32_t precision;
  int32_t C;              // features per vertex
  int32_t H;
  int32_t n_hidden;
  int32_t viewdir;        // decoder input [psi | d] (width C + 3)
  const float* params;
  // forward outputs
  float* rgb;
  float* depth;
  float* acc;
  // backward inputs
  const float* g_rgb;
  const float* g_depth;
  const float* g_acc;
  // train-step inputs
  const float* t_rgb;
  const float* t_depth;
  float lambda_depth;
  float loss_scale;
  float* loss_out;
  // backward outputs
  float* grad_params;
  float* ws_partials;     // [grid][n_params] per-block dW partial sums
  float* ws_loss;         // [grid] per-block loss partial sums
  int64_t n_params;
  float* gxu;             // deterministic mode: [n][K][C + 4] (u, dL/dx) per hit, else null
  int32_t* item_counter;  // zeroed before the launch: hands out the last work items (nullable)
};

// Deterministic feature-gradient reduction (detgrad.hip): the order step
// (needs only the hit lists) sorts the hits by leaf, stably in slot order,
// and builds the vertex-to-leaf table; the sum step (after the backward has
// written the per-hit records gxu) sums per vertex over its (up to 8)
// adjacent leaves in a fixed order.
size_t detgrad_bytes(int64_t n_rays, int K, int C, int64_t n_leaves, int64_t n_vertices);
hipError_t launch_detgrad_order(const DevScene& sc, const HitRec* hits, const int32_t* cnt,
                                int64_t n_rays, int K, int C, void* scratch, int64_t n_leaves,
                                int64_t n_vertices, hipStream_t s);
hipError_t launch_detgrad_sum(const DevScene& sc, int64_t n_rays, int K, int C, const float* gxu,
                              void* scratch, int64_t n_leaves, int64_t n_vertices, hipStream_t s);

enum ShadeMode { kForward = 0, kBackward = 1, kTrain = 2 };

// ---------------------------------------------------------------- light field
// The paper's two-decoder function (svlf_lf_*): per-hit state written by the
// density kernel and read by the colour kernel.
struct LfHit {
  float us[3];            // surface point in cell units (unclamped)
  float ts;               // its ray parameter
  float alpha;            // 1 - e^-tau
  float e;                // e^-tau
  float dtau;             // d tau / d o_T0 (0 where the ReLU is off)
  float eta;
};

// Train-mode losses of the light-field path: the photometric + depth loss of
// the single-decoder train step, or the paper's staged loss (Eq. 4) on the
// voxel holding the target surface point (surface stage) or with the
// composited colour (volumetric stages).
enum LfLossKind { kLfLossDefault = 0, kLfLossSurface = 1, kLfLossVolume = 2 };

// Supported light-field decoders: C_T = 64, C_C = 32, H = 128, one hidden
// layer in the density decoder and three in the colour decoder.
constexpr int kLfCT = 64, kLfCC = 32, kLfH = 128, kLfNHT = 1, kLfNHC = 3;
int lf_grid_limit();      // blocks of each light-field kernel (workspace partials)
int64_t lf_params_density();
int64_t lf_params_color(int viewdir);
size_t lf_pack_bytes(int precision, int viewdir);   // both decoders' MFMA packs
int lf_x_row();           // BF16 elements of one saved density-decoder input row

struct LfArgs {
  SceneTable tab;
  const float* o;
  const float* d;
  const HitRec* hits;
  const int32_t* cnt;
  int32_t K;
  int32_t tau_mode;
  int32_t precision;
  int32_t viewdir;
  const float* params;    // FP32 masters: density layers then colour layers
  LfHit* st;              // [n][K]
  float* gT;              // [n][K][2]: dL/d(o_T0, o_T1)
  uint16_t* xsave;        // [n][K][lf_x_row()] BF16 density-decoder inputs written by
                          // the forward density pass for the backward one (nullable)
  void* packs;            // lf_pack_bytes()
  float* rgb;
  float* depth;
  float* acc;
  const float* g_rgb;
  const float* g_depth;
  const float* g_acc;
  const float* t_rgb;
  const float* t_depth;
  float lambda_depth;
  float loss_scale;
  float* loss_out;
  float* grad_params;
  int32_t loss_kind;      // kLfLoss*: train-mode loss
  float lambda_eta;       // staged losses: weight of (eta - eta_target)^2
  float lambda_tau;       // staged losses: weight of e^{-2 tau}
  int32_t freeze_color;   // nonzero: no gradients for Z_C and the colour decoder
  int32_t* item_counters; // [3] zeroed before the kernels: density forward, colour,
                          // density backward; each hands out its launch's last items
  float* partT;           // [grid][params_density]
  float* partC;           // [grid][params_color]
  float* ws_loss;         // [grid]
};

// Occupied leaves from depth maps (occupancy.hip).
size_t occupancy_bitmap_words(int level);
hipError_t launch_occupancy(const float* o, const float* d, const float* t, int64_t n, int level,
                            uint32_t* bitmap, int* counts, int32_t* leaf_ijk, int64_t cap,
                            int64_t* n_out, hipStream_t s);

// Runs packing, the density kernel, the colour kernel and (backward / train)
// the density backward and the reductions of the decoder gradients.
hipError_t launch_lf(const LfArgs& a, int mode, hipStream_t s);

hipError_t launch_shade(const ShadeArgs& a, int mode, hipStream_t s, int* grid_used);
int shade_grid_limit();   // rows of the workspace's per-block partials
int shade_grid_rows();    // most blocks of a launch that writes them

hipError_t launch_reduce_partials(const float* partials, int rows, int64_t n, float* out,
                                  const float* loss_partials, float* loss_out, hipStream_t s);

hipError_t launch_adam(float* p, float* g, float* m, float* v, int64_t n, float lr, float b1,
                       float b2, float eps, float bc1, float bc2, uint16_t* bf16, int zero,
                       hipStream_t s);
hipError_t launch_to_bf16(const float* src, uint16_t* dst, int64_t n, hipStream_t s);
hipError_t launch_fill(float* dst, float v, int64_t n, hipStream_t s);
hipError_t launch_lazy_adam(float* p, float* g, float* m, float* v, int64_t n_rows, int row_len,
                            float lr, float b1, float b2, float eps, float bc1, float bc2,
                            uint16_t* bf16, int zero, hipStream_t s);
hipError_t launch_mlp_forward(const float* params, int C, int H, int n_hidden, int viewdir,
                              int precision, const float* X, int64_t n, float* out,
                              hipStream_t s);

// This device's copy of the library's scratch array of
// svlf_train_step_noalloc (util.hip; SVLF_NOALLOC_SCRATCH_BYTES).
hipError_t noalloc_scratch(void** ptr);

// Host octree build (octree_build.cpp).
struct HostOctree {
  svlf_octree_sizes sizes;
  std::vector<svlf_node> nodes;
  std::vector<int32_t> leaf_corners;
  std::vector<int32_t> leaf_ijk_sorted;
};
int build_octree_host(const int32_t* ijk, int64_t n, int depth, HostOctree* out,
                      bool want_arrays);

}  // namespace svlf
