// Shading kernels of the SVLF per-ray path (gfx950).
//
// For every hit (leaf, t_in, t_out) found by the traversal: trilinear
// interpolation of the leaf's corner features at the segment midpoint
// (section 4.1), one ReLU decoder C -> H ... -> 4 (section 4.5), optical
// thickness from sigma (section 4 footnote) and front-to-back alpha
// compositing (Eq. 3); the backward and train modes recompute all of it and
// propagate dL/d(rgb, depth, acc) to the decoder parameters (per-block partial
// sums, reduced deterministically) and the features (FP32 atomics, or per-hit
// records for the deterministic reduction).
//
// One block = 4 waves, persistent over work items, in hit windows that never
// split a ray, so compositing and its backward are window-local.  What bounds
// these kernels is waiting: for the three dependent gathers (record, corner
// ids, rows), for the chain of small layers, and in the backward for the
// memory side's atomics, which take 324 G FP32 additions a second however
// they are issued (one per clock and memory channel; measured with random
// rows of 64 to 256 bytes over tables of 2 MB to 1 GB).  So a block is kept
// small enough that others run on its CU meanwhile, and adds as few rows as it
// can:
//  * one thread per hit computes the window's records (cell coordinates,
//    corner ids), then 16 bytes of a row per thread;
//  * the waves form a grid of H / 32 output-feature groups x 4 / (H / 32) hit
//    groups; a wave computes its features of its hits.  Its weights sit in
//    registers, built through LDS once per launch;
//  * activations are LDS tiles that are MFMA operands as stored (tiles.hpp),
//    dL/dz replaces them in place, and weight gradients read the same tiles
//    with the hits along K (LDS transpose read in BF16).  Forward with H = 32 a
//    lane would read back just what it stored, so they stay in registers (a
//    2200^2 FP32 view, C = 8: 592 us of shading through LDS, 495 so);
//  * blocks per CU, by registers (launch_bounds) as far as the LDS, which grows
//    with K, leaves room: forward 4 (H = 32; BF16 with C = 16: a 2200^2 view 716 us
//    with three, 665 so, and three from K = 11 on), 3 (BF16 with C = 32: four made
//    an 800^2 view on reused hits 97 -> 109 us) or 2 (FP32; with 64-hit windows 3
//    fit, 137 instead of 130 us for an 800^2 view); backward 2, but with C = 32 and
//    the view direction one from K = 9 on (82,384 of 81,920 bytes).  The FP32
//    backward with H = 64 needs twice the registers: one block (two with the
//    weights read per window took 374 instead of 348 us for a 262,144-ray train
//    step), and a window's atomics are issued after the next window's gather, whose
//    loads would otherwise queue behind them.  At 256 registers the BF16 backward
//    with H = 64 spills 11 to 37, forward with C = 16 at 128 11;
//  * a row that consecutive hits of a ray share is added once (CornerCarry).
// Measured against one 124 KB block per CU with the packs in LDS (2^20 rays, C =
// 32, BF16): train kernel 1.18 -> 1.03 ms, of which 0.5 ms without atomics
// (1.00 before); 100,003-ray pass without atomics 262 -> 159 us; a 1600^2
// BF16 view 388 -> 360 us; backward of 20,011 rays at H = 32 FP32 63 -> 33 us.
#include <hip/hip_runtime.h>

#include <atomic>

#include "svlf_internal.hpp"
#include "tiles.hpp"

namespace svlf {
namespace {

using namespace detail;

template <int P, int C_, int H_, int NH_, int MODE_, int VD_>
struct Cfg {
  static constexpr bool BF = P == 1;
  static constexpr int C = C_, H = H_, NH = NH_, MODE = MODE_, VD = VD_, OUT = 4;
  static constexpr int EB = BF ? 2 : 4;
  static constexpr int CIN = C + 3 * VD;                 // decoder inputs
  static constexpr int CI = BF ? align16(CIN) : align8(CIN);
  static constexpr bool BWD = MODE != kForward;
  static constexpr bool NARROW = BF || H == 32;          // a wave's weights take <= 80 registers
  static constexpr bool DEFER = BWD && !NARROW;
  static constexpr int WIN = 128;
  static constexpr int BLOCKS = BWD ? (NARROW ? 2 : 1) : (H == 32 || (BF && C == 16) ? 4 : NARROW ? 3 : 2);   // per CU, by registers
  static constexpr int NT = WIN / 32;                    // 32-hit tiles
  static constexpr int MG = H / 32, NG = kWaves / MG;    // wave grid
  static constexpr int TPW = NT / NG;                    // tiles of a wave's hits
  static constexpr int NF0 = CI / kFragK<BF>, NFH = H / kFragK<BF>;
  static constexpr int NTX = (CIN + 31) / 32;            // dW tiles along the inputs
  using El = typename Types<BF>::Elem;
  static_assert(TPW >= 1 && MG * NG == kWaves && NTX <= (NG > 1 ? 2 : 1), "wave grid");
  static_assert(C <= 32 && (H == 64 || NTX == 1), "input layer");
  // parameters
  static constexpr bool REG = MG == 1 && !BWD;           // activations stay in registers
  static constexpr int NACT = BWD ? NH : REG ? 0 : 1;    // forward: each layer takes the previous one's place
  static constexpr int act_of(int l) { return BWD ? l : 0; }
  static constexpr int in_r(int l) { return l == 0 ? CIN : H; }
  static constexpr int out_r(int l) { return l == NH ? OUT : H; }
  static constexpr int par_w(int l) {
    int o = 0;
    for (int i = 0; i < l; ++i) o += out_r(i) * in_r(i) + out_r(i);
    return o;
  }
  static constexpr int par_b(int l) { return par_w(l) + out_r(l) * in_r(l); }
  static constexpr int NPARAMS = par_w(NH + 1);
  // packs, fragments of 1024 bytes: [forward layers 0 .. NH-1][transposed
  // layers 1 .. NH] (the output layer's has its 4 real K positions in fragment 0)
  static constexpr int pk_fwd(int l) { return l == 0 ? 0 : MG * (NF0 + (l - 1) * NFH); }
  static constexpr int pk_bwd(int l) { return pk_fwd(NH) + MG * (l - 1) * NFH; }
  static constexpr int PACK = (BWD ? pk_bwd(NH) + MG : pk_fwd(NH)) * 1024;
  // LDS: kept for the launch, then the window's data, where the packs are
  // built first
  static constexpr int ROWH = H * EB;
  static constexpr int ROWX = CI > 32 ? (BF ? 96 : 192) : 32 * EB;
  static constexpr int ROWG = C * 4;
  static constexpr int GOS = WIN * EB;
  static constexpr int ACT = WIN * ROWH;
  static constexpr int L_W3 = 0;                         // output layer, 4 rows
  static constexpr int L_B0 = L_W3 + OUT * H * EB;       // transposed input layer (dL/dx)
  static constexpr int L_BIAS = L_B0 + (BWD ? NFH * 1024 : 0);
  static constexpr int L_SCR = L_BIAS + (NH * H + OUT) * 4;   // (rows past the output's 4 read on)
  static constexpr int L_SHARE = L_SCR + 64;             // corners shared with the next hit [2][WIN] uint8
  static constexpr int L_X = L_SHARE + (BWD ? (DEFER ? 2 : 1) * WIN : 0);
  static constexpr int L_ACT = L_X + WIN * ROWX;
  static constexpr int L_LAST = L_ACT + (NACT - 1) * ACT;
  static constexpr int L_GX = L_LAST;                    // dL/dx takes the last layer's place
  static constexpr int L_ID = L_ACT + NACT * ACT;        // corner ids [2][WIN] int4
  static constexpr int L_U = L_ID + (DEFER ? 2 : 1) * WIN * 32;     // cell coordinates [3][WIN]
  static constexpr int L_OUT = L_U + (DEFER ? 2 : 1) * WIN * 12;
  static constexpr int L_GO = L_OUT + WIN * 32;          // dL/do [4][WIN]
  static constexpr int L_MAP = L_GO + (BWD ? OUT * GOS : 0);   // [256 K] uint16
  static constexpr int lds_bytes(int K) {
    const int map = kThreads * K * 2, live = kLiveItemRays * (K * 2 + 4);   // (live: the item's rays after it)
    const int win = L_MAP + (map > live ? map : live), pack = L_X + PACK, part = BWD ? L_X + NPARAMS * 4 : 0;
    const int m = win > pack ? win : pack;
    return m > part ? m : part;
  }
  static_assert(lds_bytes(SVLF_MAX_K) <= 160 * 1024, "LDS");
  static_assert(WIN * ROWG <= ACT && L_X % 16 == 0 && L_MAP % 16 == 0, "LDS layout");
};

// Packs, output layer, transposed input layer and biases from the FP32
// parameters (all read at once, in order); padding stays zero.  Ends with a
// barrier.
template <class CF>
__device__ __forceinline__ void build_packs(const float* __restrict__ params) {
  constexpr bool BF = CF::BF;
  constexpr int N = (CF::NPARAMS + kThreads - 1) / kThreads;
  using El = typename CF::El;
  const int tid = threadIdx.x;
  float v[N];
#pragma unroll
  for (int i = 0; i < N; ++i) v[i] = i * kThreads + tid < CF::NPARAMS ? params[i * kThreads + tid] : 0.0f;
  uint4* z = reinterpret_cast<uint4*>(g_lds);
  for (int e = tid; e < (CF::L_X + CF::PACK) / 16; e += kThreads) z[e] = make_uint4(0u, 0u, 0u, 0u);
  __syncthreads();
  auto put = [&](int frag_base, int nf, int r, int i, int g, int j, El w) {
    // row r of a packed matrix whose first fragment is at byte frag_base
    *reinterpret_cast<El*>(g_lds + frag_base + ((r >> 5) * nf + i) * 1024 + ((r & 31) + 32 * g) * 16 + j * CF::EB) = w;
  };
  auto pos_d = [](int k, int& i, int& g, int& j) {
    i = BF ? k >> 4 : k >> 3;
    g = (k >> 2) & 1;
    j = BF ? ((k >> 1) & 4) | (k & 3) : k & 3;
  };
  static_for<N>([&](auto ic) {
    constexpr int it = decltype(ic)::value;
    const int idx = it * kThreads + tid;
    static_for<CF::NH + 1>([&](auto lc) {
      constexpr int l = decltype(lc)::value;
      constexpr int PW = CF::par_w(l), PB = CF::par_b(l), IR = CF::in_r(l), OR = CF::out_r(l);
      if constexpr (PW < (it + 1) * kThreads && PB > it * kThreads) {
        if (idx >= PW && idx < PB) {
          const int m = (idx - PW) / IR, k = (idx - PW) % IR;
          const El w = to_el<BF>(v[it]);
          int i, g, j;
          if constexpr (l == 0) {
            i = BF ? k >> 4 : k >> 3;
            g = BF ? (k >> 3) & 1 : (k >> 2) & 1;
            j = BF ? k & 7 : k & 3;
          } else {
            pos_d(k, i, g, j);
          }
          if constexpr (l == CF::NH)
            *reinterpret_cast<El*>(g_lds + CF::L_W3 + (m * 2 * CF::NFH + 2 * i + g) * 16 + j * CF::EB) = w;
          else
            put(CF::L_X + CF::pk_fwd(l) * 1024, l == 0 ? CF::NF0 : CF::NFH, m, i, g, j, w);
          pos_d(m, i, g, j);
          if constexpr (!CF::BWD) {
          } else if constexpr (l == 0) {
            if (k < CF::C) put(CF::L_B0, CF::NFH, k, i, g, j, w);
          } else {
            put(CF::L_X + CF::pk_bwd(l) * 1024, l == CF::NH ? 1 : CF::NFH, k, i, g, j, w);
          }
        }
      }
      if constexpr (PB < (it + 1) * kThreads && PB + OR > it * kThreads) {
        if (idx >= PB && idx < PB + OR)
          *reinterpret_cast<float*>(g_lds + CF::L_BIAS + (l * CF::H + idx - PB) * 4) = v[it];
      }
    });
  });
  __syncthreads();
}

template <int N>
__device__ __forceinline__ void lds_frags(frag_t (&w)[N], int base, int mt, int lane) {
#pragma unroll
  for (int i = 0; i < N; ++i) w[i] = *reinterpret_cast<const frag_t*>(g_lds + base + ((mt * N + i) * 64 + lane) * 16);
}

__device__ __forceinline__ f32x16 lds_bias(int base, int g) {
  f32x16 t;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(g_lds + base + (8 * q + 4 * g) * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) t[4 * q + e] = v[e];
  }
  return t;
}

// dw += (tile ta of A)^T x (tile tb of B) over the 16-hit steps [k0, k1);
// bs += the sum of A's row, added up by step and window first: bs runs over the
// whole launch (2^19 equal hits added to it one by one came out 265 x 2^-24 off,
// 4.4 so).
template <bool BF, int ROWA, int ROWB>
__device__ __forceinline__ void dw_steps(f32x16& dw, float& bs, int base_a, int ta, int base_b, int tb, int k0, int k1,
                                         int lane) {
  lane = here(lane);
  float win = 0.0f;
  for (int k = k0; k < k1; ++k) {
    float sum = 0.0f;
    if constexpr (BF) {
      const s16x8 a = hits_operand_bf16<ROWA>(base_a, ta, k, lane);
      dw = mma(a, hits_operand_bf16<ROWB>(base_b, tb, k, lane), dw);
#pragma unroll
      for (int j = 0; j < 8; ++j) sum += bf16_f32(static_cast<uint16_t>(a[j]));
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = hits_operand_fp32<ROWA>(base_a, ta, 8 * k + j, lane);
        dw = mma(a, hits_operand_fp32<ROWB>(base_b, tb, 8 * k + j, lane), dw);
        sum += a;
      }
    }
    win += sum;
  }
  bs += win;
}

// The forward weights of a wave: its 32 features of every hidden layer.
template <class CF>
struct Weights {
  frag_t w0[CF::NF0], wh[CF::NH - 1][CF::NFH];
  __device__ __forceinline__ void load(int mg, int lane) {
    lds_frags(w0, CF::L_X, mg, lane);
    static_for<CF::NH - 1>([&](auto lc) {
      constexpr int l = decltype(lc)::value + 1;
      lds_frags(wh[l - 1], CF::L_X + CF::pk_fwd(l) * 1024, mg, lane);
    });
  }
};

// The last hidden layer's activations of a wave's hits as operand fragments,
// where they stay in registers (Cfg::REG).
template <class CF>
using Frags = frag_t[CF::REG ? CF::NFH : 1];

// Hidden layers of the window's first tp hits (a multiple of 64): wave (mg, ng)
// computes its features of its hits.  Called by all threads; ends with a
// barrier.  REG: a wave owns its hits' whole rows and reads back only what its
// lanes wrote, so the activations stay in registers, and there is no barrier.
template <class CF>
__device__ __forceinline__ void hidden_layers(const Weights<CF>& W, int tp, int mg, int ng, int lane, Frags<CF>& act) {
  constexpr bool BF = CF::BF;
  constexpr int TPW = CF::TPW;
  const int g = lane >> 5, t0 = TPW * ng;
  const bool mine = 32 * t0 < tp;
  static_for<CF::NH>([&](auto lc) {
    constexpr int l = decltype(lc)::value;
    constexpr int SRC = CF::L_ACT + CF::act_of(l > 0 ? l - 1 : 0) * CF::ACT, DST = CF::L_ACT + CF::act_of(l) * CF::ACT;
    constexpr bool IN_PLACE = l > 0 && SRC == DST && CF::MG > 1;   // all waves have read before any writes
    f32x16 acc[TPW];
    if (mine) {
      const int ln = here(lane), hit = 32 * t0 + (ln & 31);
      const f32x16 b = lds_bias(CF::L_BIAS + (l * CF::H + 32 * mg) * 4, g);
#pragma unroll
      for (int t = 0; t < TPW; ++t) acc[t] = b;
      if constexpr (l == 0) {
#pragma unroll
        for (int i = 0; i < CF::NF0; ++i)
#pragma unroll
          for (int t = 0; t < TPW; ++t)
            acc[t] = mma_frag<BF>(W.w0[i], frag_at<CF::ROWX>(CF::L_X, hit + 32 * t, 2 * i + g), acc[t]);
      } else {
#pragma unroll
        for (int i = 0; i < CF::NFH; ++i)
#pragma unroll
          for (int t = 0; t < TPW; ++t)
            acc[t] = mma_frag<BF>(W.wh[l - 1][i], CF::REG ? act[CF::REG ? i : 0] : frag_at<CF::ROWH>(SRC, hit + 32 * t, 2 * i + g),
                                  acc[t]);
      }
    }
    if constexpr (IN_PLACE) __syncthreads();
    if (mine) {
#pragma unroll
      for (int t = 0; t < TPW; ++t) {
        relu16(acc[t]);
        if constexpr (CF::REG) {
#pragma unroll
          for (int q = 0; q < CF::NFH; ++q) act[q] = pack_chunk<BF>(acc[t], q);
        } else {
          store_tile<BF, CF::ROWH>(DST, mg, 32 * (t0 + t) + (lane & 31), g, acc[t]);
        }
      }
    }
    if constexpr (!CF::REG) __syncthreads();
  });
}

// Output layer of the 32 hits from n0: raw o_0 .. o_3 of hit n0 + lane in
// registers 0 .. 3 of lanes 0 .. 31.
template <class CF>
__device__ __forceinline__ f32x16 output_layer(int n0, int lane, const Frags<CF>& act) {
  const int ln = here(lane), g = lane >> 5;
  f32x16 o = lds_bias(CF::L_BIAS + CF::NH * CF::H * 4, g);
#pragma unroll
  for (int i = 0; i < CF::NFH; ++i) {
    frag_t wf = {0, 0, 0, 0};
    if ((ln & 31) < 4) wf = *reinterpret_cast<const frag_t*>(g_lds + CF::L_W3 + ((ln & 31) * 2 * CF::NFH + 2 * i + g) * 16);
    o = mma_frag<CF::BF>(wf, CF::REG ? act[CF::REG ? i : 0] : frag_at<CF::ROWH>(CF::L_LAST, n0 + (ln & 31), 2 * i + g), o);
  }
  return o;
}

template <class CF>
__global__ __launch_bounds__(kThreads, CF::BLOCKS) void k_shade(ShadeArgs a) {
  constexpr bool BF = CF::BF;
  constexpr int H = CF::H, NH = CF::NH, MG = CF::MG, TPW = CF::TPW, NB = CF::BWD ? NH - 1 : 1;
  using El = typename CF::El;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, row = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mg = wave % MG, ng = wave / MG;
  int* scr = reinterpret_cast<int*>(g_lds + CF::L_SCR);
  float* out = reinterpret_cast<float*>(g_lds + CF::L_OUT);
  uint16_t* imap = reinterpret_cast<uint16_t*>(g_lds + CF::L_MAP);

  // this wave's weights, for the launch
  Weights<CF> W;
  frag_t bh[NB][CF::NFH], bo[1];               // transposed, backward
  build_packs<CF>(a.params);
  W.load(mg, lane);
  if constexpr (CF::BWD) {
    static_for<NH - 1>([&](auto lc) {
      constexpr int l = decltype(lc)::value + 1;
      lds_frags(bh[l - 1], CF::L_X + CF::pk_bwd(l) * 1024, mg, lane);
    });
    lds_frags(bo, CF::L_X + CF::pk_bwd(NH) * 1024, mg, lane);
  }
  __syncthreads();

  // Decoder gradients.  H = 64: wave (mg, ng) owns tile (mg, ng) of a hidden
  // layer, over all hits; H = 32 (one tile) and the output layer: every wave
  // sums its own hits.
  f32x16 dwh[NB], dw0 = zero16(), dwo = zero16();
#pragma unroll
  for (int l = 0; l < NB; ++l) dwh[l] = zero16();
  float bs[NH], gob[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
  for (int l = 0; l < NH; ++l) bs[l] = 0.0f;
  float loss_acc = 0.0f;

  int rb = 0, pend_tw = 0;
  float* pend_grad = nullptr;
  auto ids = [&](int b) { return reinterpret_cast<int4*>(g_lds + CF::L_ID + b * CF::WIN * 32); };
  auto us = [&](int b) { return reinterpret_cast<float*>(g_lds + CF::L_U + b * CF::WIN * 12); };
  auto share = [&](int b) { return reinterpret_cast<uint8_t*>(g_lds + CF::L_SHARE + b * CF::WIN); };
  // The feature gradients of a window's hits: the lanes of one atomic
  // instruction cover whole feature rows (lane = channel).  A group of C lanes
  // takes GH consecutive hits; what a hit adds to a corner that the ray's next
  // hit has as well is carried over and added there (CornerCarry).
  constexpr int HW = CF::WIN / kWaves, GH = HW * CF::C / 64;   // hits per wave, per lane group
  auto scatter = [&](int b) {
    const int c = lane % CF::C, h0 = HW * wave + GH * (lane / CF::C);
    const int4* id = ids(b);
    const float* u = us(b);
    CornerCarry carry;
    for (int hh = h0; hh < h0 + GH; ++hh) {
      if (hh < pend_tw) {
        const int4 v0 = id[hh], v1 = id[CF::WIN + hh];
        const int vid[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        float w[8];
        trilinear(u[hh], u[CF::WIN + hh], u[2 * CF::WIN + hh], w);
        const float gv = *reinterpret_cast<const float*>(tile_at<CF::ROWG>(CF::L_GX, hh, c >> 2) + (c & 3) * 4);
#pragma unroll
        for (int j = 0; j < 8; ++j) carry.v[j] += w[j] * gv;
        carry.flush(share(b)[hh], [&](int j, float x) {
          unsafeAtomicAdd(pend_grad + static_cast<int64_t>(vid[j]) * CF::C + c, x);
        });
      }
    }
    pend_tw = 0;
  };

  // work items over the live rays, or over all
  const bool compact = a.tab.live_n != nullptr;
  LiveRays lr = {};
  if (compact) lr = live_rays(a.tab, scr);
  int* ray_ids = reinterpret_cast<int*>(g_lds + CF::L_MAP + kLiveItemRays * a.K * 2);
  ItemDeal deal(compact ? lr.items : a.tab.n_items, a.item_counter);
  for (int item = deal.first(scr); item < deal.nb; item = deal.next(item, scr)) {
    const DevScene& sc = a.tab.s[compact ? 0 : scene_of(a.tab, item)];
    const ItemRays ir = item_rays(a.tab, sc, item);
    int64_t r;
    bool live;
    if (compact) {
      const int q = find_rays(a.tab, lr, item, reinterpret_cast<int*>(g_lds + CF::L_X), ray_ids);
      r = sc.ray_begin + q;
      live = q >= 0;
    } else {
      r = ir.ray(tid);
      live = tid < ir.n && r < sc.ray_end;
    }
    auto ray_of = [&](int lane) { return compact ? sc.ray_begin + ray_ids[lane] : ir.ray(lane); };
    const int count = live ? a.cnt[r] : 0;
    // the ray's target (train) or upstream gradient (backward)
    float tg0 = 0.0f, tg1 = 0.0f, tg2 = 0.0f, tg3 = 0.0f, tg4 = 0.0f;
    if (CF::MODE == kTrain && live) {
      tg0 = a.t_rgb[3 * r]; tg1 = a.t_rgb[3 * r + 1]; tg2 = a.t_rgb[3 * r + 2]; tg3 = a.t_depth[r];
    } else if (CF::MODE == kBackward && live) {
      tg0 = a.g_rgb[3 * r]; tg1 = a.g_rgb[3 * r + 1]; tg2 = a.g_rgb[3 * r + 2]; tg3 = a.g_depth[r];
      tg4 = a.g_acc ? a.g_acc[r] : 0.0f;
    }
    const float h = __int_as_float((128 - sc.depth) << 23);       // 2^(1-depth)
    const float inv_h = __int_as_float((126 + sc.depth) << 23);   // 2^(depth-1)
    int total;
    const int off = block_excl_scan<kWaves>(count, scr, total, [&](int o) {
      for (int q = 0; q < count; ++q) imap[o + q] = static_cast<uint16_t>(tid | (q << 8));
    });
    float cr = 0.0f, cg = 0.0f, cb = 0.0f, dep = 0.0f, acc_w = 0.0f;
    for (int s0 = 0; s0 < total;) {
      bool in_win;
      const int s1 = open_window<CF::WIN>(s0, total, off, count, imap, in_win);
      const uint16_t* wmap = imap + s0;
      const int tw = s1 - s0;
      const int tp = (tw + 63) & ~63;              // rows that the layers touch
      // records: one thread per hit
      if (tid < tp) {
        float rd[3] = {0.0f, 0.0f, 0.0f};
        int mp = -1;
        uint32_t ijk = 0;
        if (tid < tw) {
          mp = wmap[tid];
          const int64_t ray = ray_of(mp & 0xFF);
          const HitRec hr = a.hits[ray * a.K + (mp >> 8)];
          const float ro[3] = {a.o[3 * ray], a.o[3 * ray + 1], a.o[3 * ray + 2]};
          rd[0] = a.d[3 * ray]; rd[1] = a.d[3 * ray + 1]; rd[2] = a.d[3 * ray + 2];
          const int4* lc = reinterpret_cast<const int4*>(sc.leaf_corners + 8 * static_cast<int64_t>(hr.leaf));
          ids(rb)[tid] = lc[0];
          ids(rb)[CF::WIN + tid] = lc[1];
          float tm, tml;
          midpoint2(hr.tin, hr.tout, tm, tml);
          const float lo[3] = {-1.0f + static_cast<float>(hr.ijk & 1023u) * h,
                               -1.0f + static_cast<float>((hr.ijk >> 10) & 1023u) * h,
                               -1.0f + static_cast<float>(hr.ijk >> 20) * h};
#pragma unroll
          for (int x = 0; x < 3; ++x)
            us(rb)[x * CF::WIN + tid] = clamp01(cell_coord(ro[x], rd[x], tm, tml, lo[x], inv_h));
          out[8 * tid + 6] = tm;
          out[8 * tid + 7] = hr.tout - hr.tin;
          ijk = hr.ijk;
        }
        if constexpr (CF::BWD) {       // (a lane group's last hit hands nothing on)
          const uint32_t sh = shared_corners(mp, ijk);
          share(rb)[tid] = static_cast<uint8_t>((tid & (GH - 1)) == GH - 1 ? 0u : sh);
        }
        // view direction and zero padding up to the K steps
        constexpr int V = kRowVals<BF>;
        if constexpr (CF::CI > CF::C) {
          float x[CF::CI - CF::C];
#pragma unroll
          for (int i = 0; i < CF::CI - CF::C; ++i) x[i] = CF::VD && i < 3 ? rd[i] : 0.0f;
#pragma unroll
          for (int i = 0; i < (CF::CI - CF::C) / V; ++i)
            *reinterpret_cast<frag_t*>(tile_at<CF::ROWX>(CF::L_X, tid, CF::C / V + i)) = pack_row<BF>(x + V * i);
        }
      }
      __syncthreads();
      {
        // thread q of a hit owns VPT channels of the interpolated feature
        constexpr int VPT = kRowVals<BF>, TPH = CF::C / VPT, HPP = kThreads / TPH;
        const int q = tid % TPH;
#pragma unroll
        for (int p = 0; p < (CF::WIN + HPP - 1) / HPP; ++p) {
          const int hh = p * HPP + tid / TPH;
          if (hh >= tp) break;
          float v[VPT];
#pragma unroll
          for (int i = 0; i < VPT; ++i) v[i] = 0.0f;
          if (hh < tw) {
            const int4 v0 = ids(rb)[hh], v1 = ids(rb)[CF::WIN + hh];
            const int vid[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
            uint4 raw[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) raw[j] = load_row<BF>(sc, 0, static_cast<int64_t>(vid[j]) * CF::C + VPT * q);
            float w[8];
            trilinear(us(rb)[hh], us(rb)[CF::WIN + hh], us(rb)[2 * CF::WIN + hh], w);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              float f[VPT];
              unpack_row<BF>(raw[j], f);
#pragma unroll
              for (int i = 0; i < VPT; ++i) v[i] += w[j] * f[i];
            }
          }
          *reinterpret_cast<frag_t*>(tile_at<CF::ROWX>(CF::L_X, hh, q)) = pack_row<BF>(v);
        }
      }
      __syncthreads();
      if (CF::DEFER && pend_tw > 0) scatter(rb ^ 1);

      Frags<CF> act;
      hidden_layers<CF>(W, tp, mg, ng, lane, act);
      const int t0 = TPW * ng;                     // first tile of this wave's hits
      const bool mine = 32 * t0 < tp;
      (void)mine;
      // output layer, split by hits; per hit the colour, opacity and
      // transmittance factor of the segment (section 4 footnote, Eq. 3)
      const int n0 = 32 * wave;
      const bool has_tile = wave < CF::NT && n0 < tw;
      if (has_tile) {
        const f32x16 o = output_layer<CF>(n0, lane, act);
        if (g == 0 && n0 + row < tw) {
          float* hp = out + 8 * (n0 + row);
          const float tmid = hp[6], dt = hp[7];
          const float ft = a.tau_mode == SVLF_TAU_VOXEL ? dt * inv_h
                           : a.tau_mode == SVLF_TAU_WORLD ? dt : 1.0f;
          const float tau = fmaxf(o[3], 0.0f) * ft;
          *reinterpret_cast<f32x4*>(hp) = f32x4{sigmoidf_(o[0]), sigmoidf_(o[1]), sigmoidf_(o[2]), -expm1f(-tau)};
          *reinterpret_cast<f32x4*>(hp + 4) = f32x4{expf(-tau), o[3] > 0.0f ? ft : 0.0f, tmid, 0.0f};
        }
      }
      __syncthreads();

      // Eq. 3 front to back (owner lanes), and its backward: dL/do, kept
      // [output][hit] in the operand type
      if (in_win) {
        const int p0 = off - s0;
        float T = 1.0f;
        for (int q = 0; q < count; ++q) {
          float* hp = out + 8 * (p0 + q);
          const f32x4 va = *reinterpret_cast<const f32x4*>(hp);
          const f32x4 vb = *reinterpret_cast<const f32x4*>(hp + 4);
          const float w = T * va[3];
          cr += w * va[0];
          cg += w * va[1];
          cb += w * va[2];
          dep += w * vb[2];
          if constexpr (CF::BWD) hp[7] = T;
          else acc_w += w;
          T *= vb[0];
        }
        if constexpr (CF::BWD) {
          float gr, gg, gb, gd, ga;
          if (CF::MODE == kTrain) {
            const float er = cr - tg0, eg = cg - tg1, eb = cb - tg2, ed = dep - tg3;
            const float k2 = a.loss_scale * (2.0f / 3.0f);
            gr = k2 * er;
            gg = k2 * eg;
            gb = k2 * eb;
            gd = a.loss_scale * a.lambda_depth * (ed > 0.0f ? 1.0f : (ed < 0.0f ? -1.0f : 0.0f));
            ga = 0.0f;
          } else {
            gr = tg0;
            gg = tg1;
            gb = tg2;
            gd = tg3;
            ga = tg4;
          }
          float Sr = 0.0f, Sg = 0.0f, Sb = 0.0f, St = 0.0f, Sa = 0.0f;
          for (int q = count - 1; q >= 0; --q) {
            const float* hp = out + 8 * (p0 + q);
            const f32x4 va = *reinterpret_cast<const f32x4*>(hp);
            const f32x4 vb = *reinterpret_cast<const f32x4*>(hp + 4);
            const float Tq = vb[3];
            const float w = Tq * va[3];
            const float Tn = Tq * vb[0];
            const float c0 = va[0], c1 = va[1], c2 = va[2], tm = vb[2];
            const float gtau = gr * (Tn * c0 - Sr) + gg * (Tn * c1 - Sg) + gb * (Tn * c2 - Sb) +
                               gd * (Tn * tm - St) + ga * (Tn - Sa);
            Sr += w * c0;
            Sg += w * c1;
            Sb += w * c2;
            St += w * tm;
            Sa += w;
            const float go[4] = {gr * w * c0 * (1.0f - c0), gg * w * c1 * (1.0f - c1), gb * w * c2 * (1.0f - c2),
                                 gtau * vb[1]};
#pragma unroll
            for (int c = 0; c < 4; ++c) {
              const El e = to_el<BF>(go[c]);
              *reinterpret_cast<El*>(g_lds + CF::L_GO + c * CF::GOS + (p0 + q) * CF::EB) = e;
              gob[c] += BF ? bf16_f32(static_cast<uint16_t>(e)) : static_cast<float>(e);
            }
          }
        }
      }
      if constexpr (CF::BWD) {
        if (tid >= tw && tid < tp) {
#pragma unroll
          for (int c = 0; c < 4; ++c) *reinterpret_cast<El*>(g_lds + CF::L_GO + c * CF::GOS + tid * CF::EB) = to_el<BF>(0.0f);
        }
        __syncthreads();

        // output layer: weight gradient over this wave's hits, then dL/dz of the
        // last hidden layer in place of its activations (own hits and features)
        constexpr int ALAST = CF::L_GX;
        const int ks = (tw + 15) >> 4;               // 16-hit steps with hits
        const int k0 = 2 * t0, k1 = k0 + 2 * TPW < ks ? k0 + 2 * TPW : ks;
        if (mine) {
          const int ln = here(lane), n = ln & 31;
          for (int k = k0; k < k1; ++k) {
            if constexpr (BF) {
              s16x8 b = {0, 0, 0, 0, 0, 0, 0, 0};
              if (n < 4) b = *reinterpret_cast<const s16x8*>(g_lds + CF::L_GO + n * CF::GOS + (16 * k + 8 * g) * 2);
              dwo = mma(hits_operand_bf16<CF::ROWH>(ALAST, mg, k, ln), b, dwo);
            } else {
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                const int st = 8 * k + j;
                const float b = n < 4 ? *reinterpret_cast<const float*>(g_lds + CF::L_GO + n * CF::GOS + (2 * st + g) * 4) : 0.0f;
                dwo = mma(hits_operand_fp32<CF::ROWH>(ALAST, mg, st, ln), b, dwo);
              }
            }
          }
#pragma unroll
          for (int t = 0; t < TPW; ++t) {
            const int hit = 32 * (t0 + t) + (ln & 31);
            frag_t gb = {0, 0, 0, 0};
            if (g == 0) {
              El e[4];
#pragma unroll
              for (int c = 0; c < 4; ++c) e[c] = *reinterpret_cast<const El*>(g_lds + CF::L_GO + c * CF::GOS + hit * CF::EB);
              if constexpr (BF) {
                gb[0] = static_cast<int>(e[0] | (static_cast<uint32_t>(e[1]) << 16));
                gb[1] = static_cast<int>(e[2] | (static_cast<uint32_t>(e[3]) << 16));
              } else {
#pragma unroll
                for (int c = 0; c < 4; ++c) gb[c] = __float_as_int(e[c]);
              }
            }
            mask_store_tile<BF, CF::ROWH>(ALAST, mg, hit, g, mma_frag<BF>(bo[0], gb, zero16()));
          }
        }
        if constexpr (MG > 1) __syncthreads();
        // hidden layers, last first: weight gradient (reads the layer's
        // inputs), then dL/dz of the layer below in place of those inputs.
        // H = 32: a wave's hits are its own throughout, no barriers.
        static_for<NH - 1>([&](auto lc) {
          constexpr int l = NH - 1 - decltype(lc)::value;
          constexpr int GZ = CF::L_ACT + l * CF::ACT, IN = CF::L_ACT + (l - 1) * CF::ACT;
          if constexpr (MG > 1) {
            dw_steps<BF, CF::ROWH, CF::ROWH>(dwh[l - 1], bs[l], GZ, mg, IN, ng, 0, ks, lane);
            __syncthreads();
          } else if (mine) {
            dw_steps<BF, CF::ROWH, CF::ROWH>(dwh[l - 1], bs[l], GZ, 0, IN, 0, k0, k1, lane);
          }
          if (mine) {
            const int ln = here(lane), hit = 32 * t0 + (ln & 31);
            f32x16 acc[TPW];
#pragma unroll
            for (int t = 0; t < TPW; ++t) acc[t] = zero16();
#pragma unroll
            for (int i = 0; i < CF::NFH; ++i)
#pragma unroll
              for (int t = 0; t < TPW; ++t)
                acc[t] = mma_frag<BF>(bh[l - 1][i], frag_at<CF::ROWH>(GZ, hit + 32 * t, 2 * i + g), acc[t]);
#pragma unroll
            for (int t = 0; t < TPW; ++t) mask_store_tile<BF, CF::ROWH>(IN, mg, hit + 32 * t, g, acc[t]);
          }
          if constexpr (MG > 1) __syncthreads();
        });
        // input layer: weight gradient; dL/dx of the features, split by hits
        if constexpr (MG > 1) {
          if (ng < CF::NTX) dw_steps<BF, CF::ROWH, CF::ROWX>(dw0, bs[0], CF::L_ACT, mg, CF::L_X, ng, 0, ks, lane);
        } else {
          if (mine) dw_steps<BF, CF::ROWH, CF::ROWX>(dw0, bs[0], CF::L_ACT, 0, CF::L_X, 0, k0, k1, lane);
        }
        f32x16 gx = zero16();
        if (has_tile) {
          const int ln = here(lane);
#pragma unroll
          for (int i = 0; i < CF::NFH; ++i)
            gx = mma_frag<BF>(*reinterpret_cast<const frag_t*>(g_lds + CF::L_B0 + (i * 64 + ln) * 16),
                              frag_at<CF::ROWH>(CF::L_ACT, n0 + (ln & 31), 2 * i + g), gx);
        }
        if constexpr (MG == 1) __syncthreads();      // the last layer's tile is taken over
        if (has_tile) {
          const int hit = n0 + here(row);
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (8 * q < CF::C)
              *reinterpret_cast<frag_t*>(tile_at<CF::ROWG>(CF::L_GX, hit, 2 * q + g)) = pack_chunk<false>(gx, q);
          }
        }
        __syncthreads();
        if (a.gxu != nullptr) {
          // deterministic mode: keep (u, dL/dx) per hit slot; the feature
          // gradient is reduced afterwards in a fixed order
          constexpr int HPI = 64 / CF::C;
          const int c = lane % CF::C, hs = lane / CF::C;
          for (int k = 0; k < HW; k += HPI) {
            const int hh = HW * wave + k + hs;
            if (hh < tw) {
              const int mp = wmap[hh];
              float* rec = a.gxu + (ray_of(mp & 0xFF) * a.K + (mp >> 8)) * (CF::C + 4);
              rec[4 + c] = *reinterpret_cast<const float*>(tile_at<CF::ROWG>(CF::L_GX, hh, c >> 2) + (c & 3) * 4);
              if (c < 3) rec[c] = us(rb)[c * CF::WIN + hh];
            }
          }
        } else {
          pend_tw = tw;
          pend_grad = sc.grad;
          if (CF::DEFER) rb ^= 1;
          else scatter(rb);
        }
      }
      __syncthreads();
      s0 = s1;
    }

    if (CF::MODE != kBackward && live) {
      if (a.rgb) {
        a.rgb[3 * r] = cr;
        a.rgb[3 * r + 1] = cg;
        a.rgb[3 * r + 2] = cb;
      }
      if (a.depth) a.depth[r] = dep;
      if (!CF::BWD && a.acc) a.acc[r] = acc_w;
    }
    if (CF::MODE == kTrain && live) {
      const float er = cr - tg0, eg = cg - tg1, eb = cb - tg2, ed = dep - tg3;
      loss_acc += a.loss_scale * ((er * er + eg * eg + eb * eb) * (1.0f / 3.0f) + a.lambda_depth * fabsf(ed));
    }
  }
  // rays without hits that no item took
  if (compact && CF::MODE != kBackward) {
    const DevScene& sc = a.tab.s[0];
    for (int64_t r = sc.ray_begin + static_cast<int64_t>(blockIdx.x) * kThreads + tid; r < sc.ray_end;
         r += static_cast<int64_t>(gridDim.x) * kThreads) {
      if (a.cnt[r] != 0) continue;
      if (a.rgb) {
        a.rgb[3 * r] = 0.0f;
        a.rgb[3 * r + 1] = 0.0f;
        a.rgb[3 * r + 2] = 0.0f;
      }
      if (a.depth) a.depth[r] = 0.0f;
      if (!CF::BWD && a.acc) a.acc[r] = 0.0f;
      if (CF::MODE == kTrain) {
        const float er = a.t_rgb[3 * r], eg = a.t_rgb[3 * r + 1], eb = a.t_rgb[3 * r + 2], ed = a.t_depth[r];
        loss_acc += a.loss_scale * ((er * er + eg * eg + eb * eb) * (1.0f / 3.0f) + a.lambda_depth * fabsf(ed));
      }
    }
  }
  if constexpr (CF::BWD) {
    if (CF::DEFER && pend_tw > 0) scatter(rb ^ 1);

    // this block's partial sums of dL/dparams: the waves' shares are added in
    // LDS in a fixed order, then written out
    float* pb = reinterpret_cast<float*>(g_lds + CF::L_X);
    __syncthreads();
    for (int i = tid; i < CF::NPARAMS; i += kThreads) pb[i] = 0.0f;
    __syncthreads();
    const int n = lane & 31;
    const float gt = block_sum<kWaves>(loss_acc, reinterpret_cast<float*>(scr));
    for (int p = 0; p < CF::NG; ++p) {
      if (ng == p) {
        auto add_tile = [&](const f32x16& dw, int base, int stride, int mt, int col, bool ok) {
          if (ok) {
#pragma unroll
            for (int i = 0; i < 16; ++i) pb[base + (32 * mt + tile_feature<BF>(drow(i, g))) * stride + col] += dw[i];
          }
        };
        static_for<NH - 1>([&](auto lc) {
          constexpr int l = decltype(lc)::value + 1;
          add_tile(dwh[l - 1], CF::par_w(l), H, mg, (MG > 1 ? 32 * ng : 0) + tile_feature<BF>(n), true);
        });
        const int col0 = (MG > 1 ? 32 * ng : 0) + n;
        add_tile(dw0, CF::par_w(0), CF::CIN, mg, col0, col0 < CF::CIN && (MG == 1 || ng < CF::NTX));
        if (n < 4) {
#pragma unroll
          for (int i = 0; i < 16; ++i) pb[CF::par_w(NH) + n * H + 32 * mg + tile_feature<BF>(drow(i, g))] += dwo[i];
        }
        if (MG == 1 || ng == 0) {
          static_for<NH>([&](auto lc) {
            constexpr int l = decltype(lc)::value;
            const float v = bs[l] + __shfl_xor(bs[l], 32, 64);
            if (lane < 32) pb[CF::par_b(l) + 32 * mg + tile_feature<BF>(lane)] += v;
          });
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const float v = block_sum<kWaves>(gob[c], reinterpret_cast<float*>(scr));
      if (tid == 0) pb[CF::par_b(NH) + c] = v;
    }
    __syncthreads();
    float* part = a.ws_partials + static_cast<int64_t>(blockIdx.x) * CF::NPARAMS;
    for (int i = tid; i < CF::NPARAMS; i += kThreads) part[i] = pb[i];
    if (tid == 0) a.ws_loss[blockIdx.x] = CF::MODE == kTrain ? gt : 0.0f;
  }
}

// Decoder alone on rows of X (diagnostics / tests): one window of rows per
// block pass.
template <class CF>
__global__ __launch_bounds__(kThreads) void k_mlp_rows(const float* __restrict__ params,
                                                       const float* __restrict__ X, int64_t n,
                                                       float* __restrict__ out) {
  constexpr bool BF = CF::BF;
  constexpr int V = kRowVals<BF>;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int mg = wave % CF::MG, ng = wave / CF::MG;
  Weights<CF> W;
  build_packs<CF>(params);
  W.load(mg, lane);
  __syncthreads();
  for (int64_t base = static_cast<int64_t>(blockIdx.x) * CF::WIN; base < n;
       base += static_cast<int64_t>(gridDim.x) * CF::WIN) {
    for (int e = tid; e < CF::WIN * (CF::CI / V); e += kThreads) {
      const int hh = e / (CF::CI / V), q = e % (CF::CI / V);
      const int64_t r = base + hh;
      float x[V];
#pragma unroll
      for (int i = 0; i < V; ++i) x[i] = r < n && V * q + i < CF::CIN ? X[r * CF::CIN + V * q + i] : 0.0f;
      *reinterpret_cast<frag_t*>(tile_at<CF::ROWX>(CF::L_X, hh, q)) = pack_row<BF>(x);
    }
    __syncthreads();
    Frags<CF> act;
    hidden_layers<CF>(W, CF::WIN, mg, ng, lane, act);
    if (wave < CF::NT) {
      const f32x16 o = output_layer<CF>(32 * wave, lane, act);
      const int64_t r = base + 32 * wave + (lane & 31);
      if (g == 0 && r < n) {
#pragma unroll
        for (int c = 0; c < 4; ++c) out[4 * r + c] = o[c];
      }
    }
    __syncthreads();
  }
}

int num_cus() {
  static int n = 0;
  if (n == 0) {
    int dev = 0, v = 0;
    n = (hipGetDevice(&dev) == hipSuccess &&
         hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
            ? v
            : 256;
  }
  return n;
}

template <class CF>
hipError_t run(ShadeArgs a, hipStream_t s, int* grid_used) {
  const auto kern = k_shade<CF>;
  const int lds = CF::lds_bytes(a.K);
  // (the limit is the process's: one value for every K, so that threads cannot
  // lower it between each other's set and launch)
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, CF::lds_bytes(SVLF_MAX_K));
  if (e != hipSuccess) return e;
  // Resident blocks per CU by registers and LDS (the hit map grows with K): the
  // persistent grid must fit in one round, or the blocks of a second round
  // would run after the rest.
  static std::atomic<int> occ[SVLF_MAX_K + 1];
  int per_cu = occ[a.K].load(std::memory_order_relaxed);
  if (per_cu == 0) {
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern), kThreads, lds) !=
            hipSuccess || per_cu < 1)
      per_cu = 1;
    occ[a.K].store(per_cu, std::memory_order_relaxed);
  }
  int grid = num_cus() * per_cu;
  const int most = CF::BWD ? shade_grid_rows() : shade_grid_limit();
  if (grid > most) grid = most;
  plan_items(&a.tab, grid, CF::BWD);
  if (grid > a.tab.n_items) grid = a.tab.n_items;
  if (grid < 1) grid = 1;
  *grid_used = grid;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, a);
  return hipGetLastError();
}

template <int P, int C, int H, int NH, int VD>
hipError_t run_mode(const ShadeArgs& a, int mode, hipStream_t s, int* grid) {
  if (mode == kForward) return run<Cfg<P, C, H, NH, kForward, VD>>(a, s, grid);
  if (mode == kBackward) return run<Cfg<P, C, H, NH, kBackward, VD>>(a, s, grid);
  return run<Cfg<P, C, H, NH, kTrain, VD>>(a, s, grid);
}

template <int P, int C, int H, int NH, int VD>
hipError_t run_mlp(const float* params, const float* X, int64_t n, float* out, hipStream_t s) {
  using CF = Cfg<P, C, H, NH, kForward, VD>;
  const auto kern = k_mlp_rows<CF>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, CF::lds_bytes(1));
  if (e != hipSuccess) return e;
  int64_t blocks = (n + CF::WIN - 1) / CF::WIN;
  if (blocks > 4096) blocks = 4096;
  hipLaunchKernelGGL(kern, dim3(static_cast<unsigned>(blocks)), dim3(kThreads), CF::lds_bytes(1), s,
                     params, X, n, out);
  return hipGetLastError();
}

// Supported decoder shapes (C, H, hidden layers, view-direction input).
#define SVLF_SHAPES(X) \
  X(8, 32, 2, 0) X(16, 64, 3, 0) X(32, 64, 3, 0) X(8, 32, 2, 1) X(32, 64, 3, 1)

}  // namespace

// The partials' last 128 rows (of at least 1,476 floats) hold the live-ray
// arrays; up to three blocks per CU of 256 stay below them.
int shade_grid_limit() { return 1024; }
int shade_grid_rows() { return 896; }
static_assert(live_bytes(kMaxLiveRays) + 256 <= 128 * 1476 * sizeof(float), "live-ray arrays");

hipError_t launch_shade(const ShadeArgs& a, int mode, hipStream_t s, int* grid_used) {
  *grid_used = 0;
  const int P = a.precision == SVLF_BF16 ? 1 : 0;
  const int vd = a.viewdir ? 1 : 0;
#define SVLF_CASE(C_, H_, NH_, VD_)                                                    \
  if (a.C == C_ && a.H == H_ && a.n_hidden == NH_ && vd == VD_)                        \
    return P ? run_mode<1, C_, H_, NH_, VD_>(a, mode, s, grid_used)                    \
             : run_mode<0, C_, H_, NH_, VD_>(a, mode, s, grid_used);
  SVLF_SHAPES(SVLF_CASE)
#undef SVLF_CASE
  return hipErrorNotSupported;
}

hipError_t launch_mlp_forward(const float* params, int C, int H, int n_hidden, int viewdir,
                              int precision, const float* X, int64_t n, float* out,
                              hipStream_t s) {
  const int P = precision == SVLF_BF16 ? 1 : 0;
  const int vd = viewdir ? 1 : 0;
#define SVLF_CASE(C_, H_, NH_, VD_)                                                    \
  if (C == C_ && H == H_ && n_hidden == NH_ && vd == VD_)                              \
    return P ? run_mlp<1, C_, H_, NH_, VD_>(params, X, n, out, s)                      \
             : run_mlp<0, C_, H_, NH_, VD_>(params, X, n, out, s);
  SVLF_SHAPES(SVLF_CASE)
#undef SVLF_CASE
  return hipErrorNotSupported;
}

}  // namespace svlf
