// Shading kernels of the paper's voxel light-field function (SVLF sections
// 4.1-4.3): per crossed voxel, a density decoder F_T reads the features
// interpolated at the entry and exit points x1, x2 together with the ray
// parameterisation r (the two points where the ray meets the voxel's
// bounding sphere, as unit vectors from its centre) and outputs the optical
// thickness tau and the mixing factor eta; a colour decoder F_C reads the
// features interpolated at the surface point x_s = eta x1 + (1 - eta) x2 with
// r (and the view direction on request) and outputs the colour; Eq. 3
// composites front to back.
//
// Each scene's feature table holds the two embedding collections as two
// blocks, Z_T [n_vertices][64] followed by Z_C [n_vertices][32] (so that one
// of them can be trained or frozen as one contiguous array).  Decoder
// inputs are ordered [features | r | (d)].
//
// Three kernels, all persistent over work items with ray-aligned hit windows
// (as the single-decoder kernels):
//  * k_density: records, gather of the 8 corner rows of Z_T (one gather
//    serves x1 and x2: both lie on the same voxel), r, F_T on MFMA, and per
//    hit tau, eta and the surface point (written to the workspace); in
//    backward mode it recomputes F_T, back-propagates dL/d(o_T0, o_T1) left
//    by the colour kernel, accumulates F_T's weight gradients and scatters
//    dL/dZ_T;
//  * k_color: gather of Z_C at the surface point, F_C on MFMA, Eq. 3, and in
//    backward / train mode the compositing backward, F_C's backward, the
//    scatter of dL/dZ_C, and dL/deta through the interpolation at x_s;
//  * k_lf_pack: MFMA operand packs of both decoders (forward and transposed)
//    from the FP32 masters.
//
// Decoder organisation.  A hidden layer is 128 x 128: its weights are far too
// many for one wave, and reading them from L2 for every 32-hit tile left the
// matrix cores idle behind the loads (and, in the backward, behind the
// gradient atomics that the vector-memory counter orders before them).  So
// the layer is split over the block's four waves by OUTPUT features: wave w
// owns features [32 w, 32 w + 32) of every hidden layer, for all hits of the
// window.
//  * the wave's share of a layer is 32 VGPRs in BF16 and 64 in FP32; it stays in
//    registers for the launch where they suffice (BF16 but the colour
//    backward) and is read once per window otherwise;
//  * activations pass through LDS, [hit][feature] in 16-byte chunks that are
//    MFMA operands as they stand (Tile), written once and read by all waves;
//  * weight gradients: wave w owns the rows of its features, accumulated in
//    registers over the whole launch; the operands need the hits along K, so
//    BF16 reads the same tiles through the LDS transpose read
//    (ds_read_b64_tr_b16) and FP32 reads them as they are;
//  * dL/dz of a layer overwrites that layer's activations in place (a wave
//    masks and replaces its own features);
//  * the narrow ends (decoder outputs, dL/dx) are split by hits instead.
// Measured against waves that each ran the whole decoder on their own hits with
// the weights read from L2 (2^20 rays, 1.41 M hits, kernel times in ms): colour
// train BF16 4.95 -> 1.97, FP32 31.0 -> 6.5; density backward 3.40 -> 1.67, 9.2
// -> 3.6; density forward 0.68 -> 0.42, 2.58 -> 1.55; colour forward of a 1600^2
// view 0.89 -> 0.61, 5.0 -> 3.2.  BF16 training is now bound by the gradient
// rows' atomics (about half of the density backward's time), FP32 by the matrix
// cores (32 to 61% busy) at one block per CU in the backward.  The colour kernels
// spill: 7 to 15 registers forward in FP32, up to 30 in the backward.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "svlf_internal.hpp"
#include "tiles.hpp"

namespace svlf {
namespace {

using namespace detail;

// ------------------------------------------------------------ decoder geometry

// A ReLU MLP IN0 -> H (NH hidden layers) -> OUT (<= 32); BM0 = number of
// leading inputs whose gradient is needed (the features).
template <bool BF, int IN0_, int H_, int NH_, int OUT_, int BM0_>
struct Mlp {
  static constexpr int IN0 = IN0_, H = H_, NH = NH_, OUT = OUT_, BM0 = BM0_;
  static constexpr int KS = BF ? 16 : 2;
  static constexpr int NL = NH + 1;
  static constexpr int IN0P = BF ? align16(IN0) : align8(IN0);
  static constexpr int MTH = H / 32;
  static constexpr int in_r(int l) { return l == 0 ? IN0 : H; }
  static constexpr int in_p(int l) { return l == 0 ? IN0P : H; }
  static constexpr int out_r(int l) { return l == NH ? OUT : H; }
  static constexpr int out_p(int l) { return l == NH ? 32 : H; }
  static constexpr int bm(int l) { return l == 0 ? BM0 : H; }
  static constexpr int fwd_off(int l) {
    int o = 0;
    for (int i = 0; i < l; ++i) o += out_p(i) * in_p(i);
    return o;
  }
  static constexpr int bwd_off(int l) {
    int o = 0;
    for (int i = 0; i < l; ++i) o += bm(i) * out_p(i);
    return o;
  }
  static constexpr int bias_off(int l) {
    int o = 0;
    for (int i = 0; i < l; ++i) o += out_p(i);
    return o;
  }
  static constexpr int par_w(int l) {
    int o = 0;
    for (int i = 0; i < l; ++i) o += out_r(i) * in_r(i) + out_r(i);
    return o;
  }
  static constexpr int par_b(int l) { return par_w(l) + out_r(l) * in_r(l); }
  static constexpr int dw_mt(int l) { return out_p(l) / 32; }
  static constexpr int dw_nt(int l) { return align32(in_r(l)) / 32; }
  static constexpr int dw_off(int l) {
    int o = 0;
    for (int i = 0; i < l; ++i) o += dw_mt(i) * dw_nt(i);
    return o;
  }
  static constexpr int NPARAMS = par_w(NL);
  static constexpr int FWD = fwd_off(NL);
  static constexpr int BWD = bwd_off(NL);
  static constexpr int BIAS = bias_off(NL);
  static constexpr int NDW = dw_off(NL);
  static constexpr int NBIAS = NH * H + OUT;
  // pack layout (elements of the operand type, then FP32 biases)
  static constexpr size_t pack_bytes(int eb) {
    return ((static_cast<size_t>(FWD + BWD) * eb + 15) / 16) * 16 + BIAS * 4;
  }
  static_assert(OUT <= 32 && H % 32 == 0 && BM0 % 32 == 0 && BM0 <= IN0, "geometry");
};

template <bool BF, int VD>
struct Dec {
  using T = Mlp<BF, 2 * kLfCT + 6, kLfH, kLfNHT, 2, 2 * kLfCT>;
  using C = Mlp<BF, kLfCC + 6 + 3 * VD, kLfH, kLfNHC, 3, kLfCC>;
};

// Weight fragments are read with buffer loads: the per-fragment offset is a
// scalar (SGPR) and only the lane offset lives in a VGPR; loads past the end
// of the pack return 0.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pack_rsrc(const void* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, bytes, 0x00020000);
}
// fragments [0, N) of M tile mt of a packed matrix with NF fragments per tile
template <int N>
__device__ __forceinline__ void load_frags(frag_t (&w)[N], __amdgpu_buffer_rsrc_t rs, int byte_base,
                                           int mt, int NF, int lane) {
#pragma unroll
  for (int i = 0; i < N; ++i)
    w[i] = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(
                                          rs, lane * 16, byte_base + (mt * NF + i) * 1024, 0));
}

__device__ __forceinline__ f32x16 gbias(const float* __restrict__ b, int mt, int g) {
  f32x16 t;
  const float* p = b + 32 * mt + 4 * g;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 v = *reinterpret_cast<const float4*>(p + 8 * q);
    t[4 * q + 0] = v.x;
    t[4 * q + 1] = v.y;
    t[4 * q + 2] = v.z;
    t[4 * q + 3] = v.w;
  }
  return t;
}

// ------------------------------------------------------------ packing

// Packs one decoder from its FP32 layers (params) into [fwd][bwd] operand
// arrays (elements) followed by the padded biases (FP32).
template <bool BF, class M>
__device__ void pack_decoder(const float* __restrict__ params, char* __restrict__ out) {
  using El = typename Types<BF>::Elem;
  constexpr int E = BF ? 8 : 4;
  El* fp = reinterpret_cast<El*>(out);
  El* bp = fp + M::FWD;
  float* bias = reinterpret_cast<float*>(out + M::pack_bytes(Types<BF>::EB) - M::BIAS * 4);
  const int stride = gridDim.x * blockDim.x;
  const int t0 = blockIdx.x * blockDim.x + threadIdx.x;
  static_for<M::NL>([&](auto lc) {
    constexpr int l = decltype(lc)::value;
    constexpr int IW = M::in_p(l), OW = M::out_p(l), IR = M::in_r(l), OR = M::out_r(l);
    constexpr int STEPS = IW / kFragK<BF>;
    const float* W = params + M::par_w(l);
    const float* b = params + M::par_b(l);
    El* f = fp + M::fwd_off(l);
    for (int e = t0; e < OW * IW; e += stride) {
      const int j = e % E, lane = (e / E) % 64, s = (e / (E * 64)) % STEPS, mt = e / (E * 64 * STEPS);
      const int m = 32 * mt + (lane & 31), g = lane >> 5;
      const int k = (l == 0) ? kfrag_x<BF>(s, g, j) : kfrag_d<BF>(s, g, j);
      f[e] = to_el<BF>((m < OR && k < IR) ? W[m * IR + k] : 0.0f);
    }
    // transposed: M = layer input (the first bm(l) only), K = layer output
    constexpr int BM = M::bm(l), BSTEPS = OW / kFragK<BF>;
    El* bb = bp + M::bwd_off(l);
    for (int e = t0; e < BM * OW; e += stride) {
      const int j = e % E, lane = (e / E) % 64, s = (e / (E * 64)) % BSTEPS, mt = e / (E * 64 * BSTEPS);
      const int m = 32 * mt + (lane & 31), g = lane >> 5;
      const int k = kfrag_d<BF>(s, g, j);
      bb[e] = to_el<BF>((m < IR && k < OR) ? W[k * IR + m] : 0.0f);
    }
    for (int r = t0; r < OW; r += stride) bias[M::bias_off(l) + r] = r < OR ? b[r] : 0.0f;
  });
}

template <bool BF, int VD>
__global__ __launch_bounds__(kThreads) void k_lf_pack(const float* __restrict__ params,
                                                      char* __restrict__ packs) {
  using D = Dec<BF, VD>;
  pack_decoder<BF, typename D::T>(params, packs);
  pack_decoder<BF, typename D::C>(params + D::T::NPARAMS,
                                  packs + D::T::pack_bytes(Types<BF>::EB));
}

// Bounding-sphere parameterisation relative to the voxel centre, from the
// entry point's offset y1 = x1 - c (small: on the voxel boundary) and the
// direction d: the sphere |y1 + s d|^2 = R^2 with R^2 = 3 h^2 / 4.
__device__ __forceinline__ void sphere_r(float y0, float y1, float y2, float dx, float dy, float dz,
                                         float h, float (&r)[6]) {
  const float a = dx * dx + dy * dy + dz * dz;
  const float b = dx * y0 + dy * y1 + dz * y2;
  const float cx = dy * y2 - dz * y1, cy = dz * y0 - dx * y2, cz = dx * y1 - dy * y0;
  const float disc = a * (0.75f * h * h) - (cx * cx + cy * cy + cz * cz);
  const float sq = sqrtf(fmaxf(disc, 0.0f));
  const float sa = (-b - sq) / a, sb = (-b + sq) / a;
  const float p[2][3] = {{y0 + sa * dx, y1 + sa * dy, y2 + sa * dz},
                         {y0 + sb * dx, y1 + sb * dy, y2 + sb * dz}};
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float inv = 1.0f / sqrtf(p[k][0] * p[k][0] + p[k][1] * p[k][1] + p[k][2] * p[k][2]);
    r[3 * k + 0] = p[k][0] * inv;
    r[3 * k + 1] = p[k][1] * inv;
    r[3 * k + 2] = p[k][2] * inv;
  }
}

// ------------------------------------------------------------ layers

// One layer's share of this wave (fragments w) over the window's hits, 64 hits
// (two independent accumulators) at a time: done(t, acc) gets each 32-hit
// tile's result.
template <bool BF, int ROWB, int NT, int NF, class Done>
__device__ __forceinline__ void layer_mma(const f32x16& init, const frag_t (&w)[NF], int base, int tw, int lane,
                                          Done&& done) {
  lane = here(lane);
  const int row = lane & 31, g = lane >> 5;
  static_for<NT / 2>([&](auto pc) {
    constexpr int p = decltype(pc)::value;
    if (64 * p < tw) {
      f32x16 acc[2] = {init, init};
#pragma unroll
      for (int i = 0; i < NF; ++i) {
#pragma unroll
        for (int t = 0; t < 2; ++t)
          acc[t] = mma_frag<BF>(w[i], frag_at<ROWB>(base, 64 * p + 32 * t + row, 2 * i + g), acc[t]);
        if constexpr (!BF) __builtin_amdgcn_sched_barrier(0);
      }
      done(2 * p, acc[0]);
      done(2 * p + 1, acc[1]);
    }
  });
}

// dw[nt] += (tile ta of A)^T x (tile nt of B) over the window's hits (hits from
// tw to the next multiple of 16 are zero in one of the two and finite in the
// other); bs += the sum of A's row (the bias gradient, half of the hits in
// each lane group), added up by step and window first: bs runs over the whole
// launch.
template <bool BF, int ROWA, int ROWB, int NT>
__device__ __forceinline__ void dw_mma(f32x16 (&dw)[NT], float& bs, int base_a, int ta, int base_b, int tw, int lane) {
  lane = here(lane);
  float win = 0.0f;
#pragma unroll 1
  for (int k = 0; k < (tw + 15) >> 4; ++k) {
    float sum = 0.0f;
    if constexpr (BF) {
      const s16x8 a = hits_operand_bf16<ROWA>(base_a, ta, k, lane);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) dw[nt] = mma(a, hits_operand_bf16<ROWB>(base_b, nt, k, lane), dw[nt]);
#pragma unroll
      for (int j = 0; j < 8; ++j) sum += bf16_f32(static_cast<uint16_t>(a[j]));
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = hits_operand_fp32<ROWA>(base_a, ta, 8 * k + j, lane);
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) dw[nt] = mma(a, hits_operand_fp32<ROWB>(base_b, nt, 8 * k + j, lane), dw[nt]);
        sum += a;
      }
    }
    win += sum;
  }
  bs += win;
}

// The output layer's gradients are kept [output][hit] (row stride GOS bytes) as
// well: dw += (tile ta of A)^T x go^T, column n = output n < OUT.
template <bool BF, int ROWA, int OUT>
__device__ __forceinline__ void dw_out_mma(f32x16& dw, int base_a, int ta, int base_go, int gos, int tw, int lane) {
  lane = here(lane);
  const int n = lane & 31, g = lane >> 5;
#pragma unroll 1
  for (int k = 0; k < (tw + 15) >> 4; ++k) {
    if constexpr (BF) {
      s16x8 b = {0, 0, 0, 0, 0, 0, 0, 0};
      if (n < OUT) b = *reinterpret_cast<const s16x8*>(g_lds + base_go + n * gos + (16 * k + 8 * g) * 2);
      dw = mma(hits_operand_bf16<ROWA>(base_a, ta, k, lane), b, dw);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int st = 8 * k + j;
        const float b = n < OUT ? *reinterpret_cast<const float*>(g_lds + base_go + n * gos + (2 * st + g) * 4) : 0.0f;
        dw = mma(hits_operand_fp32<ROWA>(base_a, ta, st, lane), b, dw);
      }
    }
  }
}

// Block partials: dW tiles of a layer whose inputs are a hidden layer's tiles
// (HID) or the decoder's input columns, and the output layer's.
template <bool BF, class M, int l, bool HID, int NT>
__device__ __forceinline__ void write_dw(const f32x16 (&dw)[NT], float* __restrict__ part, int wave, int lane) {
  const int g = lane >> 5, n = lane & 31;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int col = 32 * nt + (HID ? tile_feature<BF>(n) : n);
    if (col < M::in_r(l)) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        part[M::par_w(l) + (32 * wave + tile_feature<BF>(drow(i, g))) * M::in_r(l) + col] = dw[nt][i];
    }
  }
}
template <bool BF, class M>
__device__ __forceinline__ void write_dw_out(const f32x16& dw, float* __restrict__ part, int wave, int lane) {
  const int g = lane >> 5, n = lane & 31;
  if (n < M::OUT) {
#pragma unroll
    for (int i = 0; i < 16; ++i)
      part[M::par_w(M::NH) + n * kLfH + 32 * wave + tile_feature<BF>(drow(i, g))] = dw[i];
  }
}
// Bias gradient of a hidden layer, from dw_mma's sums.
template <bool BF, class M, int l>
__device__ __forceinline__ void write_bias(float bs, float* __restrict__ part, int wave, int lane) {
  const float v = bs + __shfl_xor(bs, 32, 64);
  if (lane < 32) part[M::par_b(l) + 32 * wave + tile_feature<BF>(lane)] = v;
}
// Bias gradient of the output layer: per-lane sums of every wave, combined
// through LDS (kWaves x OUT floats at `lds`) in wave order.  Called by all threads.
template <class M>
__device__ __forceinline__ void write_bias_out(const float (&bo)[M::OUT], float* lds, float* __restrict__ part,
                                               int wave, int lane, int tid) {
  __syncthreads();
#pragma unroll
  for (int c = 0; c < M::OUT; ++c) {
    float v = bo[c];
#pragma unroll
    for (int m = 32; m > 0; m >>= 1) v += __shfl_xor(v, m, 64);
    if (lane == 0) lds[wave * M::OUT + c] = v;
  }
  __syncthreads();
  if (tid < M::OUT) {
    float v = 0.0f;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) v += lds[w * M::OUT + tid];
    part[M::par_b(M::NH) + tid] = v;
  }
  __syncthreads();
}

// ------------------------------------------------------------ density kernel

template <int P, int MODE>
struct DCfg {
  static constexpr bool BF = P == 1;
  static constexpr bool BWD = MODE != kForward;
  using M = typename Dec<BF, 0>::T;
  using El = typename Types<BF>::Elem;
  static constexpr int EB = Types<BF>::EB;
  static constexpr int WIN = BF ? 128 : 64;
  static constexpr int NT = WIN / 32;
  static constexpr int ROWH = kLfH * EB;                 // activations
  // decoder inputs; BF16: the last dW tile's columns past the row are the next
  // row's (finite, and of no gradient entry)
  static constexpr int ROWX = BF ? M::IN0P * 2 + 16 : align32(M::IN0) * 4;
  static constexpr int ROWG = 2 * kLfCT * 4;             // dL/dx, FP32
  static constexpr int NF0 = M::IN0P / kFragK<BF>, NFH = kLfH / kFragK<BF>;
  static constexpr int GOS = (WIN + 16 / EB) * EB;
  // Forward: the activations take the inputs' place (two blocks per CU).
  // Backward: dL/dx stays until the next window's inputs have been gathered,
  // so it and the records have areas of their own.
  static constexpr int L_X = 0;
  static constexpr int L_ACT = BWD ? L_X + WIN * ROWX : L_X;
  static constexpr int L_GX = L_X + WIN * ROWX + (BWD ? WIN * ROWH : 0);
  static constexpr int REC = 64;                         // bytes of a record
  static constexpr int L_REC = L_GX + (BWD ? WIN * ROWG : 0);
  static constexpr int L_GO = L_REC + (BWD ? 2 : 1) * WIN * REC;
  static constexpr int L_WO = align16(L_GO + (BWD ? 2 * GOS : 0));
  static constexpr int L_MAP = L_WO + ((BF && !BWD) ? NFH * 1024 : 0);
  static constexpr int L_SCR = L_MAP + kThreads * SVLF_MAX_K * 2;
  static constexpr int LDS = L_SCR + 64;
  static_assert(LDS <= (BWD ? 160 : 80) * 1024, "LDS");
  static_assert(BWD || WIN * ROWH <= WIN * ROWX, "activations fit in the inputs' place");
};

// Density record: unclamped cell coordinates of x1 and x2 and the 8 corner
// ids (the surface point needs them in the forward pass, the scatter in the
// backward pass).
struct __attribute__((aligned(16))) DRec {
  float u1[3];
  float u2[3];
  uint32_t share;         // corners that the ray's next hit has as well
  uint32_t pad;
  int v[8];
};

template <int P, int MODE>
__global__ __launch_bounds__(kThreads, MODE == kForward ? 2 : 1) void k_density(LfArgs a) {
  using CF = DCfg<P, MODE>;
  using M = typename CF::M;
  constexpr bool BF = CF::BF;
  static_assert(sizeof(DRec) == CF::REC, "record size");
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, row = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar offsets and branches
  uint16_t* imap = reinterpret_cast<uint16_t*>(g_lds + CF::L_MAP);
  int* scr = reinterpret_cast<int*>(g_lds + CF::L_SCR);
  const auto rs = pack_rsrc(a.packs, static_cast<int>(M::pack_bytes(CF::EB)));
  constexpr int BWD_BASE = M::FWD * CF::EB;
  const float* bias = reinterpret_cast<const float*>(static_cast<const char*>(a.packs) +
                                                     M::pack_bytes(CF::EB) - M::BIAS * 4);

  // this wave's weights
  frag_t w0[CF::NF0], b0[CF::BWD ? CF::NFH : 1], b1[1];
  if constexpr (BF) {
    load_frags(w0, rs, 0, wave, CF::NF0, lane);
    if constexpr (CF::BWD) {
      load_frags(b0, rs, BWD_BASE + M::bwd_off(0) * CF::EB, wave, CF::NFH, lane);
      load_frags(b1, rs, BWD_BASE + M::bwd_off(1) * CF::EB, wave, 32 / kFragK<BF>, lane);
    } else {
      for (int e = tid; e < CF::NFH * 64; e += kThreads)
        *reinterpret_cast<frag_t*>(g_lds + CF::L_WO + e * 16) = __builtin_bit_cast(
            frag_t, __builtin_amdgcn_raw_buffer_load_b128(rs, e * 16, M::fwd_off(1) * CF::EB, 0));
    }
  }
  const f32x16 bias0 = gbias(bias, wave, g);

  // gradients of this wave's rows, over the whole launch
  constexpr int NX = align32(M::IN0) / 32;
  f32x16 dw0[NX], dw1 = zero16();
  float bs0 = 0.0f;
#pragma unroll
  for (int i = 0; i < NX; ++i) dw0[i] = zero16();
  float bo[2] = {0.0f, 0.0f};

  // The feature-gradient atomics of a window are issued after the next
  // window's gather, so that its loads do not queue behind them.  A wave takes
  // HW consecutive hits, one at a time (lane = channel).
  constexpr int HW = CF::WIN / kWaves;
  int rb = 0, pend_tw = 0;
  float* pend_grad = nullptr;
  auto records = [&](int b) { return reinterpret_cast<DRec*>(g_lds + CF::L_REC + b * CF::WIN * CF::REC); };
  auto scatter = [&]() {
    if constexpr (CF::BWD) {
      const DRec* rec = records(rb ^ 1);
      const int n0 = HW * wave, n1 = n0 + HW < pend_tw ? n0 + HW : pend_tw;
      CornerCarry carry;
      for (int hh = n0; hh < n1; ++hh) {
        const DRec rc = rec[hh];
        float w1[8], w2[8];
        trilinear(clamp01(rc.u1[0]), clamp01(rc.u1[1]), clamp01(rc.u1[2]), w1);
        trilinear(clamp01(rc.u2[0]), clamp01(rc.u2[1]), clamp01(rc.u2[2]), w2);
        const float g1 = *reinterpret_cast<const float*>(tile_at<CF::ROWG>(CF::L_GX, hh, lane >> 2) + (lane & 3) * 4);
        const float g2 = *reinterpret_cast<const float*>(tile_at<CF::ROWG>(CF::L_GX, hh, 16 + (lane >> 2)) + (lane & 3) * 4);
#pragma unroll
        for (int j = 0; j < 8; ++j) carry.v[j] += w1[j] * g1 + w2[j] * g2;
        carry.flush(__builtin_amdgcn_readfirstlane(rc.share), [&](int j, float x) {
          unsafeAtomicAdd(pend_grad + static_cast<int64_t>(rc.v[j]) * kLfCT + lane, x);
        });
      }
      pend_tw = 0;
    }
  };

  __syncthreads();
  // Work items over the live rays, or over all (see k_color).
  const bool compact = CF::BWD && a.tab.live_n != nullptr;
  LiveRays lr = {};
  if (compact) lr = live_rays(a.tab, scr);
  int* ray_ids = reinterpret_cast<int*>(g_lds + CF::L_MAP + kLiveItemRays * SVLF_MAX_K * 2);
  ItemDeal deal(compact ? lr.items : a.tab.n_items, a.item_counters + (CF::BWD ? 2 : 0));
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
    const float h = __int_as_float((128 - sc.depth) << 23);
    const float inv_h = __int_as_float((126 + sc.depth) << 23);
    int total;
    const int off = block_excl_scan<kWaves>(count, scr, total, [&](int o) {
      for (int q = 0; q < count; ++q) imap[o + q] = static_cast<uint16_t>(tid | (q << 8));
    });
    for (int s0 = 0; s0 < total;) {
      bool in_win;
      const int s1 = open_window<CF::WIN>(s0, total, off, count, imap, in_win);
      (void)in_win;
      const uint16_t* wmap = imap + s0;
      const int tw = s1 - s0;
      const int tp = (tw + 63) & ~63;              // rows that the layers touch
      DRec* rec = records(rb);
      auto slot_of = [&](int hh) {
        const int mp = wmap[hh];
        return ray_of(mp & 0xFF) * a.K + (mp >> 8);
      };
      // records: one thread per hit; r into the input columns
      const bool saved = BF && CF::BWD && a.xsave != nullptr;
      float2 go = make_float2(0.0f, 0.0f);         // dL/d(o_0, o_1), left by the colour kernel
      if (CF::BWD && tid < tw) go = *reinterpret_cast<const float2*>(a.gT + 2 * slot_of(tid));
      if (tid < tp) {
        float rr[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        int mp = -1;
        uint32_t ijk = 0;
        if (tid < tw) {
          mp = wmap[tid];
          const int64_t ray = ray_of(mp & 0xFF);
          const HitRec hr = a.hits[ray * a.K + (mp >> 8)];
          const float ox = a.o[3 * ray], oy = a.o[3 * ray + 1], oz = a.o[3 * ray + 2];
          const float dx = a.d[3 * ray], dy = a.d[3 * ray + 1], dz = a.d[3 * ray + 2];
          const int4* lc = reinterpret_cast<const int4*>(sc.leaf_corners + 8 * static_cast<int64_t>(hr.leaf));
          const int4 c0 = lc[0], c1 = lc[1];
          const float lx = -1.0f + static_cast<float>(hr.ijk & 1023u) * h;
          const float ly = -1.0f + static_cast<float>((hr.ijk >> 10) & 1023u) * h;
          const float lz = -1.0f + static_cast<float>(hr.ijk >> 20) * h;
          DRec rc;
          rc.u1[0] = cell_coord(ox, dx, hr.tin, 0.0f, lx, inv_h);
          rc.u1[1] = cell_coord(oy, dy, hr.tin, 0.0f, ly, inv_h);
          rc.u1[2] = cell_coord(oz, dz, hr.tin, 0.0f, lz, inv_h);
          rc.u2[0] = cell_coord(ox, dx, hr.tout, 0.0f, lx, inv_h);
          rc.u2[1] = cell_coord(oy, dy, hr.tout, 0.0f, ly, inv_h);
          rc.u2[2] = cell_coord(oz, dz, hr.tout, 0.0f, lz, inv_h);
          rc.v[0] = c0.x; rc.v[1] = c0.y; rc.v[2] = c0.z; rc.v[3] = c0.w;
          rc.v[4] = c1.x; rc.v[5] = c1.y; rc.v[6] = c1.z; rc.v[7] = c1.w;
          rec[tid] = rc;
          ijk = hr.ijk;
          if (!saved) {
            const float hc = 0.5f * h;
            float r6[6];
            sphere_r(cell_coord(ox, dx, hr.tin, 0.0f, lx + hc, 1.0f),
                     cell_coord(oy, dy, hr.tin, 0.0f, ly + hc, 1.0f),
                     cell_coord(oz, dz, hr.tin, 0.0f, lz + hc, 1.0f), dx, dy, dz, h, r6);
#pragma unroll
            for (int i = 0; i < 6; ++i) rr[i] = r6[i];
          }
        }
        if constexpr (CF::BWD) {
          const uint32_t sh = shared_corners(mp, ijk);
          if (tid < tw) rec[tid].share = (tid & (HW - 1)) == HW - 1 ? 0u : sh;
        }
        if (!saved) {
          constexpr int C0 = 2 * kLfCT / kRowVals<BF>;
          const float zero[8] = {0, 0, 0, 0, 0, 0, 0, 0};
          *reinterpret_cast<frag_t*>(tile_at<CF::ROWX>(CF::L_X, tid, C0)) = pack_row<BF>(rr);
          *reinterpret_cast<frag_t*>(tile_at<CF::ROWX>(CF::L_X, tid, C0 + 1)) = pack_row<BF>(BF ? zero : rr + 4);
        }
      }
      if (saved) {
        // the forward pass kept this window's decoder inputs
        constexpr int CPR = M::IN0P * 2 / 16;      // 16-byte chunks per row
        constexpr int N = (CF::WIN * CPR + kThreads - 1) / kThreads;
        uint4 v[N];                                // all loads in flight at once
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const int e = i * kThreads + tid, hh = e / CPR, c = e % CPR;
          v[i] = make_uint4(0u, 0u, 0u, 0u);
          if (hh < tw) v[i] = *reinterpret_cast<const uint4*>(a.xsave + slot_of(hh) * M::IN0P + 8 * c);
        }
#pragma unroll
        for (int i = 0; i < N; ++i) {
          const int e = i * kThreads + tid, hh = e / CPR, c = e % CPR;
          if (hh < tp) *reinterpret_cast<uint4*>(tile_at<CF::ROWX>(CF::L_X, hh, c)) = v[i];
        }
      } else {
        __syncthreads();
        // thread q of a hit owns VPT channels of psi(x1) and psi(x2)
        constexpr int VPT = kRowVals<BF>, TPH = kLfCT / VPT, HPP = kThreads / TPH;
        const int q = tid % TPH;
#pragma unroll 2
        for (int hh = tid / TPH; hh < tp; hh += HPP) {
          float v1[VPT], v2[VPT];
#pragma unroll
          for (int i = 0; i < VPT; ++i) v1[i] = v2[i] = 0.0f;
          if (hh < tw) {
            const DRec rc = rec[hh];
            uint4 raw[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) raw[j] = load_row<BF>(sc, 0, static_cast<int64_t>(rc.v[j]) * kLfCT + VPT * q);
            float w1[8], w2[8];
            trilinear(clamp01(rc.u1[0]), clamp01(rc.u1[1]), clamp01(rc.u1[2]), w1);
            trilinear(clamp01(rc.u2[0]), clamp01(rc.u2[1]), clamp01(rc.u2[2]), w2);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              float f[VPT];
              unpack_row<BF>(raw[j], f);
#pragma unroll
              for (int i = 0; i < VPT; ++i) {
                v1[i] += w1[j] * f[i];
                v2[i] += w2[j] * f[i];
              }
            }
          }
          *reinterpret_cast<frag_t*>(tile_at<CF::ROWX>(CF::L_X, hh, q)) = pack_row<BF>(v1);
          *reinterpret_cast<frag_t*>(tile_at<CF::ROWX>(CF::L_X, hh, TPH + q)) = pack_row<BF>(v2);
        }
      }
      if constexpr (!BF) load_frags(w0, rs, 0, wave, CF::NF0, lane);
      __syncthreads();
      if (pend_tw > 0) scatter();
      if (BF && !CF::BWD && a.xsave != nullptr) {
        // keep the window's decoder inputs for the backward pass
        constexpr int CPR = M::IN0P * 2 / 16;
        for (int e = tid; e < tw * CPR; e += kThreads) {
          const int hh = e / CPR, c = e % CPR;
          *reinterpret_cast<uint4*>(a.xsave + slot_of(hh) * M::IN0P + 8 * c) =
              *reinterpret_cast<const uint4*>(tile_at<CF::ROWX>(CF::L_X, hh, c));
        }
      }

      // hidden layer
      {
        auto store = [&](int t, f32x16& acc) {
          relu16(acc);
          store_tile<BF, CF::ROWH>(CF::L_ACT, wave, 32 * t + row, g, acc);
        };
        if constexpr (CF::BWD) {
          layer_mma<BF, CF::ROWX, CF::NT>(bias0, w0, CF::L_X, tw, lane, store);
        } else {
          f32x16 acc[CF::NT];
          layer_mma<BF, CF::ROWX, CF::NT>(bias0, w0, CF::L_X, tw, lane, [&](int t, f32x16& v) { acc[t] = v; });
          __syncthreads();                         // the inputs are overwritten
#pragma unroll
          for (int t = 0; t < CF::NT; ++t)
            if (32 * t < tp) store(t, acc[t]);
        }
      }

      if constexpr (!CF::BWD) {
        __syncthreads();
        // output layer, split by hits; per hit tau, eta and the surface point
        // (section 4.2) -> workspace
        const int n0 = 32 * wave;
        if (wave < CF::NT && n0 < tw) {
          f32x16 o = gbias(bias + M::bias_off(1), 0, g);
#pragma unroll
          for (int i = 0; i < CF::NFH; ++i) {
            frag_t wf;
            if constexpr (BF) wf = *reinterpret_cast<const frag_t*>(g_lds + CF::L_WO + (i * 64 + lane) * 16);
            else
              wf = __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(
                                                  rs, lane * 16, M::fwd_off(1) * CF::EB + i * 1024, 0));
            o = mma_frag<BF>(wf, frag_at<CF::ROWH>(CF::L_ACT, n0 + row, 2 * i + g), o);
          }
          if (g == 0 && n0 + lane < tw) {
            const int hh = n0 + lane;
            const DRec rc = rec[hh];
            const int64_t slot = slot_of(hh);
            const float tin = a.hits[slot].tin, tout = a.hits[slot].tout;
            const float dt = tout - tin;
            const float ft = a.tau_mode == SVLF_TAU_VOXEL ? dt * inv_h
                             : a.tau_mode == SVLF_TAU_WORLD ? dt : 1.0f;
            const float tau = fmaxf(o[0], 0.0f) * ft;
            const float eta = sigmoidf_(o[1]);
            LfHit st;
            st.us[0] = eta * rc.u1[0] + (1.0f - eta) * rc.u2[0];
            st.us[1] = eta * rc.u1[1] + (1.0f - eta) * rc.u2[1];
            st.us[2] = eta * rc.u1[2] + (1.0f - eta) * rc.u2[2];
            st.ts = eta * tin + (1.0f - eta) * tout;
            st.alpha = -expm1f(-tau);
            st.e = expf(-tau);
            st.dtau = o[0] > 0.0f ? ft : 0.0f;
            st.eta = eta;
            a.st[slot] = st;
          }
        }
      } else {
        // backward of F_T
        if constexpr (!BF) {
          load_frags(b1, rs, BWD_BASE + M::bwd_off(1) * CF::EB, wave, 32 / kFragK<BF>, lane);
          load_frags(b0, rs, BWD_BASE + M::bwd_off(0) * CF::EB, wave, CF::NFH, lane);
        }
        using El = typename CF::El;
        if (tid < tp) {
          const El e0 = to_el<BF>(go.x), e1 = to_el<BF>(go.y);
          *reinterpret_cast<El*>(g_lds + CF::L_GO + tid * CF::EB) = e0;
          *reinterpret_cast<El*>(g_lds + CF::L_GO + CF::GOS + tid * CF::EB) = e1;
          if constexpr (BF) {
            bo[0] += bf16_f32(e0);
            bo[1] += bf16_f32(e1);
          } else {
            bo[0] += e0;
            bo[1] += e1;
          }
        }
        __syncthreads();
        // output layer: its weight gradient (this wave's features), and dL/dz_0
        dw_out_mma<BF, CF::ROWH, 2>(dw1, CF::L_ACT, wave, CF::L_GO, CF::GOS, tw, lane);
#pragma unroll
        for (int t = 0; t < CF::NT; ++t) {
          if (32 * t < tp) {
            const int hit = 32 * t + row;
            frag_t gb = {0, 0, 0, 0};
            if (g == 0) {
              const El e0 = *reinterpret_cast<const El*>(g_lds + CF::L_GO + hit * CF::EB);
              const El e1 = *reinterpret_cast<const El*>(g_lds + CF::L_GO + CF::GOS + hit * CF::EB);
              if constexpr (BF) gb[0] = static_cast<int>(e0 | (static_cast<uint32_t>(e1) << 16));
              else {
                gb[0] = __float_as_int(e0);
                gb[1] = __float_as_int(e1);
              }
            }
            const f32x16 ga = mma_frag<BF>(b1[0], gb, zero16());
            mask_store_tile<BF, CF::ROWH>(CF::L_ACT, wave, hit, g, ga);
          }
        }
        __syncthreads();
        // input layer: weight gradient, dL/dx (wave w: input features [32 w, 32 w + 32))
        dw_mma<BF, CF::ROWH, CF::ROWX>(dw0, bs0, CF::L_ACT, wave, CF::L_X, tw, lane);
        layer_mma<BF, CF::ROWH, CF::NT>(zero16(), b0, CF::L_ACT, tw, lane, [&](int t, f32x16& gx) {
          store_tile<false, CF::ROWG>(CF::L_GX, wave, 32 * t + row, g, gx);
        });
        pend_tw = tw;
        pend_grad = sc.grad;
        rb ^= 1;
      }
      __syncthreads();
      s0 = s1;
    }
  }

  if constexpr (CF::BWD) {
    if (pend_tw > 0) scatter();
    float* part = a.partT + static_cast<int64_t>(blockIdx.x) * M::NPARAMS;
    write_dw<BF, M, 0, false>(dw0, part, wave, lane);
    write_dw_out<BF, M>(dw1, part, wave, lane);
    write_bias<BF, M, 0>(bs0, part, wave, lane);
    write_bias_out<M>(bo, reinterpret_cast<float*>(scr), part, wave, lane, tid);
  }
}

// ------------------------------------------------------------ colour kernel

template <int P, int MODE, int VD>
struct CCfg {
  static constexpr bool BF = P == 1;
  static constexpr bool BWD = MODE != kForward;
  using M = typename Dec<BF, VD>::C;
  using El = typename Types<BF>::Elem;
  static constexpr int EB = Types<BF>::EB;
  static constexpr int WIN = BF ? 128 : 64;
  static constexpr int NT = WIN / 32;
  static constexpr int ROWH = kLfH * EB;
  static constexpr int ROWX = 64 * EB;                   // decoder inputs (columns up to the dW tiles)
  static constexpr int ROWG = kLfCC * 4;                 // dL/dx, FP32
  static constexpr int NF0 = M::IN0P / kFragK<BF>, NFH = kLfH / kFragK<BF>;
  static constexpr int GOS = (WIN + 16 / EB) * EB;
  static constexpr int ACT = WIN * ROWH;                 // bytes of one layer's activations
  // Forward: one layer's activations (each layer takes the previous one's
  // place; two blocks per CU).  Backward: all three; dL/dx takes the place of
  // the last layer's, which the next window does not write before the
  // pending scatter has read it.
  static constexpr int L_X = 0;
  static constexpr int L_ACT = L_X + WIN * ROWX;
  static constexpr int L_GX = L_ACT + 2 * ACT;
  static constexpr int L_REC = L_ACT + (BWD ? 3 : 1) * ACT;
  static constexpr int L_DIR = L_REC + (BWD ? 2 : 1) * WIN * 64;
  static constexpr int L_OUT = L_DIR + (BWD ? WIN * 16 : 0);
  static constexpr int L_GO = L_OUT + WIN * 32;
  static constexpr int L_WO = align16(L_GO + (BWD ? 3 * GOS : 0));       // BF16: output layer
  static constexpr int L_B0 = L_WO + (BF ? NFH * 1024 : 0);              // BF16: transposed input layer
  static constexpr int L_MAP = L_B0 + ((BF && BWD) ? NFH * 1024 : 0);
  static constexpr int L_SCR = L_MAP + kThreads * SVLF_MAX_K * 2;
  static constexpr int LDS = L_SCR + 64;
  static_assert(LDS <= (BWD ? 160 : 80) * 1024, "LDS");
  static_assert(WIN * ROWG <= ACT && align32(M::IN0) * EB <= ROWX, "dL/dx and inputs fit");
};

// Colour record (64 B): unclamped surface point in cell units, t_in, t_out,
// eta, the hit slot (top byte: corners that the ray's next hit has as well)
// and the 8 corner ids.
struct CRec {
  float us[3];
  float tin, tout, eta;
  int64_t slot;
  int v[8];
};
static_assert(sizeof(CRec) == 64, "colour record");

__device__ __forceinline__ float quad_xor1(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ float quad_xor2(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, true));
}

template <int P, int MODE, int VD>
__global__ __launch_bounds__(kThreads, MODE == kForward ? 2 : 1) void k_color(LfArgs a) {
  using CF = CCfg<P, MODE, VD>;
  using M = typename CF::M;
  using El = typename CF::El;
  constexpr bool BF = CF::BF;
  const int tid = threadIdx.x, lane = tid & 63, g = lane >> 5, row = lane & 31;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: scalar offsets and branches
  float* out = reinterpret_cast<float*>(g_lds + CF::L_OUT);
  float4* dirs = reinterpret_cast<float4*>(g_lds + CF::L_DIR);
  uint16_t* imap = reinterpret_cast<uint16_t*>(g_lds + CF::L_MAP);
  int* scr = reinterpret_cast<int*>(g_lds + CF::L_SCR);
  using MT_ = typename Dec<BF, VD>::T;
  const char* cpack = static_cast<const char*>(a.packs) + MT_::pack_bytes(CF::EB);
  const auto rs = pack_rsrc(cpack, static_cast<int>(M::pack_bytes(CF::EB)));
  constexpr int BWD_BASE = M::FWD * CF::EB;
  const float* bias = reinterpret_cast<const float*>(cpack + M::pack_bytes(CF::EB) - M::BIAS * 4);

  // This wave's weights.  BF16 forward: kept for the launch (KEEP).  Backward:
  // the registers hold the weight gradients, so the weights are read once per
  // window, BF16 all before the pending scatter's atomics (a load issued after
  // them would wait for them), FP32, whose shares are twice as large and whose
  // windows are long, a layer ahead.
  constexpr int NFB = CF::BWD ? CF::NFH : 1;
  frag_t w0[CF::NF0], w1[CF::NFH], w2[CF::NFH], b1[NFB], b2[NFB], b3[1];
  auto load_w0 = [&]() { load_frags(w0, rs, M::fwd_off(0) * CF::EB, wave, CF::NF0, lane); };
  auto load_w1 = [&]() { load_frags(w1, rs, M::fwd_off(1) * CF::EB, wave, CF::NFH, lane); };
  auto load_w2 = [&]() { load_frags(w2, rs, M::fwd_off(2) * CF::EB, wave, CF::NFH, lane); };
  auto load_b1 = [&]() { load_frags(b1, rs, BWD_BASE + M::bwd_off(1) * CF::EB, wave, CF::NFH, lane); };
  auto load_b2 = [&]() { load_frags(b2, rs, BWD_BASE + M::bwd_off(2) * CF::EB, wave, CF::NFH, lane); };
  auto load_b3 = [&]() { load_frags(b3, rs, BWD_BASE + M::bwd_off(3) * CF::EB, wave, 32 / kFragK<BF>, lane); };
  constexpr bool KEEP = BF && !CF::BWD;
  if constexpr (KEEP) {
    load_w0();
    load_w1();
    load_w2();
  }
  if constexpr (BF) {
    for (int e = tid; e < CF::NFH * 64; e += kThreads) {
      *reinterpret_cast<frag_t*>(g_lds + CF::L_WO + e * 16) = __builtin_bit_cast(
          frag_t, __builtin_amdgcn_raw_buffer_load_b128(rs, e * 16, M::fwd_off(3) * CF::EB, 0));
      if constexpr (CF::BWD)
        *reinterpret_cast<frag_t*>(g_lds + CF::L_B0 + e * 16) = __builtin_bit_cast(
            frag_t, __builtin_amdgcn_raw_buffer_load_b128(rs, e * 16, BWD_BASE + M::bwd_off(0) * CF::EB, 0));
    }
  }
  // fragment i of a narrow (one M tile) matrix: BF16 from LDS, FP32 from L2
  auto narrow = [&](int lds, int bytes, int i) -> frag_t {
    if constexpr (BF) return *reinterpret_cast<const frag_t*>(g_lds + lds + (i * 64 + lane) * 16);
    else
      return __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(rs, lane * 16, bytes + i * 1024, 0));
  };

  f32x16 dw0[2], dw1[4], dw2[4], dw3 = zero16();
  float bs0 = 0.0f, bs1 = 0.0f, bs2 = 0.0f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    dw1[i] = dw2[i] = zero16();
    if (i < 2) dw0[i] = zero16();
  }
  float bo[3] = {0.0f, 0.0f, 0.0f};
  float loss_acc = 0.0f;

  int rb = 0, pend_tw = 0;
  float* pend_grad = nullptr;
  // scatter: hits per wave, per lane group of C_C channels
  constexpr int HW = CF::WIN / kWaves, GH = HW / 2;
  auto records = [&](int b) { return reinterpret_cast<CRec*>(g_lds + CF::L_REC + b * CF::WIN * 64); };
  auto scatter = [&]() {
    if constexpr (CF::BWD) {
      const CRec* rec = records(rb ^ 1);
      const int c = lane & 31, h0 = HW * wave + GH * (lane >> 5);
      CornerCarry carry;
      for (int hh = h0; hh < h0 + GH; ++hh) {
        if (hh < pend_tw) {
          const CRec rc = rec[hh];
          float w[8];
          trilinear(clamp01(rc.us[0]), clamp01(rc.us[1]), clamp01(rc.us[2]), w);
          const float gv = *reinterpret_cast<const float*>(tile_at<CF::ROWG>(CF::L_GX, hh, c >> 2) + (c & 3) * 4);
#pragma unroll
          for (int j = 0; j < 8; ++j) carry.v[j] += w[j] * gv;
          carry.flush(static_cast<uint32_t>(rc.slot >> 56) & 0xFFu, [&](int j, float x) {
            unsafeAtomicAdd(pend_grad + static_cast<int64_t>(rc.v[j]) * kLfCC + c, x);
          });
        }
      }
      pend_tw = 0;
    }
  };

  __syncthreads();
  // Work items over the live rays, or over all.  The forward kernels always
  // take all: they run two blocks per CU and read the hits' rays several times
  // (800^2 BF16 view 384 us, 402 us with the choice made at run time, 388
  // against 366 us over live rays); the backward kernels gain (40,009 FP32 rays:
  // 741 -> 599 us; 262,144 BF16 rays: 1263 -> 1186 us).
  const bool compact = CF::BWD && a.tab.live_n != nullptr;
  LiveRays lr = {};
  if (compact) lr = live_rays(a.tab, scr);
  int* ray_ids = reinterpret_cast<int*>(g_lds + CF::L_MAP + kLiveItemRays * SVLF_MAX_K * 2);
  ItemDeal deal(compact ? lr.items : a.tab.n_items, a.item_counters + 1);
  for (int item = deal.first(scr); item < deal.nb; item = deal.next(item, scr)) {
    const DevScene& sc = a.tab.s[compact ? 0 : scene_of(a.tab, item)];
    const int64_t zc = sc.n_vertices * kLfCT;       // Z_C follows Z_T
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
    if (MODE == kTrain && live) {
      tg0 = a.t_rgb[3 * r]; tg1 = a.t_rgb[3 * r + 1]; tg2 = a.t_rgb[3 * r + 2]; tg3 = a.t_depth[r];
    } else if (MODE == kBackward && live) {
      tg0 = a.g_rgb[3 * r]; tg1 = a.g_rgb[3 * r + 1]; tg2 = a.g_rgb[3 * r + 2]; tg3 = a.g_depth[r];
      tg4 = a.g_acc ? a.g_acc[r] : 0.0f;
    }
    const float h = __int_as_float((128 - sc.depth) << 23);
    const float inv_h = __int_as_float((126 + sc.depth) << 23);
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
      CRec* rec = records(rb);
      if constexpr (!KEEP) {
        load_w0();
        load_w1();
        if constexpr (BF) load_w2();
      }
      // records: one thread per hit; r and the direction into the input columns
      if (tid < tp) {
        float rr[16] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
        int mp = -1;
        uint32_t ijk = 0;
        if (tid < tw) {
          mp = wmap[tid];
          const int64_t ray = ray_of(mp & 0xFF);
          const int64_t slot = ray * a.K + (mp >> 8);
          const HitRec hr = a.hits[slot];
          const LfHit st = a.st[slot];
          const float ox = a.o[3 * ray], oy = a.o[3 * ray + 1], oz = a.o[3 * ray + 2];
          const float dx = a.d[3 * ray], dy = a.d[3 * ray + 1], dz = a.d[3 * ray + 2];
          const int4* lc = reinterpret_cast<const int4*>(sc.leaf_corners + 8 * static_cast<int64_t>(hr.leaf));
          const int4 c0 = lc[0], c1 = lc[1];
          CRec rc;
          rc.us[0] = st.us[0];
          rc.us[1] = st.us[1];
          rc.us[2] = st.us[2];
          rc.tin = hr.tin;
          rc.tout = hr.tout;
          rc.eta = st.eta;
          rc.slot = slot;
          rc.v[0] = c0.x; rc.v[1] = c0.y; rc.v[2] = c0.z; rc.v[3] = c0.w;
          rc.v[4] = c1.x; rc.v[5] = c1.y; rc.v[6] = c1.z; rc.v[7] = c1.w;
          rec[tid] = rc;
          ijk = hr.ijk;
          // per-hit compositing inputs: {e^-tau, dtau/do_0, t_s, alpha}
          *reinterpret_cast<f32x4*>(out + 8 * tid + 4) = f32x4{st.e, st.dtau, st.ts, st.alpha};
          if constexpr (CF::BWD) dirs[tid] = make_float4(dx, dy, dz, 0.0f);
          const float lx = -1.0f + static_cast<float>(hr.ijk & 1023u) * h;
          const float ly = -1.0f + static_cast<float>((hr.ijk >> 10) & 1023u) * h;
          const float lz = -1.0f + static_cast<float>(hr.ijk >> 20) * h;
          const float hc = 0.5f * h;
          float r6[6];
          sphere_r(cell_coord(ox, dx, hr.tin, 0.0f, lx + hc, 1.0f),
                   cell_coord(oy, dy, hr.tin, 0.0f, ly + hc, 1.0f),
                   cell_coord(oz, dz, hr.tin, 0.0f, lz + hc, 1.0f), dx, dy, dz, h, r6);
#pragma unroll
          for (int i = 0; i < 6; ++i) rr[i] = r6[i];
          if (VD) {
            rr[6] = dx;
            rr[7] = dy;
            rr[8] = dz;
          }
        }
        if constexpr (CF::BWD) {
          const uint32_t sh = shared_corners(mp, ijk);
          if (tid < tw && (tid & (GH - 1)) != GH - 1) rec[tid].slot |= static_cast<int64_t>(sh) << 56;
        }
        constexpr int C0 = kLfCC / kRowVals<BF>, NC = (M::IN0P - kLfCC) / kRowVals<BF>;
#pragma unroll
        for (int c = 0; c < NC; ++c)
          *reinterpret_cast<frag_t*>(tile_at<CF::ROWX>(CF::L_X, tid, C0 + c)) = pack_row<BF>(rr + kRowVals<BF> * c);
      }
      __syncthreads();
      {
        // thread q of a hit owns VPT channels of psi(x_s)
        constexpr int VPT = kRowVals<BF>, TPH = kLfCC / VPT, HPP = kThreads / TPH;
        const int q = tid % TPH;
#pragma unroll 2
        for (int hh = tid / TPH; hh < tp; hh += HPP) {
          float v[VPT];
#pragma unroll
          for (int i = 0; i < VPT; ++i) v[i] = 0.0f;
          if (hh < tw) {
            const CRec rc = rec[hh];
            uint4 raw[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) raw[j] = load_row<BF>(sc, zc, static_cast<int64_t>(rc.v[j]) * kLfCC + VPT * q);
            float w[8];
            trilinear(clamp01(rc.us[0]), clamp01(rc.us[1]), clamp01(rc.us[2]), w);
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
      if constexpr (BF && CF::BWD) {
        load_b3();
        load_b2();
        load_b1();
      }
      __syncthreads();
      if (pend_tw > 0) scatter();

      // hidden layers
      static_for<M::NH>([&](auto lc) {
        constexpr int l = decltype(lc)::value;
        const f32x16 bt = gbias(bias + M::bias_off(l), wave, g);
        constexpr int SRC = CF::L_ACT + (CF::BWD && l > 0 ? (l - 1) * CF::ACT : 0);
        constexpr int DST = CF::L_ACT + (CF::BWD ? l * CF::ACT : 0);
        if constexpr (!BF && l == 0) load_w2();
        auto store = [&](int t, f32x16& acc) {
          relu16(acc);
          store_tile<BF, CF::ROWH>(DST, wave, 32 * t + row, g, acc);
        };
        auto run = [&](auto&& done) {
          if constexpr (l == 0) layer_mma<BF, CF::ROWX, CF::NT>(bt, w0, CF::L_X, tw, lane, done);
          else if constexpr (l == 1) layer_mma<BF, CF::ROWH, CF::NT>(bt, w1, SRC, tw, lane, done);
          else layer_mma<BF, CF::ROWH, CF::NT>(bt, w2, SRC, tw, lane, done);
        };
        if constexpr (CF::BWD || l == 0) {
          run(store);
        } else {
          f32x16 acc[CF::NT];
          run([&](int t, f32x16& v) { acc[t] = v; });
          __syncthreads();                         // in place
#pragma unroll
          for (int t = 0; t < CF::NT; ++t)
            if (32 * t < tp) store(t, acc[t]);
        }
        __syncthreads();
      });
      // output layer, split by hits
      constexpr int L_LAST = CF::L_ACT + (CF::BWD ? 2 * CF::ACT : 0);
      const int n0 = 32 * wave;
      const bool has_tile = wave < CF::NT && n0 < tw;
      if (has_tile) {
        f32x16 o = gbias(bias + M::bias_off(M::NH), 0, g);
#pragma unroll
        for (int i = 0; i < CF::NFH; ++i)
          o = mma_frag<BF>(narrow(CF::L_WO, M::fwd_off(M::NH) * CF::EB, i),
                           frag_at<CF::ROWH>(L_LAST, n0 + row, 2 * i + g), o);
        if (g == 0 && n0 + row < tw)
          *reinterpret_cast<f32x4*>(out + 8 * (n0 + row)) = f32x4{sigmoidf_(o[0]), sigmoidf_(o[1]), sigmoidf_(o[2]), 0.0f};
      }
      if constexpr (!BF && CF::BWD) {
        load_b3();
        load_b2();
      }
      __syncthreads();

      // Eq. 3 front to back by the owning lanes, and its backward
      if (in_win) {
        const int p0 = off - s0;
        float T = 1.0f;
        for (int k = 0; k < count; ++k) {
          float* hp = out + 8 * (p0 + k);
          const f32x4 va = *reinterpret_cast<const f32x4*>(hp);
          const f32x4 vb = *reinterpret_cast<const f32x4*>(hp + 4);
          const float w = T * vb[3];
          cr += w * va[0];
          cg += w * va[1];
          cb += w * va[2];
          dep += w * vb[2];
          acc_w += w;
          if constexpr (CF::BWD) hp[3] = T;
          T *= vb[0];
        }
        if constexpr (CF::BWD) {
          float gr, gg, gb, gd, ga;
          // the hit holding the target surface point (staged losses)
          int surf = -1;
          if (MODE == kTrain && a.loss_kind != kLfLossDefault) {
            for (int k = 0; k < count; ++k) {
              const CRec& rc = rec[p0 + k];
              if (rc.tin <= tg3 && tg3 < rc.tout) surf = k;
            }
          }
          if (MODE == kTrain && a.loss_kind == kLfLossSurface) {
            gr = gg = gb = gd = ga = 0.0f;
          } else if (MODE == kTrain && a.loss_kind == kLfLossVolume) {
            const float k2 = 2.0f * a.loss_scale;
            gr = k2 * (cr - tg0);
            gg = k2 * (cg - tg1);
            gb = k2 * (cb - tg2);
            gd = 0.0f;
            ga = 0.0f;
          } else if (MODE == kTrain) {
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
          float surf_loss = 0.0f;
          for (int k = count - 1; k >= 0; --k) {
            float* hp = out + 8 * (p0 + k);
            const f32x4 va = *reinterpret_cast<const f32x4*>(hp);
            const f32x4 vb = *reinterpret_cast<const f32x4*>(hp + 4);
            const float Tq = va[3];
            const float w = Tq * vb[3];
            const float Tn = Tq * vb[0];
            const float c0 = va[0], c1 = va[1], c2 = va[2], ts = vb[2];
            const float gtau = gr * (Tn * c0 - Sr) + gg * (Tn * c1 - Sg) + gb * (Tn * c2 - Sb) +
                               gd * (Tn * ts - St) + ga * (Tn - Sa);
            Sr += w * c0;
            Sg += w * c1;
            Sb += w * c2;
            St += w * ts;
            Sa += w;
            // direct terms of the staged losses on the surface hit: colour
            // (surface stage), eta against the target's within-voxel depth,
            // and the opacity term lambda_tau e^{-2 tau}
            float gc0 = gr * w, gc1 = gg * w, gc2 = gb * w, gt = gtau, geta = 0.0f;
            if (k == surf) {
              const CRec& rc = rec[p0 + k];
              const float ls2 = 2.0f * a.loss_scale;
              const float eta_gt = (rc.tout - tg3) / (rc.tout - rc.tin);
              const float e2 = vb[0] * vb[0];
              if (a.loss_kind == kLfLossSurface) {
                gc0 = ls2 * (c0 - tg0);
                gc1 = ls2 * (c1 - tg1);
                gc2 = ls2 * (c2 - tg2);
                surf_loss += (c0 - tg0) * (c0 - tg0) + (c1 - tg1) * (c1 - tg1) +
                             (c2 - tg2) * (c2 - tg2);
              }
              geta = ls2 * a.lambda_eta * (rc.eta - eta_gt);
              gt -= ls2 * a.lambda_tau * e2;
              surf_loss += a.lambda_eta * (rc.eta - eta_gt) * (rc.eta - eta_gt) + a.lambda_tau * e2;
            }
            const float z0 = gc0 * c0 * (1.0f - c0), z1 = gc1 * c1 * (1.0f - c1), z2 = gc2 * c2 * (1.0f - c2);
            *reinterpret_cast<f32x4*>(hp) = f32x4{z0, z1, z2, gt * vb[1]};
            hp[4] = w * gd;                     // dL/dt_s
            hp[5] = geta;                       // direct dL/deta
          }
          // surface-voxel terms of the staged losses (the photometric term
          // of the volume kind is added for every ray below, hits or not)
          if (MODE == kTrain && a.loss_kind != kLfLossDefault) loss_acc += a.loss_scale * surf_loss;
        }
      }

      if constexpr (CF::BWD) {
        __syncthreads();
        const int tw_dw = a.freeze_color ? 0 : tw;    // hits of the colour side's weight gradients
        constexpr int A0 = CF::L_ACT, A1 = CF::L_ACT + CF::ACT, A2 = CF::L_ACT + 2 * CF::ACT;
        if constexpr (!BF) load_b1();
        // output layer: dL/do [output][hit] for its weight gradient
        if (tid < tp) {
          f32x4 go = {0.0f, 0.0f, 0.0f, 0.0f};
          if (tid < tw) go = *reinterpret_cast<const f32x4*>(out + 8 * tid);
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const El e = to_el<BF>(go[c]);
            *reinterpret_cast<El*>(g_lds + CF::L_GO + c * CF::GOS + tid * CF::EB) = e;
            if (!a.freeze_color) bo[c] += BF ? bf16_f32(static_cast<uint16_t>(e)) : static_cast<float>(e);
          }
        }
        __syncthreads();
        dw_out_mma<BF, CF::ROWH, 3>(dw3, A2, wave, CF::L_GO, CF::GOS, tw_dw, lane);
        // dL/dz_2 (the output's gradient fills 3 of the K positions, all in lane group 0)
#pragma unroll
        for (int t = 0; t < CF::NT; ++t) {
          if (32 * t < tp) {
            const int hit = 32 * t + row;
            frag_t gb = {0, 0, 0, 0};
            if (g == 0) {
              El e[3];
#pragma unroll
              for (int c = 0; c < 3; ++c) e[c] = *reinterpret_cast<const El*>(g_lds + CF::L_GO + c * CF::GOS + hit * CF::EB);
              if constexpr (BF) {
                gb[0] = static_cast<int>(e[0] | (static_cast<uint32_t>(e[1]) << 16));
                gb[1] = static_cast<int>(e[2]);
              } else {
#pragma unroll
                for (int c = 0; c < 3; ++c) gb[c] = __float_as_int(e[c]);
              }
            }
            const f32x16 ga = mma_frag<BF>(b3[0], gb, zero16());
            mask_store_tile<BF, CF::ROWH>(A2, wave, hit, g, ga);
          }
        }
        __syncthreads();
        // layers 2 and 1: weight gradient (reads the layer's inputs), then
        // dL/dz of the layer below, in place of those inputs
        auto hidden = [&](f32x16 (&dw)[4], float& bs, const frag_t (&bw)[NFB], int gz, int in) {
          dw_mma<BF, CF::ROWH, CF::ROWH>(dw, bs, gz, wave, in, tw_dw, lane);
          __syncthreads();
          layer_mma<BF, CF::ROWH, CF::NT>(zero16(), bw, gz, tw, lane, [&](int t, f32x16& acc) {
            mask_store_tile<BF, CF::ROWH>(in, wave, 32 * t + row, g, acc);
          });
          __syncthreads();
        };
        hidden(dw2, bs2, b2, A2, A1);
        hidden(dw1, bs1, b1, A1, A0);
        dw_mma<BF, CF::ROWH, CF::ROWX>(dw0, bs0, A0, wave, CF::L_X, tw_dw, lane);
        // dL/dx of the features, split by hits: the wave that makes a hit's
        // row also uses it below
        if (has_tile) {
          f32x16 gx = zero16();
#pragma unroll
          for (int i = 0; i < CF::NFH; ++i)
            gx = mma_frag<BF>(narrow(CF::L_B0, BWD_BASE + M::bwd_off(0) * CF::EB, i),
                              frag_at<CF::ROWH>(A0, n0 + row, 2 * i + g), gx);
          store_tile<false, CF::ROWG>(CF::L_GX, 0, n0 + row, g, gx);
          // dL/deta through the interpolation at x_s: per corner, dL/dx . Z_C
          // summed in a fixed tree over the channels (channels 16, 8, 4, 2 and
          // 1 apart), in the gather's layout (16 bytes of a row per lane)
          constexpr int VPT = kRowVals<BF>, TPH = kLfCC / VPT, HPW = 64 / TPH;
          const int q = lane % TPH, hl = lane / TPH;
          uint4 raw[8];
          auto issue = [&](int p, uint4 (&rw)[8]) {
            const int hh = n0 + p * HPW + hl;
            if (hh < tw) {
              const CRec& rc = rec[hh];
#pragma unroll
              for (int j = 0; j < 8; ++j) rw[j] = load_row<BF>(sc, zc, static_cast<int64_t>(rc.v[j]) * kLfCC + VPT * q);
            }
          };
          auto project = [&](int p, const uint4 (&rw)[8]) {
            const int hh = n0 + p * HPW + hl;
            float proj[8], gv[VPT];
            const bool ok = hh < tw;
#pragma unroll
            for (int i = 0; i < VPT / 4; ++i) {
              const f32x4 v = __builtin_bit_cast(f32x4, frag_at<CF::ROWG>(CF::L_GX, ok ? hh : n0, (VPT / 4) * q + i));
#pragma unroll
              for (int e = 0; e < 4; ++e) gv[4 * i + e] = v[e];
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) {
#pragma clang fp contract(off)
              float f[VPT], s[VPT];
              unpack_row<BF>(rw[j], f);
#pragma unroll
              for (int i = 0; i < VPT; ++i) s[i] = ok ? f[i] * gv[i] : 0.0f;
              if constexpr (BF) {
#pragma unroll
                for (int i = 0; i < 8; ++i) s[i] = s[i] + quad_xor2(s[i]);
#pragma unroll
                for (int i = 0; i < 8; ++i) s[i] = s[i] + quad_xor1(s[i]);
#pragma unroll
                for (int m = 4; m > 0; m >>= 1)
#pragma unroll
                  for (int i = 0; i < m; ++i) s[i] = s[i] + s[i + m];
              } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) s[i] = s[i] + __shfl_xor(s[i], 4, 64);
#pragma unroll
                for (int i = 0; i < 4; ++i) s[i] = s[i] + quad_xor2(s[i]);
#pragma unroll
                for (int i = 0; i < 4; ++i) s[i] = s[i] + quad_xor1(s[i]);
#pragma unroll
                for (int m = 2; m > 0; m >>= 1)
#pragma unroll
                  for (int i = 0; i < m; ++i) s[i] = s[i] + s[i + m];
              }
              proj[j] = s[0];
            }
            if (ok && q == 0) {
              // dL/du_s from the trilinear weights' derivatives
              const CRec& rc = rec[hh];
              const float u[3] = {clamp01(rc.us[0]), clamp01(rc.us[1]), clamp01(rc.us[2])};
              float gu[3] = {0.0f, 0.0f, 0.0f};
#pragma unroll
              for (int j = 0; j < 8; ++j) {
#pragma unroll
                for (int ax = 0; ax < 3; ++ax) {
                  float dwv = ((j >> ax) & 1) ? 1.0f : -1.0f;
#pragma unroll
                  for (int bx = 0; bx < 3; ++bx)
                    if (bx != ax) dwv *= ((j >> bx) & 1) ? u[bx] : 1.0f - u[bx];
                  gu[ax] += dwv * proj[j];
                }
              }
              const float4 dv = dirs[hh];
              const float dir[3] = {dv.x, dv.y, dv.z};
              float gx_d = 0.0f;
#pragma unroll
              for (int ax = 0; ax < 3; ++ax) {
                const bool inside = rc.us[ax] >= 0.0f && rc.us[ax] <= 1.0f;
                gx_d += inside ? gu[ax] * dir[ax] : 0.0f;
              }
              const float* hp = out + 8 * hh;
              const float g_eta = (rc.tin - rc.tout) * (hp[4] + gx_d * inv_h) + hp[5];
              const int64_t slot = rc.slot & ((int64_t(1) << 56) - 1);
              *reinterpret_cast<float2*>(a.gT + 2 * slot) = make_float2(hp[3], g_eta * rc.eta * (1.0f - rc.eta));
            }
          };
#pragma unroll 1
          for (int p = 0; p < 32 / HPW; ++p) {
            issue(p, raw);
            project(p, raw);
          }
        }
        if (!a.freeze_color) {
          pend_tw = tw;
          pend_grad = sc.grad + zc;
        }
        rb ^= 1;
      }
      __syncthreads();
      s0 = s1;
    }

    if (live) {
      if (MODE != kBackward) {
        if (a.rgb) {
          a.rgb[3 * r] = cr;
          a.rgb[3 * r + 1] = cg;
          a.rgb[3 * r + 2] = cb;
        }
        if (a.depth) a.depth[r] = dep;
        if (a.acc) a.acc[r] = acc_w;
      }
      if (MODE == kTrain && a.loss_kind == kLfLossDefault) {
        const float er = cr - tg0, eg = cg - tg1, eb = cb - tg2, ed = dep - tg3;
        loss_acc += a.loss_scale * ((er * er + eg * eg + eb * eb) * (1.0f / 3.0f) +
                                    a.lambda_depth * fabsf(ed));
      } else if (MODE == kTrain && a.loss_kind == kLfLossVolume) {
        const float er = cr - tg0, eg = cg - tg1, eb = cb - tg2;
        loss_acc += a.loss_scale * (er * er + eg * eg + eb * eb);
      }
    }
  }

  // rays without hits that no item took
  if (compact && MODE != kBackward) {
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
      if (a.acc) a.acc[r] = 0.0f;
      if (MODE == kTrain && a.loss_kind != kLfLossSurface) {
        const float er = a.t_rgb[3 * r], eg = a.t_rgb[3 * r + 1], eb = a.t_rgb[3 * r + 2];
        const float sq = er * er + eg * eg + eb * eb;
        loss_acc += a.loss_scale * (a.loss_kind == kLfLossVolume
                                        ? sq : sq * (1.0f / 3.0f) + a.lambda_depth * fabsf(a.t_depth[r]));
      }
    }
  }
  if constexpr (CF::BWD) {
    if (pend_tw > 0) scatter();
    float* part = a.partC + static_cast<int64_t>(blockIdx.x) * M::NPARAMS;
    write_dw<BF, M, 0, false>(dw0, part, wave, lane);
    write_dw<BF, M, 1, true>(dw1, part, wave, lane);
    write_dw<BF, M, 2, true>(dw2, part, wave, lane);
    write_dw_out<BF, M>(dw3, part, wave, lane);
    write_bias<BF, M, 0>(bs0, part, wave, lane);
    write_bias<BF, M, 1>(bs1, part, wave, lane);
    write_bias<BF, M, 2>(bs2, part, wave, lane);
    write_bias_out<M>(bo, reinterpret_cast<float*>(scr), part, wave, lane, tid);
    if (MODE == kTrain) {
      const float tot = block_sum<kWaves>(loss_acc, reinterpret_cast<float*>(scr));
      if (tid == 0) a.ws_loss[blockIdx.x] = tot;
    } else if (tid == 0) {
      a.ws_loss[blockIdx.x] = 0.0f;
    }
  }
}

// ------------------------------------------------------------ dispatch

int lf_num_cus() {
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

// Persistent launch: as many blocks as fit on the device at once (registers
// and LDS), at most `cap` (the backward kernels' partial sums are sized for
// lf_grid_limit() blocks).
template <class K>
hipError_t launch_persistent(K kern, int lds, LfArgs a, hipStream_t s, int* grid_out, int cap, bool backward) {
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, lds);
  if (e != hipSuccess) return e;
  int per_cu = 1;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern),
                                                   kThreads, lds) != hipSuccess || per_cu < 1)
    per_cu = 1;
  int grid = lf_num_cus() * per_cu;
  if (grid > cap) grid = cap;
  plan_items(&a.tab, grid, backward);
  if (grid > a.tab.n_items) grid = a.tab.n_items;
  if (grid < 1) grid = 1;
  *grid_out = grid;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(kThreads), lds, s, a);
  return hipGetLastError();
}

template <int P, int VD>
hipError_t run_lf(const LfArgs& a, int mode, hipStream_t s) {
  constexpr bool BF = P == 1;
  using D = Dec<BF, VD>;
  hipLaunchKernelGGL((k_lf_pack<BF, VD>), dim3(64), dim3(kThreads), 0, s, a.params,
                     static_cast<char*>(a.packs));
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  int g1 = 0, g2 = 0, g3 = 0;
  const int fwd_cap = 4096, bwd_cap = lf_grid_limit();
  e = launch_persistent(k_density<P, kForward>, DCfg<P, kForward>::LDS, a, s, &g1, fwd_cap, false);
  if (e != hipSuccess) return e;
  if (mode == kForward)
    return launch_persistent(k_color<P, kForward, VD>, CCfg<P, kForward, VD>::LDS, a, s, &g2,
                             fwd_cap, false);
  if (mode == kTrain)
    e = launch_persistent(k_color<P, kTrain, VD>, CCfg<P, kTrain, VD>::LDS, a, s, &g2, bwd_cap, true);
  else
    e = launch_persistent(k_color<P, kBackward, VD>, CCfg<P, kBackward, VD>::LDS, a, s, &g2,
                          bwd_cap, true);
  if (e != hipSuccess) return e;
  e = launch_persistent(k_density<P, kBackward>, DCfg<P, kBackward>::LDS, a, s, &g3, bwd_cap, true);
  if (e != hipSuccess) return e;
  e = launch_reduce_partials(a.partT, g3, D::T::NPARAMS, a.grad_params, nullptr, nullptr, s);
  if (e != hipSuccess) return e;
  return launch_reduce_partials(a.partC, g2, D::C::NPARAMS, a.grad_params + D::T::NPARAMS,
                                a.ws_loss, mode == kTrain ? a.loss_out : nullptr, s);
}

}  // namespace

int lf_grid_limit() { return 256; }
int lf_x_row() { return Dec<true, 0>::T::IN0P; }
int64_t lf_params_density() { return Dec<true, 0>::T::NPARAMS; }
int64_t lf_params_color(int viewdir) {
  return viewdir ? Dec<true, 1>::C::NPARAMS : Dec<true, 0>::C::NPARAMS;
}
size_t lf_pack_bytes(int precision, int viewdir) {
  const bool bf = precision == SVLF_BF16;
  if (bf) {
    return viewdir ? Dec<true, 1>::T::pack_bytes(2) + Dec<true, 1>::C::pack_bytes(2)
                   : Dec<true, 0>::T::pack_bytes(2) + Dec<true, 0>::C::pack_bytes(2);
  }
  return viewdir ? Dec<false, 1>::T::pack_bytes(4) + Dec<false, 1>::C::pack_bytes(4)
                 : Dec<false, 0>::T::pack_bytes(4) + Dec<false, 0>::C::pack_bytes(4);
}

hipError_t launch_lf(const LfArgs& a, int mode, hipStream_t s) {
  const int P = a.precision == SVLF_BF16 ? 1 : 0;
  if (P) return a.viewdir ? run_lf<1, 1>(a, mode, s) : run_lf<1, 0>(a, mode, s);
  return a.viewdir ? run_lf<0, 1>(a, mode, s) : run_lf<0, 0>(a, mode, s);
}

}  // namespace svlf
