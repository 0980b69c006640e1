// Backward of the splat rasterizer.
//
// blend_bwd: one workgroup per (pose, tile).  Each pixel starts from its
// saved final transmittance and list length and walks its tile list back to
// front, recovering T_j = T_{j+1} / (1 - alpha_j) instead of storing
// per-pixel lists.  With h_j = gC.c_j + gZ z_j + gF.f_j and the suffix sum
// S_j = sum_{k>j} w_k h_k,
//   dL/dalpha_j = T_j h_j - (S_j + gT T_final) / (1 - alpha_j),
// where gT collects the outputs' direct dependence on T_final (background,
// depth normalisation, alpha).  Per-splat sums are formed per wave, then per
// workgroup, before one atomic per value.
//
// project_bwd: one thread per visible (pose, Gaussian): chains the splat
// gradients through the conic inverse, the EWA covariance, the clamped
// pinhole Jacobian, the camera transform and the SH view direction, into
// dL/d(mean, opacity, scales, rotation, SH) and the pose's left-perturbation
// tangent (rho, phi), block-reduced per pose.
#include <type_traits>

#include "hgsr_device.hpp"
#include "launch.hpp"

namespace hgsr {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short shortx4 __attribute__((ext_vector_type(4)));

constexpr int kBwdGroup = 16;   // splats per matrix-core product
constexpr int kBwdHalf = 8;     // splats per transposed reduction
constexpr int kBwdRow = 68;     // words per LDS row of 64 pixels (16-byte reads of 8 rows hit 32 banks)
constexpr int kBwdGcRow = 8;    // words per row of 8 pixel gradients

// Item order of a grid launch whose poses share one target: a run's target
// block (16 tiles: 0.6 MB at 32 channels) is then fetched once per block of
// poses into the XCD's L2, whose poses still pass over neighbouring tiles
// close together (records and half lines of the maps).  64 poses at 960x540:
// 3,285 -> 3,230 us, 16 at 480x270: 254 -> 249 us; all poses per run 3-5 %
// slower than pose after pose, runs of 60 tiles no faster.
constexpr int kPoseBlock = 8;
constexpr int kTileRun = 16;

// Transpose of a 4x4 block whose one index is the register and whose other is
// the row of 16 lanes: afterwards register k of lane row m holds what register
// m of lane row k held.
__device__ __forceinline__ void transpose_rows(uint32_t& r0, uint32_t& r1, uint32_t& r2, uint32_t& r3) {
  const auto a = __builtin_amdgcn_permlane32_swap(r0, r2, false, false);
  const auto b = __builtin_amdgcn_permlane32_swap(r1, r3, false, false);
  const auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  r0 = c[0];
  r1 = c[1];
  r2 = d[0];
  r3 = d[1];
}

// Sum over the four rows of 16 lanes, in every lane.
__device__ __forceinline__ float row_quad_sum(float v) {
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float t = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// v of each row of 16 lanes, in every row.
__device__ __forceinline__ void row_broadcast(float v, float out[4]) {
  const auto h = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const auto a = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
  out[0] = __uint_as_float(a[0]);
  out[1] = __uint_as_float(a[1]);
  out[2] = __uint_as_float(b[0]);
  out[3] = __uint_as_float(b[1]);
}

// Sums eight per-lane values over the eight lane octets (lanes that agree in
// lane % 8): on return the lane holds the total of value lane / 8.
__device__ __forceinline__ float octet_scatter8(const float v[8], int lane) {
  float b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[4 + i]), false, false);
    b[i] = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  }
  const auto s0 = __builtin_amdgcn_permlane16_swap(__float_as_uint(b[0]), __float_as_uint(b[2]), false, false);
  const auto s1 = __builtin_amdgcn_permlane16_swap(__float_as_uint(b[1]), __float_as_uint(b[3]), false, false);
  const float c0 = __uint_as_float(s0[0]) + __uint_as_float(s0[1]);
  const float c1 = __uint_as_float(s1[0]) + __uint_as_float(s1[1]);
  const bool odd = (lane & 8) != 0;
  return (odd ? c1 : c0) + row_ror<8>(odd ? c0 : c1);
}

// The same for two values: lanes 0-7 end with the total of a, lanes 32-39 with
// that of b.
__device__ __forceinline__ float octet_sum2(float a, float b) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  const float t = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  const auto u = __builtin_amdgcn_permlane16_swap(__float_as_uint(t), __float_as_uint(t), false, false);
  const float w = __uint_as_float(u[0]) + __uint_as_float(u[1]);
  return w + row_ror<8>(w);
}

// Element of a plane at a byte offset.
template <class E>
__device__ __forceinline__ E plane_at(const E* base, uint32_t bytes) {
  return *reinterpret_cast<const E*>(reinterpret_cast<const char*>(base) + bytes);
}

__device__ __forceinline__ bool finite_bits(float v) { return (__float_as_uint(v) & 0x7f800000u) != 0x7f800000u; }

// The reverse replay of one (pose, tile) or tile quadrant.
//
// Bound by the VALU (2,630 instructions per wave at 64 poses of 960x540, waves
// waiting 38 % of their cycles) beside the feature maps' traffic.  A
// splat's gradient sums over a wave's 64 pixels are not reduced across lanes
// splat by splat: each lane writes two numbers per splat to LDS, dL/dpower d
// and the blend weight w, and after eight splats the wave reads them back
// transposed -- a lane takes one splat's row of eight pixels -- and forms the
// sums there, every lane busy, with one cross-lane step per eight splats.  With
// the conic (a, b, c) those kept per record are d (a dx + b dy), d (b dx + c dy),
// the mean's gradient, the moments d dx^2, d dx dy, d dy^2, d, and w gZ, w gC;
// the projection backward turns the moments into conic and opacity gradients.
// The mean's two sums are formed per pixel: along a needle a dx and b dy cancel
// there, and sums of d dx and d dy combined at the end miss the 64-bit value by
// up to 48 x 2^-24 of the terms (needles of 60 px), these by less than 0.1, for
// four more instructions per splat (no features, tile 16, 8 poses of 480x270:
// 181 -> 194 us).  The waves keep their sums apart in LDS until the flush: float
// atomics there take about a cycle per lane (300 of 3,700 us at 64 poses).
//
// The feature part of h_j = gF . f_j is, for 16 splats and 64 pixels, a matrix
// product on the matrix cores (v_mfma_f32_16x16x32_bf16; 16x16x16 for up to 16
// channels): the splats' stored bf16 features enter exactly, the FP32 pixel
// gradient in three exact bf16 parts kept in registers for the whole tile, so
// products are exact and only the order of the sum differs from the FP32 dot
// product.  The FP32 matrix form (16x16x4, no split) took 400 us more at 64
// poses.  The pixel gradients are loaded in the operand's own layout, every
// load issued before the first wait (flags, tile range and list follow), and a
// splat's geometry and colour are read from LDS a step ahead.
//
// FEATGRAD: a splat's feature gradient sum_p w_p gF_p is the product of the
// weights (16 splats x 64 pixels, read transposed from LDS) with the FP32 pixel
// gradients in registers, in FP32 on the matrix cores
// (v_mfma_f32_16x16x4_f32), summed per workgroup in LDS before the global
// atomics; the form it replaces summed every channel over the wave by shuffles
// and added it to memory from one lane.
//
// Before and after, blend backward alone: 64 poses at 960x540, 32 channels,
// pose only: 3,810 -> 3,230 us; 16 poses at 480x270: 290 -> 249 us; one pose
// at 480x270: 98 -> 64 us; one 640x480 view with all Gaussian gradients: 710 ->
// 138 us.  Pose only, up to 32 channels, tile 16 and 32: held to four waves per
// SIMD, which takes all 128 registers and spills none (12 spilled, the staged
// record among them: 230 us instead of 222 at one 1920x1080 pose); five waves
// (96 registers) spill: 5,040 us at 64 poses.
//
// Non-finite output gradients reach only the splats blended at their pixels:
// a wave that holds any (`bad`) leaves zero weights out of its sums.
//
// PO (pose only, residual loss): neither the opacity nor the depth sum is
// formed (the residual has no depth term and no opacity gradient was asked
// for).
template <int TILE, int D, bool FEATGRAD, bool RES, bool PO>
__device__ __forceinline__ void blend_bwd_item(const BackArgs& a, const int item) {
  using Sh = BlockShape<TILE>;
  constexpr int NT = Sh::kThreads, NW = Sh::kWaves, NB = kListRound, ROW = kBwdRow;
  constexpr int DV = D / 8;                    // 16-byte bf16 vectors per feature
  constexpr int CG = D / 4;                    // channels per lane row of the matrix operands
  constexpr int CGA = CG > 0 ? CG : 1;
  constexpr int KW = CG > 4 ? 4 : 2;           // words per operand of one matrix step (16x16x32 or x16)
  constexpr int KS = CG > 8 ? CG / 8 : 1;      // matrix steps
  constexpr int NV = PO ? 8 : 10;              // moment sums per splat
  constexpr int GR = NB + 1;                   // words per row of sums (one row per value)
  constexpr int NBL = FEATGRAD ? (D + 15) / 16 : 1;    // FEATGRAD: blocks of 16 channels
  constexpr int SHARE = NT / NB;               // threads staging one splat
  constexpr int FBS = D > 0 ? D / 2 + 4 : 4;   // words per staged bf16 feature vector (padded)
  constexpr int WR = FEATGRAD ? kBwdGroup : kBwdHalf;  // rows of weights kept
  constexpr int GS = D + 1;                    // FEATGRAD: words per pixel's gradient and per splat's feature sum
  struct alignas(16) Wave {                    // what a wave keeps to itself, at constant offsets from one address
    float d[kBwdHalf][ROW];                    // dL/dpower per splat (row) and pixel
    float w[WR][ROW];                          // blend weight
    float gc[PO ? 3 : 4][8 * kBwdGcRow];       // gC, gZ planes of the wave's 8x8 pixels
    float g[NV * GR];                          // per staged splat: its sums (where the wave hit it)
    uint8_t list[NB];                          // slots of the wave's hits, back to front
  };
  struct Walk {
    float4 sp[NB][4];                          // u v ca cb | cc o z gid | r g b pmin | record index
    uint32_t fb[NB * FBS];                     // bf16 feature vectors
    Wave wave[NW];
    uint64_t hits[NW];                         // the waves' hits of the round
    float gfe[FEATGRAD ? NB * GS : 1];         // FEATGRAD: feature sums per staged splat
    uint8_t mask[NB];
  };
  union Lds {
    Walk walk;
    float gf[FEATGRAD ? NW : 1][FEATGRAD ? kWave * GS : 1];  // FEATGRAD prologue: per pixel dL/d(feature map)
  };
  __shared__ __align__(16) Lds s_u;
  __shared__ uint32_t s_max;
  __shared__ uint32_t s_odd;  // ODD: a staged feature of the round is not finite
  __shared__ float s_lw[NW];
  auto& s_sp = s_u.walk.sp;
  auto& s_fb = s_u.walk.fb;
  auto& s_hits = s_u.walk.hits;
  auto& s_gfe = s_u.walk.gfe;
  auto& s_mask = s_u.walk.mask;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  Wave& own = s_u.walk.wave[wave];
  const int W = a.c.W, H = a.c.H;
  const int64_t HW = static_cast<int64_t>(W) * H;
  const int part = item % Sh::kParts, titem = item / Sh::kParts;
  int pose, tile;
  if (a.schedule == kSchedTileMajor) {
    tile = titem / a.P;
    pose = titem - tile * a.P;
  } else if (a.share_target) {
    // blocks of kPoseBlock poses; within one, runs of kTileRun neighbouring
    // tiles, each run for the block's poses in turn
    const int tiles = a.c.tiles_per_pose;
    const int block = titem / (kPoseBlock * tiles), r = titem - block * kPoseBlock * tiles;
    const int np = min(kPoseBlock, a.P - block * kPoseBlock);
    const int run = r / (kTileRun * np), r2 = r - run * kTileRun * np;
    const int size = min(kTileRun, tiles - run * kTileRun);
    const int pi = r2 / size;
    pose = block * kPoseBlock + pi;
    tile = run * kTileRun + (r2 - pi * size);
  } else {
    pose = titem / a.c.tiles_per_pose;
    tile = titem - pose * a.c.tiles_per_pose;
  }
  const int ty = tile / a.c.ntx, tx = tile - ty * a.c.ntx;
  const int bx0 = tx * TILE + (part & 1) * 16 + (wave & 1) * 8, by0 = ty * TILE + (part >> 1) * 16 + (wave >> 1) * 8;
  const int mask_bit = TILE == 32 ? part : wave;  // the list masks' block that holds this wave's pixels

  // a round's staging: list entry, then record and feature vector, dealt to
  // the splat's SHARE threads and held in registers until the LDS is free
  constexpr int RV = (3 + SHARE - 1) / SHARE, FV = DV > 0 ? (DV + SHARE - 1) / SHARE : 1;
  // Infinities in the feature term, where the caller gives the gradients (the
  // residual's own are NaN wherever a map is not finite): an FP32 product gives
  // an infinity, the parts' products 0 times infinity as well.  A part of an
  // infinite gradient beyond the first is zero, and beside such a feature the
  // second and third parts meet a zero instead.
  constexpr bool ODD = !RES && D > 0;
  constexpr bool AHEAD = FV <= 4;  // 64 channels at tile 8: a thread's 32 words of features would cost a wave
  const int st_e = tid / SHARE, st_sub = tid % SHARE;
  uint32_t st_lv = 0;
  // the thread's quads and features as vector values (arrays of float4 would be kept in scratch memory)
  floatx4 st_rec0 = {}, st_rec1 = {}, st_rec2 = {};
  typedef uint32_t featv __attribute__((ext_vector_type(AHEAD ? 4 * FV : 1)));
  featv st_feat = {};
  auto stage_index = [&](uint2 range, uint32_t b0) -> uint32_t {  // the Gaussian's index
    const uint32_t j = range.x + b0 + st_e;
    uint32_t gid = 0;
    if (j < range.y) {
      st_lv = a.list[j];
      if constexpr (DV > 0 && AHEAD) gid = a.list_gid[j];
    }
    return gid;
  };
  auto stage_load = [&](uint2 range, uint32_t b0, uint32_t gid) {
    if (range.x + b0 + st_e < range.y) {
      // keeps the two 64-bit addresses inside the round, out of the walk's registers
      int sub = st_sub;
      asm volatile("" : "+v"(sub));
      const floatx4* sp = reinterpret_cast<const floatx4*>(a.recs + (st_lv & kRecMask));
      if (sub < 3) st_rec0 = sp[sub];
      if (RV > 1 && sub + SHARE < 3) st_rec1 = sp[sub + SHARE];
      if (RV > 2) st_rec2 = sp[2];
      if constexpr (DV > 0 && AHEAD) {
        const uint4* fv = reinterpret_cast<const uint4*>(a.feat) + static_cast<int64_t>(gid) * DV;
#pragma unroll
        for (int q = 0; q < FV; ++q)
          if (q * SHARE + sub < DV) {
            const uint4 f = fv[q * SHARE + sub];
            st_feat[4 * q] = f.x;
            st_feat[4 * q + 1] = f.y;
            st_feat[4 * q + 2] = f.z;
            st_feat[4 * q + 3] = f.w;
          }
      }
    }
  };
  auto stage_store = [&](int nb) {
    if (st_e < nb) {
      floatx4* sp = reinterpret_cast<floatx4*>(s_sp[st_e]);
      if (st_sub < 3) sp[st_sub] = st_rec0;
      if (RV > 1 && st_sub + SHARE < 3) sp[st_sub + SHARE] = st_rec1;
      if (RV > 2) sp[2] = st_rec2;
      if constexpr (!AHEAD) {  // a thread stages a whole splat: its record holds the Gaussian's index
        const int64_t gid = __float_as_uint(st_rec1[3]);
        const uint4* fv = reinterpret_cast<const uint4*>(a.feat) + gid * DV;
#pragma unroll
        for (int q = 0; q < DV; ++q) {
          const uint4 f = fv[q];
          if (ODD && nonfinite_bf16x8(f)) s_odd = 1;
          reinterpret_cast<uint4*>(&s_fb[st_e * FBS])[q] = f;
        }
      } else if constexpr (DV > 0) {
#pragma unroll
        for (int q = 0; q < FV; ++q)
          if (q * SHARE + st_sub < DV) {
            const uint4 f = make_uint4(st_feat[4 * q], st_feat[4 * q + 1], st_feat[4 * q + 2], st_feat[4 * q + 3]);
            if (ODD && nonfinite_bf16x8(f)) s_odd = 1;
            reinterpret_cast<uint4*>(&s_fb[st_e * FBS])[q * SHARE + st_sub] = f;
          }
      }
      if (st_sub == SHARE - 1) {
        s_sp[st_e][3].x = __uint_as_float(st_lv & kRecMask);
        s_mask[st_e] = static_cast<uint8_t>(st_lv >> kRecBits);  // blocks the support meets
      }
    }
  };
  if (tid == 0) s_max = 0;
  if (ODD && tid == 0) s_odd = 0;
  const int px = bx0 + (lane & 7), py = by0 + (lane >> 3);
  const float pxf = static_cast<float>(px) + 0.5f, pyf = static_cast<float>(py) + 0.5f;
  const int64_t po = static_cast<int64_t>(pose) * HW;
  const int64_t tp = RES ? static_cast<int64_t>(pose) * a.res_t_stride : 0;
  const bool inside = px < W && py < H;

  // Every load that the list does not order goes out first: this pixel's saved
  // state and colours, and the feature maps, so that one memory round trip
  // covers them (the flags, the range and the list's first entries follow).
  uint32_t last = 0;
  float T = 1.f, Tf = 1.f, gC[3] = {0.f, 0.f, 0.f}, GZ = 0.f, gT = 0.f;
  float cf[3] = {0.f, 0.f, 0.f}, ct[3] = {0.f, 0.f, 0.f};
  // planes are read at a wave-uniform base plus one 32-bit byte offset (an
  // image has at most 2^28 pixels)
  const uint32_t pix = 4u * (static_cast<uint32_t>(min(py, H - 1)) * static_cast<uint32_t>(W) +
                             static_cast<uint32_t>(min(px, W - 1)));
  if (inside) {
    last = plane_at(a.n_used + po, pix);
    Tf = plane_at(a.final_T + po, pix);
    if constexpr (RES) {
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        cf[ch] = plane_at(a.fwd_rgb + (3 * po + ch * HW), pix);
        ct[ch] = plane_at(a.res_rgb_t + (3 * tp + ch) * HW, pix);
      }
    } else if (a.g_rgb) {
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) gC[ch] = plane_at(a.g_rgb + (3 * po + ch * HW), pix);
    }
  }
  // B operands of the feature term, loaded in their own layout: lane l holds
  // channels CG (l / 16) + s of pixel 16 b + l % 16 (a pixel outside the image
  // reads the nearest one inside: it blends nothing)
  float gb[CGA][4] = {};
  float gt[RES ? CGA : 1][4];
  bool have_gf = false;
  if constexpr (D > 0) have_gf = RES || a.g_feat != nullptr;
  if constexpr (D > 0) {
    // per pixel block the lane's element of channel s: a uniform base (plane s)
    // plus 32-bit element offsets, where the lane rows' planes lie within reach
    uint32_t xy[4];
    auto load_operands = [&](int64_t row) {
      if constexpr (RES) {
        const float* tb = a.res_feat_t + tp * D * HW + row;
#pragma unroll
        for (int s = 0; s < CG; ++s)
#pragma unroll
          for (int b = 0; b < 4; ++b) gt[s][b] = plane_at(tb + s * HW, xy[b]);
        if (a.fwd_feat_bf16) {
          const uint16_t* fb = static_cast<const uint16_t*>(a.fwd_feat) + D * po + row;
#pragma unroll
          for (int s = 0; s < CG; ++s)
#pragma unroll
            for (int b = 0; b < 4; ++b) gb[s][b] = bf16_lo(plane_at(fb + s * HW, xy[b] / 2));
        } else {
          const float* fb = static_cast<const float*>(a.fwd_feat) + D * po + row;
#pragma unroll
          for (int s = 0; s < CG; ++s)
#pragma unroll
            for (int b = 0; b < 4; ++b) gb[s][b] = plane_at(fb + s * HW, xy[b]);
        }
      } else if (have_gf) {
        const float* gp = a.g_feat + D * po + row;
#pragma unroll
        for (int s = 0; s < CG; ++s)
#pragma unroll
          for (int b = 0; b < 4; ++b) gb[s][b] = plane_at(gp + s * HW, xy[b]);
      }
    };
#pragma unroll
    for (int b = 0; b < 4; ++b)
      xy[b] = static_cast<uint32_t>(min(by0 + 2 * b + ((lane >> 3) & 1), H - 1)) * static_cast<uint32_t>(W) +
              static_cast<uint32_t>(min(bx0 + (lane & 7), W - 1));
    if (static_cast<int64_t>(D) * HW < (1ll << 30)) {
      const uint32_t row = static_cast<uint32_t>(CG * (lane >> 4)) * static_cast<uint32_t>(HW);
#pragma unroll
      for (int b = 0; b < 4; ++b) xy[b] = (xy[b] + row) * 4u;
      load_operands(0);
    } else {
#pragma unroll
      for (int b = 0; b < 4; ++b) xy[b] *= 4u;
      load_operands(CG * (lane >> 4) * HW);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  if (a.flags[0] & 3) return;  // uniform: the render overflowed, its lists are not valid
  const uint2 range = a.ranges[static_cast<int64_t>(pose) * a.c.tiles_per_pose + tile];
  // the list's last round is the first one walked, unless every pixel stopped
  // before it
  uint32_t staged = range.y > range.x ? (range.y - range.x - 1) / NB * NB : 0u;
  const uint32_t gid0 = range.y > range.x ? stage_index(range, staged) : 0u;
  __builtin_amdgcn_sched_barrier(0);

  T = Tf;
  float lsum = 0.f;  // this thread's residual terms (RES)
  if (inside) {
    const float A = 1.f - Tf;
    if constexpr (RES) {
      const float inv = a.res_inv_hw;
#pragma unroll
      for (int ch = 0; ch < 3; ++ch) {
        const float d = cf[ch] - ct[ch];
        lsum += fabsf(d);
        gC[ch] = d > 0.f ? inv : (d < 0.f ? -inv : 0.f);
      }
    }
    gT = gC[0] * a.bg[0] + gC[1] * a.bg[1] + gC[2] * a.bg[2];
    if (a.g_depth && A > 0.f) {
      const float gd = plane_at(a.g_depth + po, pix);
      GZ = gd / A;
      gT += gd * plane_at(a.fwd_depth + po, pix) / A;
    }
    if (a.g_alpha) gT -= plane_at(a.g_alpha + po, pix);
  }
  if constexpr (RES && D > 0) {
    // the residual's gradient (the definition the residual kernel evaluates):
    // sums over this lane's channels, then over the four lane rows; the lane
    // row b then forms block b's factors for all four
    float dot = 0.f, na = 0.f, nb = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b) {
      float d = 0.f, n = 0.f, m = 0.f;
#pragma unroll
      for (int s = 0; s < CG; ++s) {
        d = fmaf(gb[s][b], gt[s][b], d);
        n = fmaf(gb[s][b], gb[s][b], n);
        m = fmaf(gt[s][b], gt[s][b], m);
      }
      d = row_quad_sum(d);
      n = row_quad_sum(n);
      m = row_quad_sum(m);
      const bool mine = (lane >> 4) == b;
      dot = mine ? d : dot;
      na = mine ? n : na;
      nb = mine ? m : nb;
    }
    na = sqrtf(na);
    nb = sqrtf(nb);
    const float n = na * nb + kCosEps;
    const float inv = a.res_inv_hw;
    if (inside) lsum += a.res_lam * (1.f - dot / n);
    const float s1 = -a.res_lam * inv / n;
    const float s2 = na > 0.f ? a.res_lam * inv * dot * nb / (n * n * na) : 0.f;
    float f1[4], f2[4];
    row_broadcast(s1, f1);
    row_broadcast(s2, f2);
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int s = 0; s < CG; ++s) gb[s][b] = fmaf(f1[b], gt[s][b], f2[b] * gb[s][b]);
  }
  if (range.y > range.x) stage_load(range, staged, gid0);  // its records travel while the prologue ends
  // the gradients in three bf16 parts that sum to them exactly (top, middle and
  // last 8 significant bits)
  uint32_t gq[KS][3][4][KW] = {};
  auto split_operands = [&](auto inf) {
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int s = 0; s < CG; s += 2) {
        float x = gb[s][b], y = gb[s + 1 < CGA ? s + 1 : 0][b];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
          gq[s / 8][q][b][(s % 8) / 2] =
              __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);  // the top halves
          const float hx = __uint_as_float(__float_as_uint(x) & 0xffff0000u);
          const float hy = __uint_as_float(__float_as_uint(y) & 0xffff0000u);
          x = inf.value && x == hx ? 0.f : x - hx;
          y = inf.value && y == hy ? 0.f : y - hy;
        }
      }
  };
  bool odd_gf = false;  // uniform: a feature gradient of the wave's block is not finite
  if constexpr (ODD) {
    float zero = 0.f;
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int s = 0; s < CG; ++s) zero = fmaf(gb[s][b], 0.f, zero);
    odd_gf = __any(zero != zero);
    if (odd_gf) split_operands(std::true_type{});
    else split_operands(std::false_type{});
  } else if constexpr (D > 0) {
    split_operands(std::false_type{});
  }
  // list positions this wave must visit: below the largest saved length
  uint32_t wave_max = last;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1)
    wave_max = max(wave_max, static_cast<uint32_t>(__shfl_xor(wave_max, off, kWave)));
  bool nonfinite = !(finite_bits(gC[0]) && finite_bits(gC[1]) && finite_bits(gC[2]) && finite_bits(GZ));
  // FEATGRAD: B operands of the feature sums: channel 16 bl + l % 16 of pixel
  // 16 (l / 16) + i, exchanged through LDS
  float gB[NBL][16] = {};
  if constexpr (FEATGRAD) {
    if (have_gf) {
      float* gf = s_u.gf[wave];
#pragma unroll
      for (int b = 0; b < 4; ++b)
#pragma unroll
        for (int s = 0; s < CG; ++s) gf[(16 * b + (lane & 15)) * GS + CG * (lane >> 4) + s] = gb[s][b];
      wave_lds_fence();
#pragma unroll
      for (int bl = 0; bl < NBL; ++bl)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int c = 16 * bl + (lane & 15);
          if (c < D) gB[bl][i] = gf[(16 * (lane >> 4) + i) * GS + c];
        }
      if (RES || odd_gf) {
#pragma unroll 4
        for (int c = 0; c < D; ++c) nonfinite |= !finite_bits(gf[lane * GS + c]);
      }
    }
  }
  __syncthreads();  // s_max cleared; the walk's staging takes the LDS
  if (lane == 0) atomicMax(&s_max, wave_max);
  if constexpr (RES) {
    // this item's loss share, summed in a fixed order (lanes, then waves)
    lsum = wave_sum(lsum * a.res_inv_hw);
    if (lane == 0) s_lw[wave] = lsum;
  }
  const uint64_t bad_pix = __ballot(nonfinite);
  const bool bad = bad_pix != 0;  // uniform
  {
    const int at = (lane >> 3) * kBwdGcRow + (lane & 7);
#pragma unroll
    for (int c = 0; c < 3; ++c) own.gc[c][at] = gC[c];
    if constexpr (!PO) own.gc[PO ? 0 : 3][at] = GZ;
  }
  if constexpr (FEATGRAD) {
    for (int e = tid; e < NB * GS; e += NT) s_gfe[e] = 0.f;
  }
  __syncthreads();
  if constexpr (RES) {
    if (tid == 0) {
      float t = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) t += s_lw[w];
      a.res_part[(static_cast<int64_t>(pose) * a.c.tiles_per_pose + tile) * Sh::kParts + part] = t;
    }
  }
  const uint32_t n_max = s_max;
  if (n_max == 0) return;

  // the suffix sum; the outputs' direct dependence on the final transmittance,
  // gT Tf, is added where it is used, so that the sum's small first terms are
  // not rounded against it
  float S = 0.f;

  // batches back to front; positions are relative to range.x
  const int n_batches = static_cast<int>((n_max + NB - 1) / NB);
  for (int bi = n_batches - 1; bi >= 0; --bi) {
    const uint32_t b0 = static_cast<uint32_t>(bi) * NB;
    const int nb = static_cast<int>(min(static_cast<uint32_t>(NB), n_max - b0));
    if (staged != b0) stage_load(range, b0, stage_index(range, b0));
    stage_store(nb);
    __syncthreads();
    const bool odd = ODD && __builtin_amdgcn_readfirstlane(s_odd) != 0;
    // the batch's splats that meet this wave's block and lie below its largest
    // saved length, as a mask (the walk) and a list, back to front (the
    // per-lane lookups)
    uint64_t todo;
    int n_mine;
    {
      const bool hit = lane < nb && b0 + lane < wave_max && ((s_mask[lane] >> mask_bit) & 1u);
      todo = __ballot(hit);
      n_mine = __popcll(todo);
      if (hit) own.list[__popcll(todo >> lane) - 1] = static_cast<uint8_t>(lane);
      if (lane == 0) s_hits[wave] = todo;
    }
    wave_lds_fence();
    // the next round's splats travel while this one's are walked
    if (bi > 0) {
      staged = b0 - NB;
      stage_load(range, staged, stage_index(range, staged));
    }
    for (int g0 = 0; g0 < n_mine; g0 += kBwdGroup) {
      // h's feature part of 16 splats: hq[q] for this lane's pixel
      float hq[kBwdGroup];
#pragma unroll
      for (int q = 0; q < kBwdGroup; ++q) hq[q] = 0.f;
      if constexpr (D > 0) {
        const int js = own.list[min(g0 + (lane & 15), n_mine - 1)];
        floatx4 acc[4] = {};
        const uint32_t* fw = &s_fb[js * FBS + (CG / 2) * (lane >> 4)];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
          uint32_t av[KW] = {};
          if constexpr (KW == 4) {
            const uint4 w = reinterpret_cast<const uint4*>(fw)[ks];
            av[0] = w.x; av[1] = w.y; av[KW - 2] = w.z; av[KW - 1] = w.w;
          } else {
            av[0] = fw[0];
            if constexpr (CG > 2) av[1] = fw[1];
          }
          auto product = [&](const uint32_t (&a0)[KW], const uint32_t (&a12)[KW]) {
#pragma unroll
            for (int q = 2; q >= 0; --q)
#pragma unroll
              for (int b = 0; b < 4; ++b) {
                if constexpr (KW == 4) {
                  bf16x8 A, B;
                  __builtin_memcpy(&A, q ? a12 : a0, 16);
                  __builtin_memcpy(&B, gq[ks][q][b], 16);
                  acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B, acc[b], 0, 0, 0);
                } else {
                  shortx4 A, B;
                  __builtin_memcpy(&A, q ? a12 : a0, 8);
                  __builtin_memcpy(&B, gq[ks][q][b], 8);
                  acc[b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(A, B, acc[b], 0, 0, 0);
                }
              }
          };
          if (odd) {  // uniform
            uint32_t finite[KW];
#pragma unroll
            for (int t = 0; t < KW; ++t)
              finite[t] = av[t] & (((av[t] & 0x7f80u) == 0x7f80u ? 0u : 0xffffu) |
                                   ((av[t] & 0x7f800000u) == 0x7f800000u ? 0u : 0xffff0000u));
            product(av, finite);
          } else {
            product(av, av);
          }
        }
        // lane l, register r of block b: splat 4 (l / 16) + r, pixel
        // 16 b + l % 16 -> this lane's pixel
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          uint32_t t[4];
#pragma unroll
          for (int b = 0; b < 4; ++b) t[b] = __float_as_uint(acc[b][r]);
          transpose_rows(t[0], t[1], t[2], t[3]);
#pragma unroll
          for (int k = 0; k < 4; ++k) hq[4 * k + r] = __uint_as_float(t[k]);
        }
      }
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int h0 = g0 + half * kBwdHalf;
        if (h0 >= n_mine) break;  // uniform
        const int wrow = FEATGRAD ? half * kBwdHalf : 0;
        // a splat's geometry and colour are read a step ahead: a step that waits
        // for its own LDS reads takes twice as long
        int jn = 63 - __builtin_clzll(todo);
        float4 geo_n = s_sp[jn][0], opz_n = s_sp[jn][1], col_n = s_sp[jn][2];
#pragma unroll
        for (int q = 0; q < kBwdHalf; ++q) {
          if (todo == 0) break;  // uniform
          const int jj = jn;
          const float4 geo = geo_n, opz = opz_n, col = col_n;
          todo &= ~(1ull << jj);
          if (q + 1 < kBwdHalf) {
            jn = todo ? 63 - __builtin_clzll(todo) : jj;
            geo_n = s_sp[jn][0];
            opz_n = s_sp[jn][1];
            col_n = s_sp[jn][2];
            __atomic_signal_fence(__ATOMIC_SEQ_CST);  // issued here, not where they are used
          }
          const float dx = pxf - geo.x, dy = pyf - geo.y;
          const float power = pair_power(dx, dy, geo.z, geo.w, opz.x);
          const float oG = opz.y * __expf(power);
          const float alpha = fminf(kAlphaMax, oG);
          float dpow = 0.f, w = 0.f;
          if (b0 + jj < last && !(power > 0.f) && !(alpha < kAlphaMin)) {
            const float iom = __builtin_amdgcn_rcpf(1.f - alpha);  // alpha <= 0.99
            T *= iom;
            w = alpha * T;
            // gradient arithmetic (not a blend decision): fused multiply-adds
            float h = fmaf(gC[0], col.x, fmaf(gC[1], col.y, fmaf(gC[2], col.z, hq[half * kBwdHalf + q])));
            if constexpr (!PO) h = fmaf(GZ, opz.z, h);
            const float dA = fmaf(T, h, -(fmaf(gT, Tf, S) * iom));
            S = fmaf(w, h, S);
            dpow = oG <= kAlphaMax ? dA * alpha : 0.f;
          }
          own.d[q][lane] = dpow;
          own.w[wrow + q][lane] = w;
        }
        wave_lds_fence();
        // transposed: lane l takes splat l % 8's pixel row l / 8 of the block
        {
          const int s = lane & 7, row = lane >> 3;
          const int e = h0 + s;
          const int slot = own.list[min(e, n_mine - 1)];
          const float4 geo = s_sp[slot][0];
          const float x0 = static_cast<float>(bx0) + 0.5f - geo.x;
          const float dy = static_cast<float>(by0 + row) + 0.5f - geo.y;
          const float bdy = geo.w * dy, cdy = s_sp[slot][1].x * dy;
          float m0 = 0.f, m1 = 0.f, m2 = 0.f, su = 0.f, sv = 0.f, c[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int i4 = 0; i4 < 2; ++i4) {
            const float4 d4 = *reinterpret_cast<const float4*>(&own.d[s][8 * row + 4 * i4]);
            const float4 w4 = *reinterpret_cast<const float4*>(&own.w[wrow + s][8 * row + 4 * i4]);
            const float dv[4] = {d4.x, d4.y, d4.z, d4.w}, wv[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float dx = x0 + static_cast<float>(4 * i4 + i);
              const float t = dv[i] * dx;
              m0 += dv[i];
              m1 += t;
              m2 = fmaf(t, dx, m2);
              su = fmaf(dv[i], fmaf(geo.z, dx, bdy), su);
              sv = fmaf(dv[i], fmaf(geo.w, dx, cdy), sv);
            }
#pragma unroll
            for (int k = 0; k < (PO ? 3 : 4); ++k) {
              const float4 g4 = *reinterpret_cast<const float4*>(&own.gc[k][row * kBwdGcRow + 4 * i4]);
              const float gv[4] = {g4.x, g4.y, g4.z, g4.w};
              if (!bad) {
#pragma unroll
                for (int i = 0; i < 4; ++i) c[k] = fmaf(wv[i], gv[i], c[k]);
              } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) c[k] = wv[i] != 0.f ? fmaf(wv[i], gv[i], c[k]) : c[k];
              }
            }
          }
          const float v[8] = {su, sv, m2, m1 * dy, m0 * dy * dy, c[0], c[1], c[2]};
          const float tot = octet_scatter8(v, lane);
          const int k = lane >> 3;
          if (e < n_mine) own.g[k * GR + slot] = tot;
          if constexpr (!PO) {
            const float t2 = octet_sum2(m0, c[3]);
            if ((lane & 31) < 8 && e < n_mine) own.g[(lane < 32 ? NV - 2 : NV - 1) * GR + slot] = t2;
          }
        }
        wave_lds_fence();  // the rows are rewritten by the next half
      }
      if constexpr (FEATGRAD) {
        // rows of splats past the list hold stale weights: their sums are dropped
        const int q4 = lane >> 4, ch = lane & 15;
        floatx4 acc[NBL] = {};
#pragma unroll
        for (int i4 = 0; i4 < 4; ++i4) {
          const float4 w4 = *reinterpret_cast<const float4*>(&own.w[ch][16 * q4 + 4 * i4]);
          const float wv[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int bl = 0; bl < NBL; ++bl) {
              float g = gB[bl][4 * i4 + i];
              if (bad) g = ((bad_pix >> (16 * q4 + 4 * i4 + i)) & 1u) ? 0.f : g;
              acc[bl] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[i], g, acc[bl], 0, 0, 0);
            }
        }
        // lane l, register r: splat 4 (l / 16) + r, channel 16 bl + l % 16
        if (bad) {  // uniform; pixels with non-finite gradients, for the splats blended there
#pragma unroll
          for (int i = 0; i < 16; ++i)
            for (int k = 0; k < 4; ++k) {
              const int p = 16 * k + i;
              if (!((bad_pix >> p) & 1u)) continue;
#pragma unroll
              for (int bl = 0; bl < NBL; ++bl) {
                const float g = __shfl(gB[bl][i], 16 * k + ch, kWave);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                  const float wv = own.w[4 * q4 + r][p];
                  if (wv != 0.f) acc[bl][r] = fmaf(wv, g, acc[bl][r]);
                }
              }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int e = g0 + 4 * q4 + r;
          if (e < n_mine) {
            const int slot = own.list[e];
#pragma unroll
            for (int bl = 0; bl < NBL; ++bl)
              if (16 * bl + ch < D) atomicAdd(&s_gfe[slot * GS + 16 * bl + ch], acc[bl][r]);
          }
        }
        wave_lds_fence();
      }
    }
    __syncthreads();
    if (ODD && tid == 0) s_odd = 0;  // read by every wave; the next round's staging waits below
    // one global atomic per nonzero sum of the round: the waves that hit the
    // splat, in order
    int first = tid;
    asm volatile("" : "+v"(first));  // keeps what follows from it inside the round
    for (int e = first; e < nb * NV; e += NT) {
      const int slot = e / NV, k = e - slot * NV;
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w)
        if ((s_hits[w] >> slot) & 1u) v += s_u.walk.wave[w].g[k * GR + slot];
      // rows: d (a dx + b dy), d (b dx + c dy), d dx^2, d dx dy, d dy^2, w gC (3), d, w gZ
      const int at = k < 5 ? k : (k < 8 ? k + 2 : k - 3);
      if (v != 0.f)
        atomicAdd(a.g_rec + static_cast<int64_t>(__float_as_uint(s_sp[slot][3].x)) * kGradRecStride + at, v);
    }
    if constexpr (FEATGRAD) {
      for (int e = first; e < nb * D; e += NT) {
        const int slot = e / D, d = e - slot * D;
        const float v = s_gfe[slot * GS + d];
        if (v != 0.f) {
          atomicAdd(a.g_featvec + static_cast<int64_t>(__float_as_uint(s_sp[slot][1].w)) * D + d, v);
          s_gfe[slot * GS + d] = 0.f;
        }
      }
    }
    __syncthreads();  // the next batch's staging overwrites s_sp
  }
}

// One workgroup per item ((pose, tile), or a quadrant of a 32-pixel tile), or
// (PERSIST) a grid of workgroups claiming runs of kQueueChunk items from a
// device counter until it passes the item count.
template <int TILE, int D, bool FEATGRAD, bool RES, bool PERSIST, bool PO = false>
__global__ __launch_bounds__(BlockShape<TILE>::kThreads, (PO && D <= 32 && !PERSIST && TILE != 8) ? 4 : 1) void
blend_bwd_kernel(BackArgs a) {
  if constexpr (PERSIST) {
    if (a.flags[0] & 3) return;
    __shared__ int s_item;
    for (;;) {
      if (threadIdx.x == 0) s_item = static_cast<int>(atomicAdd(a.queue, static_cast<uint32_t>(kQueueChunk)));
      __syncthreads();
      const int first = s_item;
      __syncthreads();
      if (first >= a.n_items) break;
      const int last = min(first + kQueueChunk, a.n_items);
      for (int item = first; item < last; ++item) {
        blend_bwd_item<TILE, D, FEATGRAD, RES, PO>(a, item);
        __syncthreads();  // the item's LDS is reused by the next one
      }
    }
  } else {
    blend_bwd_item<TILE, D, FEATGRAD, RES, PO>(a, xcd_item(blockIdx.x, gridDim.x));
  }
}

// Per-pose loss from the per-tile shares, in a fixed order (deterministic).
__global__ __launch_bounds__(256) void loss_reduce_kernel(const float* part, int32_t tiles_per_pose, float* loss) {
  __shared__ float s_r[256];
  const int pose = blockIdx.x;
  const float* p = part + static_cast<int64_t>(pose) * tiles_per_pose;
  float v = 0.f;
  for (int t = threadIdx.x; t < tiles_per_pose; t += 256) v += p[t];
  s_r[threadIdx.x] = v;
  __syncthreads();
  for (int st = 128; st > 0; st >>= 1) {
    if (threadIdx.x < st) s_r[threadIdx.x] += s_r[threadIdx.x + st];
    __syncthreads();
  }
  if (threadIdx.x == 0) loss[pose] = s_r[0];
}

void launch_loss_reduce(const float* part, int32_t tiles_per_pose, int32_t P, float* loss, hipStream_t s) {
  hipLaunchKernelGGL(loss_reduce_kernel, dim3(P), dim3(256), 0, s, part, tiles_per_pose, loss);
}

template <int TILE, int D, bool PERSIST>
static void launch_bwd_tdp(const BackArgs& a, int n_ctas, hipStream_t s) {
  constexpr int NT = BlockShape<TILE>::kThreads;
  constexpr bool F = D > 0;  // without features there is no feature gradient
  if (a.res_rgb_t) {
    if (F && a.g_featvec)
      hipLaunchKernelGGL((blend_bwd_kernel<TILE, D, F, true, PERSIST>), dim3(n_ctas), dim3(NT), 0, s, a);
    else if (a.pose_only)
      hipLaunchKernelGGL((blend_bwd_kernel<TILE, D, false, true, PERSIST, true>), dim3(n_ctas), dim3(NT), 0, s, a);
    else
      hipLaunchKernelGGL((blend_bwd_kernel<TILE, D, false, true, PERSIST>), dim3(n_ctas), dim3(NT), 0, s, a);
  } else {
    if (F && a.g_featvec)
      hipLaunchKernelGGL((blend_bwd_kernel<TILE, D, F, false, PERSIST>), dim3(n_ctas), dim3(NT), 0, s, a);
    else
      hipLaunchKernelGGL((blend_bwd_kernel<TILE, D, false, false, PERSIST>), dim3(n_ctas), dim3(NT), 0, s, a);
  }
}

template <int TILE, int D>
static void launch_bwd_td(const BackArgs& a, hipStream_t s) {
  if (a.schedule != kSchedGrid) launch_bwd_tdp<TILE, D, true>(a, a.n_ctas, s);
  else launch_bwd_tdp<TILE, D, false>(a, a.n_items, s);
}

template <int TILE>
static void launch_bwd_t(const BackArgs& a, hipStream_t s) {
  switch (a.D) {
    case 0: launch_bwd_td<TILE, 0>(a, s); break;
    case 8: launch_bwd_td<TILE, 8>(a, s); break;
    case 16: launch_bwd_td<TILE, 16>(a, s); break;
    case 32: launch_bwd_td<TILE, 32>(a, s); break;
    default: launch_bwd_td<TILE, 64>(a, s); break;
  }
}

void launch_blend_bwd(const BackArgs& a, hipStream_t s) {
  switch (a.c.tile) {
    case 8: launch_bwd_t<8>(a, s); break;
    case 32: launch_bwd_t<32>(a, s); break;
    default: launch_bwd_t<16>(a, s); break;
  }
}

// ------------------------------------------------------------ projection backward
// Gradient of the real SH basis polynomials (as functions on R^3) contracted
// with per-basis weights c[k] (one colour channel): returns sum_k c_k grad Y_k.
template <int DEG>
__device__ __forceinline__ void sh_grad_dir(const float* c, float x, float y, float z, float g[3]) {
  g[0] = g[1] = g[2] = 0.f;
  if constexpr (DEG >= 1) {
    const float C1 = 0.48860251190291987f;
    g[1] += -C1 * c[1];
    g[2] += C1 * c[2];
    g[0] += -C1 * c[3];
  }
  if constexpr (DEG >= 2) {
    const float A = 1.0925484305920792f, B = 0.31539156525252005f, Cc = 0.5462742152960396f;
    g[0] += c[4] * A * y;
    g[1] += c[4] * A * x;
    g[1] += -c[5] * A * z;
    g[2] += -c[5] * A * y;
    g[0] += -2.f * c[6] * B * x;
    g[1] += -2.f * c[6] * B * y;
    g[2] += 4.f * c[6] * B * z;
    g[0] += -c[7] * A * z;
    g[2] += -c[7] * A * x;
    g[0] += 2.f * c[8] * Cc * x;
    g[1] += -2.f * c[8] * Cc * y;
  }
  if constexpr (DEG >= 3) {
    const float a3 = 0.5900435899266435f, b3 = 2.890611442640554f, c3 = 0.4570457994644658f,
                d3 = 0.3731763325901154f, e3 = 1.445305721320277f;
    const float xx = x * x, yy = y * y, zz = z * z;
    g[0] += c[9] * (-6.f * a3 * x * y);
    g[1] += c[9] * (-a3 * (3.f * xx - 3.f * yy));
    g[0] += c[10] * b3 * y * z;
    g[1] += c[10] * b3 * x * z;
    g[2] += c[10] * b3 * x * y;
    g[0] += c[11] * (2.f * c3 * x * y);
    g[1] += c[11] * (-c3 * (4.f * zz - xx - 3.f * yy));
    g[2] += c[11] * (-8.f * c3 * y * z);
    g[0] += c[12] * (-6.f * d3 * x * z);
    g[1] += c[12] * (-6.f * d3 * y * z);
    g[2] += c[12] * (d3 * (6.f * zz - 3.f * xx - 3.f * yy));
    g[0] += c[13] * (-c3 * (4.f * zz - 3.f * xx - yy));
    g[1] += c[13] * (2.f * c3 * x * y);
    g[2] += c[13] * (-8.f * c3 * x * z);
    g[0] += c[14] * (2.f * e3 * x * z);
    g[1] += c[14] * (-2.f * e3 * y * z);
    g[2] += c[14] * (e3 * (xx - yy));
    g[0] += c[15] * (-a3 * (3.f * xx - 3.f * yy));
    g[1] += c[15] * (6.f * a3 * x * y);
  }
}

// The Gaussian's SH coefficients (3 (DEG+1)^2 floats), read once for the
// colour and its direction gradient (16-byte loads when the array allows).
template <int DEG>
__device__ __forceinline__ void load_sh(const float* sh, int64_t i, float* v) {
  constexpr int N = 3 * (DEG + 1) * (DEG + 1);
  const float* c = sh + static_cast<int64_t>(N) * i;
  if constexpr (N % 4 == 0) {
    if ((reinterpret_cast<uintptr_t>(sh) & 15) == 0) {
#pragma unroll
      for (int q = 0; q < N / 4; ++q) {
        const float4 f = reinterpret_cast<const float4*>(c)[q];
        v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
      }
      return;
    }
  }
#pragma unroll
  for (int k = 0; k < N; ++k) v[k] = c[k];
}

// One record's gradients: the pose tangent's six components are added to gp;
// GAUSS: the Gaussian's own gradients (means, opacity, scales, rotation, SH)
// where their arrays are given.
template <int DEG, bool GAUSS>
__device__ __forceinline__ void record_grad(const ProjBackArgs& a, const int pose, const uint32_t slot, float gp[6]) {
  constexpr int K = (DEG + 1) * (DEG + 1);
  {
    const int64_t idx = static_cast<int64_t>(pose) * a.rec_cap + slot;
    const float* gr = a.g_rec + idx * kGradRecStride;
    const Splat sp = a.recs[idx];
    // from the sums of dL/dpower over the splat's pixels: power is
    // -(ca dx^2 + cc dy^2) / 2 - cb dx dy with dx, dy from the mean, and
    // alpha = o e^power
    const float g_u = gr[0], g_v = gr[1];
    const float g_ca = -0.5f * gr[2], g_cb = -gr[3], g_cc = -0.5f * gr[4], g_o = gr[5] / sp.o, g_z = gr[6];
    const float gcol[3] = {gr[7], gr[8], gr[9]};
    const int64_t i = sp.gid;
    const float* Pm = a.poses + 12 * pose;
    const float mu[3] = {a.g.means[3 * i], a.g.means[3 * i + 1], a.g.means[3 * i + 2]};
    const float4 q4 = reinterpret_cast<const float4*>(a.g.quats)[i];
    const float ls[3] = {a.g.log_scales[3 * i], a.g.log_scales[3 * i + 1], a.g.log_scales[3 * i + 2]};
    float Sw[6];
    cov3_from(q4, ls, Sw);
    float mc[3];
    to_camera(Pm, mu, mc);
    const float x = mc[0], y = mc[1], z = mc[2];
    const float iz = 1.f / z;
    const float xz = x / z, yz = y / z;
    const bool clx = fabsf(xz) > a.c.limx, cly = fabsf(yz) > a.c.limy;
    const float xh = fminf(fmaxf(xz, -a.c.limx), a.c.limx);
    const float yh = fminf(fmaxf(yz, -a.c.limy), a.c.limy);
    const float fx = a.c.fx, fy = a.c.fy;
    const float J00 = fx * iz, J02 = -fx * xh * iz, J11 = fy * iz, J12 = -fy * yh * iz;
    // M = J R (rows m0, m1)
    const float m0[3] = {J00 * Pm[0] + J02 * Pm[8], J00 * Pm[1] + J02 * Pm[9], J00 * Pm[2] + J02 * Pm[10]};
    const float m1[3] = {J11 * Pm[4] + J12 * Pm[8], J11 * Pm[5] + J12 * Pm[9], J11 * Pm[6] + J12 * Pm[10]};
    // dL/dSigma' = -C G C with G = [[g_ca, g_cb/2], [g_cb/2, g_cc]]
    const float ca = sp.ca, cb = sp.cb, cc = sp.cc;
    const float h01 = 0.5f * g_cb;
    // C G
    const float t00 = ca * g_ca + cb * h01, t01 = ca * h01 + cb * g_cc;
    const float t10 = cb * g_ca + cc * h01, t11 = cb * h01 + cc * g_cc;
    const float Gs00 = -(t00 * ca + t01 * cb);
    const float Gs01 = -(t00 * cb + t01 * cc);
    const float Gs11 = -(t10 * cb + t11 * cc);
    // dL/dM = 2 Gs M Sw (2x3)
    float SM0[3], SM1[3];  // Sw m0, Sw m1
    SM0[0] = Sw[0] * m0[0] + Sw[1] * m0[1] + Sw[2] * m0[2];
    SM0[1] = Sw[1] * m0[0] + Sw[3] * m0[1] + Sw[4] * m0[2];
    SM0[2] = Sw[2] * m0[0] + Sw[4] * m0[1] + Sw[5] * m0[2];
    SM1[0] = Sw[0] * m1[0] + Sw[1] * m1[1] + Sw[2] * m1[2];
    SM1[1] = Sw[1] * m1[0] + Sw[3] * m1[1] + Sw[4] * m1[2];
    SM1[2] = Sw[2] * m1[0] + Sw[4] * m1[1] + Sw[5] * m1[2];
    float gM0[3], gM1[3];
    for (int k = 0; k < 3; ++k) {
      gM0[k] = 2.f * (Gs00 * SM0[k] + Gs01 * SM1[k]);
      gM1[k] = 2.f * (Gs01 * SM0[k] + Gs11 * SM1[k]);
    }
    // dL/dJ = dL/dM R^T (only the structurally non-zero entries)
    const float gJ00 = gM0[0] * Pm[0] + gM0[1] * Pm[1] + gM0[2] * Pm[2];
    const float gJ02 = gM0[0] * Pm[8] + gM0[1] * Pm[9] + gM0[2] * Pm[10];
    const float gJ11 = gM1[0] * Pm[4] + gM1[1] * Pm[5] + gM1[2] * Pm[6];
    const float gJ12 = gM1[0] * Pm[8] + gM1[1] * Pm[9] + gM1[2] * Pm[10];
    // dL/dmc
    const float iz2 = iz * iz;
    float gmc[3];
    gmc[0] = g_u * fx * iz;
    gmc[1] = g_v * fy * iz;
    gmc[2] = -g_u * fx * x * iz2 - g_v * fy * y * iz2 + g_z;
    gmc[2] += -gJ00 * fx * iz2 - gJ11 * fy * iz2;
    if (!clx) {
      gmc[0] += -gJ02 * fx * iz2;
      gmc[2] += 2.f * gJ02 * fx * x * iz2 * iz;
    } else {
      gmc[2] += gJ02 * fx * xh * iz2;
    }
    if (!cly) {
      gmc[1] += -gJ12 * fy * iz2;
      gmc[2] += 2.f * gJ12 * fy * y * iz2 * iz;
    } else {
      gmc[2] += gJ12 * fy * yh * iz2;
    }
    // dL/dR through the covariance: Jcol^T dL/dM, i.e. GRc[r][c] = sum_a J[a][r] gM[a][c]
    float GRc[3][3];
    for (int c2 = 0; c2 < 3; ++c2) {
      GRc[0][c2] = J00 * gM0[c2];
      GRc[1][c2] = J11 * gM1[c2];
      GRc[2][c2] = J02 * gM0[c2] + J12 * gM1[c2];
    }
    // B = R GRc^T ; dL/dphi (covariance part) = (B12 - B21, B20 - B02, B01 - B10)
    float B[3][3];
    for (int r = 0; r < 3; ++r)
      for (int c2 = 0; c2 < 3; ++c2)
        B[r][c2] = Pm[4 * r + 0] * GRc[c2][0] + Pm[4 * r + 1] * GRc[c2][1] + Pm[4 * r + 2] * GRc[c2][2];
    // SH view direction
    const float Cx = -(Pm[0] * Pm[3] + Pm[4] * Pm[7] + Pm[8] * Pm[11]);
    const float Cy = -(Pm[1] * Pm[3] + Pm[5] * Pm[7] + Pm[9] * Pm[11]);
    const float Cz = -(Pm[2] * Pm[3] + Pm[6] * Pm[7] + Pm[10] * Pm[11]);
    float dir[3] = {mu[0] - Cx, mu[1] - Cy, mu[2] - Cz};
    const float inv = rsqrtf(dir[0] * dir[0] + dir[1] * dir[1] + dir[2] * dir[2]);
    const float n0 = dir[0] * inv, n1 = dir[1] * inv, n2 = dir[2] * inv;
    // the forward's unclamped colour (the sums of sh_colour_raw, in its
    // order), from coefficients read once
    float shv[3 * K];
    load_sh<DEG>(a.g.sh, i, shv);
    float Y[K];
    sh_basis<DEG>(n0, n1, n2, Y);
    float raw[3] = {0.5f, 0.5f, 0.5f};
#pragma unroll
    for (int k = 0; k < K; ++k) {
      raw[0] = fmaf(shv[3 * k + 0], Y[k], raw[0]);
      raw[1] = fmaf(shv[3 * k + 1], Y[k], raw[1]);
      raw[2] = fmaf(shv[3 * k + 2], Y[k], raw[2]);
    }
    float graw[3];
    for (int c2 = 0; c2 < 3; ++c2) graw[c2] = raw[c2] > 0.f ? gcol[c2] : 0.f;
    float gdir[3] = {0.f, 0.f, 0.f};
    if constexpr (DEG >= 1) {
      for (int c2 = 0; c2 < 3; ++c2) {
        if (graw[c2] == 0.f) continue;
        float cch[K];
        for (int k = 0; k < K; ++k) cch[k] = shv[3 * k + c2];
        float gg[3];
        sh_grad_dir<DEG>(cch, n0, n1, n2, gg);
        const float nd = gg[0] * n0 + gg[1] * n1 + gg[2] * n2;
        gdir[0] += graw[c2] * (gg[0] - n0 * nd) * inv;
        gdir[1] += graw[c2] * (gg[1] - n1 * nd) * inv;
        gdir[2] += graw[c2] * (gg[2] - n2 * nd) * inv;
      }
    }
    if (GAUSS && a.g_sh) {
      float* gs = a.g_sh + static_cast<int64_t>(K) * 3 * i;
      for (int k = 0; k < K; ++k)
        for (int c2 = 0; c2 < 3; ++c2)
          if (graw[c2] != 0.f) atomicAdd(gs + 3 * k + c2, graw[c2] * Y[k]);
    }
    // Gaussian gradients
    if (GAUSS && a.g_means) {
      for (int c2 = 0; c2 < 3; ++c2) {
        const float gm = Pm[c2] * gmc[0] + Pm[4 + c2] * gmc[1] + Pm[8 + c2] * gmc[2] + gdir[c2];
        atomicAdd(a.g_means + 3 * i + c2, gm);
      }
    }
    if (GAUSS && a.g_opac) atomicAdd(a.g_opac + i, g_o);
    if (GAUSS && (a.g_log_scales || a.g_quats)) {
      // dL/dSigma_w = M^T Gs M
      float Gw[3][3];
      for (int r = 0; r < 3; ++r)
        for (int c2 = 0; c2 < 3; ++c2)
          Gw[r][c2] = m0[r] * (Gs00 * m0[c2] + Gs01 * m1[c2]) + m1[r] * (Gs01 * m0[c2] + Gs11 * m1[c2]);
      const float qn = rsqrtf(q4.x * q4.x + q4.y * q4.y + q4.z * q4.z + q4.w * q4.w);
      const float w = q4.x * qn, qx = q4.y * qn, qy = q4.z * qn, qz = q4.w * qn;
      const float Rq[3][3] = {{1.f - 2.f * (qy * qy + qz * qz), 2.f * (qx * qy - w * qz), 2.f * (qx * qz + w * qy)},
                              {2.f * (qx * qy + w * qz), 1.f - 2.f * (qx * qx + qz * qz), 2.f * (qy * qz - w * qx)},
                              {2.f * (qx * qz - w * qy), 2.f * (qy * qz + w * qx), 1.f - 2.f * (qx * qx + qy * qy)}};
      const float s2[3] = {__expf(2.f * ls[0]), __expf(2.f * ls[1]), __expf(2.f * ls[2])};
      if (a.g_log_scales) {
        for (int k = 0; k < 3; ++k) {
          float acc = 0.f;
          for (int r = 0; r < 3; ++r)
            for (int c2 = 0; c2 < 3; ++c2) acc += Rq[r][k] * Gw[r][c2] * Rq[c2][k];
          atomicAdd(a.g_log_scales + 3 * i + k, 2.f * s2[k] * acc);
        }
      }
      if (a.g_quats) {
        // dL/dRq = 2 Gw Rq S^2
        float G[3][3];
        for (int r = 0; r < 3; ++r)
          for (int c2 = 0; c2 < 3; ++c2)
            G[r][c2] = 2.f * (Gw[r][0] * Rq[0][c2] + Gw[r][1] * Rq[1][c2] + Gw[r][2] * Rq[2][c2]) * s2[c2];
        const float gw = 2.f * (-qz * G[0][1] + qy * G[0][2] + qz * G[1][0] - qx * G[1][2] - qy * G[2][0] + qx * G[2][1]);
        const float gx = 2.f * (qy * G[0][1] + qz * G[0][2] + qy * G[1][0] - 2.f * qx * G[1][1] - w * G[1][2] +
                                qz * G[2][0] + w * G[2][1] - 2.f * qx * G[2][2]);
        const float gy = 2.f * (-2.f * qy * G[0][0] + qx * G[0][1] + w * G[0][2] + qx * G[1][0] + qz * G[1][2] -
                                w * G[2][0] + qz * G[2][1] - 2.f * qy * G[2][2]);
        const float gz = 2.f * (-2.f * qz * G[0][0] - w * G[0][1] + qx * G[0][2] + w * G[1][0] - 2.f * qz * G[1][1] +
                                qy * G[1][2] + qx * G[2][0] + qy * G[2][1]);
        const float dq = gw * w + gx * qx + gy * qy + gz * qz;
        atomicAdd(a.g_quats + 4 * i + 0, (gw - w * dq) * qn);
        atomicAdd(a.g_quats + 4 * i + 1, (gx - qx * dq) * qn);
        atomicAdd(a.g_quats + 4 * i + 2, (gy - qy * dq) * qn);
        atomicAdd(a.g_quats + 4 * i + 3, (gz - qz * dq) * qn);
      }
    }
    // pose tangent (rho, phi)
    gp[0] += gmc[0] + Pm[0] * gdir[0] + Pm[1] * gdir[1] + Pm[2] * gdir[2];
    gp[1] += gmc[1] + Pm[4] * gdir[0] + Pm[5] * gdir[1] + Pm[6] * gdir[2];
    gp[2] += gmc[2] + Pm[8] * gdir[0] + Pm[9] * gdir[1] + Pm[10] * gdir[2];
    gp[3] += (y * gmc[2] - z * gmc[1]) + (B[1][2] - B[2][1]);
    gp[4] += (z * gmc[0] - x * gmc[2]) + (B[2][0] - B[0][2]);
    gp[5] += (x * gmc[1] - y * gmc[0]) + (B[0][1] - B[1][0]);
  }
}

// Records of one pose per blockIdx.y, walked compacted (the in-use slots of
// the kSub sub-segments, through the prefix of their counters) by a grid of
// workgroups; each thread sums its records' pose tangents, the workgroup
// reduces them (wave sums, then four waves) and adds them once per pose.
template <int DEG, bool GAUSS>
__global__ __launch_bounds__(256) void project_bwd_kernel(ProjBackArgs a) {
  __shared__ uint32_t s_pre[kSub + 1];
  __shared__ float s_red[4][6];
  if (a.flags[0] & 3) return;
  const int pose = blockIdx.y;
  const uint32_t sub_cap = a.rec_cap / kSub;
  if (threadIdx.x < kWave) {
    const int l = threadIdx.x;
    uint32_t v = l < kSub ? min(a.pose_count[pose * kSub + l], sub_cap) : 0u;
#pragma unroll
    for (int off = 1; off < kSub; off <<= 1) {
      const uint32_t u = __shfl_up(v, off, kWave);
      if (l >= off) v += u;
    }
    if (l < kSub) s_pre[l + 1] = v;
    if (l == 0) s_pre[0] = 0;
  }
  __syncthreads();
  const uint32_t total = s_pre[kSub];
  float gp[6] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (uint32_t c = blockIdx.x * 256 + threadIdx.x; c < total; c += gridDim.x * 256) {
    int lo = 0, hi = kSub;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_pre[mid] <= c) lo = mid;
      else hi = mid;
    }
    record_grad<DEG, GAUSS>(a, pose, static_cast<uint32_t>(lo) * sub_cap + (c - s_pre[lo]), gp);
  }
  if (!a.g_pose) return;
  const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < 6; ++k) {
    float v = gp[k];
    for (int off = kWave / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    if (lane == 0) s_red[wave][k] = v;
  }
  __syncthreads();
  if (threadIdx.x < 6) {
    const int k = threadIdx.x;
    const float v = (s_red[0][k] + s_red[1][k]) + (s_red[2][k] + s_red[3][k]);
    if (v != 0.f) atomicAdd(a.g_pose + 6 * pose + k, v);
  }
}

// The gradient sums of the in-use records, cleared before the blend backward
// adds into them: a grid per pose walking the compacted slots.
__global__ __launch_bounds__(256) void zero_grad_rec_kernel(float* g, const uint32_t* pose_count, uint32_t rec_cap) {
  __shared__ uint32_t s_pre[kSub + 1];
  const int pose = blockIdx.y;
  const uint32_t sub_cap = rec_cap / kSub;
  if (threadIdx.x < kWave) {
    const int l = threadIdx.x;
    uint32_t v = l < kSub ? min(pose_count[pose * kSub + l], sub_cap) : 0u;
#pragma unroll
    for (int off = 1; off < kSub; off <<= 1) {
      const uint32_t u = __shfl_up(v, off, kWave);
      if (l >= off) v += u;
    }
    if (l < kSub) s_pre[l + 1] = v;
    if (l == 0) s_pre[0] = 0;
  }
  __syncthreads();
  const uint32_t total = s_pre[kSub];
  const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
  for (uint32_t c = blockIdx.x * 256 + threadIdx.x; c < total; c += gridDim.x * 256) {
    int lo = 0, hi = kSub;
    while (hi - lo > 1) {
      const int mid = (lo + hi) >> 1;
      if (s_pre[mid] <= c) lo = mid;
      else hi = mid;
    }
    const uint32_t slot = static_cast<uint32_t>(lo) * sub_cap + (c - s_pre[lo]);
    float4* d = reinterpret_cast<float4*>(g + (static_cast<int64_t>(pose) * rec_cap + slot) * kGradRecStride);
    d[0] = z; d[1] = z; d[2] = z;
  }
}

void launch_zero_grad_rec(float* g, const uint32_t* pose_count, uint32_t rec_cap, int P, hipStream_t s) {
  const dim3 grid(std::min<uint32_t>((rec_cap + 255) / 256, 512), P);
  hipLaunchKernelGGL(zero_grad_rec_kernel, grid, dim3(256), 0, s, g, pose_count, rec_cap);
}

template <bool GAUSS>
static void launch_project_bwd_g(const ProjBackArgs& a, hipStream_t s) {
  // enough workgroups per pose for its slots at one record per thread, at
  // most kProjBwdBlocks (the walk strides over the rest)
  constexpr uint32_t kProjBwdBlocks = 512;
  const dim3 grid(std::min<uint32_t>((a.rec_cap + 255) / 256, kProjBwdBlocks), a.P);
  switch (a.g.sh_degree) {
    case 0: hipLaunchKernelGGL((project_bwd_kernel<0, GAUSS>), grid, dim3(256), 0, s, a); break;
    case 1: hipLaunchKernelGGL((project_bwd_kernel<1, GAUSS>), grid, dim3(256), 0, s, a); break;
    case 2: hipLaunchKernelGGL((project_bwd_kernel<2, GAUSS>), grid, dim3(256), 0, s, a); break;
    default: hipLaunchKernelGGL((project_bwd_kernel<3, GAUSS>), grid, dim3(256), 0, s, a); break;
  }
}

void launch_project_bwd(const ProjBackArgs& a, hipStream_t s) {
  // without per-Gaussian gradients the kernel carries none of their code
  if (a.g_means || a.g_opac || a.g_log_scales || a.g_quats || a.g_sh) launch_project_bwd_g<true>(a, s);
  else launch_project_bwd_g<false>(a, s);
}

}  // namespace hgsr
