// Front-to-back alpha blend, one workgroup per (pose, tile).
//
// Each wave owns an 8x8 block of pixels, one per lane, and a workgroup a 16x16
// block (tile 8: 8x8; a 32x32 tile is four workgroups, one per quadrant, that
// walk the same list); compact blocks keep the lanes' blend decisions coherent.
// The workgroup walks the tile's depth-ordered list in rounds: each splat
// (record, bf16 feature vector) is staged into LDS by one thread or by four,
// its loads sent off a round ahead and the list entry's two rounds ahead (the
// record's address comes from the entry, its feature's from the Gaussian index
// beside it); each wave takes the staged splats whose support meets its block
// as 64-bit masks and runs its pixels through them, reading each splat as an
// LDS broadcast one step ahead.  A pixel stops at the first splat that would
// take its transmittance below 1e-4; the round loop ends when every pixel of
// the block has stopped.  Outputs are planar per pose.
//
// What bounds it: with 32 channels, at 64 poses of 960x540 over a million
// Gaussians, the walk's vector instructions (1,700 per wave); the launch takes
// 1.61 ms without a feature buffer, and the stores of its 4.2 GB of feature
// planes add 0.74 ms to that, part of them under the walk.  2.50 -> 2.35 ms, one
// 1920x1080 pose 137 -> 103 us, one 480x270 pose 67 -> 42 us against batches of
// 128 with the feature FMAs on the VALU.  A fifth wave per SIMD spills (3.2 ms);
// planes written through LDS as 64-byte rows cost more in LDS and barriers
// (+0.27 ms) than they give.
#include "hgsr_device.hpp"
#include "launch.hpp"

namespace hgsr {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kMfGroup = 16;   // splats per matrix-core step of the feature sum

// Splats staged per round: one per thread with up to 16 channels, where a
// round fits the LDS and registers that the occupancy leaves (16 channels,
// lists of some 500: rounds of 64 splats 98 us, 128 91, 256 84; without
// features, one short list per tile: 20 -> 16).  32 and 64 channels take
// kListRound: 128 need 136 registers and lose the fourth wave per SIMD
// (1920x1080: 102 -> 116 us).
template <int TILE, int D>
constexpr int kRound = D <= 16 ? BlockShape<TILE>::kThreads : kListRound;
constexpr int kFeatRound = 4;  // 16-byte feature reads per round of the FMA form

// MF: the feature sum of 32 or 64 channels on the matrix cores.  Per 16 splats
// of the walk, F[32 ch x 64 px] += Feat[32 x 16] W[16 x 64] in two
// v_mfma_f32_32x32x16_bf16 per part of the weights: the stored bf16 features
// enter exactly, each FP32 weight in three bf16 parts that sum to it exactly
// (top, middle and last 8 significant bits), so the products are exact and only
// the order of the FP32 sum differs from one FMA per splat and channel.  The
// FMA form spends 32 of 70 VALU instructions and 8 of 11 LDS reads per splat
// on the features (both units near their limits); this one about 7 and 1.  It
// takes 0.67 to 0.89 of the FMA form's time with 32 channels and 0.47 to 0.85
// with 64 over the tile sizes and views measured (64 channels, tile 16, 8 poses
// of 480x270: 431 -> 224 us; one of 1920x1080: 286 -> 225 us), though with 64 it
// takes 168 registers against 140.
// A piece of eight channels that holds a non-finite value enters the product as
// zeros and is summed apart, at the pixels that blend its splat (a zero weight
// times infinity would reach the others).
template <int TILE, int D, bool BF16, bool MF, bool PERSIST>
__global__ __launch_bounds__(BlockShape<TILE>::kThreads, 1) void blend_fwd_kernel(BlendArgs a) {
  using S = BlockShape<TILE>;
  constexpr int NT = S::kThreads, NW = S::kWaves, NB = kRound<TILE, D>;
  constexpr int DV = D / 8;                            // 16-byte bf16 vectors per feature
  constexpr bool F32 = D > 0 && D <= 32 && !MF;        // features as FP32 in LDS (else raw bf16)
  constexpr int FS = D == 0 ? 4 : (F32 ? D : D / 2) + 4;  // words per staged feature vector (padded)
  constexpr int NA = MF ? D / 32 : 1;                  // blocks of 32 channels
  constexpr int FA = (D > 0 && !MF) ? D : 1;
  constexpr int SHARE = NT / NB;                       // threads staging one splat
  constexpr int RV = (3 + SHARE - 1) / SHARE, FV = DV > 0 ? (DV + SHARE - 1) / SHARE : 1;
  __shared__ float4 s_sp[NB][3];                       // u v ca cb | cc o z gid | r g b pmin
  __shared__ __align__(16) uint32_t s_fw[NB * FS];
  __shared__ uint8_t s_mask[NB];
  __shared__ __align__(16) uint16_t s_list[MF ? NW : 1][MF ? NB + kMfGroup : 1];  // MF: feature offsets of the wave's hits
  __shared__ float s_wt[MF ? NW : 1][MF ? kMfGroup : 1][MF ? kWave : 1];  // MF: weights, for non-finite features
  __shared__ uint32_t s_odd[NB / 32];                  // MF: staged splats with a non-finite feature
  __shared__ int s_item;
  if (a.flags[0] & 3) return;
  const int tid = threadIdx.x;
  const int lane = tid & (kWave - 1), wave = tid >> 6;
  const int W = a.c.W, H = a.c.H;
  const int64_t HW = static_cast<int64_t>(W) * H;
  int chunk_next = 0, chunk_left = 0;  // PERSIST: the claimed run of items

  for (int iter = 0;; ++iter) {
    int item;
    if constexpr (PERSIST) {
      if (chunk_left == 0) {
        if (tid == 0) s_item = static_cast<int>(atomicAdd(a.queue, static_cast<uint32_t>(kQueueChunk)));
        __syncthreads();
        chunk_next = s_item;
        chunk_left = kQueueChunk;
        __syncthreads();
      }
      item = chunk_next++;
      --chunk_left;
      if (item >= a.n_items) break;
    } else {
      if (iter > 0) break;
      item = xcd_item(blockIdx.x, gridDim.x);
    }
    const int part = item % S::kParts, titem = item / S::kParts;
    int pose, tile;
    if (a.schedule == kSchedTileMajor) {
      tile = titem / a.P;
      pose = titem - tile * a.P;
    } else {
      pose = titem / a.c.tiles_per_pose;
      tile = titem - pose * a.c.tiles_per_pose;
    }
    const int ty = tile / a.c.ntx, tx = tile - ty * a.c.ntx;
    const uint2 range = a.ranges[static_cast<int64_t>(pose) * a.c.tiles_per_pose + tile];
    // this wave's pixel block
    const int bx0 = tx * TILE + (part & 1) * 16 + (wave & 1) * 8, by0 = ty * TILE + (part >> 1) * 16 + (wave >> 1) * 8;
    const int mask_bit = TILE == 32 ? part : wave;  // the list masks' block that holds it
    const int px = bx0 + (lane & 7), py = by0 + (lane >> 3);
    const bool inside = px < W && py < H;
    const float pxf = static_cast<float>(px) + 0.5f, pyf = static_cast<float>(py) + 0.5f;
    float T = 1.f, C[3] = {0.f, 0.f, 0.f}, Z = 0.f;
    // the gate 1/255, or infinity once the pixel has stopped
    float gate = inside ? kAlphaMin : INFINITY;
    uint32_t used = 0;
    float F[FA];
#pragma unroll
    for (int d = 0; d < FA; ++d) F[d] = 0.f;
    floatx16 acc[NA][2] = {};

    const int st_e = tid / SHARE, st_sub = tid % SHARE;
    uint32_t st_lv = 0, st_lv1 = 0, st_gid1 = 0;  // entry staged next; and of the round after it
    auto stage_list = [&](uint32_t b0) {
      const uint32_t j = b0 + st_e;
      if (j < range.y) {
        st_lv1 = a.list[j];
        if constexpr (DV > 0) st_gid1 = a.list_gid[j];
      }
    };
    float4 st_rec0 = {}, st_rec1 = {}, st_rec2 = {};  // the thread's quads of the record (an array of them would be kept in scratch memory)
    uint4 st_feat[FV] = {};
    auto stage_load = [&](uint32_t b0) {
      if (b0 + st_e < range.y) {
        st_lv = st_lv1;
        const float4* sp = reinterpret_cast<const float4*>(a.recs + (st_lv & kRecMask)) + st_sub;
        if (st_sub < 3) st_rec0 = sp[0];
        if (RV > 1 && st_sub + SHARE < 3) st_rec1 = sp[SHARE];
        if (RV > 2) st_rec2 = sp[2];
        if constexpr (DV > 0) {
          const uint4* fv = reinterpret_cast<const uint4*>(a.feat) + static_cast<int64_t>(st_gid1) * DV;
#pragma unroll
          for (int q = 0; q < FV; ++q)
            if (q * SHARE + st_sub < DV) st_feat[q] = fv[q * SHARE + st_sub];
        }
      }
      stage_list(b0 + NB);
    };
    stage_list(range.x);
    stage_load(range.x);
    for (uint32_t b0 = range.x; b0 < range.y; b0 += NB) {
      if (b0 > range.x && __syncthreads_and(gate > 1.f)) break;  // every pixel of the block has stopped
      const int nb = static_cast<int>(min(static_cast<uint32_t>(NB), range.y - b0));
      if (MF && tid < NB / 32) s_odd[tid] = 0;
      if (st_e < nb) {
        if (st_sub < 3) s_sp[st_e][st_sub] = st_rec0;
        if (RV > 1 && st_sub + SHARE < 3) s_sp[st_e][st_sub + SHARE] = st_rec1;
        if (RV > 2) s_sp[st_e][2] = st_rec2;
        if (st_sub == SHARE - 1) s_mask[st_e] = static_cast<uint8_t>(st_lv >> kRecBits);  // blocks the support meets
      }
      if constexpr (MF) __syncthreads();  // s_odd cleared
      if constexpr (DV > 0) {
        if (st_e < nb) {
#pragma unroll
          for (int q = 0; q < FV; ++q) {
            const int v = q * SHARE + st_sub;
            if (v >= DV) continue;
            uint4 f = st_feat[q];
            if constexpr (F32) {
              uint4* dst = reinterpret_cast<uint4*>(&s_fw[st_e * FS + 8 * v]);
              dst[0] = make_uint4(f.x << 16, f.x & 0xffff0000u, f.y << 16, f.y & 0xffff0000u);
              dst[1] = make_uint4(f.z << 16, f.z & 0xffff0000u, f.w << 16, f.w & 0xffff0000u);
            } else {
              if constexpr (MF) {
                if (nonfinite_bf16x8(f)) {
                  atomicOr(&s_odd[st_e >> 5], 1u << (st_e & 31));
                  f = make_uint4(0u, 0u, 0u, 0u);
                }
              }
              reinterpret_cast<uint4*>(&s_fw[st_e * FS])[v] = f;
            }
          }
        }
      }
      __syncthreads();
      if (b0 + NB < range.y) stage_load(b0 + NB);  // the next round travels while this one is walked
      // the round's splats that meet this wave's block, as a mask (the walk)
      // and, MF, a list of feature offsets in order (the per-lane lookups)
#pragma unroll 1
      for (int k0 = 0; k0 < nb; k0 += kWave) {
        const bool hit = k0 + lane < nb && ((s_mask[k0 + lane] >> mask_bit) & 1u);
        uint64_t todo = __ballot(hit);
        if (todo == 0) continue;  // (the next round's barrier still orders the staging)
        const uint32_t base = b0 - range.x + 1 + k0;
        const uint64_t odd = MF ? (static_cast<uint64_t>(s_odd[k0 / 32 + 1]) << 32) | s_odd[k0 / 32] : 0ull;  // uniform
        [[maybe_unused]] const int n_mine = __popcll(todo);
        if constexpr (MF) {
          if (hit) s_list[wave][__popcll(todo & ((1ull << lane) - 1ull))] = static_cast<uint16_t>((k0 + lane) * FS * 4);
          if (lane < kMfGroup) s_list[wave][n_mine + lane] = 0;  // a group's missing splats read slot 0, weights 0
          wave_lds_fence();
        }
        // one splat at this lane's pixel, in order: its weight (0 when not blended)
        auto blend = [&](int jj, const float4& opz, const float4& col, float power, float alpha) -> float {
          const float Tn = T * (1.f - alpha);
          const bool pass = !(power > 0.f) && !(alpha < gate), stop = pass && Tn < kTMin;
          gate = stop ? INFINITY : gate;
          float w = 0.f;
          if (pass && !stop) {
            w = alpha * T;
            C[0] = fmaf(w, col.x, C[0]);
            C[1] = fmaf(w, col.y, C[1]);
            C[2] = fmaf(w, col.z, C[2]);
            Z = fmaf(w, opz.z, Z);
            T = Tn;
            used = base + jj;
            if constexpr (F32) {
              const float4* fsrc = reinterpret_cast<const float4*>(&s_fw[(k0 + jj) * FS]);
              constexpr int FR = (D / 4 > kFeatRound) ? kFeatRound : D / 4;  // reads per round
#pragma unroll
              for (int q0 = 0; q0 < D / 4; q0 += FR) {
                float4 fq[FR];
#pragma unroll
                for (int q = 0; q < FR; ++q) fq[q] = fsrc[q0 + q];
                __builtin_amdgcn_sched_barrier(0);  // the round's reads issued before its FMAs
#pragma unroll
                for (int q = 0; q < FR; ++q) {
                  const float4 f = fq[q];
                  const int d = 4 * (q0 + q);
                  F[d + 0] = fmaf(w, f.x, F[d + 0]);
                  F[d + 1] = fmaf(w, f.y, F[d + 1]);
                  F[d + 2] = fmaf(w, f.z, F[d + 2]);
                  F[d + 3] = fmaf(w, f.w, F[d + 3]);
                }
              }
            } else if constexpr (D > 0 && !MF) {
              const uint4* fq = reinterpret_cast<const uint4*>(&s_fw[(k0 + jj) * FS]);
#pragma unroll
              for (int q = 0; q < D / 8; ++q) {
                const uint4 f = fq[q];
                F[8 * q + 0] = fmaf(w, bf16_lo(f.x), F[8 * q + 0]);
                F[8 * q + 1] = fmaf(w, bf16_hi(f.x), F[8 * q + 1]);
                F[8 * q + 2] = fmaf(w, bf16_lo(f.y), F[8 * q + 2]);
                F[8 * q + 3] = fmaf(w, bf16_hi(f.y), F[8 * q + 3]);
                F[8 * q + 4] = fmaf(w, bf16_lo(f.z), F[8 * q + 4]);
                F[8 * q + 5] = fmaf(w, bf16_hi(f.z), F[8 * q + 5]);
                F[8 * q + 6] = fmaf(w, bf16_lo(f.w), F[8 * q + 6]);
                F[8 * q + 7] = fmaf(w, bf16_hi(f.w), F[8 * q + 7]);
              }
            }
          }
          return w;
        };
        // the next AHEAD splats of the mask, read a step ahead of their use;
        // without features two at once, whose alphas do not wait for each
        // other (16.1 -> 15.0 us where few waves share a SIMD; with 16
        // channels the registers cost a wave: 98 -> 104)
        constexpr int AHEAD = D == 0 ? 2 : 1;
        int jn[AHEAD];
        float4 geo_n[AHEAD], opz_n[AHEAD], col_n[AHEAD];
        int left = n_mine;  // not yet walked
        [[maybe_unused]] uint64_t rest = todo;
        auto fetch = [&]() {
#pragma unroll
          for (int i = 0; i < AHEAD; ++i) {
            jn[i] = todo ? __builtin_ctzll(todo) : 0;
            todo &= todo - 1ull;
            geo_n[i] = s_sp[k0 + jn[i]][0];
            opz_n[i] = s_sp[k0 + jn[i]][1];
            col_n[i] = s_sp[k0 + jn[i]][2];
          }
          __atomic_signal_fence(__ATOMIC_SEQ_CST);  // issued here, a step ahead of their use
        };
        fetch();
        auto step = [&]() -> float {
          int jj[AHEAD];
          float4 opz[AHEAD], col[AHEAD], geo[AHEAD];
          float power[AHEAD], alpha[AHEAD];
#pragma unroll
          for (int i = 0; i < AHEAD; ++i) {
            jj[i] = jn[i];
            geo[i] = geo_n[i];
            opz[i] = opz_n[i];
            col[i] = col_n[i];
          }
          fetch();
#pragma unroll
          for (int i = 0; i < AHEAD; ++i) {
            power[i] = pair_power(pxf - geo[i].x, pyf - geo[i].y, geo[i].z, geo[i].w, opz[i].x);
            alpha[i] = pair_alpha(opz[i].y, power[i]);
          }
          const float w = blend(jj[0], opz[0], col[0], power[0], alpha[0]);
          if constexpr (AHEAD > 1)
            if (left > 1) (void)blend(jj[1], opz[1], col[1], power[1], alpha[1]);  // uniform
          left -= AHEAD;
          return w;
        };
        if constexpr (!MF) {
          while (left > 0) {  // uniform
            (void)step();
            if (!__any(gate < 1.f)) break;
          }
        } else {
          for (int g0 = 0; g0 < n_mine; g0 += kMfGroup) {
            if (!__any(gate < 1.f)) break;  // uniform
            const uint64_t rest0 = rest;
            float w[kMfGroup];
#pragma unroll
            for (int q = 0; q < kMfGroup; ++q) {
              w[q] = 0.f;
              if (left > 0) w[q] = step();  // uniform
            }
            rest = left > 0 ? todo | (1ull << jn[0]) : 0ull;
            uint64_t odd_g = rest0 & ~rest & odd;  // the group's splats with a non-finite feature
            if (odd_g) {
#pragma unroll
              for (int q = 0; q < kMfGroup; ++q) s_wt[wave][q][lane] = w[q];
              wave_lds_fence();
            }
            // A operands: channel l % 32 (+ 32 n) of splats 8 (l / 32) + 0..7;
            // B: weights of the same splats at pixel l % 32 (and 32 + l % 32),
            // one lane-half exchange per two splats
            const uint4 lo4 = *reinterpret_cast<const uint4*>(&s_list[wave][g0 + 8 * (lane >> 5)]);
            const uint32_t lw[4] = {lo4.x, lo4.y, lo4.z, lo4.w};
            uint32_t ap[NA][4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
              const char* fb = reinterpret_cast<const char*>(s_fw) + 2 * (lane & 31);
              const char* f0 = fb + (lw[t] & 0xffffu);
              const char* f1 = fb + (lw[t] >> 16);
#pragma unroll
              for (int n = 0; n < NA; ++n) {
                const uint32_t x = *reinterpret_cast<const uint16_t*>(f0 + 64 * n);
                const uint32_t y = *reinterpret_cast<const uint16_t*>(f1 + 64 * n);
                ap[n][t] = x | (y << 16);
              }
            }
            float r[2][8];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
              const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(w[t]), __float_as_uint(w[8 + t]), false,
                                                               false);
              r[0][t] = __uint_as_float(sw[0]);
              r[1][t] = __uint_as_float(sw[1]);
            }
#pragma unroll
            for (int side = 0; side < 2; ++side) {
              uint32_t bp[3][4];
#pragma unroll
              for (int t = 0; t < 4; ++t) {
                float x = r[side][2 * t], y = r[side][2 * t + 1];
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                  bp[k][t] = __builtin_amdgcn_perm(__float_as_uint(y), __float_as_uint(x), 0x07060302u);  // top halves
                  x -= __uint_as_float(__float_as_uint(x) & 0xffff0000u);
                  y -= __uint_as_float(__float_as_uint(y) & 0xffff0000u);
                }
              }
#pragma unroll
              for (int k = 2; k >= 0; --k)
#pragma unroll
                for (int n = 0; n < NA; ++n) {
                  bf16x8 av, bv;
                  __builtin_memcpy(&av, ap[n], 16);
                  __builtin_memcpy(&bv, bp[k], 16);
                  acc[n][side] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc[n][side], 0, 0, 0);
                }
            }
            // accumulator layout: lane l, register r holds channel
            // 8 (r / 4) + 4 (l / 32) + r % 4 of pixel l % 32 (+ 32 for side 1)
            while (odd_g) {  // uniform, normally empty
              const int jj = __builtin_ctzll(odd_g);
              odd_g &= odd_g - 1ull;
              const int q = __popcll(rest0 & ((1ull << jj) - 1ull));
              // the pieces of eight channels that were staged as zeros; the
              // others of this splat are in the products above
              const uint4* f = reinterpret_cast<const uint4*>(a.feat) +
                               static_cast<int64_t>(__float_as_uint(s_sp[k0 + jj][1].w)) * DV;
#pragma unroll
              for (int v = 0; v < DV; ++v) {
                const uint4 x = f[v];
                if (!nonfinite_bf16x8(x)) continue;  // uniform
                const uint32_t x0 = lane < 32 ? x.x : x.z, x1 = lane < 32 ? x.y : x.w;
                const float c[4] = {bf16_lo(x0), bf16_hi(x0), bf16_lo(x1), bf16_hi(x1)};
#pragma unroll
                for (int side = 0; side < 2; ++side) {
                  const float wq = s_wt[wave][q][(lane & 31) + 32 * side];
                  if (wq == 0.f) continue;
#pragma unroll
                  for (int k = 0; k < 4; ++k) {
                    const int i = 4 * (v % 4) + k;
                    acc[v / 4][side][i] = fmaf(wq, c[k], acc[v / 4][side][i]);
                  }
                }
              }
            }
          }
        }
      }
    }

    const int64_t po = static_cast<int64_t>(pose) * HW;
    const int64_t pix = static_cast<int64_t>(py) * W + px;
    if (inside) {
      const int64_t o = po + pix, o3 = 3 * po + pix;
      a.rgb[o3] = fmaf(T, a.bg[0], C[0]);
      a.rgb[o3 + HW] = fmaf(T, a.bg[1], C[1]);
      a.rgb[o3 + 2 * HW] = fmaf(T, a.bg[2], C[2]);
      const float A = 1.f - T;
      a.alpha[o] = A;
      a.depth[o] = A > 0.f ? Z / A : 0.f;
      a.final_T[o] = T;
      a.n_used[o] = used;
      if constexpr (D > 0 && !MF) {
        if (a.out_feat) {
          const int64_t of = D * po + pix;
          if constexpr (BF16) {
            uint16_t* fo = static_cast<uint16_t*>(a.out_feat);
#pragma unroll
            for (int d = 0; d < D; ++d) fo[of + d * HW] = f32_to_bf16_rne(F[d]);
          } else {
            float* fo = static_cast<float*>(a.out_feat);
#pragma unroll
            for (int d = 0; d < D; ++d) fo[of + d * HW] = F[d];
          }
        }
      }
    }
    if constexpr (MF) {
      if (a.out_feat) {
#pragma unroll
        for (int side = 0; side < 2; ++side) {
          const int x = bx0 + (lane & 7), y = by0 + 4 * side + ((lane >> 3) & 3);
          if (x < W && y < H) {
            const int64_t of = D * po + 4 * (lane >> 5) * HW + static_cast<int64_t>(y) * W + x;
#pragma unroll
            for (int n = 0; n < NA; ++n)
#pragma unroll
              for (int k = 0; k < 16; ++k) {
                const int64_t o = of + (32 * n + 8 * (k / 4) + (k % 4)) * HW;
                if constexpr (BF16) static_cast<uint16_t*>(a.out_feat)[o] = f32_to_bf16_rne(acc[n][side][k]);
                else static_cast<float*>(a.out_feat)[o] = acc[n][side][k];
              }
          }
        }
      }
    }
    if constexpr (PERSIST) __syncthreads();
  }
}

template <int TILE, int D, bool BF16, bool PERSIST>
static void launch_p(const BlendArgs& a, int n_ctas, hipStream_t s) {
  constexpr int NT = BlockShape<TILE>::kThreads;
  constexpr bool MFOK = D == 32 || D == 64;
  if (MFOK && a.feat_mfma)
    hipLaunchKernelGGL((blend_fwd_kernel<TILE, D, BF16, MFOK, PERSIST>), dim3(n_ctas), dim3(NT), 0, s, a);
  else
    hipLaunchKernelGGL((blend_fwd_kernel<TILE, D, BF16, false, PERSIST>), dim3(n_ctas), dim3(NT), 0, s, a);
}

template <int TILE, int D, bool BF16>
static void launch_t(const BlendArgs& a, int n_ctas, hipStream_t s) {
  if (a.schedule != kSchedGrid) launch_p<TILE, D, BF16, true>(a, n_ctas, s);
  else launch_p<TILE, D, BF16, false>(a, a.n_items, s);
}

template <int TILE, int D>
static void launch_td(const BlendArgs& a, bool bf16, int n_ctas, hipStream_t s) {
  if (bf16) launch_t<TILE, D, true>(a, n_ctas, s);
  else launch_t<TILE, D, false>(a, n_ctas, s);
}

template <int TILE>
static void launch_tile(const BlendArgs& a, int D, bool bf16, int n_ctas, hipStream_t s) {
  switch (D) {
    case 0: launch_t<TILE, 0, false>(a, n_ctas, s); break;
    case 8: launch_td<TILE, 8>(a, bf16, n_ctas, s); break;
    case 16: launch_td<TILE, 16>(a, bf16, n_ctas, s); break;
    case 32: launch_td<TILE, 32>(a, bf16, n_ctas, s); break;
    default: launch_td<TILE, 64>(a, bf16, n_ctas, s); break;
  }
}

int blend_parts(int tile) { return tile == 32 ? BlockShape<32>::kParts : 1; }

void launch_blend_fwd(const BlendArgs& a, int D, bool bf16_out, int n_ctas, hipStream_t s) {
  switch (a.c.tile) {
    case 8: launch_tile<8>(a, D, bf16_out, n_ctas, s); break;
    case 32: launch_tile<32>(a, D, bf16_out, n_ctas, s); break;
    default: launch_tile<16>(a, D, bf16_out, n_ctas, s); break;
  }
}

}  // namespace hgsr
