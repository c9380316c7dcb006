// Internal device-side definitions of the gfx950 rasterizer: per-face record layout, the
// per-call view table, and wave64 primitives.  Included by the .hip sources only.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tsr.h"

namespace tsr {

constexpr int kTile = TSR_TILE;          // 16x16 pixel tiles
constexpr int kBlock = 256;              // one pixel per lane, 4 waves of 8x8 pixels per tile
constexpr int kWave = 64;

// Per-(view, face) setup record, 24 dwords (96 B), written by the projection kernel for
// visible faces only.  Coordinates are face-local: dx = u - u0, dy = v - v0 with (u0, v0)
// the top-left pixel of the face's pixel rectangle, so per-pixel FP32 math works on small
// exact integers.
//   E_k(p) = a_k dx + b_k dy + c_k = -L_k(p) / r  (eq. 2 edge function over phi(s) = -r)
//   rho(p) = min_k E_k(p) = phi(p) / phi(s)      (eq. 3 before ReLU and exponent)
//   colour_ch(p) = P_ch dx + Q_ch dy + R_ch        (barycentric interpolation is affine in p)
enum RecordField : int {
  kRecEdge = 0,      // [3][3] a_k, b_k, c_k
  kRecCol = 9,       // [3][3] P_ch, Q_ch, R_ch
  kRecOpa = 18,      // o_F
  kRecZ = 19,        // z_F
  kRecU0 = 20,       // u0 as a float (an exact integer)
  kRecV0 = 21,       // v0 as a float (an exact integer)
  kRecMid = 22,      // int (u0 + u1) | (v0 + v1) << 16, (u1, v1) the rectangle's last pixel: twice its
                     // middle (image sizes are at most 16384); bit 31: a colour plane is not finite
  kRecSigma = 23,    // the face's window exponent sigma (eq. 3)
  kRecDwords = 24
};
// With perspective-correct interpolation the colour planes hold the numerators N_ch of the
// perspective-correct colour, sum_k lambda_k c_k / z_k, and three dwords the plane of the
// denominator W = sum_k lambda_k / z_k (W = 1 / depth of the face's plane along the ray); the
// depth z_F, the rectangle's end and the per-face exponent are not stored.
enum PerspField : int { kRecWa = kRecZ, kRecWb = kRecMid, kRecWc = kRecSigma };

// Per-(view, face) gradient accumulator, 20 values, filled by the backward blend:
// dL/d(a_k, b_k, c_k) for the three edges, dL/d(P, Q, R) per channel, dL/do_F, dL/dz_F.
// Wave partial sums are FP32; they are accumulated across waves and tiles in acc_t.
// The planes' moments are about the anchor (u0, v0) or, where tiles may be split between two workgroups
// (and a face then takes up to twice as many additions), about the rectangle's middle: the chain rule
// combines the three of a plane with cancellation, and about the middle they are half as large.
enum GradField : int { kGEdge = 0, kGCol = 9, kGOpa = 18, kGZ = 19, kGradDwords = 20 };
// Perspective-correct mode: the colour slots hold dL/d(N_ch plane), kGZ dL/d(constant of the W
// plane); the W plane's two slopes go to a second per-(view, face) accumulator of 2 floats.
enum GradPerspField : int { kGWc = kGZ };
#ifndef TSR_ACC_F64
#define TSR_ACC_F64 0
#endif
#if TSR_ACC_F64
typedef double acc_t;
#else
typedef float acc_t;
#endif

struct ViewDesc {
  int32_t width, height, tiles_x, tiles_y;
  int32_t tile_off;        // first global tile id of this view
  int32_t pad;
  int64_t pix_off;         // first packed pixel of this view
  float fx, fy, cx, cy;
};

struct ViewTable {
  ViewDesc v[TSR_MAX_VIEWS];
  int32_t n_views;
  int32_t n_tiles;         // total tiles
  int64_t n_faces;         // M
  int32_t face_sigma;      // the scene has per-face window exponents (records hold each face's)
  int32_t pad;
};

// View of a global tile id.  Unused table entries hold a tile_off above every tile id, so the
// entries are compared eight at a time (their scalar loads overlap).
__device__ __forceinline__ int view_of_tile(const ViewTable& vt, int tile) {
  if (vt.n_views == 1) return 0;
  int v = 0;
  for (int i0 = 0; i0 < vt.n_views; i0 += 8) {
#pragma unroll
    for (int i = 0; i < 8; ++i) v += (int)((uint32_t)(vt.v[i0 + i].tile_off - 1 - tile) >> 31);   // tile >= tile_off
  }
  return v - 1;
}

// ---------------------------------------------------------------------------- wave64 DPP
// Row-wise DPP butterflies, then the legacy gfx9 row broadcasts, leave the wave total in
// lane 63.  Every lane must be active.

#define TSR_DPP(v, ctrl, rmask, bmask)                                                     \
  __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), ctrl, rmask, bmask, false))

__device__ __forceinline__ float wave_sum_to_lane63(float v) {
  v += TSR_DPP(v, 0xB1, 0xF, 0xF);     // quad_perm [1,0,3,2]
  v += TSR_DPP(v, 0x4E, 0xF, 0xF);     // quad_perm [2,3,0,1]
  v += TSR_DPP(v, 0x124, 0xF, 0xF);    // row_ror:4
  v += TSR_DPP(v, 0x128, 0xF, 0xF);    // row_ror:8  -> every lane holds its row's sum
  v += TSR_DPP(v, 0x142, 0xA, 0xF);    // row_bcast:15 into rows 1 and 3
  v += TSR_DPP(v, 0x143, 0xC, 0xF);    // row_bcast:31 into rows 2 and 3
  return v;
}

__device__ __forceinline__ float wave_sum(float v) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wave_sum_to_lane63(v)), 63));
}

// Sums of per-pixel gradient terms over the pixels of a wave's 8x8 quadrant, for two faces at a time,
// one per half of the wave: a lane's terms are already the sums of two pixels of a row, lane bits 2
// and 3 are x and bits 0, 1 and 4 y.  The sums are taken in the order x, then y, so that a term's
// moment with respect to y is formed after its sum over x (one product per row of pixels); every
// level is a transposing butterfly: a pair of vectors (a, b) becomes one, the lanes on one side of
// the level's partner bit keeping a summed with their partner and the others keeping b.
//
// On gfx950 a wave64 v_permlane*_swap or reciprocal takes 8 cycles of a SIMD; a DPP add, a compare, a
// select, a minimum or an integer instruction 4; an add, multiply or FMA 4 alone and 2.4 where those of
// two waves issue together (a microbenchmark of each kind, many waves).  The x levels are pairs of DPP
// row rotations that write only the banks of their side (a bank is four lanes; no select needed),
// lane bits 1 and 0 quad permutes and a select, and only the last level, on the two vectors that are
// left, a swap.  A lane that holds two pixels halves the sums' share of the work.
//
// The levels are asm blocks: the compiler cannot fold a masked DPP move into an add, and inside a
// block the two wait states between a write and a DPP read of the same register are kept by the
// order of the instructions (the hazard tables do not look inside asm: the leading s_nop covers
// what was written just before).

constexpr unsigned long long kLaneBit1 = 0xccccccccccccccccull, kLaneBit0 = 0xaaaaaaaaaaaaaaaaull;

// Sums over x.  With b2, b3 the lane's bits: a[0] holds value 2 b2 + b3 of a, a[4] value 4 + 2 b2 +
// b3; c[0] value 2 b2 + b3 of c, c[4] value 4 + b3 where b2 is 0, else value 6 if there are seven.
// Every lane must be active.
__device__ __forceinline__ void sum_x(float (&a)[8], float (&c)[6]) {
  asm volatile(
      "s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %4, %4, %4 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %6, %6, %6 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %8, %8, %8 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %10, %10, %10 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %12, %12, %12 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %2, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %4, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %6, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %8, %9, %9 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %10, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %12, %13, %13 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %4, %4, %4 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %8, %8, %8 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %12, %12, %12 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %0, %2, %2 row_ror:4 row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %4, %6, %6 row_ror:4 row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %8, %10, %10 row_ror:4 row_mask:0xf bank_mask:0xa"
      : "+&v"(a[0]), "+&v"(a[1]), "+&v"(a[2]), "+&v"(a[3]), "+&v"(a[4]), "+&v"(a[5]), "+&v"(a[6]), "+&v"(a[7]),
        "+&v"(c[0]), "+&v"(c[1]), "+&v"(c[2]), "+&v"(c[3]), "+&v"(c[4]), "+&v"(c[5]));
}

__device__ __forceinline__ void sum_x(float (&a)[8], float (&c)[7]) {
  asm volatile(
      "s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %4, %4, %4 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %6, %6, %6 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %8, %8, %8 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %10, %10, %10 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %12, %12, %12 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %14, %14, %14 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %2, %3, %3 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %4, %5, %5 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %6, %7, %7 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %8, %9, %9 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %10, %11, %11 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %12, %13, %13 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %4, %4, %4 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %8, %8, %8 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %12, %12, %12 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %0, %2, %2 row_ror:4 row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %4, %6, %6 row_ror:4 row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %8, %10, %10 row_ror:4 row_mask:0xf bank_mask:0xa\n\t"
      "v_add_f32_dpp %12, %14, %14 row_ror:4 row_mask:0xf bank_mask:0xa"
      : "+&v"(a[0]), "+&v"(a[1]), "+&v"(a[2]), "+&v"(a[3]), "+&v"(a[4]), "+&v"(a[5]), "+&v"(a[6]), "+&v"(a[7]),
        "+&v"(c[0]), "+&v"(c[1]), "+&v"(c[2]), "+&v"(c[3]), "+&v"(c[4]), "+&v"(c[5]), "+&v"(c[6]));
}

// The same for three values: c[0] holds value b3 where b2 is 0, else value 2.
__device__ __forceinline__ void sum_x(float (&c)[3]) {
  asm volatile(
      "s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
      "v_add_f32_dpp %2, %2, %2 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %1, %1 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
      "s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 row_ror:12 row_mask:0xf bank_mask:0x5\n\t"
      "v_add_f32_dpp %0, %2, %2 row_ror:4 row_mask:0xf bank_mask:0xa"
      : "+&v"(c[0]), "+&v"(c[1]), "+&v"(c[2]));
}

// Lane bit 4: even rows of 16 lanes keep a, odd rows b.
__device__ __forceinline__ float sum_bit4(float a, float b) {
#pragma clang fp contract(off)
  const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// Sums over y of (a0, a1), (c0, c1) and (q0, q1), each pair's second taken where lane bit 1 is set;
// then the a's where lane bits 4 and 0 are 0, the c's where bit 0 is set, the q's where bit 4 is, and
// the n's (if given) where both are.  The trailing s_nop is for the swap that reads the results.
__device__ __forceinline__ float sum_y(float a0, float a1, float c0, float c1, float q0, float q1) {
  asm volatile(
      "s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %3, %3, %3 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %4, %4, %4 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %5, %5, %5 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_e64 %0, %0, %1, %6\n\t"
      "v_cndmask_b32_e64 %2, %2, %3, %6\n\t"
      "v_cndmask_b32_e64 %4, %4, %5, %6\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %2, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %4, %4, %4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_e64 %0, %0, %2, %7\n\t"
      "s_nop 1"
      : "+&v"(a0), "+&v"(a1), "+&v"(c0), "+&v"(c1), "+&v"(q0), "+&v"(q1)
      : "s"(kLaneBit1), "s"(kLaneBit0));
  return sum_bit4(a0, q0);
}

__device__ __forceinline__ float sum_y(float a0, float a1, float c0, float c1, float q0, float q1, float n) {
  asm volatile(
      "s_nop 1\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %2, %2, %2 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %3, %3, %3 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %4, %4, %4 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %5, %5, %5 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %6, %6, %6 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_cndmask_b32_e64 %0, %0, %1, %7\n\t"
      "v_cndmask_b32_e64 %2, %2, %3, %7\n\t"
      "v_cndmask_b32_e64 %4, %4, %5, %7\n\t"
      "v_add_f32_dpp %6, %6, %6 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %2, %2, %2 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_add_f32_dpp %4, %4, %4 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_cndmask_b32_e64 %0, %0, %2, %8\n\t"
      "v_cndmask_b32_e64 %4, %4, %6, %8\n\t"
      "s_nop 1"
      : "+&v"(a0), "+&v"(a1), "+&v"(c0), "+&v"(c1), "+&v"(q0), "+&v"(q1), "+&v"(n)
      : "s"(kLaneBit1), "s"(kLaneBit0));
  return sum_bit4(a0, q0);
}

// Largest value of the wave, in every lane (row-wise DPP steps and broadcasts, no LDS).
__device__ __forceinline__ int wave_max_int(int v) {
#define TSR_DPP_MAX(ctrl, rmask) v = max(v, __builtin_amdgcn_update_dpp(v, v, ctrl, rmask, 0xF, false))
  TSR_DPP_MAX(0xB1, 0xF);      // quad_perm [1,0,3,2]
  TSR_DPP_MAX(0x4E, 0xF);      // quad_perm [2,3,0,1]
  TSR_DPP_MAX(0x124, 0xF);     // row_ror:4
  TSR_DPP_MAX(0x128, 0xF);     // row_ror:8
  TSR_DPP_MAX(0x142, 0xA);     // row_bcast:15 into rows 1 and 3
  TSR_DPP_MAX(0x143, 0xC);     // row_bcast:31 into rows 2 and 3
#undef TSR_DPP_MAX
  return __builtin_amdgcn_readlane(v, 63);
}

__device__ __forceinline__ int uniform_int(int v) { return __builtin_amdgcn_readfirstlane(v); }

__device__ __forceinline__ unsigned long long uniform_u64(unsigned long long v) {
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}

// Wave ballot of a predicate, taken as a lane mask directly (no conversion to an integer first).
__device__ __forceinline__ unsigned long long ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// Inclusive prefix sum over the 64 lanes of a wave.
__device__ __forceinline__ unsigned long long wave_incl_scan_u64(unsigned long long v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long y = __shfl_up(v, (unsigned)o, 64);
    if (lane >= o) v += y;
  }
  return v;
}

// Exclusive prefix sum of one value per thread over the workgroup (blockDim.x a multiple of
// 64, at most 1024), and the workgroup total.  `wsum` is 16 shared slots.  Every thread of the
// workgroup must call it; it contains two barriers, after which `wsum` may be reused.
__device__ __forceinline__ unsigned long long block_excl_scan_u64(unsigned long long s, unsigned long long* wsum,
                                                                  unsigned long long* total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  const unsigned long long inc = wave_incl_scan_u64(s);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  unsigned long long before = 0, tot = 0;
  for (int i = 0; i < nw; ++i) {
    const unsigned long long x = wsum[i];
    if (i < w) before += x;
    tot += x;
  }
  __syncthreads();
  *total = tot;
  return before + inc - s;
}

}  // namespace tsr
