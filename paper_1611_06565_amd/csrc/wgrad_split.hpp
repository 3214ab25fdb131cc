// Weight gradient of F(2^3, 3^3) with both transforms inside the product, on
// the bf16 matrix cores (fp32 operands split into three bf16 each, see
// gemm_split.hpp): V and D (the transformed input and output gradients) are
// formed in LDS, split as they are written, and never reach memory.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "gemm_split.hpp"
#include "kernels.hpp"
#include "synth.hpp"
#include "transforms.hpp"

namespace wino {

// Division by a launch constant d >= 1 of values below 2^31 by a multiplication
// (T. Granlund, P. L. Montgomery, "Division by Invariant Integers using
// Multiplication", PLDI 1994): with l = ceil(log2 d) and m = ceil(2^(31 + l) / d),
// v / d = (v m) >> (31 + l).
struct FastDiv {
  uint32_t d, m, s;     // s = l - 1; d = 1: the quotient is v
};

inline FastDiv fast_div(uint32_t d) {
  FastDiv f{d, 0, 0};
  if (d > 1) {
    uint32_t l = 0;
    while ((uint64_t(1) << l) < d) ++l;
    f.m = uint32_t(((uint64_t(1) << (31 + l)) + d - 1) / d);
    f.s = l - 1;
  }
  return f;
}

__device__ __forceinline__ int quot(int v, const FastDiv& f) {
  return f.d == 1 ? v : int(__umulhi(uint32_t(v), f.m) >> f.s);
}

struct WgSplitArgs {
  float* part;          // M: [nsplit][64][kp][cpn]
  FastDiv tiles[3];
  int32_t X[3], pad[3], Y[3];
  int32_t T, K, C;
  int32_t kp, cpn;      // kernels and channels of M, multiples of 64
  int32_t nkb, ncb;     // kernel and channel blocks
  int32_t nsplit, nsteps;   // tile ranges; 16-tile steps in all
  uint32_t xbytes, xstride, ybytes, ystride;   // bytes in all and of a channel (a kernel)
};

// One work-group: KB kernels x 64 channels of M for the eight elements of pass
// p (xi0 = p / 2, xi1 = 2 (p % 2) + {0, 1}, xi2 = 0..3) over a range of
// tiles; wave w owns element w, the contraction runs over the tiles, 16 a
// step.
//   produce: thread = (two neighbouring tiles, channel) for V and, KB / 64
//     times, (two neighbouring tiles, kernel) for D: window rows are one
//     aligned 16-byte load each, the outer columns of V come from the
//     neighbouring lanes.  The transforms run axis by axis; a word holds the
//     pair's two tiles of one row, so split values go straight to
//     planes[element][h, m, l][8-tile half][row][16 bytes].
//   consume: the wave's KB / 32 x 2 blocks of 32 x 32, six products each.
// The next step's loads run under the products.
//
// Why KB = 128 (for more than 64 kernels): the 128 accumulators fit, V is
// formed once instead of twice, and D's rows outnumber V's.  What bounds it
// (8 x 64 x 16 x 56 x 56, K = 128: 567 us with the sum and A'^T, 1069 with V
// and D in memory): producing and products take turns between the barriers;
// of the time the vector ALU is busy 47%, addresses 34%, matrix cores 21%, LDS
// 13%.  Stripped copies: without the loads 415, without the producing 240.  256
// registers, one of them spilled.
template <int KB>
__global__ void __launch_bounds__(512, 2) k_wgrad_split(const float* __restrict__ x, const float* __restrict__ dy,
                                                        WgSplitArgs a) {
  constexpr int MM = 2, R = 3, E = 8, CB = 64, KI = KB / 64;
  constexpr int ROWS = KB + CB;                   // D's rows, then V's
  constexpr int HALF = ROWS * 16 + 64;            // the two halves of a row in different banks
  constexpr int PLANE = 2 * HALF;
  __shared__ __attribute__((aligned(16))) char lds[E * 3 * PLANE];

  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;

  // The eight passes (and the blocks) of a range are neighbours on one XCD, so
  // that they run together and its L2 fetches their rows of x and dy once
  // (with a pass per XCD every XCD read all of both: 790 us in place of 567 on
  // 8 x 64 x 16 x 56 x 56, K = 128).
  int u = xcd_remap(int(blockIdx.x), int(gridDim.x));
  const int p = u % E; u /= E;
  const int kb = u % a.nkb; u /= a.nkb;
  const int cb = u % a.ncb, sp = u / a.ncb;
  if (sp >= a.nsplit) return;
  const int s0 = int(int64_t(a.nsteps) * sp / a.nsplit), s1 = int(int64_t(a.nsteps) * (sp + 1) / a.nsplit);

  const int i0 = p >> 1, hh = p & 1;
  const int P0 = i0 == 0 ? 0 : i0 == 2 ? 2 : 1, P1 = i0 == 3 ? 3 : i0 == 2 ? 1 : 2;
  const int rr3[3] = {hh ? 2 : 0, hh ? 3 : 1, hh ? 1 : 2};
  const float g0 = i0 == 1 ? 1.0f : -1.0f, g1 = hh ? -1.0f : 1.0f;   // see k_fwd_split
  const MatRef<Which::G, true, R, MM> Gp{nullptr};                   // G' of F(3, 2): 4 x 2
  float ga[2], gb[2][2];                          // axis 0 (row xi0), axis 1 (the two xi1)
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    ga[o] = i0 == 0 ? Gp(0, o) : i0 == 1 ? Gp(1, o) : i0 == 2 ? Gp(2, o) : Gp(3, o);
    gb[0][o] = hh ? Gp(2, o) : Gp(0, o);
    gb[1][o] = hh ? Gp(3, o) : Gp(1, o);
  }

  // lane: pair j of the step's eight, row 8 w + lane / 8 of each 64-row group
  const int pj = lane & 7, prow = 8 * wave + (lane >> 3);
  const int c = cb * CB + prow;
  // ends: slot 16 r + 2 s + e = value left (e = 0) / right (e = 1) of the
  // eight pairs in window row r of the wave's channel s; rows 0..3 in the
  // first load, 4 and 5 in the second
  const int es = (lane >> 1) & 7, ee = lane & 1, er = lane >> 4;
  const int ec = cb * CB + 8 * wave + es;
  const int epick = 4 * (2 * (lane >> 3) + (pj == 7 ? 1 : 0));
  const bool first = pj == 0, last = pj == 7;
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, int(a.xbytes), 0x00020000);
  const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(dy), 0, int(a.ybytes), 0x00020000);
  constexpr uint32_t kOut = 0x80000000u;          // past every buffer's end: the load returns 0

  f32x4 xr[2][3], dr[KI][2][2];
  float xe[2];
  bool has_left, has_right;                       // of the loaded step's pair
  auto load = [&](int s) {
    int ti[3], te[3];
    auto decode = [&](int t, int (&q)[3]) {
      const int a1 = quot(t, a.tiles[2]);
      q[2] = t - a1 * int(a.tiles[2].d);
      const int a0 = quot(a1, a.tiles[1]);
      q[1] = a1 - a0 * int(a.tiles[1].d);
      const int n = quot(a0, a.tiles[0]);
      q[0] = a0 - n * int(a.tiles[0].d);
      return n;
    };
    const int t = 16 * s + 2 * pj, t_e = 16 * s + 14 * ee;
    const bool live = t < a.T, elive = (t_e < a.T) & (ec < a.C);
    const int n = decode(live ? t : 0, ti), ne = decode(elive ? t_e : 0, te);
    has_left = ti[2] > 0;
    has_right = ti[2] + 2 < int(a.tiles[2].d);
    const uint32_t xb = (uint32_t(n) * uint32_t(a.C) + uint32_t(c)) * a.xstride + uint32_t(ti[2]) * 8u;
    const uint32_t eb = (uint32_t(ne) * uint32_t(a.C) + uint32_t(ec)) * a.xstride + uint32_t(te[2]) * 8u +
                        (ee ? 16u : uint32_t(-4));
    const bool ein = elive & (ee ? te[2] + 2 < int(a.tiles[2].d) : te[2] > 0);
    auto x_at = [&](const int (&q)[3], bool in, uint32_t base, int w0, int w1) {
      const int q0 = 2 * q[0] - a.pad[0] + w0, q1 = 2 * q[1] - a.pad[1] + w1;
      in = in & (unsigned(q0) < unsigned(a.X[0])) & (unsigned(q1) < unsigned(a.X[1]));
      return in ? base + uint32_t(q0 * a.X[1] + q1) * uint32_t(a.X[2]) * 4u : kOut;
    };
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
      for (int r = 0; r < 3; ++r)
        xr[pl][r] = __builtin_bit_cast(
            f32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, int(x_at(ti, live & (c < a.C), xb, pl ? P1 : P0, rr3[r])), 0, 0));
    // window row r = 3 plane + row
    const uint32_t e0 = x_at(te, ein, eb, er < 3 ? P0 : P1, er == 0 || er == 3 ? rr3[0] : er == 1 ? rr3[1] : rr3[2]);
    const uint32_t e1 = x_at(te, ein & (er < 2), eb, P1, er == 0 ? rr3[1] : rr3[2]);
    xe[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, int(e0), 0, 0));
    xe[1] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, int(e1), 0, 0));
#pragma unroll
    for (int i = 0; i < KI; ++i) {
      const int k = kb * KB + 64 * i + prow;
      const uint32_t yb = (uint32_t(n) * uint32_t(a.K) + uint32_t(k)) * a.ystride + uint32_t(ti[2]) * 8u;
#pragma unroll
      for (int o0 = 0; o0 < 2; ++o0)
#pragma unroll
        for (int o1 = 0; o1 < 2; ++o1) {
          const int y0 = 2 * ti[0] + o0, y1 = 2 * ti[1] + o1;
          const bool in = live & (k < a.K) & (y0 < a.Y[0]) & (y1 < a.Y[1]);
          dr[i][o0][o1] = __builtin_bit_cast(
              f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                         ry, int(in ? yb + uint32_t(y0 * a.Y[1] + y1) * uint32_t(a.Y[2]) * 4u : kOut), 0, 0));
        }
    }
  };
  // split element e of the pair's two tiles and write it to a row
  char* const pw = lds + (pj >> 2) * HALF + prow * 16 + (pj & 3) * 4;
  auto put = [&](char* dst, int e, float u0, float u1) {
    uint32_t h, m, l;
    split2(u0, u1, h, m, l);
    *reinterpret_cast<uint32_t*>(dst + (e * 3 + 0) * PLANE) = h;
    *reinterpret_cast<uint32_t*>(dst + (e * 3 + 1) * PLANE) = m;
    *reinterpret_cast<uint32_t*>(dst + (e * 3 + 2) * PLANE) = l;
  };
  auto produce = [&]() {
#pragma unroll
    for (int i = 0; i < KI; ++i) {
      f32x4 q[2];                                 // axis 0 done, [o1]
#pragma unroll
      for (int o1 = 0; o1 < 2; ++o1)
#pragma unroll
        for (int k = 0; k < 4; ++k) q[o1][k] = __builtin_fmaf(ga[1], dr[i][1][o1][k], ga[0] * dr[i][0][o1][k]);
      char* dst = pw + i * 64 * 16;
#pragma unroll
      for (int rr = 0; rr < 2; ++rr) {
        float w[4];                               // axis 1 done: outputs of tile 2j, 2j + 1
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = __builtin_fmaf(gb[rr][1], q[1][k], gb[rr][0] * q[0][k]);
        float u0[4], u1[4];
        apply_axis<1, MM, 4, 1>(w, u0, Gp);
        apply_axis<1, MM, 4, 1>(w + 2, u1, Gp);
#pragma unroll
        for (int e = 0; e < 4; ++e) put(dst, rr * 4 + e, u0[e], u1[e]);
      }
    }
    float d[3][5];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const int r1 = 3 + r;
      const float e0 = __int_as_float(__builtin_amdgcn_ds_bpermute(epick + 64 * r, __float_as_int(xe[0])));
      const float e1 = __int_as_float(__builtin_amdgcn_ds_bpermute(epick + 64 * (r1 & 3), __float_as_int(xe[r1 >> 2])));
#pragma unroll
      for (int k = 0; k < 4; ++k) d[r][k] = __builtin_fmaf(g0, xr[1][r][k], xr[0][r][k]);
      d[r][4] = __builtin_fmaf(g0, e1, e0);
    }
#pragma unroll
    for (int rr = 0; rr < 2; ++rr) {
      float w[5];
#pragma unroll
      for (int k = 0; k < 5; ++k) w[k] = rr == 0 ? d[0][k] - d[2][k] : __builtin_fmaf(g1, d[1][k], d[2][k]);
      float lv = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(w[3]), 0x111, 0xf, 0xf, false));
      float rv = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(w[0]), 0x101, 0xf, 0xf, false));
      // the eight pairs' ends were loaded (0 outside the row); inside, a
      // neighbour in another row of tiles stands for a value outside x
      lv = first ? w[4] : has_left ? lv : 0.0f;
      rv = last ? w[4] : has_right ? rv : 0.0f;
      const float u0[4] = {lv - w[1], w[0] + w[1], w[1] - w[0], w[0] - w[2]};
      const float u1[4] = {w[1] - w[3], w[2] + w[3], w[3] - w[2], w[2] - rv};
#pragma unroll
      for (int e = 0; e < 4; ++e) put(pw + KB * 16, rr * 4 + e, u0[e], u1[e]);
    }
  };

  f32x16 acc[KB / 32][2];
#pragma unroll
  for (int i = 0; i < KB / 32; ++i)
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) acc[i][jb] = f32x16{};
  const char* const rd = lds + wave * 3 * PLANE + half * HALF + col * 16;

  if (s0 < s1) load(s0);
#pragma unroll 1
  for (int s = s0; s < s1; ++s) {
    produce();
    load(s + 1 < s1 ? s + 1 : s);
    stage_barrier();
    bf16x8 B[2][3];
#pragma unroll
    for (int jb = 0; jb < 2; ++jb)
#pragma unroll
      for (int k = 0; k < 3; ++k) B[jb][k] = *reinterpret_cast<const bf16x8*>(rd + k * PLANE + (KB + 32 * jb) * 16);
#pragma unroll
    for (int i = 0; i < KB / 32; ++i) {
      bf16x8 A[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) A[k] = *reinterpret_cast<const bf16x8*>(rd + k * PLANE + 32 * i * 16);
      // the small terms first; 0, 1, 2 = h, m, l
      constexpr int SA[6] = {2, 0, 1, 1, 0, 0}, SB[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
      for (int k = 0; k < 6; ++k)
#pragma unroll
        for (int jb = 0; jb < 2; ++jb) acc[i][jb] = mfma_bf16(A[SA[k]], B[jb][SB[k]], acc[i][jb]);
    }
    stage_barrier();
  }

  // partial M: lanes over channels
  float* const out = a.part + (int64_t(sp) * 64 + p * E + wave) * a.kp * a.cpn;
#pragma unroll
  for (int i = 0; i < KB / 32; ++i)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int k = kb * KB + 32 * i + 8 * (r >> 2) + 4 * half + (r & 3);
      if (k >= a.kp) continue;
#pragma unroll
      for (int jb = 0; jb < 2; ++jb) out[int64_t(k) * a.cpn + cb * CB + 32 * jb + col] = acc[i][jb][r];
    }
}

}  // namespace wino
