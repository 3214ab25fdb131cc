// Batched GEMM with the inverse transform of F(4^2, 3^2) on the bf16 matrix
// cores (fp32 operands split into three bf16 each, gemm_split.hpp), all 36
// elements resident.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "gemm_acc.hpp"
#include "gemm_split.hpp"
#include "kernels.hpp"
#include "synth.hpp"
#include "transforms.hpp"

namespace wino {

template <int N, int MM, int R>
struct Split4Geom {
  static constexpr int A = MM + R - 1;
  static constexpr int NXI = ipow(A, N);
  static constexpr int NOUT = ipow(MM, N);
  static constexpr int TB = 64, KB = 32;          // tiles and kernels per work-group
  static constexpr int NW = 12, NT = 768;
  static constexpr int E = NXI / NW;              // elements per wave
  static constexpr int SC = 16;                   // channels per step
  static constexpr int HT = 32;                   // tiles per epilogue round
  static constexpr int LDK = HT * MM + 4;         // stitch: floats per (o0, kernel), padded
  static_assert(N == 2 && MM == 4 && A == 6 && E * NW == NXI, "F(4^2, 3^2)");
  static_assert(MM * KB * LDK <= NXI * HT * KB, "the stitch fits the exchange");
};

// out[o * os] = sum_i AT[o][i] v[i * vs] of the default points, the terms in
// pairs (0, 1), (2, 3), .. added in order.  The sums and differences that the
// columns of points a and -a share (apply_vec) take 10 operations for F(4, 3)
// instead of 14, but round more: on one channel's products (float64 beside
// them) they leave a relative error of 3.3e-7, this 2.6e-7 and k_gemm_acc4's
// running sum 2.7e-7.  Over many channels that is below the products' own
// rounding, and the 4 operations are 0.5% of a layer's time.
template <int MM, int R>
__device__ __forceinline__ void at_pairs(const float* v, int vs, float* out, int os) {
  constexpr int A = MM + R - 1;
  unroll<MM>([&](auto O) {
    constexpr int o = decltype(O)::value;
    float sum = 0.0f;
    bool any = false;                             // folds away: every entry is a constant
    unroll<A / 2>([&](auto P) {
      constexpr float c0 = const_entry<Which::AT, MM, R>(o, 2 * decltype(P)::value);
      constexpr float c1 = const_entry<Which::AT, MM, R>(o, 2 * decltype(P)::value + 1);
      const float v0 = v[2 * decltype(P)::value * vs], v1 = v[(2 * decltype(P)::value + 1) * vs];
      if constexpr (c0 == 0.0f && c1 == 0.0f) return;
      else {
        float pair;
        if constexpr (c1 == 0.0f) pair = c0 * v0;
        else if constexpr (c0 == 0.0f) pair = c1 * v1;
        else pair = __builtin_fmaf(c1, v1, c0 * v0);
        sum = any ? sum + pair : pair;
        any = true;
      }
    });
    out[o * os] = sum;
  });
}

// One work-group: 64 tiles x 32 kernels, twelve waves; wave w owns elements
// 3w .. 3w + 2 (96 accumulators), so every V and U value of the block is
// loaded and split by exactly one wave, straight from global memory to
// registers: lane (row r, half h) takes channels 8h .. 8h + 7 of a 16-channel
// step for both operands.  No barrier until the channels are done.  Then the
// products of 32 tiles at a time meet in LDS (144 KB), a thread applies A^T to
// two (tile, kernel) pairs, and the outputs go through LDS once more so that
// neighbouring lanes store neighbouring tiles' rows, 16 bytes each, or (rows of
// no whole 16-byte units) neighbouring outputs.
//
// FEW (at most four channels): one channel group, lane half h takes channels
// 2h and 2h + 1 and multiplies them in fp32 (two k-steps an element).  The
// terms that the split leaves out weigh more there than the roundings it saves:
// against float64 (2-norm, 2 x C x 48 x 64, K = 64) the split products show
// 1.18, 1.12, 1.07 and 1.04 times k_gemm_acc4's error for 1 to 4 channels, 1.00
// for 5, 0.97 for 6 and 0.77 for 16; FEW, with at_pairs, 0.98 to 1.00.  FEW also
// has no splits to make: the forward of 32 x 3 x 224 x 224, K = 64, 247 -> 214
// us (k_gemm_acc4 297).
//
// What bounds it: the sum of its parts, which hardly overlap (on 64 x 256 x
// 56 x 56, K = 256, 535-575 us: matrix work 200 at the clock it falls to, the
// splits' vector work about 135, the loads' addresses about 160, the
// epilogues about 60).  A 64 x 64 block would take a third off the loads and
// splits, but its 36 elements do not fit the registers.  Against the fp32
// passes of k_gemm_acc4 (us, there / here): that layer 581 / 536;
// 64 x 512 x 28 x 28, K = 128, 205 / 133; 16 x 16 x 112 x 112, K = 64, 43 / 31;
// 1 x 3 x 224 x 224, K = 64, 39 / 16.  V is loaded temporally while
// several kernel blocks re-read it (570 -> 531 us against non-temporal loads;
// the next input transform then finds less of x in the memory-side cache and
// gives the 40 us back where x is the same tensor each time), and
// non-temporally with ONE kernel block, where a V past that cache's 256 MB only
// displaces x and itself.  The whole forward with K = 32 (us, k_gemm_acc4 /
// temporal / non-temporal): 64 channels, 32768 tiles 155 / 187 / 148; 160
// channels, 12288 tiles 147 / 164 / 126; 256 channels, 8320 tiles 180 / 185 / 151.
template <int N, int MM, int R, bool FEW, bool ONE>
__global__ void __launch_bounds__(768, 3) k_gemm_split4(const float* __restrict__ V, const float* __restrict__ U,
                                                        float* __restrict__ y, AccArgs g) {
  using G = Split4Geom<N, MM, R>;
  constexpr int NXI = G::NXI, NOUT = G::NOUT, TB = G::TB, KB = G::KB, E = G::E, HT = G::HT;
  __shared__ __attribute__((aligned(16))) float ex[NXI * HT * KB];

  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;

  // Work unit -> (block, channel stages): blocks and tail blocks as in
  // k_gemm_acc, a tail block's parts are runs of its channel stages (the
  // inverse transform is linear in them).
  const int xcd = int(blockIdx.x) & 7, j = int(blockIdx.x) >> 3;
  const int xn = g.xn[xcd], xs = g.xs[xcd], np = g.nparts;
  const int nwhole = xn - xs;
  if (j >= nwhole + xs * np) return;
  const bool tail = np > 1 && j >= nwhole;
  const int tj = j >= nwhole ? j - nwhole : 0;
  const int blk = g.xb0[xcd] + (j >= nwhole ? nwhole + tj / np : j);
  const int nstage = g.C_pad / G::SC;
  const int q = tail ? tj % np : 0;
  const int s0 = tail ? nstage * q / np : 0;
  const int s1 = tail ? nstage * (q + 1) / np : nstage;
  const int64_t pslot = tail ? int64_t(g.xt0[xcd]) * np + tj : 0;
  const int tb = blk / g.nkb, kb = blk % g.nkb;

  constexpr int64_t VX = TB * 4, VG = int64_t(NXI) * TB * 4;      // V element / group strides (floats)
  const int64_t UG = int64_t(g.K_pad) * 4;                        // U group stride
  using Vec = std::conditional_t<FEW, float2, f32x4>;             // channels of one load
  constexpr int HG = FEW ? 1 : 2;                                 // loads per lane half and row
  const uint32_t hoff = FEW ? 8u : uint32_t(2 * VG * 4);
  const uint32_t vlane = uint32_t(half) * hoff + uint32_t(col) * 16u;
  const uint32_t ulane = uint32_t(half) * (FEW ? 8u : uint32_t(2 * UG * 4)) + uint32_t(col) * 16u;
  const float* const vblk = V + int64_t(tb) * g.vblock + wave * E * VX;
  const float* const ublk = U + int64_t(kb) * (KB * 4) + wave * E * g.uplane;

  Vec ra[2 * HG], rb[HG];                         // [32-tile half][load of the lane's half]
  auto load = [&](int st, int e) {
    const char* us = reinterpret_cast<const char*>(ublk + e * g.uplane + int64_t(st) * 4 * UG);
    const char* vs = reinterpret_cast<const char*>(vblk + e * VX + int64_t(st) * 4 * VG);
#pragma unroll
    for (int jj = 0; jj < HG; ++jj) rb[jj] = *reinterpret_cast<const Vec*>(us + jj * UG * 4 + ulane);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int jj = 0; jj < HG; ++jj) {
        const char* at = vs + jj * VG * 4 + vlane + i * 512;
        if constexpr (ONE) ra[HG * i + jj] = __builtin_nontemporal_load(reinterpret_cast<const Vec*>(at));
        else ra[HG * i + jj] = *reinterpret_cast<const Vec*>(at);
      }
  };

  f32x16 acc[E][2];
#pragma unroll
  for (int e = 0; e < E; ++e)
#pragma unroll
    for (int i = 0; i < 2; ++i) acc[e][i] = f32x16{};

  if (s0 < s1) load(s0, 0);
#pragma unroll 1
  for (int st = s0; st < s1; ++st) {
    // the loads past the last step read the last stage again
    const int nx = st + 1 < s1 ? st + 1 : st;
    static_for<E>([&](auto I) {
      constexpr int e = decltype(I)::value;
      f32x16 c0 = acc[e][0], c1 = acc[e][1];
      if constexpr (FEW) {
        // k-step j: channel j in the lower lanes, 2 + j in the upper ones
        const float2 b = rb[0], a0 = ra[0], a1 = ra[1];
        load(e + 1 < E ? st : nx, (e + 1) % E);
        c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.x, b.x, c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.x, b.x, c1, 0, 0, 0);
        c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(a0.y, b.y, c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_32x32x2f32(a1.y, b.y, c1, 0, 0, 0);
        acc[e][0] = c0;
        acc[e][1] = c1;
      } else {
        const Split8 b = split8(rb[0], rb[1]);
        const Split8 a0 = split8(ra[0], ra[1]), a1 = split8(ra[2], ra[3]);
        load(e + 1 < E ? st : nx, (e + 1) % E);
        // the small terms first
        c0 = mfma_bf16(a0.l, b.h, c0);
        c1 = mfma_bf16(a1.l, b.h, c1);
        c0 = mfma_bf16(a0.h, b.l, c0);
        c1 = mfma_bf16(a1.h, b.l, c1);
        c0 = mfma_bf16(a0.m, b.m, c0);
        c1 = mfma_bf16(a1.m, b.m, c1);
        c0 = mfma_bf16(a0.m, b.h, c0);
        c1 = mfma_bf16(a1.m, b.h, c1);
        c0 = mfma_bf16(a0.h, b.m, c0);
        c1 = mfma_bf16(a1.h, b.m, c1);
        acc[e][0] = mfma_bf16(a0.h, b.h, c0);
        acc[e][1] = mfma_bf16(a1.h, b.h, c1);
      }
    });
  }

  const MatRef<Which::AT, true, MM, R> AT{nullptr};
  const bool quad = g.Y[1] % 4 == 0;              // rows of whole 16-byte units
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    if (!tail && tb * TB + i * HT >= g.T) break;  // no tile of this half
    if (i == 1) __syncthreads();                  // the first half's stores have read ex
    // exchange: ex[element][slot q][lane][4], slot q of a wave's block = rows
    // 8q + 4 half + 0..3 (tiles) of kernel col
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
      for (int qq = 0; qq < 4; ++qq) {
        const f32x16& c = acc[e][i];
        *reinterpret_cast<f32x4*>(ex + (wave * E + e) * (HT * KB) + qq * 256 + lane * 4) =
            f32x4{c[4 * qq], c[4 * qq + 1], c[4 * qq + 2], c[4 * qq + 3]};
      }
    __syncthreads();
    // thread (q, lane, two rows): pairs (tiles t2, t2 + 1, kernel col)
    const bool works = wave < 8;                  // 512 threads finish 1024 pairs
    const int t2 = 8 * (wave >> 1) + 4 * half + 2 * (wave & 1);
    float out[2][NOUT];
    if (works) {
      float m[2][NXI];
#pragma unroll
      for (int x = 0; x < NXI; ++x) {
        const float2 v = *reinterpret_cast<const float2*>(ex + x * (HT * KB) + (wave >> 1) * 256 + lane * 4 + 2 * (wave & 1));
        m[0][x] = v.x;
        m[1][x] = v.y;
      }
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        if constexpr (FEW) {
          float t[MM * G::A];
#pragma unroll
          for (int c = 0; c < G::A; ++c) at_pairs<MM, R>(m[p] + c, G::A, t + c, G::A);
#pragma unroll
          for (int o = 0; o < MM; ++o) at_pairs<MM, R>(t + o * G::A, 1, out[p] + o * MM, 1);
        } else {
          transform_nd<N, G::A, MM>(m[p], out[p], AT);
        }
      }
    }
    if (tail) {
      // partial outputs of this unit: part[pslot][o][t][k], lanes over k
      if (works) {
        float* pp = g.part + pslot * NOUT * (TB * KB);
#pragma unroll
        for (int o = 0; o < NOUT; ++o)
#pragma unroll
          for (int p = 0; p < 2; ++p) pp[(o * TB + i * HT + t2 + p) * KB + col] = out[p][o];
      }
      continue;
    }
    __syncthreads();                              // the products are read
    if (works) {
#pragma unroll
      for (int o0 = 0; o0 < MM; ++o0)
#pragma unroll
        for (int p = 0; p < 2; ++p)
          *reinterpret_cast<f32x4*>(ex + (o0 * KB + col) * G::LDK + (t2 + p) * MM) =
              f32x4{out[p][o0 * MM], out[p][o0 * MM + 1], out[p][o0 * MM + 2], out[p][o0 * MM + 3]};
    }
    __syncthreads();
    if (!quad) {
      // Rows that are no whole 16-byte units: lanes over the outputs of 16
      // tiles, so that a store covers a run of a row.  (With a tile's four
      // outputs stored by its lane, each store wrote a quarter of every line it
      // touched: the forward of 62 x 17 x 138 x 11, K = 161, took 322 us and of
      // 20 x 4 x 71 x 17, K = 440, 159; so 79 and 39, the fp32 passes 142 and 72.)
      float* yt[2];
      int rows[2];                                // output rows of the tile inside y; 0: nothing to store
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int t = tb * TB + i * HT + 16 * h + (lane >> 2);
        int ti[3] = {0, 0, 0};
        const int n = split_tile<N>(t < g.T ? t : 0, g.tiles, ti);
        const int ylast = ti[1] * MM + (lane & 3);
        yt[h] = y + (int64_t(n) * g.K + kb * KB) * g.ystride_k + int64_t(ti[0] * MM) * g.Y[1] + ylast;
        rows[h] = t < g.T && ylast < g.Y[1] ? g.Y[0] - ti[0] * MM : 0;
      }
      const int n_it = MM * (g.K - kb * KB < KB ? g.K - kb * KB : KB);   // (kernel, output row) pairs
      constexpr int BATCH = 4;                    // reads of LDS ahead of the stores
      static_assert(((MM - 1) * KB + (MM * KB + BATCH * G::NW) / MM) * G::LDK + HT * MM <= NXI * HT * KB,
                    "the reads past the last pair stay inside ex");
#pragma unroll 1
      for (int it0 = wave; it0 < n_it; it0 += BATCH * G::NW) {
        float v[BATCH][2];
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {         // past the last pair: other words of ex
          const int it = it0 + b * G::NW, o0 = it % MM, kl = it / MM;
#pragma unroll
          for (int h = 0; h < 2; ++h) v[b][h] = ex[(o0 * KB + kl) * G::LDK + lane + 64 * h];
        }
#pragma unroll
        for (int b = 0; b < BATCH; ++b) {
          const int it = it0 + b * G::NW, o0 = it % MM, kl = it / MM;
          if (it >= n_it) break;
          const float bk = g.bias != nullptr ? g.bias[kb * KB + kl] : 0.0f;
          const int64_t off = int64_t(kl) * g.ystride_k + int64_t(o0) * g.Y[1];
#pragma unroll
          for (int h = 0; h < 2; ++h) {
            float u = v[b][h];
            if (g.bias != nullptr) u += bk;
            u = activate(u, g.act, g.slope);
            if (o0 < rows[h]) __builtin_nontemporal_store(u, yt[h] + off);
          }
        }
      }
      continue;
    }
    // thread = (tile, then kernel and output row): lanes over tiles, 16 bytes each
    const int tl = tid % HT;
    const int t = tb * TB + i * HT + tl;
    if (t < g.T) {
      int ti[3] = {0, 0, 0};
      const int n = split_tile<N>(t, g.tiles, ti);
      float* const yt = y + int64_t(n) * g.K * g.ystride_k + int64_t(ti[0] * MM) * g.Y[1] + ti[1] * MM;
#pragma unroll 1
      for (int it = tid / HT; it < MM * KB; it += G::NT / HT) {
        const int o0 = it / KB, kl = it % KB, kg = kb * KB + kl;
        if (kg >= g.K || ti[0] * MM + o0 >= g.Y[0]) continue;
        f32x4 v = *reinterpret_cast<const f32x4*>(ex + it * G::LDK + tl * MM);
        const float bk = g.bias != nullptr ? g.bias[kg] : 0.0f;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          if (g.bias != nullptr) v[k] += bk;
          v[k] = activate(v[k], g.act, g.slope);
        }
        __builtin_nontemporal_store(
            v, reinterpret_cast<f32x4*>(yt + int64_t(kg) * g.ystride_k + int64_t(o0) * g.Y[1]));
      }
    }
  }
}

}  // namespace wino
