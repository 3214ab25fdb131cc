// The F(2^3, 3^3) forward in one kernel (k_fwd_split), on the bf16 matrix
// cores with fp32 operands split into three bf16 numbers each.
//
// The split (of fp32 values into three bf16 and products of their leading
// terms: G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the bfloat16
// Artificial Intelligence Datatype For Higher-Precision Computations", ARITH
// 2019).  a = a1 + a2 + a3: a1 the upper 16 bits of a (truncated: it never
// overflows), a2 the bf16 nearest to a - a1, a3 the bf16 nearest to the rest;
// the subtractions are exact, and so is the sum (8 + 16 bits, of which a2 takes
// 8 and its sign leaves 8) while a3 is a normal bf16 number: for |a| from about
// 2^-112 up.  Below, a3 loses bits, to 2^-133 absolute.  A product a b is the sum of
// the six terms a1 b1, a1 b2, a2 b1, a1 b3, a2 b2, a3 b1, each exact; what is left
// out (a2 b3, a3 b2, a3 b3) is below 2^-22 |a b|, about 2^-26 in the mean and of
// random sign.  Small terms are not flushed: errors are the same with every
// product near 2^-120.  An infinity's remainder a - a1 is a NaN.
//
// The sums stay in fp32 MFMA accumulators.  One v_mfma_f32_32x32x16_bf16 sums
// 16 channels with fewer roundings of the accumulator than the eight
// v_mfma_f32_32x32x2_f32 it replaces; six of them, against float64, products over
// 64 / 256 / 512 channels of normal values: relative error (2-norm) of 1.1e-7 /
// 2.4e-7 / 3.4e-7 where the fp32 instruction shows 1.4e-7 / 2.9e-7 / 4.1e-7, and
// the forward of 8 x 64 x 16 x 56 x 56, K = 128, 2.5e-7 against 3.0e-7.  Over fewer
// than about six terms the ones left out weigh more than the roundings saved;
// such layers take the fp32 products.
//
// Why.  Dense peaks: fp32 MFMA 157 TFLOP/s, bf16 2.5 PFLOP/s, 419 at six products
// a term.  Plain loops of the instructions reach 142 and 1.8 PFLOP/s / 6 = 300 (on
// random values the clock falls to 1.7 GHz), a large library matrix product 153
// and 1.16 PFLOP/s / 6 = 193.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>
#include <utility>

#include "gemm_acc.hpp"
#include "kernels.hpp"
#include "synth.hpp"
#include "transforms.hpp"

namespace wino {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// f(0), f(1), .. f(N - 1) with the index as a compile-time constant
template <int N, class F, int... I>
__device__ __forceinline__ void static_for_seq(F& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F f) {
  static_for_seq<N>(f, std::make_integer_sequence<int, N>{});
}

// Eight fp32 values (consecutive k of one row) as three bf16 operand registers
// of four words each.
struct Split8 {
  bf16x8 h, m, l;
};

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  bf16x2 r;
  r.x = static_cast<__bf16>(a);
  r.y = static_cast<__bf16>(b);
  return __builtin_bit_cast(uint32_t, r);
}

// Two values -> one word of each operand register.
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  const uint32_t ua = __builtin_bit_cast(uint32_t, a), ub = __builtin_bit_cast(uint32_t, b);
  h = __builtin_amdgcn_perm(ub, ua, 0x07060302);    // the upper halves
  const float ra = a - __builtin_bit_cast(float, ua & 0xffff0000u);
  const float rb = b - __builtin_bit_cast(float, ub & 0xffff0000u);
  m = pack_bf16(ra, rb);
  const float sa = ra - __builtin_bit_cast(float, m << 16);
  const float sb = rb - __builtin_bit_cast(float, m & 0xffff0000u);
  l = pack_bf16(sa, sb);
}

__device__ __forceinline__ Split8 split8(const f32x4& a, const f32x4& b) {
  u32x4 h, m, l;
  uint32_t th, tm, tl;
  split2(a[0], a[1], th, tm, tl); h[0] = th; m[0] = tm; l[0] = tl;
  split2(a[2], a[3], th, tm, tl); h[1] = th; m[1] = tm; l[1] = tl;
  split2(b[0], b[1], th, tm, tl); h[2] = th; m[2] = tm; l[2] = tl;
  split2(b[2], b[3], th, tm, tl); h[3] = th; m[3] = tm; l[3] = tl;
  return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}

__device__ __forceinline__ f32x16 mfma_bf16(const bf16x8& a, const bf16x8& b, const f32x16& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

template <int N, int MM, int R>
struct SplitGeom {
  static constexpr int A = MM + R - 1;
  static constexpr int NXI = ipow(A, N);
  static constexpr int NW = 8, NT = 512;          // wave w owns element w of a pass
  static constexpr int E = 8;                     // elements per pass: two rows of the last axis
  static constexpr int NPASS = NXI / E;
  static constexpr int NOUT = ipow(MM, N);        // outputs per (tile, kernel)
  static constexpr int NLEAD = NOUT / MM;
  static constexpr int TB = 64, KB = 64;          // tiles and kernels per work-group
  static constexpr int SC = 16;                   // channels per step
  static constexpr int POS = TB * KB / NT;        // (tile, kernel) pairs a thread finishes
  static_assert(MM == 2 && A == 4 && NXI % E == 0 && E == 2 * A, "m = 2, r = 3");
};

// The end of a 64-tile x 64-kernel block whose thread holds the outputs
// yacc[o][p] of its pairs p = (tile tile_of(p), kernel kern_of(p)), both local
// to the block: partial outputs of a tail unit (part != null), the pooled
// store, or bias, activation and the store of every output.  ex: the
// work-group's LDS, NOUT * 64 * 66 floats, free after a barrier.  The rows of
// y are whole 16-byte units and a pair of neighbouring tiles (2j, 2j + 1)
// starts one, so their outputs of a row are one 16-byte store: a wave's store
// takes 16 cycles of addresses whatever its width, and 16 stores a thread
// instead of 64 took the forward of 8 x 64 x 16 x 56 x 56, K = 128, from 544
// to 530 us.
template <int N, int MM, int POOL, int NOUT, int POS, class TileOf, class KernOf>
__device__ __forceinline__ void split_finish(const float (&yacc)[NOUT][POS], TileOf tile_of, KernOf kern_of,
                                             float* ex, float* __restrict__ y, const AccArgs& g, int tb, int kb,
                                             float* part) {
  constexpr int TB = 64, KB = 64, NT = TB * KB / POS, NLEAD = NOUT / MM;
  const int tid = int(threadIdx.x);
  if (part != nullptr) {
    // part[o][t][k], lanes over k
#pragma unroll
    for (int o = 0; o < NOUT; ++o)
#pragma unroll
      for (int p = 0; p < POS; ++p) part[(o * TB + tile_of(p)) * KB + kern_of(p)] = yacc[o][p];
    return;
  }

  if constexpr (POOL != 0) {
    // Window (2, 2, 2), stride 2: a tile of 2 is one window, whose 8 outputs
    // are this thread's.  Bias, activation and the maximum in registers,
    // scanned in the stand-alone pool's order (first axis slowest, strict
    // comparison from -inf), so the result has the bits of the forward
    // followed by that pool; floor rounding drops the tiles cut by the
    // output's end.
    static_assert(N == 3 && MM == 2, "the pooled epilogue takes 3-D tiles of 2");
#pragma unroll
    for (int p = 0; p < POS; ++p) {
      const int kg = kb * KB + kern_of(p);
      const int t = tb * TB + tile_of(p);
      if (kg >= g.K || t >= g.T) continue;
      int ti[3] = {0, 0, 0};
      const int n = split_tile<N>(t, g.tiles, ti);
      if (ti[0] >= g.Yp[0] || ti[1] >= g.Yp[1] || ti[2] >= g.Yp[2]) continue;
      const float bk = g.bias != nullptr ? g.bias[kg] : 0.0f;
      float best = -__builtin_inff();
#pragma unroll
      for (int o = 0; o < NOUT; ++o) {
        float v = yacc[o][p];
        if (g.bias != nullptr) v += bk;
        v = activate(v, g.act, g.slope);
        best = v > best ? v : best;
      }
      y[(int64_t(n) * g.K + kg) * g.ystride_p + (int64_t(ti[0]) * g.Yp[1] + ti[1]) * g.Yp[2] + ti[2]] = best;
    }
    return;
  }

  constexpr int LD = TB + 2;                    // row stride: lanes over k spread over the banks
  __syncthreads();
#pragma unroll
  for (int o = 0; o < NOUT; ++o)
#pragma unroll
    for (int p = 0; p < POS; ++p) ex[(o * KB + kern_of(p)) * LD + tile_of(p)] = yacc[o][p];
  __syncthreads();
  const int tj = tid % (TB / 2);                // tile pair
  const int t = tb * TB + 2 * tj;
  if (t >= g.T) return;
  int ti[3] = {0, 0, 0};
  const int n = split_tile<N>(t, g.tiles, ti);
  float* const yn = y + int64_t(n) * g.K * g.ystride_k;
  constexpr int KS = NT / (TB / 2);
#pragma unroll
  for (int orest = 0; orest < NLEAD; ++orest) {
    int64_t off = 0;
    bool in = true;
#pragma unroll
    for (int ax = 0; ax < N - 1; ++ax) {
      const int yc = ti[ax] * MM + (orest / ipow(MM, N - 2 - ax)) % MM;
      in = in && yc < g.Y[ax];
      off = off * g.Y[ax] + yc;
    }
    if (!in) continue;
    float* const yo = yn + off * g.Y[N - 1] + ti[N - 1] * MM;
    const float* pl = ex + (orest * MM) * (KB * LD) + 2 * tj;
#pragma unroll
    for (int kk = tid / (TB / 2); kk < KB; kk += KS) {
      const int kg = kb * KB + kk;
      if (kg >= g.K) break;
      const float2 a = *reinterpret_cast<const float2*>(pl + kk * LD);
      const float2 b = *reinterpret_cast<const float2*>(pl + (KB + kk) * LD);
      f32x4 v = {a.x, b.x, a.y, b.y};
      const float bk = g.bias != nullptr ? g.bias[kg] : 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (g.bias != nullptr) v[i] += bk;
        v[i] = activate(v[i], g.act, g.slope);
      }
      __builtin_nontemporal_store(v, reinterpret_cast<f32x4*>(yo + int64_t(kg) * g.ystride_k));
    }
  }
}

// U (fp32, U[xi][C_pad/4][K_pad][4]) as three bf16 operand planes,
// P[xi][C_pad/8][3][K_pad][8]: one thread per (xi, 8 channels, kernel).
static __global__ void __launch_bounds__(256) k_split_u(const float* __restrict__ U, u32x4* __restrict__ P,
                                                        int64_t n, int32_t K_pad) {
  const int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x;   // (xi, c8, k)
  if (i >= n) return;
  const int64_t row = i / K_pad;
  const int k = int(i % K_pad);
  const f32x4* src = reinterpret_cast<const f32x4*>(U) + row * 2 * K_pad + k;
  const Split8 t = split8(src[0], src[K_pad]);
  u32x4* dst = P + row * 3 * K_pad + k;
  dst[0] = __builtin_bit_cast(u32x4, t.h);
  dst[K_pad] = __builtin_bit_cast(u32x4, t.m);
  dst[2 * K_pad] = __builtin_bit_cast(u32x4, t.l);
}

// A^T of F(2, 3) for the pass epilogue, which indexes it with the
// wave-uniform pass (scalar loads).
struct SplitAT {
  float at[2][4];
};
constexpr SplitAT make_split_at() {
  SplitAT t{};
  for (int o = 0; o < 2; ++o)
    for (int e = 0; e < 4; ++e) t.at[o][e] = kDefaultF<2, 3>.AT[o][e];
  return t;
}
static __constant__ SplitAT kSplitAT = make_split_at();

struct FuseArgs {
  AccArgs g;
  int32_t X[3], pad[3];
  int32_t C;
  uint32_t xbytes;    // bytes of x (at most 2^29)
  uint32_t xstride;   // bytes of one channel of one sample
};

// The F(2^3, 3^3) forward in one kernel: V is formed in LDS, split as it is
// written, and never reaches memory.  One work-group: 64 tiles x 64 kernels,
// eight waves.  It walks eight passes of eight elements, xi0 = p / 2,
// xi1 = 2 (p % 2) + {0, 1}, xi2 = 0..3, which take two planes and three rows
// of each 4 x 4 x 4 window; a step is 16 channels of a pass.
//   produce: thread = (two neighbouring tiles, channel): the six window rows
//     are one aligned 16-byte load each, the outer columns come from the
//     neighbouring lanes by DPP.  B^T axis by axis, then v_permlane32_swap
//     trades tiles for channels between the lane halves, so that a thread
//     splits and writes one word (two channels of a tile) per element and
//     operand register to planes[element][h, m, l][8-channel half][row][16 bytes].
//   consume: wave w multiplies element w, all 64 x 64: A from those planes, B
//     (the split kernels, k_split_u) straight from global memory, so every
//     operand is loaded by one wave only.
//   end of a pass: the eight products meet in LDS, one kernel half after the
//     other; each thread applies A^T for its eight (tile, kernel) pairs and
//     adds the result into their eight outputs, which stay in registers.
// The planes are double-buffered, so a step's producing (vector ALU) and the
// previous step's products (matrix cores) share the step between two
// barriers, part by part behind the products.
//
// What bounds it (8 x 64 x 16 x 56 x 56, K = 128, stripped copies): 530-545 us;
// without the x and B loads 410, without the pass epilogue 480, without the
// final stores 475, matrix work and producing alone 260, matrix work alone
// 180.  The latencies of a step, which all eight waves share through its
// barrier, not the rate of a unit: vector ALU 47%, addresses 39%, LDS 29%,
// matrix cores 27% busy.  252 of 256 registers leave no room to load further
// ahead.  The two-stage form takes 150 us for V and 500 for the product.
template <int POOL>
__global__ void __launch_bounds__(512, 2) k_fwd_split(const float* __restrict__ x, const u32x4* __restrict__ P,
                                                      float* __restrict__ y, FuseArgs a) {
  constexpr int N = 3, MM = 2, R = 3;
  using G = SplitGeom<N, MM, R>;
  constexpr int NOUT = G::NOUT, NLEAD = G::NLEAD, TB = G::TB, KB = G::KB, POS = G::POS;
  constexpr int PLANE = 2048;                     // bytes of one (element, operand register)
  constexpr int BUF = G::E * 3 * PLANE;           // 48 KB
  constexpr int EX = 2 * BUF;                     // exchange region: 64 KB
  __shared__ __attribute__((aligned(16))) char lds[EX + G::E * TB * KB * 2];
  const AccArgs& g = a.g;

  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col = lane & 31, half = lane >> 5;

  const int xcd = int(blockIdx.x) & 7, j = int(blockIdx.x) >> 3;
  const int xn = g.xn[xcd], xs = g.xs[xcd], np = g.nparts;
  const int nwhole = xn - xs;
  if (j >= nwhole + xs * np) return;
  const bool tail = j >= nwhole;
  const int tj = tail ? j - nwhole : 0;
  const int blk = g.xb0[xcd] + (tail ? nwhole + tj / np : j);
  const int nstage = g.C_pad / G::SC;
  const int total = G::NPASS * nstage;
  const int q = tail ? tj % np : 0;
  const int s0 = tail ? int(int64_t(total) * q / np) : 0;
  const int s1 = tail ? int(int64_t(total) * (q + 1) / np) : total;
  const int64_t pslot = tail ? int64_t(g.xt0[xcd]) * np + tj : 0;
  const int tb = blk / g.nkb, kb = blk % g.nkb;

  // ---- producing: this thread's channel and pair of tiles.  Wave w takes the
  // 32 tiles of half w / 4 and the channel pairs 2 (w % 4) + {0, 1}; lane
  // (par, cpx, j): channel par of pair cpx, tiles 2j and 2j + 1.
  const int pi = wave >> 2, par = lane >> 5, pj = lane & 15;
  const int cp = 2 * (wave & 3) + ((lane >> 4) & 1);
  // offset of a tile pair's first own column in channel c of the step
  auto pair_at = [&](int jj, int c, int (&ti)[3], bool& live) {
    const int t = tb * TB + 32 * pi + 2 * jj;
    live = t < g.T;
    const int n = split_tile<N>(live ? t : 0, g.tiles, ti);
    return (uint32_t(n) * uint32_t(a.C) + uint32_t(c)) * a.xstride + uint32_t(ti[2]) * 8u;
  };
  int ti[3], te[3];
  bool live, elive;
  const uint32_t xbase = pair_at(pj, 2 * cp + par, ti, live);
  const bool has_left = ti[2] > 0, has_right = ti[2] + 2 < g.tiles[2];
  // The ends of the wave's 16-lane rows miss one value each.  One load fetches
  // them all: lane 8 r + 2 d + e the value left (e = 0) or right (e = 1) of
  // 16-lane row d in window row r, handed out by ds_bpermute.
  const int er = lane >> 3, ed = (lane >> 1) & 3, ee = lane & 1;
  const uint32_t ebase = pair_at(ee * 15, 2 * (2 * (wave & 3) + (ed & 1)) + (ed >> 1), te, elive) +
                         (ee ? 16u : uint32_t(-4));
  elive = elive & (er < 6) & (ee ? te[2] + 2 < g.tiles[2] : te[2] > 0);
  const int epick = 4 * (2 * (lane >> 4) + (pj == 15 ? 1 : 0));
  const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(x), 0, int(a.xbytes), 0x00020000);
  // the pair's slots of an operand plane: rows par * 16 + j of its 32-tile half
  char* const pw = lds + (cp >> 2) * 1024 + pi * 512 + (par * 16 + pj) * 16 + (cp & 3) * 4;

  f32x4 xr[2][3];                                 // [plane][row]: columns of both tiles
  float xe;
  uint32_t ro[2][3], reo;                         // row offsets of the pass being loaded
  int lp = s0 / nstage, lst = s0 % nstage;        // load cursor
  auto rows = [&](int p) {
    const int i0 = p >> 1, hh = p & 1;
    const int P0 = i0 == 0 ? 0 : i0 == 2 ? 2 : 1, P1 = i0 == 3 ? 3 : i0 == 2 ? 1 : 2;
    const int rr[3] = {hh ? 2 : 0, hh ? 3 : 1, hh ? 1 : 2};
    auto row_at = [&](const int (&tt)[3], bool in, uint32_t base, int w0, int w1) {
      const int q0 = 2 * tt[0] - a.pad[0] + w0, q1 = 2 * tt[1] - a.pad[1] + w1;
      in = in & (unsigned(q0) < unsigned(a.X[0])) & (unsigned(q1) < unsigned(a.X[1]));
      return in ? base + uint32_t(q0 * a.X[1] + q1) * uint32_t(a.X[2]) * 4u : 0x80000000u;   // past the end: 0
    };
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
#pragma unroll
      for (int r = 0; r < 3; ++r) ro[pl][r] = row_at(ti, live, xbase, pl == 0 ? P0 : P1, rr[r]);
    const int e3 = er % 3;
    reo = row_at(te, elive, ebase, er < 3 ? P0 : P1, e3 == 0 ? rr[0] : e3 == 1 ? rr[1] : rr[2]);
  };
  // window row r of both planes, for the cursor's step; with the last, the ends
  auto load_row = [&](int r) {
    const int so = int(uint32_t(lst * G::SC) * a.xstride);
#pragma unroll
    for (int pl = 0; pl < 2; ++pl)
      xr[pl][r] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rx, int(ro[pl][r]), so, 0));
    if (r == 2) xe = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, int(reo), so, 0));
  };
  auto load_x = [&]() {
#pragma unroll
    for (int r = 0; r < 3; ++r) load_row(r);
  };
  // the load cursor's next step; it stays on the block's last one
  auto next_x = [&]() {
    const bool wrap = lst + 1 == nstage, last = lp + 1 == G::NPASS;
    if (wrap && !last) {
      ++lp;
      lst = 0;
      rows(lp);
    } else if (!wrap) {
      ++lst;
    }
  };
  // B^T of pass p on the loaded rows, in eleven parts that can stand between the
  // products: v[0 / 1][e], the two channels of the pair for one tile
  // (2j + par) after the exchange between the lane halves.
  float v[2][G::E];
  float d[3][5];                                  // axis 0 done: [row][four columns, end]
  float w[5], lv, rv;                             // axis 1 done
  auto transform = [&](int p, auto K) {
    constexpr int k = decltype(K)::value;
    if constexpr (k < 3) {
      const float g0 = p >> 1 == 1 ? 1.0f : -1.0f;               // d_P0 - d_P1, + for xi0 = 1
      const float e0 = __int_as_float(__builtin_amdgcn_ds_bpermute(epick + 32 * k, __float_as_int(xe)));
      const float e1 = __int_as_float(__builtin_amdgcn_ds_bpermute(epick + 32 * (3 + k), __float_as_int(xe)));
#pragma unroll
      for (int i = 0; i < 4; ++i) d[k][i] = __builtin_fmaf(g0, xr[1][k][i], xr[0][k][i]);
      d[k][4] = __builtin_fmaf(g0, e1, e0);
    } else {
      constexpr int rr = k >= 7 ? 1 : 0, q = (k - 3) % 4;
      if constexpr (q == 0) {
        const float g1 = p & 1 ? -1.0f : 1.0f;                   // a - c and c +- b
#pragma unroll
        for (int i = 0; i < 5; ++i) w[i] = rr == 0 ? d[0][i] - d[2][i] : __builtin_fmaf(g1, d[1][i], d[2][i]);
      } else if constexpr (q == 1) {
        // row_shr:1 / row_shl:1: lane i takes lane i -+ 1's value, the row's end keeps w[4]
        lv = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(w[4]), __float_as_int(w[3]), 0x111, 0xf, 0xf, false));
        rv = __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(w[4]), __float_as_int(w[0]), 0x101, 0xf, 0xf, false));
        lv = has_left ? lv : 0.0f;
        rv = has_right ? rv : 0.0f;
      } else {
        // tile 2j: columns lv, w0, w1, w2; tile 2j + 1: w1, w2, w3, rv
        const float u0[4] = {lv - w[1], w[0] + w[1], w[1] - w[0], w[0] - w[2]};
        const float u1[4] = {w[1] - w[3], w[2] + w[3], w[3] - w[2], w[2] - rv};
#pragma unroll
        for (int e = 2 * (q - 2); e < 2 * (q - 2) + 2; ++e) {
          // the upper lanes' (channel 1) tile 2j against the lower lanes' tile 2j + 1
          const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(uint32_t, u0[e]),
                                                           __builtin_bit_cast(uint32_t, u1[e]), false, false);
          v[0][rr * 4 + e] = __builtin_bit_cast(float, uint32_t(sw[0]));
          v[1][rr * 4 + e] = __builtin_bit_cast(float, uint32_t(sw[1]));
        }
      }
    }
  };
  constexpr int TPARTS = 11;                      // 3 rows, then 4 parts for each of the two xi1

  // Split element e and write it to buffer b, in three parts so that they can
  // stand between the products: k = 0 h, 1 m, 2 l.
  uint32_t sm;
  float sr[2];
  auto put = [&](int b, int e, int k) {
    uint32_t w;
    if (k == 0) {
      const uint32_t u0 = __builtin_bit_cast(uint32_t, v[0][e]), u1 = __builtin_bit_cast(uint32_t, v[1][e]);
      w = __builtin_amdgcn_perm(u1, u0, 0x07060302);
      sr[0] = v[0][e] - __builtin_bit_cast(float, u0 & 0xffff0000u);
      sr[1] = v[1][e] - __builtin_bit_cast(float, u1 & 0xffff0000u);
    } else if (k == 1) {
      w = sm = pack_bf16(sr[0], sr[1]);
    } else {
      w = pack_bf16(sr[0] - __builtin_bit_cast(float, sm << 16), sr[1] - __builtin_bit_cast(float, sm & 0xffff0000u));
    }
    *reinterpret_cast<uint32_t*>(pw + b * BUF + (e * 3 + k) * PLANE) = w;
  };

  // ---- consuming
  // B planes P[xi][stage * 2 + half][3][K_pad]: uniform base + lane offset
  const int64_t pstep = int64_t(6) * g.K_pad;                       // a stage, in 16-byte words
  const u32x4* const pblk = P + (int64_t(wave) * nstage) * pstep + kb * KB;
  const uint32_t plane_off = (uint32_t(half) * 3u * uint32_t(g.K_pad) + uint32_t(col)) * 16u;
  int bp = s0 / nstage, bst = s0 % nstage;        // B cursor
  bf16x8 B[2][3];
  auto load_b = [&](int jb) {
    const char* src = reinterpret_cast<const char*>(pblk + (int64_t(bp) * G::E * nstage + bst) * pstep);
#pragma unroll
    for (int s = 0; s < 3; ++s)
      B[jb][s] = *reinterpret_cast<const bf16x8*>(src + int64_t(s) * g.K_pad * 16 + plane_off + jb * 512);
  };
  auto next_b = [&]() {
    const bool wrap = bst + 1 == nstage, last = bp + 1 == G::NPASS;
    bst = wrap ? (last ? bst : 0) : bst + 1;
    bp += wrap && !last ? 1 : 0;
  };
  const char* const ar = lds + wave * 3 * PLANE + half * 1024 + col * 16;

  f32x16 acc[2][2];                               // [tile half][kernel half]
#pragma unroll
  for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = f32x16{};
  float yacc[NOUT][POS];
#pragma unroll
  for (int o = 0; o < NOUT; ++o)
#pragma unroll
    for (int p = 0; p < POS; ++p) yacc[o][p] = 0.0f;
  const MatRef<Which::AT, true, MM, R> AT{nullptr};

  // end of a pass: one kernel half after the other meets in the exchange
  // region; slot 4i + q of a wave's half holds rows 8q + 4 half + 0..3 of tile
  // half i; thread (w, lane) finishes slot w of both halves
  auto epilogue = [&](int p) {
    // A^T's columns of the pass: xi0 over o0, xi1 = 2 (p % 2) + {0, 1} over o1
    const float c00 = kSplitAT.at[0][p >> 1], c01 = kSplitAT.at[1][p >> 1];
    float c1[2][MM];
#pragma unroll
    for (int rr = 0; rr < 2; ++rr)
#pragma unroll
      for (int o = 0; o < MM; ++o) c1[rr][o] = kSplitAT.at[o][2 * (p & 1) + rr];
    float* const ex = reinterpret_cast<float*>(lds + EX);
#pragma unroll
    for (int jb = 0; jb < 2; ++jb) {
      if (jb == 1) stage_barrier();               // round 0's reads are done
      float* mine = ex + wave * 2048 + lane * 4;
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int qq = 0; qq < 4; ++qq) {
          const f32x16& c = acc[i][jb];
          *reinterpret_cast<f32x4*>(mine + (i * 4 + qq) * 256) =
              f32x4{c[4 * qq], c[4 * qq + 1], c[4 * qq + 2], c[4 * qq + 3]};
        }
      acc[0][jb] = f32x16{};
      acc[1][jb] = f32x16{};
      stage_barrier();
      const float* theirs = ex + wave * 256 + lane * 4;
      f32x4 m4[G::E];
#pragma unroll
      for (int e = 0; e < G::E; ++e) m4[e] = *reinterpret_cast<const f32x4*>(theirs + e * 2048);
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float rv[2][MM];
#pragma unroll
        for (int rr = 0; rr < 2; ++rr) {
          float t[G::A];
#pragma unroll
          for (int e = 0; e < G::A; ++e) t[e] = m4[rr * G::A + e][k];
#pragma unroll
          for (int ol = 0; ol < MM; ++ol) rv[rr][ol] = dot_row<G::A>(AT, ol, t, 1);
        }
#pragma unroll
        for (int o1 = 0; o1 < MM; ++o1)
#pragma unroll
          for (int ol = 0; ol < MM; ++ol) {
            const float t = __builtin_fmaf(c1[1][o1], rv[1][ol], c1[0][o1] * rv[0][ol]);
            float& y0 = yacc[o1 * MM + ol][jb * 4 + k];
            float& y1 = yacc[NLEAD + o1 * MM + ol][jb * 4 + k];
            y0 = __builtin_fmaf(c00, t, y0);
            y1 = __builtin_fmaf(c01, t, y1);
          }
      }
    }
  };

  if (s0 < s1) {
    int cp = lp, cst = lst;                       // step being multiplied
    int pp = lp, pst = lst;                       // step being produced
    auto next_p = [&]() {
      const bool wrap = pst + 1 == nstage;
      pst = wrap ? 0 : pst + 1;
      pp += wrap ? 1 : 0;
    };
    rows(lp);
    load_x();
    next_x();
    load_b(0);
    load_b(1);
    next_b();
    static_for<TPARTS>([&](auto K) { transform(pp, K); });
    next_p();
    load_x();
    next_x();
#pragma unroll
    for (int m = 0; m < 3 * G::E; ++m) put(0, m / 3, m % 3);
    stage_barrier();
    // A step is one straight run of code: the loads and the producing of the
    // steps past the last one run too (on the last step's operands, into the
    // buffer nobody reads), so that the products and the producing interleave
    // and every wait counts exactly the loads behind it.
#pragma unroll 1
    for (int s = s0; s < s1; ++s) {
      const int cur = (s - s0) & 1;
      bf16x8 A[2][3];
      const char* src = ar + cur * BUF;
#pragma unroll
      for (int sp = 2; sp >= 0; --sp)
#pragma unroll
        for (int i = 0; i < 2; ++i) A[i][sp] = *reinterpret_cast<const bf16x8*>(src + sp * PLANE + i * 512);
      // 24 products, the small terms first (registers 0, 1, 2 = h, m, l), with
      // the next step's producing between them: a part of the transform behind
      // each of the first, two thirds of an element's split behind each of the
      // others.  The fences keep them so.
      constexpr int SA[6] = {2, 0, 1, 1, 0, 0}, SB[6] = {0, 2, 1, 0, 1, 0};
      static_assert(TPARTS == 11 && 3 * G::E == 2 * 12, "parts behind the products");
      static_for<24>([&](auto M) {
        constexpr int m = decltype(M)::value, jb = m / 12, p = m % 12 / 2, i = m % 2;
        acc[i][jb] = mfma_bf16(A[i][SA[p]], B[jb][SB[p]], acc[i][jb]);
        if constexpr (m < TPARTS) {
          transform(pp, M);
          if constexpr (m < 3) load_row(m);
        } else if constexpr (m > 11) {
          put(cur ^ 1, (2 * (m - 12)) / 3, (2 * (m - 12)) % 3);
          put(cur ^ 1, (2 * (m - 12) + 1) / 3, (2 * (m - 12) + 1) % 3);
        }
        if constexpr (m % 12 == 11) load_b(jb);
        __builtin_amdgcn_sched_barrier(0);
      });
      next_b();
      next_p();
      stage_barrier();
      next_x();
      if (++cst == nstage || s + 1 == s1) {
        epilogue(cp);
        cst = 0;
        ++cp;
      }
    }
  }

  // row r of a 32-tile half is its tile 2 (r % 16) + r / 16
  const int r0 = 8 * (wave & 3) + 4 * half;
  const int tl0 = 32 * (wave >> 2) + 2 * (r0 & 15) + (r0 >> 4);
  split_finish<N, MM, POOL>(
      yacc, [&](int p) { return tl0 + 2 * (p & 3); }, [&](int p) { return 32 * (p >> 2) + col; },
      reinterpret_cast<float*>(lds), y, g, tb, kb, tail ? g.part + pslot * NOUT * (TB * KB) : nullptr);
}

}  // namespace wino
