// Integer-only network layers on gfx950 int8 MFMA (Sec. 3.3, Eq. 13-14):
//   * gather-GEMM for the 3x3x3 submanifold convolutions (indexed linear
//     transforms over a kernel map), the stride-2 child convolution of the
//     re-densification (Eq. 4) and dense linear layers;
//   * upsampling + pruning (Eq. 6/9/11): Linear(C+8 -> 8C) + PReLU per parent,
//     only occupied child slots are written, in Morton order;
//   * the occupancy embedding;
//   * the predictor (Eq. 7) fused with the integer softmax (Eq. 15) and the
//     16-bit frequency table that drives the range coder.
// The products run on v_mfma_i32_16x16x64_i8, weights as rows; int32
// accumulation is exact, so any summation order gives the same result.
#include "lpcc_internal.h"

namespace lpcc {

// Lane layout of v_mfma_i32_16x16x64_i8 used throughout: A lane l holds row
// l%16, 16 consecutive k of group l/16; B lane l holds column l%16, the same
// k; the accumulator lane l holds rows 4(l/16)+i (i = 0..3) of column l%16.

__device__ __forceinline__ v4i ld16(const int8_t* p) { return *(const GAS v4i*)p; }

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// N int8 values (N a multiple of 4; p aligned to 4 N bytes up to 16) as one
// vector access of N/4 32-bit words
template <int N>
struct Words;
template <>
struct Words<4> { typedef int T __attribute__((ext_vector_type(1))); };
template <>
struct Words<8> { typedef int T __attribute__((ext_vector_type(2))); };
template <>
struct Words<16> { typedef int T __attribute__((ext_vector_type(4))); };

// Workgroups are dispatched round-robin over the 8 XCDs (block b on XCD
// b % 8), each with its own L2.  Tile t of a launch goes to the block that
// gives every XCD one contiguous run of tiles: neighbouring tiles (close in
// Morton order, sharing most of their 3x3x3 neighbours) then hit one L2.
constexpr int kXcds = 8;
__device__ __forceinline__ int xcd_tile() {
  const int G = (int)gridDim.x, b = (int)blockIdx.x;
  const int q = G / kXcds, rem = G % kXcds, x = b % kXcds;
  return x * q + min(x, rem) + b / kXcds;
}

// The block's segment, layer and first row: from the kernel arguments for a
// single-segment launch, else from the tile and segment arrays.
__device__ __forceinline__ int pick_seg(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                        const GemmArg& A, GemmSeg& S, LayerDev& L, int tile_rows = 64) {
  const int t = xcd_tile();
  if (A.one) {
    S = A.seg;
    L = A.L;
    return t * tile_rows;
  }
  const Tile tl = tiles[t];
  S = segs[tl.seg];
  L = load_layer(S.L);
  return tl.row0;
}

// ---------------------------------------------------------------------------
// All sparse and dense layers of width C form their products transposed: the
// weights are the MFMA row operand, the gathered rows its columns.  The row
// order of the packed weights (out_channel) leaves lane (r, g) with the C/4
// consecutive channels C/4 g .. of ONE output row, r, so a lane requantises
// and writes its share of the row directly, whole vectors at a time, with no
// LDS stage, and the biases start in the accumulators.
//
// FL is the launch's flavour: F_FAST: requant_top serves every
// segment, no input zero points; F_GENERAL: any requantisation, no input zero
// points; F_ANY: anything.  Absent inputs must contribute nothing, also with a
// zero point z (Eq. 13: present inputs contribute (q - z) W).  Their rows are
// gathered as zeros, or as z with F_ANY, and then every row's sum over the taps
// the wave multiplies is too large by z times those taps' weights, one number
// per channel (zc), not per row.
// ---------------------------------------------------------------------------
enum { F_GENERAL = 0, F_FAST = 1, F_ANY = 2 };

template <bool TOP>
__device__ __forceinline__ uint32_t pack4(int y0, int y1, int y2, int y3) {  // low or top bytes
  const uint32_t lo = __builtin_amdgcn_perm((uint32_t)y1, (uint32_t)y0, TOP ? 0x0C0C0703u : 0x0C0C0400u);
  const uint32_t hi = __builtin_amdgcn_perm((uint32_t)y3, (uint32_t)y2, TOP ? 0x0C0C0703u : 0x0C0C0400u);
  return lo | (hi << 16);
}

// C/4 bytes of a row
template <int C>
struct RowPart {
  typedef typename Words<C / 4>::T T;
};

// Buffer descriptor of `bytes` bytes at p (below 2^31, wave-uniform): loads
// past the end return 0 and touch no memory, which is how absent rows are
// gathered.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void* p, int64_t bytes) {
  const uint64_t a = (uint64_t)p;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
  const int n = __builtin_amdgcn_readfirstlane((int)bytes);
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), 0, n, 0x00027000);
}
// offset past the end of every descriptor
constexpr uint32_t kNoRow = 0x80000000u;
// byte offset of row `row` of width C in an array below 2^31 bytes, kNoRow for -1
template <int C>
__device__ __forceinline__ uint32_t row_off(int row) {
  return min((uint32_t)row, kNoRow / (uint32_t)C) * (uint32_t)C;
}
// F_ANY: 16 bytes from channel c of row `row` of an array of any size; zs for
// an absent row (-1), 0 for padding (-2)
template <int C>
__device__ __forceinline__ v4i any_row(const int8_t* in, int row, uint32_t c, int zs) {
  v4i x = ld16(in + (int64_t)max(row, 0) * C + c);
  const int f = row == -1 ? zs : 0;
#pragma unroll
  for (int q = 0; q < 4; q++) x[q] = row >= 0 ? x[q] : f;
  return x;
}

// Epilogue of one row block: the row's share of this lane, requantised, the
// residual (when res is given) added and clamped.
template <int C, int FL, bool PRELU>
__device__ __forceinline__ typename RowPart<C>::T row_out(const v4i (&acc)[C / 16], const LayerDev& L, bool has_res,
                                                          typename RowPart<C>::T res) {
  typename RowPart<C>::T w;
#pragma unroll
  for (int nb = 0; nb < C / 16; nb++) {
    int y[4];
#pragma unroll
    for (int i = 0; i < 4; i++)
      y[i] = FL == F_FAST ? requant_top<PRELU>(acc[nb][i], L) : requant_l(acc[nb][i], L);
    if (has_res) {
#pragma unroll
      for (int i = 0; i < 4; i++) {
        if (FL == F_FAST) {  // the scaled sum saturates where the int8 one does
          y[i] = __builtin_elementwise_add_sat(y[i], (int)((uint32_t)res[nb] << (24 - 8 * i) & 0xFF000000u));
        } else {
          y[i] += (int)(int8_t)((uint32_t)res[nb] >> (8 * i));
          y[i] = min(max(y[i], -128), 127);
        }
      }
    }
    w[nb] = (int)pack4<FL == F_FAST>(y[0], y[1], y[2], y[3]);
  }
  return w;
}

// Accumulators of a lane's channels, started with bias (+ extra).
template <int C>
__device__ __forceinline__ void acc_bias(v4i (&acc)[C / 16], const int32_t* bias, int g) {
#pragma unroll
  for (int nb = 0; nb < C / 16; nb++) acc[nb] = *(const GAS v4i*)(bias + C / 4 * g + 4 * nb);
}

// ---------------------------------------------------------------------------
// 3x3x3 submanifold convolution over the present taps only, and dense layers:
// out[row] = rq(bias + sum_t in[kmap[t][row]] W[t]) (+ resid), in = one array
// (CIN = C) or two side by side (CIN = 2 C: [in | in2]).
//
// A wave owns 16 RB output rows.  Every row has a mask of its present taps
// (stored after the 27 tap rows); the OR over the wave's rows lists the taps
// the wave multiplies, in rank order (the tap of rank i sits in lane i of a
// register, read with readlane); a tap that no row has costs nothing.  The
// table rows of the present taps are staged straight from global memory into
// LDS.  A step is one MFMA depth (64): 64 / C taps (one for C = 64) of one
// input array.  Steps are software-pipelined: the gathers and weights of step
// v + 1 are in flight behind the products of step v, and the table rows of the
// step after are read ahead of them.
//
// Bound: the 64 bytes per clock between a CU and its L1.  Gathers and weights
// take half each (4 KB per 64 rows and 64 of K); the texture units are busy
// 97 % of the time, the matrix cores 27 %.  The 7.0 M rows of 8 128-beam
// frames' deep depths, 128 -> 64 channels: 1.13 ms; 1.52 ms with the gathered
// rows as the row operand, the accumulators staged through LDS, the 64-bit
// requantisation and selects that zeroed absent rows and weights (2640 vector
// instructions per wave of 64 rows).  With the weights in LDS instead (one
// block of 16 waves per CU) the CU cycles fall by a quarter, but the launches
// end unevenly and the calls gain nothing.
// ---------------------------------------------------------------------------
template <int MODE>
struct Taps;
template <>
struct Taps<G_CONV> { static constexpr int n = 27; };
template <>
struct Taps<G_DENSE> { static constexpr int n = 1; };

template <int MODE, int CIN, int C, int RB, int FL>
__global__ __launch_bounds__(256) void k_conv(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                              const GemmArg A) {
  constexpr int TAPS = Taps<MODE>::n;
  constexpr int NB = C / 16;
  constexpr int NA = CIN / C;     // input arrays
  constexpr int TPS = 64 / C;     // taps per step
  constexpr int WR = 16 * RB;     // rows per wave
  static_assert((CIN == C || CIN == 2 * C) && (C == 16 || C == 32 || C == 64) && WR <= 64, "shape");
  __shared__ int32_t skm_all[MODE == G_CONV ? 4 * 28 * WR : 1];

  GemmSeg S;
  LayerDev L;
  const int tile_row0 = pick_seg(segs, tiles, A, S, L, 4 * WR);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int wrow0 = tile_row0 + wave * WR;
  int32_t* skm = skm_all + (MODE == G_CONV ? wave * 28 * WR : 0);  // [rank][WR], one rank of padding

  // the union of the rows' taps, and lane i: the tap of rank i
  const int myrow = wrow0 + lane;
  uint32_t U = MODE == G_DENSE ? 1u : 0u;
  int tapof = 0;
  if (MODE == G_CONV) {
    if (lane < WR && myrow < S.rows) U = (uint32_t)gp(S.kmap)[27 * S.kstride + myrow];
    if (A.all) U = (1u << 27) - 1u;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) U |= (uint32_t)__shfl_xor((int)U, o);
    U = (uint32_t)__builtin_amdgcn_readfirstlane((int)U);
  }
  const int nt = __popc(U);
  if (MODE == G_CONV) {
    // the owner of each set bit sends its tap to the lane of its rank
    const bool own = lane < TAPS && ((U >> (lane & 31)) & 1u);
    const int rk = __popc(U & ((1u << (lane & 31)) - 1u));
    const int got = __builtin_amdgcn_ds_permute((own ? rk : 63) * 4, lane);
    tapof = lane < nt ? got : 0;
    // table rows of the present taps, straight into LDS (rows past the end
    // read the last row; they are never written out)
    const int crow = min(myrow, S.rows - 1);
    uint32_t rem = U;
    if (lane < WR) {
      for (int i = 0; i < nt; i++) {
        const int t = __builtin_ctz(rem);
        rem &= rem - 1u;
        __builtin_amdgcn_global_load_lds((const GAS void*)(gp(S.kmap) + (int64_t)t * S.kstride + crow),
                                         (__attribute__((address_space(3))) void*)(skm + i * WR), 4, 0, 0);
      }
    }
  }

  // accumulators: biases, with zero points the correction of the wave's taps
  v4i acc[RB][NB];
  acc_bias<C>(acc[0], L.bias, g);
  if (MODE == G_CONV && FL == F_ANY && L.zc != nullptr) {
    for (int i = 0; i < nt; i++) {
      const int32_t* z = L.zc + (int64_t)__builtin_amdgcn_readlane(tapof, i) * L.npad;
      v4i zz[NB];
      acc_bias<C>(zz, z, g);
#pragma unroll
      for (int nb = 0; nb < NB; nb++) acc[0][nb] += zz[nb];
    }
  }
#pragma unroll
  for (int rb = 1; rb < RB; rb++)
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[rb][nb] = acc[0][nb];
  const int zs = FL == F_ANY ? (L.z_in & 0xFF) * 0x01010101 : 0;

  // a dense layer's descriptors cover the wave's rows alone
  const int dbase = MODE == G_DENSE ? min(wrow0, S.rows) : 0;
  const int64_t in_bytes = (int64_t)(MODE == G_DENSE ? min(S.rows - dbase, WR) : S.rows) * C;
  const __amdgpu_buffer_rsrc_t b1 = rsrc_of(S.in + (int64_t)dbase * C, in_bytes);
  const __amdgpu_buffer_rsrc_t b2 = rsrc_of((NA == 2 ? S.in2 : S.in) + (int64_t)dbase * C, in_bytes);
  const uint32_t c0 = (uint32_t)((16 * g) & (C - 1));  // first channel of this lane's slice
  const int kt = (16 * g) / C;                         // this lane's tap within the step (0 for C = 64)
  const int ng = (nt + TPS - 1) / TPS;                 // groups of TPS taps
  const int KV = ng * NA;

  if (MODE == G_CONV) __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the staged rows have landed
  wave_lds_sync();

  // byte offsets of this lane's source rows for tap group i (kNoRow for absent
  // rows and taps past the last); F_ANY: the rows (-1, -2)
  auto rows_of = [&](int i, uint32_t (&o)[RB]) {
    const int slot = min(i * TPS + kt, 27);
    const bool tv = i * TPS + kt < nt;
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      int row = MODE == G_CONV ? skm[slot * WR + 16 * rb + r] : 16 * rb + r;
      row = tv ? row : (FL == F_ANY ? -2 : -1);
      o[rb] = FL == F_ANY ? (uint32_t)row : row_off<C>(row);
    }
  };
  // this lane's weights of step (i, h): rows k = tap CIN + h C + c of the
  // packed layout
  auto weights = [&](int i, int h, v4i (&w)[NB]) {
    if (C == 64) {
      const int tap = MODE == G_CONV ? __builtin_amdgcn_readlane(tapof, min(i, 63)) : 0;
      const GAS int8_t* p = gp(L.Wp) + (int64_t)(tap * NA + h) * (NB * 1024) + 16 * (uint32_t)lane;
#pragma unroll
      for (int nb = 0; nb < NB; nb++) w[nb] = *(const GAS v4i*)(p + 1024 * nb);
    } else {
      int tap = 0;
      if (MODE == G_CONV) {
        const int base = min(i * TPS, 60);
        tap = __builtin_amdgcn_readlane(tapof, base);
#pragma unroll
        for (int q = 1; q < TPS; q++) {
          const int tq = __builtin_amdgcn_readlane(tapof, base + q);
          tap = kt == q ? tq : tap;
        }
      }
      const int k = tap * CIN + h * C + (int)c0;
      const GAS int8_t* p = gp(L.Wp) + (int64_t)(k >> 6) * (NB * 1024) + (((k >> 4) & 3) * 16 + r) * 16;
#pragma unroll
      for (int nb = 0; nb < NB; nb++) w[nb] = *(const GAS v4i*)(p + 1024 * nb);
    }
  };
  auto gather = [&](int h, const uint32_t (&o)[RB], v4i (&x)[RB]) {
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      if (FL == F_ANY) x[rb] = any_row<C>(h == 0 ? S.in : S.in2, (int)o[rb], c0, zs);
      else x[rb] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(h == 0 ? b1 : b2, o[rb] + c0, 0, 0);
    }
  };

  // two steps per iteration (for two arrays: both arrays of one tap group;
  // else two groups), each loading the next one's operands first
  uint32_t o0[RB], o1[RB];
  v4i x0[RB], x1[RB], w0[NB], w1[NB];
  auto mul = [&](const v4i (&x)[RB], const v4i (&w)[NB]) {
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++) acc[rb][nb] = mfma16(w[nb], x[rb], acc[rb][nb]);
  };
  rows_of(0, o0);
  weights(0, 0, w0);
  gather(0, o0, x0);
  for (int v = 0; v < KV; v += 2) {
    if (NA == 2) {
      weights(v / 2, 1, w1);
      gather(1, o0, x1);
      rows_of(v / 2 + 1, o0);
      mul(x0, w0);
      weights(v / 2 + 1, 0, w0);
      gather(0, o0, x0);
      mul(x1, w1);
    } else {
      rows_of(v + 1, o1);
      weights(v + 1, 0, w1);
      gather(0, o1, x1);
      mul(x0, w0);
      rows_of(v + 2, o0);
      weights(v + 2, 0, w0);
      gather(0, o0, x0);
      mul(x1, w1);
    }
  }

  typedef typename RowPart<C>::T P;
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
    const int row = wrow0 + 16 * rb + r;
    if (row >= S.rows) continue;
    const int64_t at = (int64_t)row * C + C / 4 * g;
    P res;
    if (S.resid != nullptr) res = *(const GAS P*)(gp(S.resid) + at);
    const P w = S.resid != nullptr ? row_out<C, FL, false>(acc[rb], L, true, res)
                                   : row_out<C, FL, false>(acc[rb], L, false, res);
    *(GAS P*)(gp(S.out) + at) = w;
  }
}

// The same convolution for launches of few rows: a block owns 16 RB rows and
// its four waves share the taps (tap groups w, w + 4, ...; every tap, present
// or not), so the serial chain of gathers is a quarter as long and the chip
// has four times the waves.  The partial sums meet in LDS.
template <int CIN, int C, int RB, int FL>
__global__ __launch_bounds__(256) void k_conv_split(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                                    const GemmArg A) {
  constexpr int NB = C / 16;
  constexpr int NA = CIN / C;
  constexpr int TPS = 64 / C;
  constexpr int WR = 16 * RB;
  constexpr int NG = (27 + TPS - 1) / TPS;   // groups of TPS taps
  constexpr int GW = (NG + 3) / 4;           // groups per wave
  static_assert((CIN == C || CIN == 2 * C) && (C == 16 || C == 32 || C == 64), "shape");
  __shared__ v4i part[3][RB][NB][64];

  GemmSeg S;
  LayerDev L;
  const int row0 = pick_seg(segs, tiles, A, S, L, WR);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const uint32_t c0 = (uint32_t)((16 * g) & (C - 1));
  const int kt = (16 * g) / C;
  const int zs = FL == F_ANY ? (L.z_in & 0xFF) * 0x01010101 : 0;
  const int64_t in_bytes = (int64_t)S.rows * C;
  const __amdgpu_buffer_rsrc_t b1 = rsrc_of(S.in, in_bytes);
  const __amdgpu_buffer_rsrc_t b2 = rsrc_of(NA == 2 ? S.in2 : S.in, in_bytes);

  // source rows of all the wave's groups first (one round trip)
  uint32_t o[GW][RB];
#pragma unroll
  for (int q = 0; q < GW; q++) {
    const int tap = (wave + 4 * q) * TPS + kt;
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      const int row = row0 + 16 * rb + r;
      const int src = tap < 27 && row < S.rows ? gp(S.kmap)[(int64_t)tap * S.kstride + row] : (tap < 27 ? -1 : -2);
      o[q][rb] = FL == F_ANY ? (uint32_t)src : row_off<C>(src);
    }
  }
  v4i acc[RB][NB];
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[rb][nb] = v4i{0, 0, 0, 0};
    if (wave == 0) acc_bias<C>(acc[rb], FL == F_ANY ? L.biasz : L.bias, g);
  }
#pragma unroll
  for (int q = 0; q < GW; q++) {
    const int tap = min((wave + 4 * q) * TPS + kt, 26);
#pragma unroll
    for (int h = 0; h < NA; h++) {
      const int k = tap * CIN + h * C + (int)c0;
      const GAS int8_t* p = gp(L.Wp) + (int64_t)(k >> 6) * (NB * 1024) + (((k >> 4) & 3) * 16 + r) * 16;
      v4i w[NB];
#pragma unroll
      for (int nb = 0; nb < NB; nb++) w[nb] = *(const GAS v4i*)(p + 1024 * nb);
#pragma unroll
      for (int rb = 0; rb < RB; rb++) {
        v4i x;
        if (FL == F_ANY) x = any_row<C>(h == 0 ? S.in : S.in2, (int)o[q][rb], c0, zs);
        else x = (v4i)__builtin_amdgcn_raw_buffer_load_b128(h == 0 ? b1 : b2, o[q][rb] + c0, 0, 0);
#pragma unroll
        for (int nb = 0; nb < NB; nb++) acc[rb][nb] = mfma16(w[nb], x, acc[rb][nb]);
      }
    }
  }
  if (wave > 0) {
#pragma unroll
    for (int rb = 0; rb < RB; rb++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++) part[wave - 1][rb][nb][lane] = acc[rb][nb];
  }
  __syncthreads();
  if (wave > 0) return;
  typedef typename RowPart<C>::T P;
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int w = 0; w < 3; w++) acc[rb][nb] += part[w][rb][nb][lane];
    const int row = row0 + 16 * rb + r;
    if (row >= S.rows) continue;
    const int64_t at = (int64_t)row * C + C / 4 * g;
    P res;
    if (S.resid != nullptr) res = *(const GAS P*)(gp(S.resid) + at);
    const P w = S.resid != nullptr ? row_out<C, FL, false>(acc[rb], L, true, res)
                                   : row_out<C, FL, false>(acc[rb], L, false, res);
    *(GAS P*)(gp(S.out) + at) = w;
  }
}

// ---------------------------------------------------------------------------
// Child convolution (the stride-2 step of the re-densification, Eq. 4):
// out[q] = rq(b + sum over children c of q of in[c] W[slot(c)]).  With `ccode`
// set, child c reads row ccode[c] of `in`: the occupancy embedding of depth j
// depends on the code alone, so the first step reads a 256-row table.
//
// A wave keeps the whole layer (8 slots: 8 C^2 bytes, 128 registers at C = 64)
// and takes 16 parents at a time, one per column, over all eight slots: an
// absent child is gathered as zeros, at no memory cost.  The zeros cost matrix
// cycles (1.1 to 2 of 8 slots are occupied; 512 cycles per 16 parents at C =
// 64), but no compaction, no LDS and no atomics.  The weights leave two waves
// per SIMD, so the gathers are pipelined: a slot's row of the next tile is
// requested as soon as the slot's products have read this one's, and codes,
// child positions and table rows are read one and two tiles further ahead.
//
// 14 M parents (8 128-beam frames, 18 levels, C = 64): 0.85 ms, against 1.70
// ms when a tile's gathers were issued together after the products (latency:
// 32 % of the vector issue slots and 20 % of the matrix cycles used).  Bound
// now: the texture units, busy 97 % of the time with the gathers.  Two tiles of
// gathers in flight, the children through LDS, and the weights in LDS with
// four waves per SIMD were each no faster end to end.
// ---------------------------------------------------------------------------
template <int C, int FL, bool TABLE>
__global__ __launch_bounds__(256, 2) void k_down(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                                 const GemmArg A) {
  constexpr int NB = C / 16;
  constexpr int SPS = 64 / C;       // slots per step
  constexpr int KS = 8 / SPS;       // steps
  static_assert(C == 16 || C == 32 || C == 64, "C");
  GemmSeg S;
  LayerDev L;
  const int q0 = pick_seg(segs, tiles, A, S, L, 64 * A.tpw);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const uint32_t c0 = (uint32_t)((16 * g) & (C - 1));
  const int kt = (16 * g) / C;      // this lane's slot within a step
  const int wrow0 = q0 + wave * 16 * A.tpw;
  const int nrow = min(S.rows - wrow0, 16 * A.tpw);
  if (nrow <= 0) return;            // wave-uniform, no barrier below
  // the children of consecutive parents are consecutive rows: descriptors of
  // the wave's parents and children alone (at most 8 per parent; children past
  // the depth in a corrupt stream are past the end)
  const int cbase = min(__builtin_amdgcn_readfirstlane(gp(S.cstart)[wrow0]), S.child_rows);
  const int crows = min(S.child_rows - cbase, 8 * nrow);
  const __amdgpu_buffer_rsrc_t bin =
      TABLE ? rsrc_of(S.in, 256 * C) : rsrc_of(S.in + (int64_t)cbase * C, (int64_t)crows * C);
  const __amdgpu_buffer_rsrc_t bcc = rsrc_of(TABLE ? S.ccode + cbase : S.code, TABLE ? crows : 0);
  const __amdgpu_buffer_rsrc_t bcode = rsrc_of(S.code + wrow0, nrow);
  const __amdgpu_buffer_rsrc_t bcst = rsrc_of(S.cstart + wrow0, 4ll * nrow);
  const int zs = FL == F_ANY ? (L.z_in & 0xFF) * 0x01010101 : 0;

  v4i w[KS][NB], bias[NB];
  {
    const GAS int8_t* p = gp(L.Wp) + 16 * (uint32_t)lane;
#pragma unroll
    for (int s = 0; s < KS; s++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++) w[s][nb] = *(const GAS v4i*)(p + 1024 * (s * NB + nb));
  }
  acc_bias<C>(bias, FL == F_ANY ? L.biasz : L.bias, g);

  // code (0 past the wave's rows) and first child of column r of tile t
  auto parent = [&](int t, uint32_t& code, uint32_t& first) {
    const uint32_t q = (uint32_t)(16 * t + r);
    code = (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(bcode, q, 0, 0);
    first = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(bcst, 4 * q, 0, 0);
  };
  // by step: the lane's child (row index times `scale`, plus c), kNoRow added
  // where it is absent
  auto absent = [&](uint32_t code, int s) { return (~code << (31 - s * SPS - kt)) & kNoRow; };
  auto children = [&](uint32_t code, uint32_t first, uint32_t scale, uint32_t c, uint32_t (&o)[KS]) {
    uint32_t at = (first - (uint32_t)cbase) * scale + c;
    if (SPS > 1) at += (uint32_t)__popc(code & ((1u << kt) - 1u)) * scale;
#pragma unroll
    for (int s = 0; s < KS; s++) {
      o[s] = at | absent(code, s);
      const uint32_t next = code >> (s * SPS + kt);  // bits of the slots passed on the way to the next step
      at += (SPS == 1 ? next & 1u : (uint32_t)__popc(next & ((1u << SPS) - 1u))) * scale;
    }
  };
  auto row = [&](uint32_t o) { return (v4i)__builtin_amdgcn_raw_buffer_load_b128(bin, o, 0, 0); };

  // code0: tile t, code1 / first1: tile t + 1, code2 / first2: t + 2 (TABLE
  // alone), e: table rows of tile t + 1 (in flight)
  uint32_t code0, code1, code2, first0, first1, first2, o[KS], e[KS];
  v4i x[KS];
  auto table_rows = [&](uint32_t code, uint32_t first) {
    uint32_t ce[KS];
    children(code, first, 1u, 0u, ce);
#pragma unroll
    for (int s = 0; s < KS; s++) e[s] = (uint32_t)(uint8_t)__builtin_amdgcn_raw_buffer_load_b8(bcc, ce[s], 0, 0);
  };
  auto offsets = [&](uint32_t code, uint32_t first) {
    if (TABLE) {
#pragma unroll
      for (int s = 0; s < KS; s++) o[s] = (e[s] * (uint32_t)C + c0) | absent(code, s);
    } else {
      children(code, first, (uint32_t)C, c0, o);
    }
  };
  parent(0, code0, first0);
  parent(1, code1, first1);
  if (TABLE) {
    parent(2, code2, first2);
    table_rows(code0, first0);
  }
  offsets(code0, first0);
#pragma unroll
  for (int s = 0; s < KS; s++) x[s] = row(o[s]);
  if (TABLE) table_rows(code1, first1);

  typedef typename RowPart<C>::T P;
  const int nt = (nrow + 15) >> 4;
  for (int t = 0; t < nt; t++) {
    offsets(code1, first1);
    uint32_t code, first;
    if (TABLE) {
      table_rows(code2, first2);
      parent(t + 3, code, first);
    } else {
      parent(t + 2, code, first);
    }
    v4i acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[nb] = bias[nb];
#pragma unroll
    for (int s = 0; s < KS; s++) {
      if (FL == F_ANY) {
#pragma unroll
        for (int z = 0; z < 4; z++) x[s][z] = absent(code0, s) ? zs : x[s][z];
      }
#pragma unroll
      for (int nb = 0; nb < NB; nb++) acc[nb] = mfma16(w[s][nb], x[s], acc[nb]);
      x[s] = row(o[s]);
      __builtin_amdgcn_sched_barrier(0);  // else the gathers sink below all the products
    }
    code0 = code1;
    if (TABLE) {
      code1 = code2;
      first1 = first2;
      code2 = code;
      first2 = first;
    } else {
      code1 = code;
      first1 = first;
    }
    if (16 * t + r < nrow) {
      P none;
      *(GAS P*)(gp(S.out) + (int64_t)(wrow0 + 16 * t + r) * C + C / 4 * g) = row_out<C, FL, false>(acc, L, false, none);
    }
  }
}

// flavour of a launch's layers
#define LPCC_FL(K, ...)                                                                                    \
  if (A.fl == F_FAST) hipLaunchKernelGGL((K<__VA_ARGS__, F_FAST>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A); \
  else if (A.fl == F_ANY) hipLaunchKernelGGL((K<__VA_ARGS__, F_ANY>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A); \
  else hipLaunchKernelGGL((K<__VA_ARGS__, F_GENERAL>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);      \
  return hipGetLastError();

hipError_t launch_conv(int cin, int cout, const GemmSeg* segs, const Tile* tiles, int ntiles, const GemmArg& A, int rb,
                       hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
#define LPCC_C(CI, CO)                                                     \
  if (cin == CI && cout == CO) {                                           \
    if (rb == 4) { LPCC_FL(k_conv, G_CONV, CI, CO, 4) }                    \
    if (rb == 2) { LPCC_FL(k_conv, G_CONV, CI, CO, 2) }                    \
    LPCC_FL(k_conv, G_CONV, CI, CO, 1)                                     \
  }
  LPCC_C(16, 16) LPCC_C(32, 16) LPCC_C(32, 32) LPCC_C(64, 32) LPCC_C(64, 64) LPCC_C(128, 64)
#undef LPCC_C
  return hipErrorInvalidValue;
}

hipError_t launch_conv_split(int cin, int cout, const GemmSeg* segs, const Tile* tiles, int ntiles, const GemmArg& A,
                             int rb, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
#define LPCC_C(CI, CO)                                                     \
  if (cin == CI && cout == CO) {                                           \
    if (rb == 4) { LPCC_FL(k_conv_split, CI, CO, 4) }                      \
    if (rb == 2) { LPCC_FL(k_conv_split, CI, CO, 2) }                      \
    LPCC_FL(k_conv_split, CI, CO, 1)                                       \
  }
  LPCC_C(16, 16) LPCC_C(32, 16) LPCC_C(32, 32) LPCC_C(64, 32) LPCC_C(64, 64) LPCC_C(128, 64)
#undef LPCC_C
  return hipErrorInvalidValue;
}

hipError_t launch_dense(int cin, int cout, const GemmSeg* segs, const Tile* tiles, int ntiles, const GemmArg& A,
                        int rb, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  // a dense layer's zero point is in its bias
#define LPCC_C(CI, CO, R)                                                                                       \
  if (cin == CI && cout == CO && rb == R) {                                                                     \
    if (A.fl == F_FAST)                                                                                         \
      hipLaunchKernelGGL((k_conv<G_DENSE, CI, CO, R, F_FAST>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);  \
    else                                                                                                        \
      hipLaunchKernelGGL((k_conv<G_DENSE, CI, CO, R, F_GENERAL>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A); \
    return hipGetLastError();                                                                                   \
  }
  LPCC_C(32, 16, 1) LPCC_C(32, 16, 2) LPCC_C(32, 16, 4) LPCC_C(64, 32, 1) LPCC_C(64, 32, 2) LPCC_C(64, 32, 4)
  LPCC_C(128, 64, 1) LPCC_C(128, 64, 2) LPCC_C(128, 64, 4)
#undef LPCC_C
  return hipErrorInvalidValue;
}

hipError_t launch_down(int C, const GemmSeg* segs, const Tile* tiles, int ntiles, const GemmArg& A, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
#define LPCC_D(CC)                                                                                          \
  if (C == CC) {                                                                                            \
    if (A.table) {                                                                                          \
      if (A.fl == F_FAST)                                                                                   \
        hipLaunchKernelGGL((k_down<CC, F_FAST, true>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);      \
      else if (A.fl == F_ANY)                                                                               \
        hipLaunchKernelGGL((k_down<CC, F_ANY, true>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);       \
      else                                                                                                  \
        hipLaunchKernelGGL((k_down<CC, F_GENERAL, true>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);   \
    } else {                                                                                                \
      if (A.fl == F_FAST)                                                                                   \
        hipLaunchKernelGGL((k_down<CC, F_FAST, false>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);     \
      else if (A.fl == F_ANY)                                                                               \
        hipLaunchKernelGGL((k_down<CC, F_ANY, false>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);      \
      else                                                                                                  \
        hipLaunchKernelGGL((k_down<CC, F_GENERAL, false>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);  \
    }                                                                                                       \
    return hipGetLastError();                                                                               \
  }
  LPCC_D(16) LPCC_D(32) LPCC_D(64)
#undef LPCC_D
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Upsampling + pruning: per parent p, A = [Z[p] (C) | bits(X[p]) (8)],
// out block o (columns oC..oC+C-1) is child slot o; occupied slots only,
// child row = cstart[p] + rank of o among the set bits.
//
// Two forms: every slot of every parent (small launches), and the occupied
// children only.
// ---------------------------------------------------------------------------
__device__ __forceinline__ v4i occupancy(uint32_t code) {  // bits as int8 {0, 127}
  uint32_t w0 = 0, w1 = 0;
#pragma unroll
  for (int b = 0; b < 4; b++) {
    if ((code >> b) & 1u) w0 |= 127u << (8 * b);
    if ((code >> (b + 4)) & 1u) w1 |= 127u << (8 * b);
  }
  return v4i{(int)w0, (int)w1, 0, 0};
}

template <int C, int RB, int FL>
__global__ __launch_bounds__(256) void k_up(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                            const GemmArg A) {
  constexpr int KS = (C + 8 + 63) / 64;
  constexpr int NBS = C / 16;          // column blocks per child slot
  constexpr int NBT = 8 * NBS;         // column blocks of the layer
  constexpr int WR = 16 * RB;          // parent rows per wave
  static_assert(C % 16 == 0, "C");

  GemmSeg S;
  LayerDev L;
  const int tile_row0 = pick_seg(segs, tiles, A, S, L, 4 * WR);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int wrow0 = tile_row0 + wave * WR;
  // lane (r, g) serves parent row wrow0 + 16 rb + r
  uint32_t code[RB];
  int first[RB];
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
    const int row = wrow0 + 16 * rb + r;
    code[rb] = row < S.rows ? gp(S.code)[row] : 0u;
    first[rb] = row < S.rows ? gp(S.cstart)[row] : 0;
  }

  // column operand: k-slice 16g..16g+15 of the parent's input row
  v4i a[RB][KS];
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
    const int row = wrow0 + 16 * rb + r;
    const bool rv = row < S.rows;
#pragma unroll
    for (int s = 0; s < KS; s++) {
      const int k0 = 64 * s + 16 * g;
      a[rb][s] = v4i{0, 0, 0, 0};
      if (rv && k0 < C) {
        a[rb][s] = ld16(S.in + (int64_t)row * C + k0);
      } else if (rv && k0 == C) {  // occupancy bits as int8 {0,127}, then zeros
        a[rb][s] = occupancy(code[rb]);
      }
    }
  }
  const GAS v4i* Wp = (const GAS v4i*)L.Wp;
  // weights and biases of slot o+1 are in flight while slot o is computed
  v4i wb[2][KS][NBS], bb[2][NBS];
#pragma unroll
  for (int s = 0; s < KS; s++)
#pragma unroll
    for (int nb = 0; nb < NBS; nb++) wb[0][s][nb] = Wp[((int64_t)s * NBT + nb) * 64 + lane];
  acc_bias<C>(bb[0], L.bias, g);

#pragma unroll
  for (int o = 0; o < 8; o++) {
    if (o + 1 < 8) {
#pragma unroll
      for (int s = 0; s < KS; s++)
#pragma unroll
        for (int nb = 0; nb < NBS; nb++)
          wb[(o + 1) & 1][s][nb] = Wp[((int64_t)s * NBT + (o + 1) * NBS + nb) * 64 + lane];
      acc_bias<C>(bb[(o + 1) & 1], L.bias + (o + 1) * C, g);
    }
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      const bool has = (code[rb] >> o) & 1u;
      if (__ballot(has) == 0ull) continue;  // no parent of the block has child o
      v4i acc[NBS];
#pragma unroll
      for (int nb = 0; nb < NBS; nb++) acc[nb] = bb[o & 1][nb];
#pragma unroll
      for (int s = 0; s < KS; s++)
#pragma unroll
        for (int nb = 0; nb < NBS; nb++) acc[nb] = mfma16(wb[o & 1][s][nb], a[rb][s], acc[nb]);
      if (!has) continue;
      const int crow = first[rb] + __popc(code[rb] & ((1u << o) - 1u));
      if (crow >= S.child_rows) continue;  // only for a corrupt stream
      typedef typename RowPart<C>::T P;
      P none;
      *(GAS P*)(gp(S.out) + (int64_t)crow * C + C / 4 * g) = row_out<C, FL, true>(acc, L, false, none);
    }
  }
}

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {  // set bits of m below this lane
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Upsampling + pruning over the occupied children only.  A block takes a range
// of 64 A.tpw consecutive parents, and each of its eight waves ONE child slot
// of it: the wave loads the slot's weights once, scans the parents' codes,
// lists those that have the child in a list of its own (by ballots), and
// multiplies the list in groups of 16: the weights are the row operand, the
// parents' inputs [Z | bits(X)] the columns, and a lane writes its C/4 channels
// of one child.  No barrier: the waves share nothing but the caches (the same
// parents' rows, and the two halves of an output line).  A list entry holds
// all a group needs: the parent (10 bits), its code (8) and the child's row
// relative to the batch's first child (14; padding and children out of range
// have the largest value, which is past the end of every output descriptor).
// The inputs of three groups are in flight behind the products, and the codes
// of the next batch (1024 parents) behind a batch's groups.
//
// Bound: memory and vector issue together (64-byte rows read and written: 1.1 ms
// of the figure below without the arithmetic, 0.9 ms without the reads or
// without the writes).  The 28 M children of 8 128-beam frames (18 levels, C =
// 64) take 1.38 ms; a block's waves sharing one list of all slots, built
// between barriers, with the weights reloaded at each change of slot, took 1.69
// ms.  Tiles of 512 / 1024 / 2048 parents: 1.39 / 1.38 / 1.38 ms, and 1.44 /
// 1.46 / 1.57 ms in the smaller launches of a decode of the same frames; tiles
// of 256 are for launches that would leave compute units idle.  With the tiles
// in use, 256 and 1024, the loop over batches runs once.  It stays because the
// kernel without it is slower: half the registers at C = 32, so four blocks
// instead of two share a compute unit's caches, 0.86 -> 0.89 ms for the
// encode of 8 such frames and 0.297 -> 0.317 ms for 32 uneven ones (0.303 ms
// with the waves held at four per SIMD).
constexpr uint32_t kNoChild = 0x3FFFu << 18;
constexpr int kUpBatch = 1024;

template <int C, int FL>
__global__ __launch_bounds__(512, 4) void k_up_slots(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                                     const GemmArg A) {
  constexpr int KS = (C + 8 + 63) / 64;
  constexpr int NBS = C / 16;          // column blocks per child slot
  constexpr int NBT = 8 * NBS;         // column blocks of the layer
  constexpr int Q = kUpBatch / 256;    // lane l holds parents 256 q + 4 l .. + 3
  static_assert(C == 16 || C == 32 || C == 64, "C");
  __shared__ uint32_t lists[8][kUpBatch + 16];

  GemmSeg S;
  LayerDev L;
  int p0 = pick_seg(segs, tiles, A, S, L, 64 * A.tpw);
  const int o = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int pend = min(S.rows, p0 + 64 * A.tpw);
  uint32_t* list = lists[o];

  v4i wb[KS][NBS], bb[NBS];
  {
    const GAS v4i* w = (const GAS v4i*)L.Wp + (int64_t)o * NBS * 64 + lane;
#pragma unroll
    for (int s = 0; s < KS; s++)
#pragma unroll
      for (int nb = 0; nb < NBS; nb++) wb[s][nb] = w[(s * NBT + nb) * 64];
    acc_bias<C>(bb, L.bias + o * C, g);
  }
  // codes and first children of the lane's parents of the batch at p (the
  // arrays are readable to a multiple of 16 bytes past a depth's last row)
  uint32_t code[Q];
  v4i first[Q];
  auto parents = [&](int p) {
    const int np = min(pend - p, kUpBatch);
    const __amdgpu_buffer_rsrc_t bcode = rsrc_of(S.code + p, (np + 3) & ~3);
    const __amdgpu_buffer_rsrc_t bcst = rsrc_of(S.cstart + p, 4ll * ((np + 3) & ~3));
#pragma unroll
    for (int q = 0; q < Q; q++) {
      const uint32_t t = 256u * q + 4u * lane;
      code[q] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b32(bcode, t, 0, 0);
      first[q] = (v4i)__builtin_amdgcn_raw_buffer_load_b128(bcst, 4 * t, 0, 0);
    }
  };
  // lanes of the input row's channels, and the lane with the occupancy bits
  const uint32_t c0 = 16 * g < C ? 16u * g : kNoRow;
  const uint32_t om = g == (C & 63) / 16 ? 0xFFu : 0u;
  const uint32_t st0 = (uint32_t)(C / 4 * g);
  const uint32_t below = (1u << o) - 1u;

  parents(p0);
  for (; p0 < pend; p0 += kUpBatch) {
    const int np = min(pend - p0, kUpBatch);
    const int cfirst = __builtin_amdgcn_readfirstlane(first[0][0]);
    const int cbase = min(max(cfirst, 0), S.child_rows);
    const __amdgpu_buffer_rsrc_t bin = rsrc_of(S.in + (int64_t)p0 * C, (int64_t)np * C);
    const __amdgpu_buffer_rsrc_t bout =
        rsrc_of(S.out + (int64_t)cbase * C, (int64_t)min(S.child_rows - cbase, 8 * kUpBatch) * C);
    int n = 0;
#pragma unroll
    for (int q = 0; q < Q; q++) {
      if (256 * q >= np) break;
      const int left = np - (256 * q + 4 * lane);  // parents of this lane inside the batch
      const uint32_t cw = left >= 4 ? code[q] : (left <= 0 ? 0u : code[q] & ((1u << (8 * left)) - 1u));
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const uint32_t cd = (cw >> (8 * i)) & 0xFFu;
        const bool has = (cd >> o) & 1u;
        const uint64_t m = __ballot(has);
        const uint32_t at = (uint32_t)(first[q][i] - cbase) + (uint32_t)__popc(cd & below);
        if (has) list[n + (int)lanes_below(m)] = (256u * q + 4u * lane + i) | (cd << 10) | (min(at, 0x3FFFu) << 18);
        n += __popcll(m);
      }
    }
    if (lane < 16) list[n + lane] = kNoChild;
    wave_lds_sync();
    if (p0 + kUpBatch < pend) parents(p0 + kUpBatch);
    const int G = (n + 15) >> 4;
    if (G == 0) continue;

    auto entry = [&](int gi) { return list[16 * min(gi, G - 1) + r]; };
    auto row = [&](uint32_t e) {
      return (v4i)__builtin_amdgcn_raw_buffer_load_b128(bin, (e & 0x3FFu) * (uint32_t)C + c0, 0, 0);
    };
    auto group = [&](uint32_t e, const v4i& x) {
      // occupancy bits as int8 {0, 127}
      const uint32_t cd = (e >> 10) & om;
      const uint32_t lo = __builtin_amdgcn_perm(0u, 0x7F00u, __umul24(cd & 15u, 0x204081u) & 0x01010101u);
      const uint32_t hi = __builtin_amdgcn_perm(0u, 0x7F00u, __umul24(cd >> 4, 0x204081u) & 0x01010101u);
      v4i acc[NBS];
#pragma unroll
      for (int nb = 0; nb < NBS; nb++) {
        if (KS == 1) {
          acc[nb] = mfma16(wb[0][nb], v4i{x[0] | (int)lo, x[1] | (int)hi, x[2], x[3]}, bb[nb]);
        } else {
          acc[nb] = mfma16(wb[KS - 1][nb], v4i{(int)lo, (int)hi, 0, 0}, bb[nb]);
          acc[nb] = mfma16(wb[0][nb], x, acc[nb]);
        }
      }
      typedef typename RowPart<C>::T T;
      T none;
      const T y = row_out<C, FL, true>(acc, L, false, none);
      const uint32_t at = (e >> 18) * (uint32_t)C + st0;
      if constexpr (C == 64) __builtin_amdgcn_raw_buffer_store_b128(y, bout, at, 0, 0);
      else if constexpr (C == 32) __builtin_amdgcn_raw_buffer_store_b64(y, bout, at, 0, 0);
      else __builtin_amdgcn_raw_buffer_store_b32(y[0], bout, at, 0, 0);
    };
    uint32_t e[3], en;
    v4i x[3];
#pragma unroll
    for (int k = 0; k < 3; k++) e[k] = entry(k);
#pragma unroll
    for (int k = 0; k < 3; k++) {
      x[k] = row(e[k]);
      __builtin_amdgcn_sched_barrier(0);  // in the order of use
    }
    int gi = 0;
    for (; gi + 3 <= G; gi += 3) {
#pragma unroll
      for (int k = 0; k < 3; k++) {
        en = entry(gi + k + 3);
        group(e[k], x[k]);
        e[k] = en;
        x[k] = row(en);
        __builtin_amdgcn_sched_barrier(0);  // else the loads sink below the next group
      }
    }
    if (gi < G) group(e[0], x[0]);
    if (gi + 1 < G) group(e[1], x[1]);
    wave_lds_sync();  // the list is written again
  }
}

hipError_t launch_up_slots(int C, const GemmSeg* segs, const Tile* tiles, int ntiles, const GemmArg& A,
                           hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
#define LPCC_U(CC)                                                                                            \
  if (C == CC) {                                                                                              \
    if (A.fl == F_FAST)                                                                                       \
      hipLaunchKernelGGL((k_up_slots<CC, F_FAST>), dim3(ntiles), dim3(512), 0, s, segs, tiles, A);            \
    else                                                                                                      \
      hipLaunchKernelGGL((k_up_slots<CC, F_GENERAL>), dim3(ntiles), dim3(512), 0, s, segs, tiles, A);         \
    return hipGetLastError();                                                                                 \
  }
  LPCC_U(16) LPCC_U(32) LPCC_U(64)
#undef LPCC_U
  return hipErrorInvalidValue;
}

hipError_t launch_up(int C, const GemmSeg* segs, const Tile* tiles, int ntiles, const GemmArg& A, int rb,
                     hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
#define LPCC_U(CC, RR)                                                                                        \
  if (C == CC && rb == RR) {                                                                                  \
    if (A.fl == F_FAST)                                                                                       \
      hipLaunchKernelGGL((k_up<CC, RR, F_FAST>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);              \
    else                                                                                                      \
      hipLaunchKernelGGL((k_up<CC, RR, F_GENERAL>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);           \
    return hipGetLastError();                                                                                 \
  }
  LPCC_U(16, 1) LPCC_U(16, 2) LPCC_U(16, 4) LPCC_U(32, 1) LPCC_U(32, 2) LPCC_U(32, 4)
  LPCC_U(64, 1) LPCC_U(64, 2) LPCC_U(64, 4)
#undef LPCC_U
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Occupancy embedding (first step of the re-densification, Eq. 4): 8 int8
// channels {0,127} from the code bits, Linear(8 -> C), ReLU requantisation.
// One thread per output element.  Tiles cover 64 rows.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_emb(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                             int C, const GemmArg A) {
  GemmSeg S;
  LayerDev L;
  const int tile_row0 = pick_seg(segs, tiles, A, S, L);
  const int cs = __builtin_ctz((unsigned)C);  // C is a power of two dividing 256
  // a thread keeps one output channel o for every row it writes, so its
  // weights and bias are loaded once; the codes of all its rows (at most 16)
  // are loaded together before any is used
  const int o = threadIdx.x & (C - 1);
  const int rstep = 256 >> cs, nrow = 64 >> (8 - cs);  // rows per pass, rows per thread
  int w[8];
#pragma unroll
  for (int b = 0; b < 8; b++) w[b] = 127 * (int)gp(L.Wr)[b * C + o];
  const int bias = gp(L.bias)[o];
  uint32_t code[16];
#pragma unroll
  for (int k = 0; k < 16; k++) {
    const int row = tile_row0 + (threadIdx.x >> cs) + k * rstep;
    code[k] = (k < nrow && row < S.rows) ? (S.code != nullptr ? (uint32_t)gp(S.code)[row] : (uint32_t)row) : 0u;
  }
#pragma unroll
  for (int k = 0; k < 16; k++) {
    const int row = tile_row0 + (threadIdx.x >> cs) + k * rstep;
    if (k >= nrow || row >= S.rows) continue;
    int acc = bias;
#pragma unroll
    for (int b = 0; b < 8; b++) acc += ((code[k] >> b) & 1u) ? w[b] : 0;
    gp(S.out)[(int64_t)row * C + o] = (int8_t)requant_l(acc, L);
  }
}

// The same for launches of many rows: a block computes the 256 possible rows
// once, into LDS, and copies one per code, 16 bytes per thread.  It pays from
// about a thousand rows per block (computed, a row costs 14 instructions per
// channel).  The launches of 8 128-beam frames (C = 64): 28 us in the decode and
// 39 us in the encode, 98 and 100 us computed row by row.
template <int C>
__global__ __launch_bounds__(256) void k_emb_rows(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                                  const GemmArg A) {
  constexpr int U = C / 16;  // 16-byte units per row
  __shared__ v4i tab[256 * U];
  GemmSeg S;
  LayerDev L;
  const int row0 = pick_seg(segs, tiles, A, S, L, kEmbRows);
  const int o = threadIdx.x & (C - 1);
  int w[8];
#pragma unroll
  for (int b = 0; b < 8; b++) w[b] = 127 * (int)gp(L.Wr)[b * C + o];
  const int bias = gp(L.bias)[o];
  for (int c = threadIdx.x / C; c < 256; c += 256 / C) {
    int acc = bias;
#pragma unroll
    for (int b = 0; b < 8; b++) acc += ((c >> b) & 1) ? w[b] : 0;
    ((int8_t*)tab)[c * C + o] = (int8_t)requant_l(acc, L);
  }
  __syncthreads();
  const int n = min(S.rows - row0, kEmbRows) * U;
  const GAS uint8_t* code = gp(S.code) + row0;
  GAS v4i* out = (GAS v4i*)(gp(S.out) + (int64_t)row0 * C);
#pragma unroll 4
  for (int i = threadIdx.x; i < n; i += 256) out[i] = tab[(int)code[i / U] * U + i % U];
}

hipError_t launch_emb_rows(const GemmSeg* segs, const Tile* tiles, int ntiles, int C, const GemmArg& A,
                           hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  if (C == 16) hipLaunchKernelGGL(k_emb_rows<16>, dim3(ntiles), dim3(256), 0, s, segs, tiles, A);
  else if (C == 32) hipLaunchKernelGGL(k_emb_rows<32>, dim3(ntiles), dim3(256), 0, s, segs, tiles, A);
  else if (C == 64) hipLaunchKernelGGL(k_emb_rows<64>, dim3(ntiles), dim3(256), 0, s, segs, tiles, A);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_emb(const GemmSeg* segs, const Tile* tiles, int ntiles, int C, const GemmArg& A, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_emb, dim3(ntiles), dim3(256), 0, s, segs, tiles, C, A);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Predictor + integer softmax + frequency table.
//   h = relu-rq(F W1 + b1)            (C -> C)
//   l = rq(h W2 + b2)                 (C -> 255 int8 logits)
//   M = max l, E_i = LUT[M - l_i], S = sum E_i
//   f_i = 1 + floor(E_i * 65281 / S), the remainder 65536 - sum f goes to the
//   lowest index holding M;  cdf[s] = sum_{i<s} f_i.
//
// Both products are formed transposed (weights as the MFMA row operand, nodes
// as columns), and the row order of the logit weights is permuted on the host
// (logit_symbol, logit_channel), so that lane (r, g) ends with the 64
// consecutive symbols 64g .. 64g + 63 of ONE node, r.  Everything per node (M,
// S, the reciprocal, the coded symbol) is then a per-lane value: the reductions run over the 4
// lanes of a node, the prefix sums are serial inside a lane, and the biases
// ride in the accumulators.  fc1's accumulators are already fc2's column
// operand (the permutation of K is in the packed weights), so no activations
// pass through LDS.
//
// The kernel is bound by vector instruction issue: this form needs 17.2
// vector instructions per 64 logits in encode mode where the one with 16 lanes
// per node needed 30.4, and for the 12.75 M nodes of 8 128-beam frames (18
// levels, C = 64) it takes 1.40 ms where that took 2.39 ms.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t recip_k(uint32_t S) {  // floor(65281 * 2^16 / S), 2^15 <= S < 2^23
  uint32_t rem = 65281u << 16;  // < 2^32
  uint32_t q = 0;
#pragma unroll
  for (int b = 16; b >= 0; b--) {
    // rem >= S 2^b  <=>  floor(rem / 2^b) >= S; then S 2^b <= rem fits 32 bits
    if ((rem >> b) >= S) {
      rem -= S << b;
      q |= 1u << b;
    }
  }
  return q;
}

// run + f with f = 1 + floor(E * 65281 / S) for E <= 2^15 (a table entry), S <
// 2^23 and K = floor(65281 2^16 / S) < 2^17.  floor(E K / 2^16) is the
// quotient or one below it (E K / 2^16 is at most E / 2^16 <= 1/2 below E
// 65281 / S), so with q1 = floor(E K / 2^16) + 1 the quotient is q1 exactly
// when q1 S <= E 65281.  The +1 rides in the product's addend: E K + 2^16 <
// 2^32 because E K <= 2^15 floor(65281 2^16 / 2^15) = 2^32 - 255 2^16, and q1
// S <= E 65281 + S < 2^32.  All unsigned (E K reaches 2^31 once S <= 65281: a
// confident head, one dominant logit).
// Five full-rate instructions: the high half of the product is read in place
// by its two users (sub-dword source selects), which the compiler does only
// for a single user, and it forms the multiply-add with the quarter-rate
// 64-bit one.  No matrix instruction is in flight here (the maximum over all
// logits comes first).  The compare's VCC may be read as a carry only two wait
// states later, and the compiler does not look inside the asm.  An s_nop costs
// the least where four waves per SIMD fill the issue slots: the encoder's
// predictor takes 1.40 ms for 8 128-beam frames, 1.43 ms with the next entry's
// instructions in between (freq_next).
__device__ __forceinline__ uint32_t freq_mad(uint32_t E, uint32_t K) {
  uint32_t m;
  asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(m) : "v"(E), "v"(K), "s"(0x10000));
  return m;
}
__device__ __forceinline__ uint32_t freq_mul(uint32_t m, uint32_t S) {
  uint32_t t;
  asm("v_mul_u32_u24_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD"
      : "=v"(t)
      : "v"(m), "v"(S));
  return t;
}
__device__ __forceinline__ uint32_t freq_end(uint32_t run, uint32_t m, uint32_t t, uint32_t p) {
  uint32_t o;
  asm("v_cmp_le_u32_e32 vcc, %1, %2\n\t"
      "s_nop 1\n\t"
      "v_addc_co_u32_sdwa %0, vcc, %3, %4, vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
      : "=v"(o)
      : "v"(t), "v"(p), "v"(run), "v"(m)
      : "vcc");
  return o;
}
__device__ __forceinline__ uint32_t freq_prod(uint32_t E) { return __umul24(E & 0xFFFFu, 65281u); }
__device__ __forceinline__ uint32_t freq_add(uint32_t run, uint32_t E, uint32_t S, uint32_t K) {
  const uint32_t m = freq_mad(E, K);
  return freq_end(run, m, freq_mul(m, S), freq_prod(E));
}

// The same over consecutive entries, with the next entry's products in between:
// 2.86 ms for the decoder of 8 128-beam frames, three waves per SIMD, 2.91 ms
// with the s_nop.
struct FreqStep {
  uint32_t m, t, p;  // of the next entry: E K + 2^16 (q1 in its high half), q1 S, E 65281
};
__device__ __forceinline__ FreqStep freq_begin(uint32_t E, uint32_t S, uint32_t K) {
  const uint32_t m = freq_mad(E, K);
  return FreqStep{m, freq_mul(m, S), freq_prod(E)};
}
// run + f of the entry begun in s; begins the entry E1 in s
__device__ __forceinline__ uint32_t freq_next(uint32_t run, FreqStep& s, uint32_t E1, uint32_t S, uint32_t K) {
  FreqStep n;
  uint32_t o;
  asm("v_cmp_le_u32_e32 vcc, %4, %5\n\t"
      "v_mad_u32_u24 %1, %6, %7, %8\n\t"
      "v_mul_u32_u24_e32 %3, %9, %6\n\t"
      "v_mul_u32_u24_sdwa %2, %1, %10 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD\n\t"
      "v_addc_co_u32_sdwa %0, vcc, %11, %12, vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
      : "=v"(o), "=&v"(n.m), "=&v"(n.t), "=&v"(n.p)
      : "v"(s.t), "v"(s.p), "v"(E1), "v"(K), "s"(0x10000), "s"(65281), "v"(S), "v"(run), "v"(s.m)
      : "vcc");
  s = n;
  return o;
}

// Reductions over the lanes of a node.  Both forms join the four lane groups
// g (16 lanes apart: gfx950's row and half swaps hand every lane its partner's
// value); the small form first joins the quad of lanes that share a node.
template <int CTRL>
__device__ __forceinline__ int dpp_mov(int v) {
  return __builtin_amdgcn_mov_dpp(v, CTRL, 0xF, 0xF, false);
}
template <bool SMALL, class Op>
__device__ __forceinline__ int node_reduce(int v, Op op) {
  if (SMALL) {
    v = op(v, dpp_mov<0xB1>(v));  // quad_perm(1, 0, 3, 2)
    v = op(v, dpp_mov<0x4E>(v));  // quad_perm(2, 3, 0, 1)
  }
  auto a = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
  v = op((int)a[0], (int)a[1]);
  a = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
  return op((int)a[0], (int)a[1]);
}
// sum of v over the lanes of the node that hold smaller symbols
template <bool SMALL>
__device__ __forceinline__ uint32_t node_before(uint32_t v, int lane) {
  uint32_t off = 0, sum = v;
  if (SMALL) {  // lanes of the quad below this one
    const int q = lane & 3;
    const uint32_t v0 = (uint32_t)dpp_mov<0x00>((int)v), v1 = (uint32_t)dpp_mov<0x55>((int)v);
    const uint32_t v2 = (uint32_t)dpp_mov<0xAA>((int)v), v3 = (uint32_t)dpp_mov<0xFF>((int)v);
    off = (q > 0 ? v0 : 0u) + (q > 1 ? v1 : 0u) + (q > 2 ? v2 : 0u);
    sum = v0 + v1 + v2 + v3;
  }
  auto a = __builtin_amdgcn_permlane16_swap(sum, sum, false, false);
  off += (lane & 16) ? (uint32_t)a[0] : 0u;
  sum = (uint32_t)a[0] + (uint32_t)a[1];
  a = __builtin_amdgcn_permlane32_swap(sum, sum, false, false);
  return off + ((lane & 32) ? (uint32_t)a[0] : 0u);
}

// Per-node results of the logits, held by each of the node's lanes.
struct NodeSum {
  uint32_t S, K;  // sum of the table entries, floor(65281 2^16 / S)
  int aord, ablk;  // lane (in the node's order) and block of 4 of the first maximum
  int ord;         // this lane's place among its node's lanes
  bool tail;       // this lane's last entry is 255, which is no symbol
};

// Table entries e[j] of this lane's NS symbols, from the column operand x
// (channels 16g .. 16g + 15 of the node).  w1(k), w2(k): this lane's packed
// weights of block k (from LDS or global memory), b1, b2: biases.
template <int C, bool SMALL, int RQ, class W1, class W2>
__device__ __forceinline__ void predict_table(W1 w1, W2 w2, const int32_t* b1, const int32_t* b2, const uint16_t* lut,
                                              const v4i x, int lane, const LayerDev& L1, const LayerDev& L2,
                                              int (&e)[SMALL ? 16 : 64], NodeSum& n) {
  constexpr int NB1 = C / 16;
  constexpr int NS = SMALL ? 16 : 64;  // symbols per lane
  constexpr int NBL = NS / 4;          // blocks of 4 symbols per lane
  constexpr int LPN = SMALL ? 16 : 4;  // lanes per node
  const int g = lane >> 4, q = lane & 3;
  n.ord = SMALL ? 4 * g + q : g;
  n.tail = n.ord == LPN - 1;
  // fc1: byte 4 nb + i of lane (r, g) is channel 16 nb + 4 g + i
  v4i h = v4i{0, 0, 0, 0};
#pragma unroll
  for (int nb = 0; nb < NB1; nb++) {
    const v4i acc = mfma16(w1(nb), x, *(const v4i*)&b1[16 * nb + 4 * g]);
    uint32_t w = 0;
#pragma unroll
    for (int i = 0; i < 4; i++) {
      const int y = RQ == 1 ? requant_f(acc[i], L1) : requant_l(acc[i], L1);
      w |= ((uint32_t)y & 0xFFu) << (8 * i);
    }
    h[nb] = (int)w;
  }
  // fc2: accumulator register i of block b is symbol 64 g + 4 b + i
  if (SMALL) {
#pragma unroll
    for (int b = 0; b < 16; b++) {
      const v4i acc = mfma16(w2(b), h, *(const v4i*)&b2[64 * g + 4 * b]);
#pragma unroll
      for (int i = 0; i < 4; i++) e[(4 * b + i) % NS] = b < 4 || q == b / 4 ? acc[i] : e[(4 * b + i) % NS];
      if (b % 4 == 3) __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < NS; j++) e[j] = RQ == 1 ? requant_f(e[j], L2) : requant_l(e[j], L2);
  } else {
    // the weights of the next two blocks are in flight while two are
    // multiplied; the scheduling barriers keep all loads from moving to the
    // front (64 registers on top of the 64 logits)
    v4i w[2][2];
#pragma unroll
    for (int k = 0; k < 2; k++) w[0][k] = w2(k);
#pragma unroll
    for (int p = 0; p < 8; p++) {
      if (p < 7) {
#pragma unroll
        for (int k = 0; k < 2; k++) w[(p + 1) & 1][k] = w2(2 * p + 2 + k);
      }
#pragma unroll
      for (int k = 0; k < 2; k++) {
        const int b = 2 * p + k;
        const v4i acc = mfma16(w[p & 1][k], h, *(const v4i*)&b2[64 * g + 4 * b]);
#pragma unroll
        for (int i = 0; i < 4; i++) e[(4 * b + i) % NS] = RQ == 1 ? requant_f(acc[i], L2) : requant_l(acc[i], L2);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // entry 255 is no symbol: the lowest logit at the highest index never
  // holds the maximum first, and its table entry is taken as 0
  if (n.tail) e[NS - 1] = -128;
  // maximum and the first block of 4 that holds it: 16 M + (15 - block),
  // then over the node's lanes 256 M + 16 (15 - lane) + (15 - block)
  int key = -(1 << 20);
#pragma unroll
  for (int b = 0; b < NBL; b++) {
    const int mb = max(max(max(e[4 * b], e[4 * b + 1]), e[4 * b + 2]), e[4 * b + 3]);
    key = max(key, mb * 16 + (15 - b));
  }
  key = ((key >> 4) << 8) | ((15 - n.ord) << 4) | (key & 15);
  key = node_reduce<SMALL>(key, [](int a, int b) { return max(a, b); });
  const int M = key >> 8;
  n.aord = 15 - ((key >> 4) & 15);
  n.ablk = 15 - (key & 15);
  // E = LUT[M - l]: entry at byte 2 M - 2 l from the table's start
  const uint8_t* lb = (const uint8_t*)lut + 2 * M;
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < NS; j++) {
    e[j] = *(const uint16_t*)(lb + __mul24(e[j], -2));
    if (j % 16 == 15) __builtin_amdgcn_sched_barrier(0);
  }
  if (n.tail) e[NS - 1] = 0;
#pragma unroll
  for (int j = 0; j < NS; j++) sum += (uint32_t)e[j];
  n.S = (uint32_t)node_reduce<SMALL>((int)sum, [](int a, int b) { return a + b; });
  n.K = recip_k(n.S);
}

// The CDF row of the node, in place: e[j] becomes the exclusive prefix inside
// the lane; p0 / p1 are the packed offsets of the pairs up to / after the
// block of the first maximum (mod 2^16), R the remainder it takes.
template <bool SMALL>
__device__ __forceinline__ void row_prefix(int (&e)[SMALL ? 16 : 64], const NodeSum& n, int lane, uint32_t& p0,
                                           uint32_t& p1, uint32_t& R) {
  constexpr int NS = SMALL ? 16 : 64;
  uint32_t run = 0;
  FreqStep fs = freq_begin((uint32_t)e[0], n.S, n.K);
#pragma unroll
  for (int j = 0; j < NS; j++) {
    const uint32_t next =
        j + 1 < NS ? freq_next(run, fs, (uint32_t)e[(j + 1) % NS], n.S, n.K) : freq_end(run, fs.m, fs.t, fs.p);
    e[j] = (int)run;
    run = next;
  }
  const uint32_t tot = n.tail ? (uint32_t)e[NS - 1] : run;
  R = 65536u - (uint32_t)node_reduce<SMALL>((int)tot, [](int a, int b) { return a + b; });
  const uint32_t o0 = node_before<SMALL>(tot, lane) + (n.aord < n.ord ? R : 0u);
  const uint32_t o1 = o0 + (n.aord == n.ord ? R : 0u);
  p0 = (o0 & 0xFFFFu) | (o0 << 16);
  p1 = (o1 & 0xFFFFu) | (o1 << 16);
}

// 8 entries of the row (chunk c of this lane's symbols) as 16-bit values;
// entry 255 comes out as 2^16 = 0
template <int NS>
__device__ __forceinline__ v4i row_chunk(const int (&e)[NS], int c, int ablk, uint32_t p0, uint32_t p1) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  v4i w;
#pragma unroll
  for (int k = 0; k < 4; k++) {
    const int j = 8 * c + 2 * k;
    const uint32_t pk = __builtin_amdgcn_perm((uint32_t)e[j + 1], (uint32_t)e[j], 0x05040100u);
    const uint32_t po = j / 4 > ablk ? p1 : p0;
    w[k] = (int)__builtin_bit_cast(uint32_t,
                                   (u16x2)(__builtin_bit_cast(u16x2, pk) + __builtin_bit_cast(u16x2, po)));
  }
  return w;
}

// The block of the first maximum (4 entries at p, not counting R yet): the
// entries after its first one of frequency fmax, the largest, take R (a
// smaller table entry gives a smaller frequency: the table falls by at least
// 1984 of 32768 from entry 0 to 1, and S < 2^23).
__device__ __forceinline__ void row_remainder(uint32_t* p, const NodeSum& n, uint32_t R) {
  const uint32_t fmax = freq_add(0u, 32768u, n.S, n.K) & 0xFFFFu;
  const uint32_t lo = p[0], hi = p[1];
  const uint32_t v0 = lo & 0xFFFFu, v1 = lo >> 16, v2 = hi & 0xFFFFu, v3 = hi >> 16;
  const bool a0 = ((v1 - v0) & 0xFFFFu) == fmax;
  const bool a1 = a0 || ((v2 - v1) & 0xFFFFu) == fmax;
  const bool a2 = a1 || ((v3 - v2) & 0xFFFFu) == fmax;
  p[0] = v0 | ((v1 + (a0 ? R : 0u)) << 16);
  p[1] = ((v2 + (a1 ? R : 0u)) & 0xFFFFu) | ((v3 + (a2 ? R : 0u)) << 16);
}

enum { P_ENCODE = 0, P_CDF32 = 2 };

// SMALL: 4 nodes per wave (columns 4n .. 4n + 3 all hold node n, lane q of
// the quad takes the blocks 4q .. 4q + 3 of its group's 64 symbols: 16 symbols
// per lane, a quarter of the serial work, so short launches finish sooner);
// else 16 nodes per wave and `groups` such groups one after the other, so the
// block's copy of the weights in LDS serves 64 x groups nodes.
template <int C, int MODE, bool SMALL, int RQ>
// at most 128 VGPRs (four waves per SIMD); the general requantisation may take
// more
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(RQ == 1 ? 4 : 3))) void k_predict(
    const PredSeg* __restrict__ segs, const Tile* __restrict__ tiles, const int32_t* __restrict__ lut_g, int groups,
    const PredArg A) {
  constexpr int NB1 = C / 16;
  constexpr int NS = SMALL ? 16 : 64;  // symbols per lane
  constexpr int NBL = NS / 4;          // blocks of 4 symbols per lane
  constexpr int NPW = SMALL ? 4 : 16;  // nodes per wave
  __shared__ uint16_t lut[256];  // E_j = round(2^15 e^(-j/16)) <= 2^15
  __shared__ v4i w2s[16 * 64];
  __shared__ v4i w1s[NB1 * 64];
  __shared__ __attribute__((aligned(16))) int32_t b2s[256];
  __shared__ __attribute__((aligned(16))) int32_t b1s[C];
  // encode: the block of 4 table entries that holds the coded symbol, per
  // lane; CDF rows: half of the symbols of the wave's nodes (NPW rows of 128
  // entries, 16-byte chunks swizzled by the node)
  constexpr int kStage = MODE == P_ENCODE ? 64 : NPW * 16;  // 16-byte units per wave
  __shared__ v4i stage[4][kStage];

  PredSeg S;
  LayerDev L1, L2;
  int tile_row0;
  if (A.one) {
    S = A.seg;
    L1 = A.fc1;
    L2 = A.fc2;
    tile_row0 = (int)blockIdx.x * (SMALL ? 16 : 64 * groups);
  } else {
    const Tile tl = tiles[blockIdx.x];
    S = segs[tl.seg];
    L1 = load_layer(S.fc1);
    L2 = load_layer(S.fc2);
    tile_row0 = tl.row0;
  }
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  {
    const GAS v4i* W1 = (const GAS v4i*)L1.Wp;
    const GAS v4i* W2 = (const GAS v4i*)L2.Wp;
    v4i t[4];
#pragma unroll
    for (int k = 0; k < 4; k++) t[k] = W2[256 * k + tid];
    const v4i u = tid < NB1 * 64 ? W1[tid] : v4i{0, 0, 0, 0};
    b2s[tid] = gp(L2.bias)[tid];
    if (tid < C) b1s[tid] = gp(L1.bias)[tid];
    lut[tid] = (uint16_t)gp(lut_g)[tid];
#pragma unroll
    for (int k = 0; k < 4; k++) w2s[256 * k + tid] = t[k];
    if (tid < NB1 * 64) w1s[tid] = u;
  }
  __syncthreads();

  const int ng = SMALL ? 1 : groups;
  for (int gi = 0; gi < ng; gi++) {
    const int row0 = tile_row0 + gi * 64 + wave * NPW;
    if (row0 >= S.rows) break;  // wave-uniform; no barrier below
    const int row = row0 + (SMALL ? r >> 2 : r);
    const bool rv = row < S.rows;
    v4i x = v4i{0, 0, 0, 0};
    if (rv && 16 * g < C) x = ld16(S.F + (int64_t)row * C + 16 * g);
    int sym = 0;
    if (MODE == P_ENCODE) sym = rv ? max((int)gp(S.code)[row] - 1, 0) : 0;
    int e[NS];
    NodeSum n;
    predict_table<C, SMALL, RQ>([&](int k) { return w1s[k * 64 + lane]; }, [&](int k) { return w2s[k * 64 + lane]; },
                                b1s, b2s, lut, x, lane, L1, L2, e, n);

    if (MODE == P_ENCODE) {
      // start = sum of f below the symbol.  The symbol's lane notes its
      // running sum before the symbol's block of 4 and the block's entries;
      // the lanes before it add their totals.
      const int sord = sym / NS, sblk = n.ord == sord ? (sym % NS) / 4 : -1;
      uint32_t run = 0, runb = 0, rlast = 0;
#pragma unroll
      for (int b = 0; b < NBL; b++) {
        if (b == sblk) {
          runb = run;
          stage[wave][lane] = v4i{e[4 * b], e[4 * b + 1], e[4 * b + 2], e[4 * b + 3]};
        }
#pragma unroll
        for (int i = 0; i < 4; i++) {
          if (4 * b + i == NS - 1) rlast = run;
          run = freq_add(run, (uint32_t)e[4 * b + i], n.S, n.K);
        }
      }
      const uint32_t tot = n.tail ? rlast : run;
      const uint32_t R =
          65536u - (uint32_t)node_reduce<SMALL>((int)tot, [](int a, int b) { return a + b; });
      const uint32_t below = node_before<SMALL>(tot, lane);
      if (n.ord == sord && rv) {
        const v4i es = stage[wave][lane];  // written by this lane
        const int si = sym & 3;
        uint32_t st = below + runb, fr = 0;
        bool lower = false, here = false;  // the maximum lies at a lower entry of the block / at the symbol
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const uint32_t f = freq_add(0u, (uint32_t)es[i], n.S, n.K);
          st += i < si ? f : 0u;
          fr = i == si ? f : fr;
          lower = lower || (i < si && es[i] == 32768);
          here = here || (i == si && es[i] == 32768);
        }
        // the remainder goes to the first maximum: block ablk of lane aord
        const int ab = 16 * n.aord + n.ablk, sb = 16 * sord + sblk;
        const bool lt = ab < sb || (ab == sb && lower);
        st += lt ? R : 0u;
        fr += ab == sb && !lower && here ? R : 0u;
        gp(S.sf)[row] = st | (fr << 16);
      }
    } else {
      uint32_t p0, p1, R;
      row_prefix<SMALL>(e, n, lane, p0, p1, R);
      // rows of all nodes in two passes of half of every lane's symbols
      // (CH 16-byte chunks of 8 entries per lane)
      constexpr int CH = NS / 16;
      const int node = SMALL ? r >> 2 : r;
#pragma unroll
      for (int hf = 0; hf < 2; hf++) {
#pragma unroll
        for (int c = 0; c < CH; c++)
          stage[wave][node * 16 + ((n.ord * CH + c) ^ node)] = row_chunk<NS>(e, hf * CH + c, n.ablk, p0, p1);
        if (n.aord == n.ord && n.ablk / (2 * CH) == hf) {
          const int bl = n.ablk % (2 * CH);
          row_remainder((uint32_t*)&stage[wave][node * 16 + ((n.ord * CH + (bl >> 1)) ^ node)] + 2 * (bl & 1), n, R);
        }
        wave_lds_sync();
        // whole rows out: chunk k of a node's half row is chunk k % CH of lane
        // k / CH, i.e. entries NS (k / CH) + NS/2 hf + 8 (k % CH)
#pragma unroll
        for (int it = 0; it < NPW / 4; it++) {
          const int nn = it * 4 + g, k = r;
          const int nrow = row0 + nn;
          const v4i w = stage[wave][nn * 16 + (k ^ nn)];
          const int at = NS * (k / CH) + NS / 2 * hf + 8 * (k % CH);
          if (nrow < S.rows) {
            GAS v4i* dst = (GAS v4i*)(S.cdf32 + (int64_t)nrow * 256 + at);
            const uint32_t u0 = (uint32_t)w[0], u1 = (uint32_t)w[1], u2 = (uint32_t)w[2], u3 = (uint32_t)w[3];
            dst[0] = v4i{(int)(u0 & 0xFFFFu), (int)(u0 >> 16), (int)(u1 & 0xFFFFu), (int)(u1 >> 16)};
            dst[1] = v4i{(int)(u2 & 0xFFFFu), (int)(u2 >> 16), (int)(u3 & 0xFFFFu),
                         at + 7 == 255 ? 65536 : (int)(u3 >> 16)};
          }
        }
        wave_lds_sync();
      }
    }
  }
}

// ---------------------------------------------------------------------------
// Decoding of one depth: predictor and range decoder in one launch.
//
// A block decodes one chunk.  Wave NP decodes; waves 0 .. NP - 1 predict: in
// step s wave w makes the CDF rows of nodes 16 (s NP + w) .. + 15 and the
// decoder takes the rows of step s - 1, through two halves of a ring in LDS,
// one barrier per step.  The rows (512 bytes per node) so never leave the
// compute unit, and the decoder's serial chain (latency) runs beside the
// predictor's arithmetic (issue), which as two launches took turns: over the
// 18 depths of 8 128-beam frames (12.75 M nodes) 2.28 + 1.92 ms became 2.86
// ms, over the 12 depths of a 16-beam frame 390 us became 245 us.
//
// Range decoder (G. N. N. Martin 1979, as in rc.hip): state code and range,
// r = range >> 16; the symbol is the last s with r cdf[s] <= code, then code
// -= r cdf[s], range = r (cdf[s+1] - cdf[s]).  Lane l of the decoding wave
// holds the boundaries b_j = cdf[4 L + j], j = 0 .. 3, of group L = 63 - l.
// With t = r b - code - 1 (mod 2^32, one 16-bit multiply-add) a boundary
// passed (r b <= code) gives t >= ~code and one not passed t < ~code, both
// increasing in b, so over the group that holds the symbol the largest t_0 ..
// t_3 is the symbol's and the smallest of t_1 .. t_4 (t_4: the next group's
// t_0, from lane l - 1) the next boundary's: code = ~max, range = min - max.
// The group is the first lane whose t_0 passed.  Entry 255, 2^16, is stored as
// 65535, and the missing r is in that lane's addend of t_3.  The state holds
// ~code, which is max itself.  Renormalisation takes 0, 1 or 2 bytes: lane p
// of `win` holds the complement of the four bytes from byte p of the block's
// part of the payload, shifted in below ~code.
// The decoder only notes code, range and lane of every symbol; the wave that
// made the rows counts the boundaries passed (the code's last two bits) before
// it overwrites them two steps later.  It also finds a corrupt stream, one
// where code >= r 2^16 at some symbol (no boundary is above it): what the
// decoder does from there on means nothing, but stays inside its buffers (a
// symbol takes at most 3 bytes, 16 of them stay inside the window).
// ---------------------------------------------------------------------------
constexpr int kRowWords = 132;  // LDS row: 256 entries of 16 bits, padded against bank conflicts

__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

struct RcDec {
  uint32_t nc, range, pos;  // ~code, range, payload bytes taken from the window's start
};

// One symbol from the group's boundaries x = b_0 | b_1 << 16, y = b_2 | b_3 <<
// 16; returns the lane of its group.
// last: 1 in the lane of group 63, else 0.
__device__ __forceinline__ int rc_symbol(RcDec& d, uint32_t x, uint32_t y, uint32_t win, uint32_t last) {
  const uint32_t nc = d.nc;
  uint32_t t0, t1, t2, t3, n3;
  // the high half of the range times the low or high half of x, y; t0 first:
  // its cross-lane use needs two instructions in between
  asm("v_mad_u32_u16 %0, %5, %7, %8 op_sel:[0,1,0,0]\n\t"
      "v_mad_u32_u16 %4, %9, %7, %8 op_sel:[0,1,0,0]\n\t"
      "v_mad_u32_u16 %1, %5, %7, %8 op_sel:[1,1,0,0]\n\t"
      "v_mad_u32_u16 %2, %6, %7, %8 op_sel:[0,1,0,0]\n\t"
      "v_mad_u32_u16 %3, %6, %7, %4 op_sel:[1,1,0,0]"
      : "=&v"(t0), "=&v"(t1), "=&v"(t2), "=v"(t3), "=&v"(n3)
      : "v"(x), "v"(y), "s"(d.range), "v"(nc), "v"(last));
  const uint64_t passed = __ballot(t0 >= nc);
  uint32_t hi = max(t0, t1), lo = min(min(t1, t2), t3);
  int lane;
  // lo takes the next group's t0 in (lane 0, group 63, has none and keeps its
  // own); the lane is the first of the mask.  In one block, so that an
  // instruction lies between each vector result and the lane reads below.
  asm("v_min_u32_dpp %0, %3, %0 wave_shr:1 row_mask:0xf bank_mask:0xf\n\t"
      "v_max3_u32 %1, %1, %4, %5\n\t"
      "s_ff1_i32_b64 %2, %6"
      : "+v"(lo), "+v"(hi), "=s"(lane)
      : "v"(t0), "v"(t2), "v"(t3), "s"(passed));
  const uint32_t mx = (uint32_t)__builtin_amdgcn_readlane((int)hi, lane);
  const uint32_t mn = (uint32_t)__builtin_amdgcn_readlane((int)lo, lane);
  d.range = mn - mx;
  uint32_t sh;  // leading zeros in whole bytes
  asm("s_flbit_i32_b32 %0, %1" : "=s"(sh) : "s"(d.range));
  sh &= 24u;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readlane((int)win, (int)(d.pos & 63u));
  d.nc = (uint32_t)(((((uint64_t)mx << 32) | w) << sh) >> 32);
  d.range <<= sh;
  d.pos += sh >> 3;
  return lane;
}

// lane k of v (k a constant) takes the wave-uniform s, a value of the scalar
// unit (no wait states are needed after those)
__device__ __forceinline__ void put_lane(uint32_t& v, uint32_t s, int k) {
  asm("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(s), "n"(k));
}

// Three waves per SIMD: LDS holds four blocks of NP = 2 (36 KB and the payload
// each) per compute unit, and the predictor takes up to 130 registers here.
template <int C, int NP, int RQ>
__global__ __launch_bounds__(64 * (NP + 1)) __attribute__((amdgpu_waves_per_eu(3))) void k_decode_chunks(
    const Chunk* __restrict__ chunks, const uint8_t* __restrict__ payload, const int32_t* __restrict__ lut_g,
    const DecArg A, uint8_t* __restrict__ codes, uint32_t* __restrict__ csum, uint32_t* __restrict__ err,
    int pay_words) {
  constexpr int NT = 64 * (NP + 1);
  __shared__ uint16_t lut[256];
  __shared__ __attribute__((aligned(16))) int32_t b2s[256];
  __shared__ __attribute__((aligned(16))) int32_t b1s[C];
  __shared__ __attribute__((aligned(16))) uint32_t ring[2][NP * 16 * kRowWords];
  __shared__ uint32_t note[2][3][NP * 16];  // ~code, range and lane of every symbol of the half
  __shared__ uint32_t kids;                 // children announced by the chunk's codes
  extern __shared__ uint32_t pay[];  // the chunk's bytes, zero padded (at least two words of zeros)

  const Chunk ch = chunks[blockIdx.x];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = ch.count;
  const int nblk = (n + 15) / 16, nstep = (nblk + NP - 1) / NP;
  for (int k = tid; k < 256; k += NT) {
    lut[k] = (uint16_t)gp(lut_g)[k];
    b2s[k] = gp(A.fc2.bias)[k];
    if (k < C) b1s[k] = gp(A.fc1.bias)[k];
  }
  {
    const uint32_t len = (uint32_t)ch.pad_;
    const GAS uint8_t* src = gp(payload) + ch.scratch;
    for (int w = tid; w < pay_words; w += NT) {
      uint32_t v = 0;
#pragma unroll
      for (int k = 0; k < 4; k++) {
        const uint32_t b = 4u * (uint32_t)w + (uint32_t)k;
        if (b < len) v |= (uint32_t)src[b] << (8 * k);
      }
      pay[w] = v;
    }
  }
  if (tid == 0) kids = 0u;
  lds_barrier();

  if (wave < NP) {
    const int r = lane & 15, g = lane >> 4;
    const GAS int8_t* F = gp(A.F) + (int64_t)ch.node0 * C + 16 * g;
    auto fetch = [&](int s) {
      const int i = 16 * (s * NP + wave) + r;
      return i < n && 16 * g < C ? *(const GAS v4i*)(F + (int64_t)i * C) : v4i{0, 0, 0, 0};
    };
    v4i x = fetch(0);
    uint32_t nkids = 0;
    // the codes of step s, whose rows and notes lie in half s & 1
    auto resolve = [&](int s) {
      const int base = 16 * (s * NP + wave);
      if (s < 0 || base + lane >= n || lane >= 16) return;
      const uint32_t* nt = &note[s & 1][0][wave * 16 + lane];
      const uint32_t sc = ~nt[0], sr = nt[NP * 16], L = 63u - (nt[2 * NP * 16] & 63u);
      const uint2 b = *(const uint2*)&ring[s & 1][(wave * 16 + lane) * kRowWords + 2 * L];
      const uint32_t rr = sr >> 16;
      uint32_t cv = 4u * L + 1u;
      cv += __umul24(rr, b.x >> 16) <= sc ? 1u : 0u;
      cv += __umul24(rr, b.y & 0xFFFFu) <= sc ? 1u : 0u;
      cv += L != 63u && __umul24(rr, b.y >> 16) <= sc ? 1u : 0u;
      if (sc >= (sr & 0xFFFF0000u)) atomicOr(err, ERR_CORRUPT);
      gp(codes)[ch.node0 + base + lane] = (uint8_t)cv;
      nkids += __popc(cv & 0xFFu);
    };
    for (int s = 0; s <= nstep; s++) {
      resolve(s - 2);
      if (s * NP + wave < nblk) {
        int e[64];
        NodeSum ns;
        // a lane offset the compiler cannot see through: it would keep the 20
        // 64-bit addresses in vector registers across the steps and spill
        uint32_t lo = 16u * (uint32_t)lane;
        asm volatile("" : "+v"(lo));
        predict_table<C, false, RQ>([&](int k) { return *(const GAS v4i*)(gp(A.fc1.Wp) + 1024 * k + lo); },
                                    [&](int k) { return *(const GAS v4i*)(gp(A.fc2.Wp) + 1024 * k + lo); }, b1s, b2s,
                                    lut, x, lane, A.fc1, A.fc2, e, ns);
        x = fetch(s + 1);
        uint32_t p0, p1, R;
        row_prefix<false>(e, ns, lane, p0, p1, R);
        uint32_t* row = &ring[s & 1][(wave * 16 + r) * kRowWords + 32 * g];
#pragma unroll
        for (int c = 0; c < 8; c++) {
          *(v4i*)&row[4 * c] = row_chunk<64>(e, c, ns.ablk, p0, p1);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (ns.aord == ns.ord) row_remainder(row + 2 * ns.ablk, ns, R);
        if (ns.tail) ((uint16_t*)row)[63] = 65535;  // entry 255, whatever the remainder made of it
      }
      lds_barrier();
    }
    resolve(nstep - 1);
    nkids = wave_scan_incl(nkids);  // lane 63: the wave's sum
    if (lane == 63) atomicAdd(&kids, nkids);
    lds_barrier();
    if (tid == 0) csum[blockIdx.x] = kids;
    return;
  }

  // the decoding wave
  int wb = 0;  // first payload byte of the window
  auto window = [&](int at) -> uint32_t {
    const int b = at + lane;
    const int w = min(b >> 2, pay_words - 2);
    const uint32_t v = __builtin_amdgcn_alignbyte(pay[w + 1], pay[w], (uint32_t)b & 3u);
    return ~__builtin_amdgcn_perm(0u, v, 0x00010203u);  // first byte on top
  };
  uint32_t win = window(0);
  // the first 5 bytes: the first is always 0
  RcDec d{(uint32_t)__builtin_amdgcn_readlane((int)win, 1), 0xFFFFFFFFu, 5u};
  const uint32_t last = lane == 0 ? 1u : 0u;
  __builtin_amdgcn_s_setprio(3);  // the chain sets the pace where waves are few
  lds_barrier();
  for (int s = 1; s <= nstep; s++) {
    for (int q = 0; q < NP; q++) {
      const int base = 16 * ((s - 1) * NP + q);
      if (base >= n) break;
      const uint32_t* rows = &ring[(s - 1) & 1][q * 16 * kRowWords];
      const uint32_t* grp = rows + 2 * (63 - lane);
      wb += (int)d.pos;
      d.pos = 0;
      win = window(wb);
      // lane k: ~code and range before symbol k and the lane of its group
      uint32_t sc = 0, sr = 0, sl = 0;
      const int cnt = min(16, n - base);
      // rows past the chunk's end (its last block) exist and decode to
      // nothing that is read
      uint2 t[16];
#pragma unroll
      for (int k = 0; k < 16; k++) t[k] = *(const uint2*)(grp + k * kRowWords);
#pragma unroll
      for (int h = 0; h < 2; h++) {
        if (8 * h >= cnt) break;
#pragma unroll
        for (int k = 8 * h; k < 8 * h + 8; k++) {
          put_lane(sc, d.nc, k);
          put_lane(sr, d.range, k);
          put_lane(sl, (uint32_t)rc_symbol(d, t[k].x, t[k].y, win, last), k);
        }
      }
      if (lane < cnt) {
        uint32_t* nt = &note[(s - 1) & 1][0][q * 16 + lane];
        nt[0] = sc;
        nt[NP * 16] = sr;
        nt[2 * NP * 16] = sl;
      }
    }
    lds_barrier();
  }
  lds_barrier();
}

// Predicting waves per decoding wave.  A full chunk of 256 nodes alone takes
// 27.5 us with 3 (the chain, 175 cycles per symbol, sets the pace), 31.5 us
// with 2 (it waits for rows; 66 us with 1) and 29 us with 5.  With thousands
// of chunks both arithmetic and chains are in flight anyway, and 2 leave a
// compute unit more chunks at once: 8 128-beam frames decode in 8.04 ms with 2
// and 8.28 ms with 3, one such frame (at most 920 chunks) in 2.12 and 2.09 ms,
// a 64-beam frame in 0.87 and 0.82 ms.  With the 64-bit requantisation the line
// lies at the same place: 8.70 and 8.92, 2.36 and 2.29, 0.92 and 0.86 ms.
constexpr int kDecodeWide = 1024;

hipError_t launch_decode_chunks(int C, const Chunk* chunks, int nchunks, const uint8_t* payload, const int32_t* lut,
                                const DecArg& A, uint8_t* codes, uint32_t* csum, uint32_t* err, size_t max_len,
                                hipStream_t s) {
  if (nchunks <= 0) return hipSuccess;
  const int words = (int)((max_len + 3) / 4) + 4;
  const int np = nchunks < kDecodeWide ? 3 : 2;
#define LPCC_DC(CC, NN, RR)                                                                                         \
  if (C == CC && np == NN && A.rqf == RR) {                                                                         \
    hipLaunchKernelGGL((k_decode_chunks<CC, NN, RR>), dim3(nchunks), dim3(64 * (NN + 1)), (size_t)words * 4, s,     \
                       chunks, payload, lut, A, codes, csum, err, words);                                           \
    return hipGetLastError();                                                                                       \
  }
#define LPCC_DC2(CC) LPCC_DC(CC, 2, 1) LPCC_DC(CC, 3, 1) LPCC_DC(CC, 2, 0) LPCC_DC(CC, 3, 0)
  LPCC_DC2(16) LPCC_DC2(32) LPCC_DC2(64)
#undef LPCC_DC2
#undef LPCC_DC
  return hipErrorInvalidValue;
}

// Nodes per block of the 16-node form: 64 x the groups of a wave.  More
// groups share one load of the weights (20 KB per block at C = 64); a launch
// keeps at least 4096 blocks (16 per compute unit, four times what runs at
// once) before a wave takes more.
int predict_groups(int64_t rows) { return rows >= (1 << 20) ? 4 : (rows >= (1 << 19) ? 2 : 1); }

hipError_t launch_predict(int C, int mode, const PredSeg* segs, const Tile* tiles, int ntiles, const int32_t* lut,
                          int groups, const PredArg& A, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  // single-segment launches of at most kPredSmall rows use 4 nodes per wave
  const bool small = A.one && A.seg.rows <= kPredSmall;
  const int grid = small ? (A.seg.rows + 15) / 16 : ntiles;
#define LPCC_P(CC, MM)                                                                                             \
  if (C == CC && mode == MM) {                                                                                     \
    if (small && A.rqf)                                                                                            \
      hipLaunchKernelGGL((k_predict<CC, MM, true, 1>), dim3(grid), dim3(256), 0, s, segs, tiles, lut, groups, A);  \
    else if (small)                                                                                                \
      hipLaunchKernelGGL((k_predict<CC, MM, true, 0>), dim3(grid), dim3(256), 0, s, segs, tiles, lut, groups, A);  \
    else if (A.rqf)                                                                                                \
      hipLaunchKernelGGL((k_predict<CC, MM, false, 1>), dim3(grid), dim3(256), 0, s, segs, tiles, lut, groups, A); \
    else                                                                                                           \
      hipLaunchKernelGGL((k_predict<CC, MM, false, 0>), dim3(grid), dim3(256), 0, s, segs, tiles, lut, groups, A); \
    return hipGetLastError();                                                                                      \
  }
  LPCC_P(16, 0) LPCC_P(16, 2) LPCC_P(32, 0) LPCC_P(32, 2) LPCC_P(64, 0) LPCC_P(64, 2)
#undef LPCC_P
  return hipErrorInvalidValue;
}

}  // namespace lpcc
