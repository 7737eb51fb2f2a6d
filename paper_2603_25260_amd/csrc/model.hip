// Integer-only network layers on gfx950 int8 MFMA (Sec. 3.3, Eq. 13-14):
//   * gather-GEMM for the 3x3x3 submanifold convolutions (indexed linear
//     transforms over a kernel map), the stride-2 child convolution of the
//     re-densification (Eq. 4) and dense linear layers;
//   * upsampling + pruning (Eq. 6/9/11): Linear(C+8 -> 8C) + PReLU per parent,
//     only occupied child slots are written, in Morton order;
//   * the occupancy embedding;
//   * the predictor (Eq. 7) fused with the integer softmax (Eq. 15) and the
//     16-bit frequency table that drives the range coder.
// One wave computes a 16-row tile with v_mfma_i32_16x16x64_i8; int32
// accumulation is exact, so any summation order gives the same result.
#include "lpcc_internal.h"

namespace lpcc {

// Lane layout of v_mfma_i32_16x16x64_i8 used throughout: A lane l holds row
// l%16, 16 consecutive k of group l/16; B lane l holds column l%16, the same
// k; the accumulator lane l holds rows 4(l/16)+i (i = 0..3) of column l%16.

__device__ __forceinline__ v4i ld16(const int8_t* p) { return *(const GAS v4i*)p; }

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

template <int N>
__device__ __forceinline__ void ld_bytes(const int8_t* p, int8_t (&v)[N]) {
  const typename Words<N>::T x = *(const GAS typename Words<N>::T*)p;
#pragma unroll
  for (int w = 0; w < N / 4; w++)
#pragma unroll
    for (int b = 0; b < 4; b++) v[4 * w + b] = (int8_t)((uint32_t)x[w] >> (8 * b));
}
template <int N>
__device__ __forceinline__ void st_bytes(int8_t* p, const int8_t (&v)[N]) {
  typename Words<N>::T x;
#pragma unroll
  for (int w = 0; w < N / 4; w++) {
    uint32_t y = 0;
#pragma unroll
    for (int b = 0; b < 4; b++) y |= ((uint32_t)(uint8_t)v[4 * w + b]) << (8 * b);
    x[w] = (int)y;
  }
  *(GAS typename Words<N>::T*)p = x;
}

// Epilogue: one wave's 16 x COUT int32 tile staged in LDS, then every lane
// handles a contiguous run of COUT/4 columns of one row.
template <int COUT>
struct Stage {
  int32_t v[16][COUT];
};

// ---------------------------------------------------------------------------
// Gather-GEMM: out[row][o] = rq(bias[o] + sum_t sum_c in[src(row,t)][c] W[t][c][o]
//                               + sum over present taps of zc[t][o]) (+ resid)
// MODE G_CONV : src(row,t) = kmap[t][row]            (27 taps)
// MODE G_DENSE: src(row,0) = row                      (1 tap)
// MODE G_DOWN : src(row,o) = child in slot o of parent row, if occupied (8 taps)
// ---------------------------------------------------------------------------
template <int MODE>
struct Taps;
template <>
struct Taps<G_CONV> { static constexpr int n = 27; };
template <>
struct Taps<G_DENSE> { static constexpr int n = 1; };
template <>
struct Taps<G_DOWN> { static constexpr int n = 8; };

template <int MODE>
__device__ __forceinline__ int src_row(const GemmSeg& S, int row, int tap) {
  if (MODE == G_CONV) return gp(S.kmap)[(int64_t)tap * S.kstride + row];
  if (MODE == G_DENSE) return row;
  uint32_t code = gp(S.code)[row];
  if (!((code >> tap) & 1u)) return -1;
  const int cr = gp(S.cstart)[row] + __popc(code & ((1u << tap) - 1u));
  if (cr >= S.child_rows) return -1;  // only for a corrupt stream
  return S.ccode != nullptr ? (int)gp(S.ccode)[cr] : cr;  // the embedding table is indexed by the child's code
}

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

template <int MODE, int CIN, int COUT>
__global__ __launch_bounds__(256) void k_gemm(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                              const GemmArg A) {
  constexpr int TAPS = Taps<MODE>::n;
  constexpr int K = TAPS * CIN;
  constexpr int KS = (K + 63) / 64;
  constexpr int NB = COUT / 16;
  static_assert(CIN % 16 == 0 && COUT % 16 == 0, "widths must be multiples of 16");
  __shared__ Stage<COUT> st[4];

  GemmSeg S;
  LayerDev L;
  const int tile_row0 = pick_seg(segs, tiles, A, S, L);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int row0 = tile_row0 + wave * 16;
  const int row = row0 + r;
  const bool rv = row < S.rows;

  // epilogue operands first, so that their latency overlaps the main loop
  constexpr int PER = COUT / 4;
  const int er = lane >> 2;           // epilogue row within the wave's 16
  const int ec = (lane & 3) * PER;    // first column
  const int orow = row0 + er;
  const bool ov = orow < S.rows;
  int bia[PER];
#pragma unroll
  for (int q = 0; q < PER; q++) bia[q] = gp(L.bias)[ec + q];
  int8_t res[PER];
#pragma unroll
  for (int q = 0; q < PER; q++) res[q] = 0;
  if (S.resid != nullptr && ov) {
    ld_bytes<PER>(S.resid + (int64_t)orow * S.resid_stride + ec, res);
  }

  v4i acc[NB];
#pragma unroll
  for (int nb = 0; nb < NB; nb++) acc[nb] = v4i{0, 0, 0, 0};

  // source row of every k-step for this lane (taps beyond TAPS are padding)
  int src[KS];
#pragma unroll
  for (int s = 0; s < KS; s++) {
    const int k0 = 64 * s + 16 * g;
    const int tap = k0 / CIN;
    src[s] = (rv && tap < TAPS) ? src_row<MODE>(S, row, tap) : -1;
  }
  const GAS v4i* Wp = (const GAS v4i*)L.Wp;
  // software pipeline: the loads of step s + PD - 1 are issued before the
  // MFMAs of step s; absent neighbours read row 0 and are zeroed afterwards
  constexpr int PD = 3;
  v4i abuf[PD], bbuf[PD][NB];
  auto load_step = [&](int s, v4i& a, v4i (&b)[NB]) {
    const int k0 = 64 * s + 16 * g;
    const int c0 = k0 % CIN;
    const int64_t ur = src[s] >= 0 ? src[s] : 0;
    const v4i v = c0 < S.split ? ld16(S.in + ur * S.in_stride + c0) : ld16(S.in2 + ur * S.in2_stride + (c0 - S.split));
    a = src[s] >= 0 ? v : v4i{0, 0, 0, 0};
#pragma unroll
    for (int nb = 0; nb < NB; nb++) b[nb] = Wp[((int64_t)s * NB + nb) * 64 + lane];
  };
#pragma unroll
  for (int p = 0; p < PD - 1; p++)
    if (p < KS) load_step(p, abuf[p], bbuf[p]);
#pragma unroll
  for (int s = 0; s < KS; s++) {
    if (s + PD - 1 < KS) load_step(s + PD - 1, abuf[(s + PD - 1) % PD], bbuf[(s + PD - 1) % PD]);
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[nb] = mfma16(abuf[s % PD], bbuf[s % PD][nb], acc[nb]);
  }

  // stage the tile, then requantise row-contiguous runs
#pragma unroll
  for (int nb = 0; nb < NB; nb++)
#pragma unroll
    for (int i = 0; i < 4; i++) st[wave].v[4 * g + i][16 * nb + r] = acc[nb][i];
  __syncthreads();
  if (ov) {
    int zsum[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) zsum[q] = 0;
    if (L.zc != nullptr) {
      for (int t = 0; t < TAPS; t++) {
        if (src_row<MODE>(S, orow, t) < 0) continue;
#pragma unroll
        for (int q = 0; q < PER; q++) zsum[q] += gp(L.zc)[t * L.npad + ec + q];
      }
    }
    int8_t outv[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) {
      int a = st[wave].v[er][ec + q] + bia[q] + zsum[q];
      int y = requant_l(a, L);
      if (S.resid != nullptr) {
        y += res[q];
        y = y < -128 ? -128 : (y > 127 ? 127 : y);
      }
      outv[q] = (int8_t)y;
    }
    st_bytes<PER>(S.out + (int64_t)orow * S.out_stride + ec, outv);
  }
}

// Register-blocked variant for large launches: a wave computes RB blocks of
// 16 rows, so every weight fragment it loads serves RB MFMAs (the weights
// are re-read from L2 by every wave; with RB = 1 that traffic exceeds the
// gathered activations several times over for C >= 32).  The neighbour
// table of the wave's rows is staged in LDS first (one coalesced load per
// tap), then each k-step gathers the RB A fragments through it.
template <int MODE, int CIN, int COUT, int RB>
__global__ __launch_bounds__(256) void k_gemm_rb(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                                 const GemmArg A) {
  constexpr int TAPS = Taps<MODE>::n;
  constexpr int K = TAPS * CIN;
  constexpr int KS = (K + 63) / 64;
  constexpr int NB = COUT / 16;
  constexpr int WR = 16 * RB;  // rows per wave
  static_assert(CIN % 16 == 0 && COUT % 16 == 0 && (CIN & (CIN - 1)) == 0, "widths");
  static_assert(WR <= 64, "at most 64 rows per wave");
  __shared__ Stage<COUT> st[4];
  __shared__ int32_t skm[MODE == G_CONV ? 4 : 1][MODE == G_CONV ? TAPS : 1][WR];

  GemmSeg S;
  LayerDev L;
  const int tile_row0 = pick_seg(segs, tiles, A, S, L, 4 * WR);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int wrow0 = tile_row0 + wave * WR;

  // epilogue operands first
  constexpr int PER = COUT / 4;
  const int er = lane >> 2, ec = (lane & 3) * PER;
  int bia[PER];
#pragma unroll
  for (int q = 0; q < PER; q++) bia[q] = gp(L.bias)[ec + q];
  int8_t res[RB][PER];
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
    const int orow = wrow0 + 16 * rb + er;
#pragma unroll
    for (int q = 0; q < PER; q++) res[rb][q] = 0;
    if (S.resid != nullptr && orow < S.rows) {
      ld_bytes<PER>(S.resid + (int64_t)orow * S.resid_stride + ec, res[rb]);
    }
  }

  // per row block: the row of this lane, and for the child convolution its
  // parent's code and first child
  uint32_t pcode[RB];
  int pcs[RB];
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
    const int row = wrow0 + 16 * rb + r;
    pcode[rb] = 0u;
    pcs[rb] = 0;
    if (MODE == G_DOWN && row < S.rows) {
      pcode[rb] = gp(S.code)[row];
      pcs[rb] = gp(S.cstart)[row];
    }
  }
  if (MODE == G_CONV) {
    if (lane < WR) {
      const int row = wrow0 + lane;
      const bool ok = row < S.rows;
#pragma unroll
      for (int t = 0; t < TAPS; t++) skm[wave][t][lane] = ok ? gp(S.kmap)[(int64_t)t * S.kstride + row] : -1;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  auto src_of = [&](int rb, int tap) -> int {
    const int row = wrow0 + 16 * rb + r;
    if (tap >= TAPS || row >= S.rows) return -1;
    if (MODE == G_CONV) return skm[MODE == G_CONV ? wave : 0][MODE == G_CONV ? tap : 0][16 * rb + r];
    if (MODE == G_DENSE) return row;
    if (!((pcode[rb] >> tap) & 1u)) return -1;
    const int cr = pcs[rb] + __popc(pcode[rb] & ((1u << tap) - 1u));
    if (cr >= S.child_rows) return -1;
    return S.ccode != nullptr ? (int)gp(S.ccode)[cr] : cr;  // the embedding table is indexed by the child's code
  };

  v4i acc[RB][NB];
#pragma unroll
  for (int rb = 0; rb < RB; rb++)
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[rb][nb] = v4i{0, 0, 0, 0};
  const GAS v4i* Wp = (const GAS v4i*)L.Wp;
  constexpr int LC = __builtin_ctz(CIN);
  // [in | in2] layers (the ResBlock at k0 on [F | G]) are exactly those with
  // cin = 2 cout, split at cout; the feature arrays stay below 2^31 bytes
  // (checked on the host), so row offsets are 32-bit
  constexpr int SPLIT = CIN == 2 * COUT ? COUT : CIN;
  const GAS int8_t* in1 = gp(S.in);
  const GAS int8_t* in2 = gp(S.in2);
  const uint32_t st1 = (uint32_t)S.in_stride, st2 = (uint32_t)S.in2_stride;
  // Software pipeline over the k-steps: the gathers and weight fragments of
  // step s + PD - 1 are issued before the MFMAs of step s, so PD - 1 steps of
  // loads are in flight behind the math instead of one load latency per
  // step.  Absent neighbours read row 0 (every launch has one) and are
  // zeroed after the load, which keeps the gathers free of branches.
  constexpr int PD = 3;
  v4i abuf[PD][RB], bbuf[PD][NB];
  auto load_step = [&](int s, v4i (&a)[RB], v4i (&b)[NB]) {
    const int k0 = 64 * s + 16 * g;
    const int tap = k0 >> LC, c0 = k0 & (CIN - 1);
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      const int sr = src_of(rb, tap);
      const uint32_t ur = sr >= 0 ? (uint32_t)sr : 0u;
      const v4i v = c0 < SPLIT ? *(const GAS v4i*)(in1 + (ur * st1 + (uint32_t)c0))
                               : *(const GAS v4i*)(in2 + (ur * st2 + (uint32_t)(c0 - SPLIT)));
      a[rb] = sr >= 0 ? v : v4i{0, 0, 0, 0};
    }
#pragma unroll
    for (int nb = 0; nb < NB; nb++) b[nb] = Wp[((int64_t)s * NB + nb) * 64 + lane];
  };
#pragma unroll
  for (int p = 0; p < PD - 1; p++)
    if (p < KS) load_step(p, abuf[p], bbuf[p]);
#pragma unroll
  for (int s = 0; s < KS; s++) {
    if (s + PD - 1 < KS) load_step(s + PD - 1, abuf[(s + PD - 1) % PD], bbuf[(s + PD - 1) % PD]);
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int rb = 0; rb < RB; rb++) acc[rb][nb] = mfma16(abuf[s % PD][rb], bbuf[s % PD][nb], acc[rb][nb]);
  }

  // epilogue, one row block at a time through the wave's LDS stage
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int i = 0; i < 4; i++) st[wave].v[4 * g + i][16 * nb + r] = acc[rb][nb][i];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int orow = wrow0 + 16 * rb + er;
    if (orow < S.rows) {
      int zsum[PER];
#pragma unroll
      for (int q = 0; q < PER; q++) zsum[q] = 0;
      if (L.zc != nullptr) {
        for (int t = 0; t < TAPS; t++) {
          int present;
          if (MODE == G_CONV) present = skm[MODE == G_CONV ? wave : 0][MODE == G_CONV ? t : 0][16 * rb + er] >= 0;
          else present = src_row<MODE>(S, orow, t) >= 0;
          if (!present) continue;
#pragma unroll
          for (int q = 0; q < PER; q++) zsum[q] += gp(L.zc)[t * L.npad + ec + q];
        }
      }
      int8_t outv[PER];
#pragma unroll
      for (int q = 0; q < PER; q++) {
        int y = requant_l(st[wave].v[er][ec + q] + bia[q] + zsum[q], L);
        if (S.resid != nullptr) {
          y += res[rb][q];
          y = y < -128 ? -128 : (y > 127 ? 127 : y);
        }
        outv[q] = (int8_t)y;
      }
      st_bytes<PER>(S.out + (int64_t)orow * S.out_stride + ec, outv);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// ---------------------------------------------------------------------------
// Gather-GEMM over the present taps only (kernel-map compaction) for the
// 3x3x3 convolution and the child convolution.  A wave owns WR = 16 RB
// output rows.  Every row has a bit mask of its present taps: the presence
// mask the neighbour-table kernel stores after the 27 tap rows, or for the
// child convolution the parent's occupancy code.  The OR of the masks over
// the wave's rows sets the wave's K dimension: its nt taps, ranked by tap
// index, times CIN channels, in k-steps of 64.  A tap that no row of the
// wave has costs nothing (no table read, weight load, gather or MFMA); rows
// without a present tap contribute a zero A fragment.  Only the table rows
// of the present taps are staged, straight from global memory into LDS.
// The tap of rank i sits in lane i of a register (read with readlane), and
// the weights of tap t, channel c are rows k = t CIN + c of the packed
// layout, so any tap's B fragment is addressed directly.  The sums are exact
// int32, so the order of the taps does not change the result.
// ---------------------------------------------------------------------------
template <int MODE, int CIN, int COUT, int RB>
__global__ __launch_bounds__(256) void k_gemm_cx(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                                 const GemmArg A) {
  constexpr int TAPS = Taps<MODE>::n;
  constexpr int NB = COUT / 16;
  constexpr int WR = 16 * RB;  // rows per wave
  static_assert(MODE == G_CONV || MODE == G_DOWN, "tap-compacted modes");
  static_assert(CIN % 16 == 0 && COUT % 16 == 0 && (CIN & (CIN - 1)) == 0, "widths");
  static_assert(WR <= 64 && TAPS <= 32, "shape");
  // Per wave, one LDS region holds first the neighbour rows of the wave's
  // rows (slot i = the tap of rank i, lane l = row wrow0 + l), then, after
  // the k-loop, the accumulator stage of the epilogue.
  constexpr int KMW = MODE == G_CONV ? TAPS * WR : 0;
  constexpr int RW = KMW > 16 * COUT ? KMW : 16 * COUT;  // words per wave
  __shared__ __attribute__((aligned(16))) int32_t smem[4 * RW];

  GemmSeg S;
  LayerDev L;
  const int tile_row0 = pick_seg(segs, tiles, A, S, L, 4 * WR);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int wrow0 = tile_row0 + wave * WR;
  int32_t* skm = smem + wave * RW;  // [slot][WR]
  Stage<COUT>* st = (Stage<COUT>*)(smem + wave * RW);

  // presence masks: the table's (one load per row) or the parents' codes
  uint32_t pcode[RB];
  int pcs[RB];
  uint32_t mine = 0u;
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
    const int row = wrow0 + 16 * rb + r;
    pcode[rb] = 0u;
    pcs[rb] = 0;
    if (MODE == G_DOWN && row < S.rows) {
      pcode[rb] = gp(S.code)[row] & 0xFFu;
      pcs[rb] = gp(S.cstart)[row];
    }
    mine |= pcode[rb];
  }
  const int myrow = wrow0 + lane;
  if (MODE == G_CONV && lane < WR && myrow < S.rows) mine = (uint32_t)gp(S.kmap)[27 * S.kstride + myrow];
  uint32_t U = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) U |= (uint32_t)__shfl_xor((int)U, o);
  U = (uint32_t)__builtin_amdgcn_readfirstlane((int)U);
  const int nt = __popc(U);
  // lane i: the tap of rank i (255 past the last); the owner of each set bit
  // sends its tap to the lane of its rank
  int tapof;
  {
    const bool own = lane < TAPS && ((U >> (lane & 31)) & 1u);
    const int rk = __popc(U & ((1u << (lane & 31)) - 1u));
    const int got = __builtin_amdgcn_ds_permute((own ? rk : 63) * 4, lane);
    tapof = lane < nt ? got : 255;
  }
  if (MODE == G_CONV) {
    // table rows of the present taps, straight into LDS (rows past the end
    // read the last row; they are never used)
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
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): the staged rows have landed
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

  // source row of block rb for the tap of rank `slot` (tap `tap`), or -1
  auto src_of = [&](int rb, int slot, int tap) -> int {
    const int row = wrow0 + 16 * rb + r;
    if (row >= S.rows) return -1;
    if (MODE == G_CONV) return skm[slot * WR + 16 * rb + r];
    if (!((pcode[rb] >> tap) & 1u)) return -1;
    const int cr = pcs[rb] + __popc(pcode[rb] & ((1u << tap) - 1u));
    if (cr >= S.child_rows) return -1;  // only for a corrupt stream
    return S.ccode != nullptr ? (int)gp(S.ccode)[cr] : cr;  // the embedding table is indexed by the child's code
  };

  v4i acc[RB][NB];
#pragma unroll
  for (int rb = 0; rb < RB; rb++)
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[rb][nb] = v4i{0, 0, 0, 0};
  const GAS v4i* Wp = (const GAS v4i*)L.Wp;
  constexpr int LC = __builtin_ctz(CIN);
  constexpr int SPLIT = CIN == 2 * COUT ? COUT : CIN;  // [in | in2] layers have cin = 2 cout
  // taps per k-step (CIN < 64: lane group g takes slot base + (16 g >> LC))
  constexpr int SPS = CIN >= 64 ? 1 : 64 / CIN;
  const GAS int8_t* in1 = gp(S.in);
  const GAS int8_t* in2 = gp(S.in2);
  const uint32_t st1 = (uint32_t)S.in_stride, st2 = (uint32_t)S.in2_stride;
  const int KV = (nt * CIN + 63) >> 6;  // k-steps over the present taps (wave-uniform)

  // Software pipeline over the k-steps, one step of loads in flight behind
  // the MFMAs.  The loop body is straight-line code: steps past the last
  // present tap, and rows without the step's tap, load from row 0 and the
  // first weight fragment and are zeroed after the load.
  constexpr int PD = 2;
  v4i abuf[PD][RB], bbuf[PD][NB];
  auto load_step = [&](int v, v4i (&a)[RB], v4i (&b)[NB]) {
    const int kk = 64 * v + 16 * g;
    const int c0 = kk & (CIN - 1);
    int slot, tap;
    if (SPS == 1) {
      slot = min((64 * v) >> LC, 31);
      tap = __builtin_amdgcn_readlane(tapof, slot);
    } else {
      const int base = min(v * SPS, 28);
      int tk[SPS];
#pragma unroll
      for (int k = 0; k < SPS; k++) tk[k] = __builtin_amdgcn_readlane(tapof, base + k);
      const int k = (16 * g) >> LC;
      slot = base + k;
      tap = tk[0];
#pragma unroll
      for (int q = 1; q < SPS; q++) tap = k == q ? tk[q] : tap;
    }
    const bool tv = tap < TAPS;
    const int ko = tv ? tap * CIN + c0 : 0;
    const GAS v4i* w = Wp + (int64_t)(ko >> 6) * NB * 64 + ((ko >> 4) & 3) * 16 + r;
#pragma unroll
    for (int nb = 0; nb < NB; nb++) {
      const v4i x = w[nb * 64];
      b[nb] = tv ? x : v4i{0, 0, 0, 0};
    }
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      const int sr = tv ? src_of(rb, slot, tap) : -1;
      const bool present = sr >= 0;
      const uint32_t ur = present ? (uint32_t)sr : 0u;
      const v4i x = c0 < SPLIT ? *(const GAS v4i*)(in1 + (ur * st1 + (uint32_t)c0))
                               : *(const GAS v4i*)(in2 + (ur * st2 + (uint32_t)(c0 - SPLIT)));
      a[rb] = present ? x : v4i{0, 0, 0, 0};
    }
  };
#pragma unroll
  for (int p = 0; p < PD - 1; p++) load_step(p, abuf[p], bbuf[p]);
  for (int v0 = 0; v0 < KV; v0 += PD) {
#pragma unroll
    for (int u = 0; u < PD; u++) {
      load_step(v0 + u + PD - 1, abuf[(u + PD - 1) % PD], bbuf[(u + PD - 1) % PD]);
#pragma unroll
      for (int rb = 0; rb < RB; rb++)
#pragma unroll
        for (int nb = 0; nb < NB; nb++) acc[rb][nb] = mfma16(abuf[u][rb], bbuf[u][nb], acc[rb][nb]);
    }
  }

  // epilogue, one row block at a time through the wave's LDS stage, which
  // reuses the region of the staged neighbour rows (its operands are loaded
  // only now: registers, not latency, bound the k-loop)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  constexpr int PER = COUT / 4;
  const int er = lane >> 2, ec = (lane & 3) * PER;
  int bia[PER];
#pragma unroll
  for (int q = 0; q < PER; q++) bia[q] = gp(L.bias)[ec + q];
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
    int8_t res[PER];
#pragma unroll
    for (int q = 0; q < PER; q++) res[q] = 0;
    if (S.resid != nullptr && wrow0 + 16 * rb + er < S.rows) {
      ld_bytes<PER>(S.resid + (int64_t)(wrow0 + 16 * rb + er) * S.resid_stride + ec, res);
    }
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int i = 0; i < 4; i++) st->v[4 * g + i][16 * nb + r] = acc[rb][nb][i];
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int orow = wrow0 + 16 * rb + er;
    // presence mask of the epilogue row (zero-point correction over its taps)
    const uint32_t omask = MODE == G_CONV ? (uint32_t)__shfl((int)mine, (16 * rb + er) & 63) : 0u;
    if (orow < S.rows) {
      int zsum[PER];
#pragma unroll
      for (int q = 0; q < PER; q++) zsum[q] = 0;
      if (L.zc != nullptr) {
        for (int t = 0; t < TAPS; t++) {
          const int present = MODE == G_CONV ? (int)((omask >> t) & 1u) : (int)(src_row<MODE>(S, orow, t) >= 0);
          if (!present) continue;
#pragma unroll
          for (int q = 0; q < PER; q++) zsum[q] += gp(L.zc)[t * L.npad + ec + q];
        }
      }
      int8_t outv[PER];
#pragma unroll
      for (int q = 0; q < PER; q++) {
        int y = requant_l(st->v[er][ec + q] + bia[q] + zsum[q], L);
        if (S.resid != nullptr) {
          y += res[q];
          y = y < -128 ? -128 : (y > 127 ? 127 : y);
        }
        outv[q] = (int8_t)y;
      }
      st_bytes<PER>(S.out + (int64_t)orow * S.out_stride + ec, outv);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

template <int MODE>
static hipError_t launch_gemm_mode(int cin, int cout, const GemmSeg* segs, const Tile* tiles, int ntiles,
                                   const GemmArg& A, int rb, hipStream_t s) {
#define LPCC_G(CI, CO)                                                                                    \
  if (cin == CI && cout == CO) {                                                                          \
    if (rb == 4)                                                                                          \
      hipLaunchKernelGGL((k_gemm_rb<MODE, CI, CO, 4>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);    \
    else if (rb == 2)                                                                                     \
      hipLaunchKernelGGL((k_gemm_rb<MODE, CI, CO, 2>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);    \
    else                                                                                                  \
      hipLaunchKernelGGL((k_gemm<MODE, CI, CO>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);          \
    return hipGetLastError();                                                                             \
  }
  LPCC_G(16, 16) LPCC_G(32, 16) LPCC_G(32, 32) LPCC_G(64, 32) LPCC_G(64, 64) LPCC_G(128, 64)
#undef LPCC_G
  return hipErrorInvalidValue;
}

// the 3x3x3 and child convolutions: (C, C) layers, and (2C, C) for the
// ResBlock's first convolution on [F | G]
template <int MODE>
static hipError_t launch_gemm_cx(int cin, int cout, const GemmSeg* segs, const Tile* tiles, int ntiles,
                                 const GemmArg& A, int rb, hipStream_t s) {
#define LPCC_C(CI, CO)                                                                                    \
  if (cin == CI && cout == CO) {                                                                          \
    if (rb == 4)                                                                                          \
      hipLaunchKernelGGL((k_gemm_cx<MODE, CI, CO, 4>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);    \
    else if (rb == 2)                                                                                     \
      hipLaunchKernelGGL((k_gemm_cx<MODE, CI, CO, 2>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);    \
    else                                                                                                  \
      hipLaunchKernelGGL((k_gemm_cx<MODE, CI, CO, 1>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);    \
    return hipGetLastError();                                                                             \
  }
  LPCC_C(16, 16) LPCC_C(32, 16) LPCC_C(32, 32) LPCC_C(64, 32) LPCC_C(64, 64) LPCC_C(128, 64)
#undef LPCC_C
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_dense(int mode, int cin, int cout, const GemmSeg* segs, const Tile* tiles, int ntiles,
                             const GemmArg& A, int rb, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  if (mode == G_CONV) return launch_gemm_mode<G_CONV>(cin, cout, segs, tiles, ntiles, A, rb, s);
  if (mode == G_DENSE) return launch_gemm_mode<G_DENSE>(cin, cout, segs, tiles, ntiles, A, rb, s);
  if (mode == G_DOWN) return launch_gemm_mode<G_DOWN>(cin, cout, segs, tiles, ntiles, A, rb, s);
  return hipErrorInvalidValue;
}

hipError_t launch_gemm(int mode, int cin, int cout, const GemmSeg* segs, const Tile* tiles, int ntiles,
                       const GemmArg& A, int rb, hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
  if (mode == G_CONV) return launch_gemm_cx<G_CONV>(cin, cout, segs, tiles, ntiles, A, rb, s);
  if (mode == G_DENSE) return launch_gemm_mode<G_DENSE>(cin, cout, segs, tiles, ntiles, A, rb, s);
  if (mode == G_DOWN) return launch_gemm_cx<G_DOWN>(cin, cout, segs, tiles, ntiles, A, rb, s);
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Upsampling + pruning: per parent p, A = [Z[p] (C) | bits(X[p]) (8)],
// out block o (columns oC..oC+C-1) is child slot o; occupied slots only,
// child row = cstart[p] + rank of o among the set bits.
//
// The product is formed transposed (weights as the MFMA row operand,
// parents as columns), so that every lane ends with four consecutive output
// channels of one parent: it requantises them and writes one 32-bit word of
// the child row directly, with no staging of the accumulators.
// ---------------------------------------------------------------------------
template <int C, int RB>
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
        a[rb][s] = ld16(S.in + (int64_t)row * S.in_stride + k0);
      } else if (rv && k0 == C) {  // occupancy bits as int8 {0,127}, then zeros
        uint32_t w0 = 0, w1 = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
          if ((code[rb] >> b) & 1u) w0 |= 127u << (8 * b);
          if ((code[rb] >> (b + 4)) & 1u) w1 |= 127u << (8 * b);
        }
        a[rb][s] = v4i{(int)w0, (int)w1, 0, 0};
      }
    }
  }
  const GAS v4i* Wp = (const GAS v4i*)L.Wp;
  const GAS v4i* Bp = (const GAS v4i*)L.bias;
  // weights and biases of slot o+1 are in flight while slot o is computed;
  // lane (r, g) holds the bias of channels 16 nb + 4g .. +3
  v4i wb[2][KS][NBS], bb[2][NBS];
#pragma unroll
  for (int s = 0; s < KS; s++)
#pragma unroll
    for (int nb = 0; nb < NBS; nb++) wb[0][s][nb] = Wp[((int64_t)s * NBT + nb) * 64 + lane];
#pragma unroll
  for (int nb = 0; nb < NBS; nb++) bb[0][nb] = Bp[(16 * nb + 4 * g) / 4];

#pragma unroll
  for (int o = 0; o < 8; o++) {
    if (o + 1 < 8) {
#pragma unroll
      for (int s = 0; s < KS; s++)
#pragma unroll
        for (int nb = 0; nb < NBS; nb++)
          wb[(o + 1) & 1][s][nb] = Wp[((int64_t)s * NBT + (o + 1) * NBS + nb) * 64 + lane];
#pragma unroll
      for (int nb = 0; nb < NBS; nb++) bb[(o + 1) & 1][nb] = Bp[((o + 1) * C + 16 * nb + 4 * g) / 4];
    }
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      const bool has = (code[rb] >> o) & 1u;
      if (__ballot(has) == 0ull) continue;  // no parent of the block has child o
      v4i acc[NBS];
#pragma unroll
      for (int nb = 0; nb < NBS; nb++) acc[nb] = v4i{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < KS; s++)
#pragma unroll
        for (int nb = 0; nb < NBS; nb++) acc[nb] = mfma16(wb[o & 1][s][nb], a[rb][s], acc[nb]);
      if (!has) continue;
      const int crow = first[rb] + __popc(code[rb] & ((1u << o) - 1u));
      if (crow >= S.child_rows) continue;  // only for a corrupt stream
      GAS uint32_t* dst = (GAS uint32_t*)(gp(S.out) + (int64_t)crow * S.out_stride + 4 * g);
#pragma unroll
      for (int nb = 0; nb < NBS; nb++) {
        uint32_t packed = 0;
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const int y = requant_l(acc[nb][i] + bb[o & 1][nb][i], L);
          packed |= ((uint32_t)y & 0xFFu) << (8 * i);
        }
        dst[4 * nb] = packed;
      }
    }
  }
}

// Staged variant for C = 64: the accumulators of a slot go through LDS and
// only the occupied (parent, slot) outputs are requantised, RPP child rows
// per pass.  At the sparse depths most slots hold few children, and this
// compaction saves more requantisation work than the staging costs; at
// C <= 32 the direct form above is faster.
template <int C, int RB>
__global__ __launch_bounds__(256) void k_up_staged(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                            const GemmArg A) {
  constexpr int KS = (C + 8 + 63) / 64;
  constexpr int NBS = C / 16;          // column blocks per child slot
  constexpr int NBT = 8 * NBS;         // column blocks of the layer
  constexpr int WR = 16 * RB;          // parent rows per wave
  // per wave: the accumulator tile of one slot, and the parents' codes / first children
  __shared__ int32_t st[4][16][C + 1];
  __shared__ uint32_t pc[4][WR];
  __shared__ int32_t ps[4][WR];

  GemmSeg S;
  LayerDev L;
  const int tile_row0 = pick_seg(segs, tiles, A, S, L, 4 * WR);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const int wrow0 = tile_row0 + wave * WR;
  uint32_t code[RB];
#pragma unroll
  for (int rb = 0; rb < RB; rb++) {
    const int row = wrow0 + 16 * rb + r;
    code[rb] = row < S.rows ? gp(S.code)[row] : 0u;
    if (g == 0) {
      pc[wave][16 * rb + r] = code[rb];
      ps[wave][16 * rb + r] = row < S.rows ? gp(S.cstart)[row] : 0;
    }
  }
  // output: 4 consecutive columns per lane, C/4 lanes per child row
  static_assert(C % 4 == 0 && 64 % (C / 4) == 0, "C");
  constexpr int LPR = C / 4, RPP = 64 / LPR;
  const int jl = lane / LPR, c4 = (lane % LPR) * 4;
  int bia[8][4];
#pragma unroll
  for (int o = 0; o < 8; o++)
#pragma unroll
    for (int q = 0; q < 4; q++) bia[o][q] = gp(L.bias)[o * C + c4 + q];

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
        a[rb][s] = ld16(S.in + (int64_t)row * S.in_stride + k0);
      } else if (rv && k0 == C) {  // occupancy bits as int8 {0,127}, then zeros
        uint32_t w0 = 0, w1 = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
          if ((code[rb] >> b) & 1u) w0 |= 127u << (8 * b);
          if ((code[rb] >> (b + 4)) & 1u) w1 |= 127u << (8 * b);
        }
        a[rb][s] = v4i{(int)w0, (int)w1, 0, 0};
      }
    }
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const GAS v4i* Wp = (const GAS v4i*)L.Wp;
  // weights of slot o+1 are in flight while slot o is computed
  v4i wb[2][KS][NBS];
#pragma unroll
  for (int s = 0; s < KS; s++)
#pragma unroll
    for (int nb = 0; nb < NBS; nb++) wb[0][s][nb] = Wp[((int64_t)s * NBT + nb) * 64 + lane];

#pragma unroll
  for (int o = 0; o < 8; o++) {
    if (o + 1 < 8) {
#pragma unroll
      for (int s = 0; s < KS; s++)
#pragma unroll
        for (int nb = 0; nb < NBS; nb++)
          wb[(o + 1) & 1][s][nb] = Wp[((int64_t)s * NBT + (o + 1) * NBS + nb) * 64 + lane];
    }
#pragma unroll
    for (int rb = 0; rb < RB; rb++) {
      // rows of this block whose parent has child slot o (wave-uniform)
      const uint32_t m = (uint32_t)(__ballot((code[rb] >> o) & 1u) & 0xFFFFull);
      if (m == 0u) continue;
      v4i acc[NBS];
#pragma unroll
      for (int nb = 0; nb < NBS; nb++) acc[nb] = v4i{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < KS; s++)
#pragma unroll
        for (int nb = 0; nb < NBS; nb++) acc[nb] = mfma16(a[rb][s], wb[o & 1][s][nb], acc[nb]);
#pragma unroll
      for (int nb = 0; nb < NBS; nb++)
#pragma unroll
        for (int i = 0; i < 4; i++) st[wave][4 * g + i][16 * nb + r] = acc[nb][i];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      // only the occupied (row, slot) outputs: k rows of C columns, RPP rows
      // per pass, 4 columns (one 32-bit store) per lane
      const int k = __popc(m);
      for (int j = jl; j < k; j += RPP) {
        // row of the j-th set bit of m
        int pos = 0;
#pragma unroll
        for (int w = 8; w >= 1; w >>= 1)
          if (__popc(m & ((1u << (pos + w)) - 1u)) <= j) pos += w;
        const uint32_t pcode = pc[wave][16 * rb + pos];
        const int crow = ps[wave][16 * rb + pos] + __popc(pcode & ((1u << o) - 1u));
        if (crow >= S.child_rows) continue;  // only for a corrupt stream
        uint32_t packed = 0;
#pragma unroll
        for (int q = 0; q < 4; q++) {
          const int y = requant_l(st[wave][pos][c4 + q] + bia[o][q], L);
          packed |= ((uint32_t)y & 0xFFu) << (8 * q);
        }
        *(GAS uint32_t*)(gp(S.out) + (int64_t)crow * S.out_stride + c4) = packed;
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
  }
}

// Upsampling + pruning over the occupied children only.  A block takes P
// (128 or 512) consecutive parents and compacts them, per child slot o, into a
// list of the parents that have child o (wave ballot and prefix count, then
// the per-wave totals: the list keeps parent order).  The lists are cut into
// groups of 16 entries; a wave computes one group with one MFMA column block
// per 16 output channels: the weights of slot o as the row operand, the 16
// parents' inputs [Z | bits(X)] as the columns, so that every lane ends with
// four consecutive output channels of one child and writes them as one word.
// Only the last group of each slot is partly empty.  Groups are dealt to the
// waves in slot order, so a wave keeps a slot's weights across its groups.

__device__ __forceinline__ uint32_t lanes_below(uint64_t m) {  // set bits of m below this lane
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

template <int C, int P>
__global__ __launch_bounds__(256) void k_up_cx(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                               const GemmArg A) {
  constexpr int KS = (C + 8 + 63) / 64;
  constexpr int NBS = C / 16;          // column blocks per child slot
  constexpr int NBT = 8 * NBS;         // column blocks of the layer
  constexpr int PPT = P >= 256 ? P / 256 : 1;  // parents per thread
  static_assert(C % 16 == 0 && (P % 256 == 0 || P == 128), "shape");
  __shared__ uint16_t list[8][P];
  __shared__ uint8_t pcode[P];
  __shared__ uint32_t wtot[8][4 * PPT];
  __shared__ uint32_t cnt[8];
  __shared__ uint32_t goff[9];
  __shared__ uint32_t ost[4][16][C / 4 + 4];  // output stage of every wave (16 rows)
  __shared__ int32_t ocrow[4][16];

  GemmSeg S;
  LayerDev L;
  const int p0 = pick_seg(segs, tiles, A, S, L, P);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;

  // compaction: parent t of the block is thread t % 256, round t / 256
  uint32_t code[PPT];
  uint32_t rank[PPT][8];
#pragma unroll
  for (int q = 0; q < PPT; q++) {
    const int t = 256 * q + (int)threadIdx.x;
    const int p = p0 + t;
    code[q] = t < P && p < S.rows ? (uint32_t)gp(S.code)[p] : 0u;
    if (t < P) pcode[t] = (uint8_t)code[q];
#pragma unroll
    for (int o = 0; o < 8; o++) {
      const uint64_t m = __ballot((code[q] >> o) & 1u);
      rank[q][o] = lanes_below(m);
      if (lane == 0) wtot[o][4 * q + wave] = (uint32_t)__popcll(m);
    }
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < PPT; q++) {
    const int t = 256 * q + (int)threadIdx.x;
#pragma unroll
    for (int o = 0; o < 8; o++) {
      if (!((code[q] >> o) & 1u)) continue;
      uint32_t before = rank[q][o];
      for (int w = 0; w < 4 * q + wave; w++) before += wtot[o][w];
      list[o][before] = (uint16_t)t;
    }
  }
  if (threadIdx.x < 8) {  // list lengths
    uint32_t n = 0;
    for (int w = 0; w < 4 * PPT; w++) n += wtot[threadIdx.x][w];
    cnt[threadIdx.x] = n;
  }
  __syncthreads();
  if (threadIdx.x == 0) {  // first group of every slot (16 entries per group)
    uint32_t gsum = 0;
    for (int o = 0; o < 8; o++) {
      goff[o] = gsum;
      gsum += (cnt[o] + 15) / 16;
    }
    goff[8] = gsum;
  }
  __syncthreads();

  const GAS v4i* Wp = (const GAS v4i*)L.Wp;
  const GAS v4i* Bp = (const GAS v4i*)L.bias;
  const int G = (int)goff[8];
  // wave w takes the contiguous groups [G w / 4, G (w + 1) / 4)
  const int gb = (G * wave) / 4, ge = (G * (wave + 1)) / 4;
  // operands of group gi: its slot, the column's parent, that parent's
  // input slice and first child (fetched one group ahead of the MFMAs)
  struct Op {
    int o, p, first;
    bool ev;
    uint32_t pc;
    v4i a[KS];
  };
  auto fetch = [&](int gi, Op& x) {
    int o = 0;
#pragma unroll
    for (int q = 1; q < 8; q++) o += gi >= (int)goff[q] ? 1 : 0;
    const int e = 16 * (gi - (int)goff[o]) + r;  // entry of column r
    x.o = o;
    x.ev = e < (int)cnt[o];
    const int t = x.ev ? (int)list[o][e] : 0;
    x.p = p0 + t;
    x.pc = pcode[t];
    // column operand: k-slice 16 g of the parent's [Z | bits(X)] row
#pragma unroll
    for (int s = 0; s < KS; s++) {
      const int k0 = 64 * s + 16 * g;
      x.a[s] = v4i{0, 0, 0, 0};
      if (x.ev && k0 < C) {
        x.a[s] = ld16(S.in + (int64_t)x.p * S.in_stride + k0);
      } else if (x.ev && k0 == C) {  // occupancy bits as int8 {0,127}, then zeros
        uint32_t w0 = 0, w1 = 0;
#pragma unroll
        for (int b = 0; b < 4; b++) {
          if ((x.pc >> b) & 1u) w0 |= 127u << (8 * b);
          if ((x.pc >> (b + 4)) & 1u) w1 |= 127u << (8 * b);
        }
        x.a[s] = v4i{(int)w0, (int)w1, 0, 0};
      }
    }
    x.first = x.ev ? gp(S.cstart)[x.p] : 0;
  };
  int cur = -1;
  v4i wb[KS][NBS], bb[NBS];
  Op nx;
  if (gb < ge) fetch(gb, nx);
  for (int gi = gb; gi < ge; gi++) {
    const Op x = nx;
    const int o = x.o;
    // weights and biases of slot o (wave-uniform), requested before the next
    // group's operands: the memory counter drains in order, so the waits for
    // these loads then leave the prefetch in flight
    if (o != cur) {
      cur = o;
#pragma unroll
      for (int s = 0; s < KS; s++)
#pragma unroll
        for (int nb = 0; nb < NBS; nb++) wb[s][nb] = Wp[((int64_t)s * NBT + o * NBS + nb) * 64 + lane];
#pragma unroll
      for (int nb = 0; nb < NBS; nb++) bb[nb] = Bp[(o * C + 16 * nb + 4 * g) / 4];
    }
    if (gi + 1 < ge) fetch(gi + 1, nx);
    const bool ev = x.ev;
    const int p = x.p;
    const uint32_t pc = x.pc;
    const int first = x.first;
    (void)p;
    v4i acc[NBS];
#pragma unroll
    for (int nb = 0; nb < NBS; nb++) acc[nb] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; s++)
#pragma unroll
      for (int nb = 0; nb < NBS; nb++) acc[nb] = mfma16(wb[s][nb], x.a[s], acc[nb]);
    // the group's 16 child rows go through the wave's LDS stage, so that
    // every row leaves as whole 16-byte stores (lane (r, g) holds channels
    // 16 nb + 4 g .. + 3 of column r)
    int crow = ev ? first + __popc(pc & ((1u << o) - 1u)) : -1;
    if (crow >= S.child_rows) crow = -1;  // only for a corrupt stream
    if (g == 0) ocrow[wave][r] = crow;
#pragma unroll
    for (int nb = 0; nb < NBS; nb++) {
      uint32_t packed = 0;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int y = requant_l(acc[nb][i] + bb[nb][i], L);
        packed |= ((uint32_t)y & 0xFFu) << (8 * i);
      }
      ost[wave][r][4 * nb + g] = packed;
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane < 16 * NBS) {
      const int row = lane / NBS, part = lane % NBS;
      const int cr = ocrow[wave][row];
      if (cr >= 0) {
        const uint32_t* w = &ost[wave][row][4 * part];
        *(GAS v4i*)(gp(S.out) + (int64_t)cr * S.out_stride + 16 * part) =
            v4i{(int)w[0], (int)w[1], (int)w[2], (int)w[3]};
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// Child convolution (the stride-2 step of the re-densification, Eq. 4) over
// the occupied children only: out[q] = rq(b + sum over children c of q of
// in[c] W[slot(c)]).  A block takes P (64 or 128) consecutive parents, compacts
// them per child slot as the upsampling does, and multiplies 16-entry groups
// of one slot (the slot's weights as the row operand, the 16 children's
// input rows as the columns).  Each lane then holds four consecutive output
// channels of one child's contribution and adds them into its parent's
// int32 accumulator row in LDS (a parent with several children collects one
// contribution per slot; integer adds, so the order does not matter).  The
// accumulators are requantised once all groups are done.  With `ccode` set,
// child c reads row ccode[c] of `in`: the occupancy embedding of depth j
// depends on the code alone, so the first step reads a 256-row table.
template <int C, int P>
__global__ __launch_bounds__(256) void k_down_cx(const GemmSeg* __restrict__ segs, const Tile* __restrict__ tiles,
                                                 const GemmArg A) {
  constexpr int NB = C / 16;
  constexpr int KS = (C + 63) / 64;
  static_assert(C % 16 == 0 && P <= 256 && P % 64 == 0, "shape");
  __shared__ int32_t accs[P][C + 1];
  __shared__ uint8_t list[8][P];
  __shared__ uint8_t pcode[P];
  __shared__ int32_t pfirst[P];
  __shared__ uint32_t wtot[8][P / 64];
  __shared__ uint32_t cnt[8];
  __shared__ uint32_t goff[9];

  GemmSeg S;
  LayerDev L;
  const int q0 = pick_seg(segs, tiles, A, S, L, P);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;

  for (int k = threadIdx.x; k < P * (C + 1); k += 256) (&accs[0][0])[k] = 0;
  uint32_t code = 0u, rk[8];
  if ((int)threadIdx.x < P) {
    const int q = q0 + (int)threadIdx.x;
    code = q < S.rows ? ((uint32_t)gp(S.code)[q] & 0xFFu) : 0u;
    pcode[threadIdx.x] = (uint8_t)code;
    pfirst[threadIdx.x] = q < S.rows ? gp(S.cstart)[q] : 0;
#pragma unroll
    for (int o = 0; o < 8; o++) {
      const uint64_t m = __ballot((code >> o) & 1u);
      rk[o] = lanes_below(m);
      if (lane == 0) wtot[o][wave] = (uint32_t)__popcll(m);
    }
  }
  __syncthreads();
  if ((int)threadIdx.x < P) {
#pragma unroll
    for (int o = 0; o < 8; o++) {
      if (!((code >> o) & 1u)) continue;
      uint32_t before = rk[o];
      for (int w = 0; w < wave; w++) before += wtot[o][w];
      list[o][before] = (uint8_t)threadIdx.x;
    }
  }
  if (threadIdx.x < 8) {
    uint32_t n = 0;
    for (int w = 0; w < P / 64; w++) n += wtot[threadIdx.x][w];
    cnt[threadIdx.x] = n;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t gsum = 0;
    for (int o = 0; o < 8; o++) {
      goff[o] = gsum;
      gsum += (cnt[o] + 15) / 16;
    }
    goff[8] = gsum;
  }
  __syncthreads();

  const GAS v4i* Wp = (const GAS v4i*)L.Wp;
  const int G = (int)goff[8];
  const int gb = (G * wave) / 4, ge = (G * (wave + 1)) / 4;
  // operands of group gi: its slot, the column's parent and child, the
  // child's input slice (fetched one group ahead of the MFMAs)
  struct Op {
    int o, t;
    bool cv;
    v4i a[KS];
  };
  auto fetch = [&](int gi, Op& x) {
    int o = 0;
#pragma unroll
    for (int q = 1; q < 8; q++) o += gi >= (int)goff[q] ? 1 : 0;
    const int e = 16 * (gi - (int)goff[o]) + r;  // entry of column r
    const bool ev = e < (int)cnt[o];
    const int t = ev ? (int)list[o][e] : 0;
    const uint32_t pc = pcode[t];
    const int c = pfirst[t] + __popc(pc & ((1u << o) - 1u));
    x.o = o;
    x.t = t;
    x.cv = ev && c < S.child_rows;  // out of range only for a corrupt stream
    const int64_t src = !x.cv ? 0 : (S.ccode != nullptr ? (int64_t)gp(S.ccode)[c] : (int64_t)c);
#pragma unroll
    for (int s = 0; s < KS; s++) {
      const int k0 = 64 * s + 16 * g;
      x.a[s] = v4i{0, 0, 0, 0};
      if (x.cv && k0 < C) x.a[s] = ld16(S.in + src * S.in_stride + k0);
    }
  };
  int cur = -1;
  v4i wb[KS][NB];
  Op nx;
  if (gb < ge) fetch(gb, nx);
  for (int gi = gb; gi < ge; gi++) {
    const Op x = nx;
    const int o = x.o;
    // the slot's weights (rows k = o C + c of the packed layout), requested
    // before the next group's operands so that waiting for them leaves the
    // prefetch in flight (the memory counter drains in order)
    if (o != cur) {
      cur = o;
#pragma unroll
      for (int s = 0; s < KS; s++) {
        const bool kv = 64 * s + 16 * g < C;
        const int ko = kv ? o * C + 64 * s + 16 * g : 0;
        const GAS v4i* w = Wp + (int64_t)(ko >> 6) * NB * 64 + ((ko >> 4) & 3) * 16 + r;
#pragma unroll
        for (int nb = 0; nb < NB; nb++) {
          const v4i y = w[kv ? nb * 64 : 0];
          wb[s][nb] = kv ? y : v4i{0, 0, 0, 0};
        }
      }
    }
    if (gi + 1 < ge) fetch(gi + 1, nx);
    const int t = x.t;
    const bool cv = x.cv;
    v4i acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; nb++) acc[nb] = v4i{0, 0, 0, 0};
#pragma unroll
    for (int s = 0; s < KS; s++)
#pragma unroll
      for (int nb = 0; nb < NB; nb++) acc[nb] = mfma16(wb[s][nb], x.a[s], acc[nb]);
    if (!cv) continue;
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
      for (int i = 0; i < 4; i++) atomicAdd(&accs[t][16 * nb + 4 * g + i], acc[nb][i]);
  }
  __syncthreads();

  // requantise: thread (row, 4-channel group), rows in steps of 256 / (C / 4)
  constexpr int LPR = C / 4;
  const int c4 = (threadIdx.x % LPR) * 4;
  int bia[4];
#pragma unroll
  for (int q = 0; q < 4; q++) bia[q] = gp(L.bias)[c4 + q];
  for (int t = threadIdx.x / LPR; t < P; t += 256 / LPR) {
    const int q = q0 + t;
    if (q >= S.rows) break;
    const uint32_t pc = pcode[t];
    uint32_t packed = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      int a = accs[t][c4 + k] + bia[k];
      if (L.zc != nullptr) {
        for (int o = 0; o < 8; o++)
          if ((pc >> o) & 1u) a += gp(L.zc)[o * L.npad + c4 + k];
      }
      packed |= ((uint32_t)requant_l(a, L) & 0xFFu) << (8 * k);
    }
    *(GAS uint32_t*)(gp(S.out) + (int64_t)q * S.out_stride + c4) = packed;
  }
}

hipError_t launch_down_cx(int C, const GemmSeg* segs, const Tile* tiles, int ntiles, const GemmArg& A, int P,
                          hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
#define LPCC_D(CC, PP)                                                                                 \
  if (C == CC && P == PP) {                                                                            \
    hipLaunchKernelGGL((k_down_cx<CC, PP>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);            \
    return hipGetLastError();                                                                          \
  }
  LPCC_D(16, 64) LPCC_D(16, 128) LPCC_D(32, 64) LPCC_D(32, 128) LPCC_D(64, 64) LPCC_D(64, 128)
#undef LPCC_D
  return hipErrorInvalidValue;
}

hipError_t launch_up_cx(int C, const GemmSeg* segs, const Tile* tiles, int ntiles, const GemmArg& A, int P,
                        hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
#define LPCC_U(CC, PP)                                                                                 \
  if (C == CC && P == PP) {                                                                            \
    hipLaunchKernelGGL((k_up_cx<CC, PP>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);              \
    return hipGetLastError();                                                                          \
  }
  LPCC_U(16, 128) LPCC_U(16, 512) LPCC_U(32, 128) LPCC_U(32, 512) LPCC_U(64, 128) LPCC_U(64, 512)
#undef LPCC_U
  return hipErrorInvalidValue;
}

hipError_t launch_up(int C, const GemmSeg* segs, const Tile* tiles, int ntiles, const GemmArg& A, int rb,
                     hipStream_t s) {
  if (ntiles <= 0) return hipSuccess;
#define LPCC_U(CC)                                                                                 \
  if (C == CC) {                                                                                   \
    if (rb == 4) hipLaunchKernelGGL((k_up<CC, 4>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A); \
    else if (rb == 2) hipLaunchKernelGGL((k_up<CC, 2>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A); \
    else hipLaunchKernelGGL((k_up<CC, 1>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);         \
    return hipGetLastError();                                                                      \
  }
  LPCC_U(16) LPCC_U(32)
#undef LPCC_U
  if (C == 64) {
    if (rb == 4) hipLaunchKernelGGL((k_up_staged<64, 4>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);
    else if (rb == 2) hipLaunchKernelGGL((k_up_staged<64, 2>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);
    else hipLaunchKernelGGL((k_up_staged<64, 1>), dim3(ntiles), dim3(256), 0, s, segs, tiles, A);
    return hipGetLastError();
  }
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
    gp(S.out)[(int64_t)row * S.out_stride + o] = (int8_t)requant_l(acc, L);
  }
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
// (pack_logits), so that lane (r, g) ends with the 64 consecutive symbols
// 64g .. 64g + 63 of ONE node, r.  Everything per node (M, S, the reciprocal,
// the coded symbol) is then a per-lane value: the reductions run over the 4
// lanes of a node, the prefix sums are serial inside a lane, and the biases
// ride in the accumulators.  fc1's accumulators are already fc2's column
// operand (the permutation of K is in the packed weights), so no activations
// pass through LDS.
//
// The kernel is bound by vector instruction issue: this form needs 17.2
// vector instructions per 64 logits in encode mode where the one with 16 lanes
// per node needed 30.4, and for the 12.75 M nodes of 8 128-beam frames (18
// levels, C = 64) it takes 1.58 ms where that took 2.39 ms.
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
// logits comes first), so the asm needs no wait states it cannot see.
__device__ __forceinline__ uint32_t freq_add(uint32_t run, uint32_t E, uint32_t S, uint32_t K) {
  uint32_t m, t, o;
  asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(m) : "v"(E), "v"(K), "s"(0x10000));
  asm("v_mul_u32_u24_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD"
      : "=v"(t)
      : "v"(m), "v"(S));
  const uint32_t p = __umul24(E & 0xFFFFu, 65281u);
  asm("v_cmp_le_u32_e32 vcc, %1, %2\n\t"
      "v_addc_co_u32_sdwa %0, vcc, %3, %4, vcc dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:WORD_1"
      : "=v"(o)
      : "v"(t), "v"(p), "v"(run), "v"(m)
      : "vcc");
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

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
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
#pragma unroll
  for (int j = 0; j < NS; j++) {
    const uint32_t next = freq_add(run, (uint32_t)e[j], n.S, n.K);
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
// at most 128 VGPRs (four waves per SIMD); the general requantisation needs more
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
// 18 depths of 8 128-beam frames (12.75 M nodes) 2.28 + 1.92 ms became 2.99
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

template <int C, int NP, int RQ>
__global__ __launch_bounds__(64 * (NP + 1)) __attribute__((amdgpu_waves_per_eu(RQ == 1 ? 4 : 3))) void k_decode_chunks(
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
// compute unit more chunks at once: the 8-frame 128-beam batch decodes in
// 10.17 ms with 2 and 10.42 ms with 3, one such frame (at most 920 chunks) in
// 2.58 and 2.54 ms.
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
