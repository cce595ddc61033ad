// Implicit-GEMM convolution over two-dimensional output tiles (gfx950): any
// stencil, any strides, any feature counts, no workspace.
//
// The paper's tile schedule (Sec. 2.1, Listing 3 with W_c = N_c): a workgroup
// keeps a tile of tk features by up to tp outputs in accumulators and walks
// the input features tc = 16 KS at a time.  The outputs of a tile are a run
// of tr whole output rows of the flattened (b, w) index (plan.tp = tr * Nh);
// where such a run holds more outputs than a workgroup's accumulators, it is
// cut into ncol bands of ct columns, one workgroup each, so that the halo of
// a wide image stays that of a two-dimensional tile.
//
// * In: a work item is 16 bytes of a row (8 columns of bf16, 4 of fp32) of each
//   of 8 channels, at any alignment of an element (h strides 1 and 2; the last
//   item of a row ends with it, so no load leaves its row), or a pair of columns
//   (larger strides, the narrowest bands), transposed in registers (v_perm) into
//   16-byte [8 channels] vectors, one a column.  LDS holds [channel group][row][column],
//   columns split by their residue modulo the h stride, so that a tap's
//   operand is a run of consecutive vectors for any stride.  Rows and
//   (1-wide stencils) columns that no output reads are not staged.
// * Ker: loaded as it lies -- the taps of two neighbouring channels (bf16) or
//   of one (fp32) of a feature, along its contiguous (c, r, s) run, at any
//   2-byte alignment -- and written in pairs of channels in the operand order
//   [tap][c/8][k][8], so no repack kernel, no workspace and no condition on
//   the feature count or the stencil.
// * Both operands of a product are then single 16-byte LDS reads.  Two LDS
//   buffers; while stage i multiplies, stage i + 1 is written to the other
//   buffer piece by piece, each piece's registers taking its share of stage
//   i + 2 at once, so that a load has a whole stage to land and the matrix
//   units do not wait for a staging phase; one barrier per stage.
// * What bounds it: LDS bandwidth and vector instruction issue beside the
//   products (64 -> 64 features at 224x224, 3x3, batch 8, bf16 Out: 41.8 us as one
//   kernel, 44 a call of many; matrix units busy 44 % of the cycles, LDS 38 %).
//   On that layer, kernel alone, from 96 us of the whole-row tiles (whose slab is
//   2.2 times the outputs): 63 with this tile and dword loads, 54 with the
//   staging between the products, 50 with 16-byte loads and Out through LDS,
//   44 with Ker in channel pairs, 42 with two workgroups per CU.
// * fp32 (CNN_F32): In and Ker values are split into three bf16 parts that
//   sum to them exactly (truncation, then two roundings: 8 + 8 + 8 bits) and
//   the six products of combined order up to 2^-16 are accumulated in fp32 by
//   the bf16 units, 16 times the rate of the fp32 ones; the leading one in a
//   sum of its own, which is rounded once for 8 channels of a tap where the
//   fp32 units round for every two.  The error against 64 bits (2-norm, uniform
//   inputs) is 0.3 to 0.8 of theirs from four products a sum on: 1.2e-7 and
//   3.5e-7 on 64 channels 3x3, 3.4e-8 and 3.9e-8 on 4 channels 1x1; with one
//   sum for all six it was 3.5e-7 there, and above theirs (4.0e-8 and 2.6e-8,
//   1x1, 1 channel; 1.9e-7 and 1.8e-7, 10 channels 3x3) for few channels or
//   few in the last eight.  What is dropped (up to 4 units of 2^-24 a
//   product) would show in shorter sums: those below eight products take the
//   fp32 units.  The parts of infinities
//   do not work that way, nor do products that overflow, and values below
//   2^-102 (other than zero) lose a part of theirs: a workgroup where that shows
//   in a sum computes its tile again on the fp32 units (64 -> 64 features 3x3 at
//   56x56, batch 16: 84 us for 30.5; the fp32 units' staging tiles 82; with unstaged
//   4-byte loads of Ker the second pass came to 98).
#pragma once

#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "common.h"

namespace cnnlib {

// What a launch fixes beyond ConvArgs (made on the host).
struct TileGeo {
  int32_t tr, ct, ncol;   // rows per tile, columns per band, bands
  int32_t rows_total;     // Nb * Nw output rows
  int32_t pitch, hp;      // LDS row pitch and columns per residue (vectors)
  int32_t SP;             // LDS vectors per channel group
  int32_t squeeze;        // 1: only the Nr rows each output row reads are staged
  int32_t nch;            // Ker items per feature and stage (1x1, runtime stencils)
  int32_t njt;            // runtime stencils: runs of taps per channel
  int32_t nst;            // stages
  int32_t units;          // (fp32) 1: computed on the fp32 units
  FastDiv kt, ncold, nw, nx, nr, nchd, njd, shd, rsd, nsd;
  FastDiv ipr, ctd;       // work items per row and columns of a band
};

__device__ __forceinline__ f32x16_t mfma_t(const u32x4_t& a, const u32x4_t& b, const f32x16_t& c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a),
                                                 __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
}

// How a row's columns are staged: in items of two (any stride; 1-wide
// stencils stage only the columns the outputs read), or in items of 16 bytes
// per channel -- 8 columns (bf16) or 4 (fp32) -- at h stride 1 or 2, and at
// stride 2 with a 1-wide stencil, where an item is that many outputs' columns.
enum { kPairs = 0, kWide1 = 1, kWide2 = 2, kGather2 = 3 };

// LDS stride of a (tap, channel group) row of Ker, and the extra bytes per 8
// taps of runtime stencils: the lanes of a staging write then meet distinct
// banks (3x3: eight features x the eight channel pairs of two groups; runtime
// stencils: four runs of 8 taps x eight channel pairs x two features; 1x1: the
// channel groups of a feature).
__host__ __device__ constexpr int tile_ker_row(int tk, int es, int taps) {
  return tk * 8 * es + (taps == 9 ? 128 : taps == 1 ? 16 : 32);
}
constexpr int kTapPad = 64;
__host__ __device__ constexpr int tile_ker_bytes(int tk, int es, int taps_fixed, int groups, int rs) {
  return rs * groups * tile_ker_row(tk, es, taps_fixed) + (taps_fixed ? 0 : (rs - 1) / 8 * kTapPad);
}

template <int N, int I = 0, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>());
    static_for<N, I + 1>(f);
  }
}

// Two fp32 values as three pairs of bf16 that sum to them exactly: the top
// 8 bits (truncated, so that the largest values do not round to infinity),
// then the rest rounded to nearest, then what that rounding left.
struct Split3 {
  uint32_t p[3];
};
__device__ __forceinline__ Split3 split3(float x, float y) {
  const uint32_t xu = __float_as_uint(x), yu = __float_as_uint(y);
  Split3 r;
  r.p[0] = __builtin_amdgcn_perm(yu, xu, 0x07060302u);
  const float x1 = x - __uint_as_float(xu & 0xffff0000u), y1 = y - __uint_as_float(yu & 0xffff0000u);
  r.p[1] = pk_bf16(x1, y1);
  r.p[2] = pk_bf16(x1 - __uint_as_float(r.p[1] << 16), y1 - __uint_as_float(r.p[1] & 0xffff0000u));
  return r;
}

// The largest of the values staged (twice its bits) in `hi`, and in `lo` the
// least other than zero: below 2^-102 its last part may be subnormal.
struct SplitRange {
  uint32_t hi = 0u, lo = ~0u;
  __device__ __forceinline__ void see(uint32_t x) {
    const uint32_t m = x << 1;
    hi = max(hi, m);
    lo = min(lo, m - 1u);  // zero becomes the largest
  }
  __device__ __forceinline__ bool small() const { return lo < (25u << 24) - 1u; }
};

// Workgroups per CU that the registers of an instantiation leave room for.  fp32
// on four waves: two, not one, within 256 registers a lane, at 19 spilled ones for
// runtime stencils (16 -> 32 features 1x1 at 94x94, batch 22: 24.6 -> 16.1 us) and
// without accumulators to be copied out for 3x3 (16 -> 129 at 60x60, batch 6: 17.5
// -> 16.4); not the gathered form, which would spill more.
template <typename TI, int NW, int OCC, int FORM> constexpr int tile_occ() {
  return std::is_same<TI, float>::value && NW == 4 && FORM != kGather2 ? 2 : OCC;
}

// TI: bf16_t or float; TO: the Out type.  WM x WN = 4 waves, MB x NB blocks
// of 32 features x 32 outputs per wave, KS K-steps of 16 channels per stage,
// NR x NS the stencil (0: any), MAXP In items and KCH Ker items per
// thread, OCC workgroups per CU.  FORM: how columns are staged (kPairs ...).
template <typename TI, typename TO, int WM, int WN, int MB, int NB, int KS, int NR, int NS,
          int MAXP, int KCH, int OCC, int FORM>
__global__ __launch_bounds__(64 * WM * WN, (tile_occ<TI, WM * WN, OCC, FORM>() * WM * WN / 4)) void conv_tile(const TI* __restrict__ In,
                                                      const TI* __restrict__ Ker,
                                                      TO* __restrict__ Out, ConvArgs a,
                                                      TileGeo t) {
  constexpr bool F32 = std::is_same<TI, float>::value;
  constexpr int ES = (int)sizeof(TI);
  constexpr int TK = 32 * WM * MB;
  constexpr int TC = 16 * KS;
  constexpr int G = 2 * KS;                 // channel groups per stage
  constexpr int GPW = G > WM * WN ? G / (WM * WN) : 1;    // groups per wave
  constexpr int WPG = G < WM * WN ? WM * WN / G : 1;    // waves per group
  constexpr int PT = 64 * WPG;              // threads sharing a group's positions
  constexpr int PL = F32 ? 3 : 1;           // bf16 planes of In in LDS
  constexpr int EPC = 16 / ES;              // Ker elements per chunk
  constexpr int KB = 8 * ES;                // bytes of 8 channels of one feature
  constexpr int ARS = tile_ker_row(TK, ES, NR * NS);  // LDS stride of a (tap, group) row of Ker
  const int Nr = NR ? NR : a.Nr, Ns = NS ? NS : a.Ns;
  const int RS = Nr * Ns;
  constexpr bool WIDE = FORM != kPairs;
  constexpr int PW = WIDE ? EPC : 2;        // columns of a work item
  constexpr int DW = PW * ES / 4;           // dwords of a channel's item
  constexpr int NL = FORM == kGather2 ? 2 : 1;  // loads of a channel's item
  const bool gather = FORM == kGather2 || (FORM == kPairs && Ns == 1 && a.sh > 1);
  constexpr int NW = WM * WN, NT = 64 * NW;
  // Ker: K9 (3x3) and K1 (1x1) stencils have staging of their own
  constexpr bool K9 = NR == 3 && NS == 3, K1 = NR == 1 && NS == 1;
  static_assert(NW == 4 || NW == 8, "four or eight waves");

  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int in_bytes = PL * G * t.SP * 16;
  const int buf_bytes = in_bytes + tile_ker_bytes(TK, ES, NR * NS, G, RS);
  // (bf16) the tensor's last element: see the ragged write below
  uint32_t ker_last = 0u;
  if constexpr (!F32) ker_last = Ker[(int64_t)a.Nk * a.Nc * RS - 1];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // (scalar: wave-uniform offsets)
  const int wm = wave / WN, wn = wave % WN;
  const int l32 = lane & 31, half = lane >> 5;

  // ---- the tile: features k0.., output rows row0.., columns h0..
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int rest = fdiv(tile, t.kt);
  const int k0 = (tile - rest * a.n_ktiles) * TK;
  const int rt = fdiv(rest, t.ncold);
  const int band = rest - rt * t.ncol;
  // (the last band may overlap its neighbour.  bf16: both store the same values
  // there; fp32: the neighbour alone stores them, as one of the two may compute
  // its tile on the fp32 units, which rounds differently)
  const int h0 = min(band * t.ct, a.Nh - t.ct);
  const int own = F32 ? band * t.ct - h0 : 0;  // first column of the tile that is stored
  const int row0 = rt * t.tr;
  const int rows = min(t.tr, t.rows_total - row0);
  const int cols = t.ct;
  const int b0 = fdiv(row0, t.nw);
  const int G0 = b0 * a.Nx + a.sw * (row0 - b0 * a.Nw);  // first input row (flattened b, x)
  int S;                                                  // staged rows
  if (t.squeeze) {
    S = rows * Nr;
  } else {
    const int rl = row0 + rows - 1;
    const int b1 = fdiv(rl, t.nw);
    S = b1 * a.Nx + a.sw * (rl - b1 * a.Nw) + Nr - G0;
  }
  const int cw = gather ? cols : a.sh * (cols - 1) + Ns;  // staged columns
  const int ipr = (cw + PW - 1) / PW;                     // work items per row
  const int nitems = S * ipr;

  // ---- In work items
  const int grp0 = WPG > 1 ? wave / WPG : wave * GPW;  // first channel group of the wave
  const int pt0 = WPG > 1 ? (wave % WPG) * 64 + lane : lane;
  const __amdgpu_buffer_rsrc_t ir = rsrc_words(In + (int64_t)b0 * a.in_img,
                                           (a.in_total - (int64_t)b0 * a.in_img) * ES);
  // Lanes write 8 consecutive vectors each, 128 bytes apart: half of them
  // write the columns of each pair in the other order, which spreads the
  // writes over twice the banks.
  constexpr bool SWAP = !F32 && (FORM == kWide1 || FORM == kWide2);
  const bool swp = (lane >> (FORM == kWide1 ? 1 : 2)) & 1;
  const uint32_t sel_e = SWAP && swp ? 0x07060302u : 0x05040100u;
  const uint32_t sel_o = SWAP && swp ? 0x05040100u : 0x07060302u;
  uint32_t voff[MAXP];
  uint32_t dst[MAXP];  // LDS vectors of the item's first two columns, 16 bits each
#pragma unroll
  for (int j = 0; j < MAXP; ++j) {
    const int q = min(pt0 + PT * j, nitems - 1);
    const int row = fdiv(q, t.ipr);
    const int col = min(PW * (q - row * ipr), cw - PW);
    int b, x;
    if (t.squeeze) {
      const int i = NR ? row / (NR ? NR : 1) : fdiv(row, t.nr);
      const int orow = row0 + i;
      b = fdiv(orow, t.nw);
      x = (orow - b * a.Nw) * a.sw + row - i * Nr;
    } else {
      const int gr = G0 + row;
      b = fdiv(gr, t.nx);
      x = gr - b * a.Nx;
    }
    const int y = a.sh * h0 + (gather ? a.sh * col : col);
    voff[j] = (uint32_t)(((int64_t)(b - b0) * a.in_img + (int64_t)x * a.Ny + y) * ES);
    int d0 = col, d1 = col + 1;
    if ((FORM == kPairs && !gather && a.sh > 1) || FORM == kWide2) {
      const int q0 = FORM == kWide2 ? d0 >> 1 : fdiv(d0, t.shd);
      const int q1 = FORM == kWide2 ? d1 >> 1 : fdiv(d1, t.shd);
      d0 = (d0 - q0 * a.sh) * t.hp + q0;
      d1 = (d1 - q1 * a.sh) * t.hp + q1;
    }
    if (SWAP && swp) {
      const int x = d0;
      d0 = d1;
      d1 = x;
    }
    dst[j] = (uint32_t)(row * t.pitch + d0) | ((uint32_t)(row * t.pitch + d1) << 16);
  }

  // ---- Ker work items, CPI channels of one feature each.  3x3: all nine taps,
  // 36 contiguous bytes.  1x1: 16 bytes of channels.  Runtime stencils: a run
  // of TPI taps (the last run of a longer stencil ends with its last tap).
  const int64_t ker_total = (int64_t)a.Nk * a.Nc * RS;
  const __amdgpu_buffer_rsrc_t kr = rsrc_words(Ker, ker_total * ES);
  constexpr int CPI = K1 ? EPC : F32 ? 1 : 2;
  constexpr int TPI = 16 / ES;
  constexpr int CI = TC / CPI;  // channel items of a stage
  constexpr int NK = K9 ? TK * CI / NT : KCH;
  static_assert(!K9 || NK * NT == TK * CI, "whole items per thread");
  // per item: byte offset in Ker (stage 0), LDS byte offset, and its feature
  // (low), channel (bits 8..15 of the high half) and first tap (low 8)
  uint32_t kdst[NK];
#pragma unroll
  for (int j = 0; j < NK; ++j) {
    if constexpr (K9) {
      const int v = tid + NT * j;
      kdst[j] = (uint32_t)(v / CI) | ((uint32_t)(v % CI * CPI) << 24);
    } else {
      const int v = min(tid + NT * j, TK * t.nch - 1);
      const int kk = fdiv(v, t.nchd);
      const int part = v - kk * t.nch;
      if constexpr (K1) {
        kdst[j] = (uint32_t)kk | ((uint32_t)(part * CPI) << 24);
      } else {
        const int ci = fdiv(part, t.njd);
        const int t0 = max(0, min(TPI * (part - ci * t.njt), RS - TPI));
        kdst[j] = (uint32_t)kk | ((uint32_t)(ci * CPI) << 24) | ((uint32_t)t0 << 16);
      }
    }
  }
  const uint32_t krow = (uint32_t)(a.Nc * RS * ES);  // bytes of a feature
  auto koff = [&](int j) -> uint32_t {
    return (uint32_t)min(k0 + (int)(kdst[j] & 0xffffu), a.Nk - 1) * krow +
           ((kdst[j] >> 24) * RS + (K9 || K1 ? 0u : (kdst[j] >> 16) & 0xffu)) * ES;
  };

  // A stage's staging is cut into NP pieces (an In item or a Ker chunk of
  // every thread), so that it can run between the products.
  constexpr int NPI = GPW * MAXP, NP = NPI + NK;
  uint32_t pre[NPI][8][NL][DW];
  uint32_t kpre[NK][K9 ? 9 : K1 || F32 ? 4 : 8];
  const uint32_t plane = (uint32_t)a.nxny * ES;

  auto load = [&](auto pc, int st) __attribute__((always_inline)) {
    constexpr int P = decltype(pc)::value;
    const int c0 = st * TC;
    if constexpr (P < NPI) {
      constexpr int g = P / MAXP, j = P % MAXP;
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        // a channel past Nc loads channel Nc - 1; the write zeroes it
        const uint32_t so = (uint32_t)min(c0 + 8 * (grp0 + g) + i, a.Nc - 1) * plane;
        if constexpr (WIDE) {
          // (gathered: outputs' columns 0, 2, 4, .. in the even elements of
          // the first load and the odd ones of the second, which starts one
          // column before the next so as not to leave the row)
#pragma unroll
          for (int l = 0; l < NL; ++l) {
            const u32x4_t d = __builtin_bit_cast(
                u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                             ir, voff[j] + l * (EPC - 1) * ES, so, 0));
#pragma unroll
            for (int e = 0; e < 4; ++e) pre[P][i][l][e] = d[e];
          }
        } else if constexpr (F32) {
          pre[P][i][0][0] = __builtin_amdgcn_raw_buffer_load_b32(ir, voff[j], so, 0);
          pre[P][i][0][1] =
              __builtin_amdgcn_raw_buffer_load_b32(ir, voff[j] + (gather ? a.sh * 4 : 4), so, 0);
        } else {
          pre[P][i][0][0] = __builtin_amdgcn_raw_buffer_load_b32(ir, voff[j], so, 0);
          if (gather) {  // the second output's column is the last of another pair
            const uint32_t hi =
                __builtin_amdgcn_raw_buffer_load_b32(ir, voff[j] + (a.sh - 1) * 2, so, 0);
            pre[P][i][0][0] = __builtin_amdgcn_perm(hi, pre[P][i][0][0], 0x07060100u);
          }
        }
      }
    } else {
      constexpr int j = P - NPI;
      const uint32_t ko = koff(j), so = (uint32_t)(c0 * RS * ES);
      const u32x4_t d =
          __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(kr, ko, so, 0));
#pragma unroll
      for (int e = 0; e < 4; ++e) kpre[j][e] = d[e];
      if constexpr (K9) {
        const u32x4_t d2 =
            __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(kr, ko + 16, so, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) kpre[j][4 + e] = d2[e];
        kpre[j][8] = __builtin_amdgcn_raw_buffer_load_b32(kr, ko + 32, so, 0);
      } else if constexpr (!K1 && !F32) {  // the second channel
        const u32x4_t d2 = __builtin_bit_cast(
            u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(kr, ko + RS * ES, so, 0));
#pragma unroll
        for (int e = 0; e < 4; ++e) kpre[j][4 + e] = d2[e];
      }
    }
  };

  // LDS offset of tap q's rows, and what tap t0 + e adds to t0's besides e rows
  auto tap_off = [&](int q) -> int { return q * G * ARS + (NR ? 0 : (q >> 3) * kTapPad); };
  auto tap_pad = [&](int t0, int e) -> int { return (((t0 & 7) + e) >> 3) * kTapPad; };

  SplitRange range;  // (fp32) of the values staged

  // RAG: the stage may hold channels past Nc (only the last one does): they
  // become zero on both sides.
  auto write = [&](auto pc, auto rg, int st, char* buf) __attribute__((always_inline)) {
    constexpr int P = decltype(pc)::value;
    constexpr bool RAG = decltype(rg)::value;
    const int c0 = st * TC;
    if constexpr (P < NPI) {
      constexpr int g = P / MAXP, j = P % MAXP;
      u32x4_t* ib = reinterpret_cast<u32x4_t*>(buf);
      const int grp = grp0 + g;
      const int left = a.Nc - c0 - 8 * grp;  // channels of the group that exist
      if (pt0 + PT * j >= nitems) return;
      // column e of the item: vector (e even ? v0 : v1) + (e / 2) * INC
      constexpr int INC = FORM == kWide2 ? 1 : 2;
      const int v0 = grp * t.SP + (int)(dst[j] & 0xffffu), v1 = grp * t.SP + (int)(dst[j] >> 16);
#pragma unroll
      for (int e = 0; e < PW; ++e) {
        const int v = ((e & 1) ? v1 : v0) + (e >> 1) * INC;
        // where column e lies in the item's loads
        const int l = NL == 2 ? e / (EPC / 2) : 0;
        const int x = NL == 2 ? 2 * (e % (EPC / 2)) + l : e;
        if constexpr (F32) {
          u32x4_t p[3];
#pragma unroll
          for (int i = 0; i < 8; i += 2) {
            float w0 = __uint_as_float(pre[P][i][l][x]), w1 = __uint_as_float(pre[P][i + 1][l][x]);
            if (RAG && i >= left) w0 = 0.f;
            if (RAG && i + 1 >= left) w1 = 0.f;
            range.see(__float_as_uint(w0));
            range.see(__float_as_uint(w1));
            const Split3 h = split3(w0, w1);
#pragma unroll
            for (int z = 0; z < 3; ++z) p[z][i >> 1] = h.p[z];
          }
#pragma unroll
          for (int z = 0; z < 3; ++z) ib[z * G * t.SP + v] = p[z];
        } else {
          u32x4_t w;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            uint32_t e0 = pre[P][2 * i][l][x >> 1], e1 = pre[P][2 * i + 1][l][x >> 1];
            if (RAG && 2 * i >= left) e0 = 0u;
            if (RAG && 2 * i + 1 >= left) e1 = 0u;
            w[i] = __builtin_amdgcn_perm(e1, e0, (x & 1) ? sel_o : sel_e);
          }
          ib[v] = w;
        }
      }
    } else {
      constexpr int j = P - NPI;
      if (!K9 && tid + NT * j >= TK * t.nch) return;
      const int kk = (int)(kdst[j] & 0xffffu), c = (int)(kdst[j] >> 24);
      char* base = buf + in_bytes + kk * KB + (c >> 3) * ARS + (c & 7) * ES;
      const int left = a.Nc - c0 - c;  // channels of the item that exist
      // the tensor's last element is lost to the range check when a dword
      // straddles the tensor's end
      const bool kend = RAG && !F32 && k0 + kk >= a.Nk - 1;
      if constexpr (K1) {
        u32x4_t w = {kpre[j][0], kpre[j][1], kpre[j][2], kpre[j][3]};
        if constexpr (RAG) {
#pragma unroll
          for (int i = 0; i < EPC; ++i) {
            if constexpr (F32) {
              if (i >= left) w[i] = 0u;
            } else {
              const uint32_t sh = 16 * (i & 1), m = 0xffffu << sh;
              if (kend && i == left - 1) w[i >> 1] = (w[i >> 1] & ~m) | (ker_last << sh);
              if (i >= left) w[i >> 1] &= ~m;
            }
          }
        }
        if constexpr (F32) {
#pragma unroll
          for (int i = 0; i < 4; ++i) range.see(w[i]);
        }
        *reinterpret_cast<u32x4_t*>(base) = w;
      } else if constexpr (F32) {
        const int t0 = K9 ? 0 : (int)((kdst[j] >> 16) & 0xffu);
        if (!K9) base += tap_off(t0);
#pragma unroll
        for (int e = 0; e < (K9 ? 9 : TPI); ++e)
          if (K9 || t0 + e < RS) {
            const uint32_t w = RAG && left < 1 ? 0u : kpre[j][e];
            range.see(w);
            *reinterpret_cast<uint32_t*>(base + e * G * ARS + (K9 ? 0 : tap_pad(t0, e))) = w;
          }
      } else {
        // tap e of the two channels: halves e and 9 + e of the 3x3 run, else
        // half e of each load
        uint32_t wl[K9 ? 9 : 8];
#pragma unroll
        for (int e = 0; e < (K9 ? 9 : 8); ++e) wl[e] = kpre[j][e];
        const int t0 = K9 ? 0 : (int)((kdst[j] >> 16) & 0xffu);
        if constexpr (RAG) {
          if constexpr (K9) {
            if (kend && left == 1) wl[4] = ker_last;
          } else if (RS < 8) {
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (kend && e == RS - 1) {
                const uint32_t sh = 16 * (e & 1), m = 0xffffu << sh;
                if (left == 1) wl[e >> 1] = (wl[e >> 1] & ~m) | (ker_last << sh);
                if (left == 2) wl[4 + (e >> 1)] = (wl[4 + (e >> 1)] & ~m) | (ker_last << sh);
              }
          }
        }
        if (!K9) base += tap_off(t0);
#pragma unroll
        for (int e = 0; e < (K9 ? 9 : 8); ++e) {
          const uint32_t lo = wl[e >> 1], hi = K9 ? wl[(9 + e) >> 1] : wl[4 + (e >> 1)];
          // both halves low or high, or (3x3) of opposite parity
          uint32_t w = __builtin_amdgcn_perm(
              hi, lo, K9 ? ((e & 1) ? 0x05040302u : 0x07060100u)
                         : ((e & 1) ? 0x07060302u : 0x05040100u));
          if (RAG && left < 2) w = left < 1 ? 0u : w & 0xffffu;
          if (K9 || t0 + e < RS)
            *reinterpret_cast<uint32_t*>(base + e * G * ARS + (K9 ? 0 : tap_pad(t0, e))) = w;
        }
      }
    }
  };

  static_for<NP>([&](auto pc) __attribute__((always_inline)) { load(pc, 0); });

  // ---- while stage 0 is on its way: a lane's LDS positions (lanes past the
  // tile's last output take its place)
  const int nout = rows * cols;
  int pix[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const int q = min((wn * NB + nb) * 32 + l32, nout - 1);
    const int i = fdiv(q, t.ctd);
    int row = i * Nr;
    if (!t.squeeze) {
      const int orow = row0 + i;
      const int b = fdiv(orow, t.nw);
      row = b * a.Nx + a.sw * (orow - b * a.Nw) - G0;
    }
    pix[nb] = row * t.pitch + q - i * cols + half * t.SP;
  }

  // (fp32: the products of the leading parts, and apart from them the small ones)
  f32x16_t acc[MB][NB], low[F32 ? MB : 1][F32 ? NB : 1];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int j = 0; j < 16; ++j) {
        acc[mb][nb][j] = 0.f;
        if constexpr (F32) low[mb][nb][j] = 0.f;
      }

  // One product step's operands: MB blocks of Ker, NB of In (fp32: the Ker
  // values as they are, split when they are used, and the parts of In).
  constexpr int PA = F32 ? 2 : 1;
  struct Ops {
    u32x4_t a[MB][PA], b[NB][PL];
  };
  auto fetch = [&](Ops& o, const char* buf, int tap, int ks, int toff) __attribute__((always_inline)) {
    const u32x4_t* src = reinterpret_cast<const u32x4_t*>(buf) + 2 * ks * t.SP + toff;
    const char* ka = buf + in_bytes + half * ARS + (wm * MB * 32 + l32) * KB + tap_off(tap) +
                     2 * ks * ARS;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int z = 0; z < PA; ++z)
        o.a[mb][z] = *reinterpret_cast<const u32x4_t*>(ka + mb * 32 * KB + 16 * z);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int z = 0; z < PL; ++z) o.b[nb][z] = src[z * G * t.SP + pix[nb]];
  };
  auto multiply = [&](const Ops& o) __attribute__((always_inline)) {
    if constexpr (F32) {
      u32x4_t av[MB][3];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const u32x4_t w = o.a[mb][i >> 1];
          const Split3 h = split3(__uint_as_float(w[2 * (i & 1)]), __uint_as_float(w[2 * (i & 1) + 1]));
#pragma unroll
          for (int z = 0; z < 3; ++z) av[mb][z][i] = h.p[z];
        }
      // the leading parts' product has its own sum, which the others would
      // round five more times (between them, so that a sum's next product is
      // not the next one issued: 30.5 us against 30.9 last, 64 -> 64 features
      // 3x3 at 56x56, batch 16)
      constexpr int za[6] = {2, 0, 1, 0, 1, 0}, zb[6] = {0, 2, 1, 0, 0, 1};
#pragma unroll
      for (int z = 0; z < 6; ++z)
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            f32x16_t& s = z == 3 ? acc[mb][nb] : low[mb][nb];
            s = mfma_t(av[mb][za[z]], o.b[nb][zb[z]], s);
          }
    } else {
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = mfma_t(o.a[mb][0], o.b[nb][0], acc[mb][nb]);
    }
  };
  // PF: the next step's operands are read before this step's products (where
  // the registers allow; a runtime stencil always does)
  constexpr bool PF = F32 ? MB * NB <= 2 : MB * NB <= 4;
  // The products of one stage; after each NP-th part of them, one piece of
  // the next stage is written to the other buffer and (MODE 2) its registers
  // take that piece of the stage after.
  auto stage = [&](auto mode, int st) __attribute__((always_inline)) {
    constexpr int MODE = decltype(mode)::value;
    char* cur = smem + (st & 1) * buf_bytes;
    char* nxt = smem + ((st + 1) & 1) * buf_bytes;
    Ops op[2];
    int q = 0, r = 0, s = 0, sm = 0, sq = 0;  // runtime stencils: tap (r, s), s % sh, s / sh
    auto next = [&]() {
      ++q, ++s;
      if (++sm == a.sh) sm = 0, ++sq;
      if (s == Ns) s = 0, sm = 0, sq = 0, ++r;
    };
    auto fetch_q = [&](auto qc) __attribute__((always_inline)) {
      constexpr int Q = decltype(qc)::value, tap = Q / KS, tr = tap / (NS ? NS : 1),
                    ts = tap % (NS ? NS : 1);
      int so = ts;
      if constexpr (FORM == kWide2) so = (ts & 1) * t.hp + (ts >> 1);
      if constexpr (FORM == kPairs) so = (ts % a.sh) * t.hp + ts / a.sh;
      fetch(op[Q & 1], cur, tap, Q % KS, tr * t.pitch + so);
    };
    if constexpr (NR == 0) {
      fetch(op[0], cur, 0, 0, 0);
      next();
    } else if constexpr (PF) {
      fetch_q(std::integral_constant<int, 0>());
    }
    static_for<NP>([&](auto pc) __attribute__((always_inline)) {
      constexpr int P = decltype(pc)::value;
      if constexpr (NR != 0) {
        constexpr int NSTEP = NR * NS * KS;
        static_for<(P + 1) * NSTEP / NP - P * NSTEP / NP>([&](auto qc) __attribute__((always_inline)) {
          constexpr int Q = P * NSTEP / NP + decltype(qc)::value;
          if constexpr (!PF) fetch_q(std::integral_constant<int, Q>());
          if constexpr (PF && Q + 1 < NSTEP) fetch_q(std::integral_constant<int, Q + 1>());
          multiply(op[Q & 1]);
          __builtin_amdgcn_sched_barrier(0);
        });
      } else {
        const int q1 = (P + 1) * RS / NP;  // taps multiplied by the end of this part
        while (q <= q1 && q < RS) {        // op[0] holds tap q - 1
          fetch(op[1], cur, q, 0, r * t.pitch + sm * t.hp + sq);
          multiply(op[0]);
          op[0] = op[1];
          next();
        }
        if (P == NP - 1) multiply(op[0]);
      }
      if constexpr (MODE >= 1) write(pc, std::integral_constant<bool, MODE == 1>(), st + 1, nxt);
      if constexpr (MODE == 2) load(pc, st + 2);
      // (keeps the pieces where they are: the scheduler otherwise gathers them)
      __builtin_amdgcn_sched_barrier(0);
    });
  };

  if (t.nst > 1) {
    static_for<NP>([&](auto pc) __attribute__((always_inline)) {
      write(pc, std::false_type(), 0, smem);
      load(pc, 1);
    });
  } else {
    static_for<NP>([&](auto pc)
                       __attribute__((always_inline)) { write(pc, std::true_type(), 0, smem); });
  }
  __syncthreads();
  int st = 0;
  for (; st + 2 < t.nst; ++st) {
    stage(std::integral_constant<int, 2>(), st);
    __syncthreads();
  }
  if (st + 1 < t.nst) {
    stage(std::integral_constant<int, 1>(), st);
    __syncthreads();
    ++st;
  }
  stage(std::integral_constant<int, 0>(), st);
  if constexpr (F32) {
    // The tile again on the fp32 units, where the parts do not give its sums:
    // any that is not finite (an infinity or a NaN among its values; or, where
    // a product overflows, a smaller one of its parts that does so with the
    // other sign: NaN for infinity), and any that the parts of values below
    // 2^-102 may have missed.  Such a value's parts lose less than 2^-125 of it
    // (what is below the least normal number), a sum of K products less than
    // K 2^-124 top, top the largest value: sums of 2^26 times that keep fp32's
    // accuracy, so one small weight or input among ordinary ones costs nothing.
    // The sums are looked at only where a value is small, or so large that K
    // products of two such may overflow.
    const int K = a.Nc * RS;
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[mb][nb][j] += low[mb][nb][j];
    // (the buffers are free: the votes there)
    uint32_t* vote = reinterpret_cast<uint32_t*>(smem);  // small values, large ones, the largest, again
    __syncthreads();
    if (tid < 4) vote[tid] = 0u;
    __syncthreads();
    if (range.small()) vote[0] = 1u;
    if (range.hi >= (uint32_t)(126 + (126 - (32 - __builtin_clz(K))) / 2) << 24) vote[1] = 1u;
    __syncthreads();
    bool again = t.units;
    if (!again && (vote[0] | vote[1])) {
      float least = __builtin_inff(), nan = 0.f;  // 0 times every sum: NaN if one is not finite
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            least = fminf(least, fabsf(acc[mb][nb][j]));
            nan = __builtin_fmaf(acc[mb][nb][j], 0.f, nan);
          }
      atomicMax(&vote[2], range.hi >> 1);
      __syncthreads();
      const float bound = vote[0] ? (float)K * 0x1p-98f * __uint_as_float(vote[2]) : 0.f;
      if (nan != 0.f || !(least >= bound)) vote[3] = 1u;
      __syncthreads();
      again = vote[3] != 0u;
    }
    if (again) {
      // Straight from memory: of the flattened (c, r, s) index of a feature, a
      // lane's half takes four elements of every eight, 16 bytes of Ker and
      // four gathers of In, two such steps ahead of the products.
      const uint32_t kmax = (uint32_t)(a.Nk - 1);
      uint32_t ko[MB], io[NB];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
        ko[mb] = min((uint32_t)(k0 + (wm * MB + mb) * 32 + l32), kmax) * krow;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const int q = min((wn * NB + nb) * 32 + l32, nout - 1);
        const int i = fdiv(q, t.ctd), orow = row0 + i, b = fdiv(orow, t.nw);
        io[nb] = (uint32_t)(((int64_t)(b - b0) * a.in_img + (int64_t)(orow - b * a.Nw) * a.sw * a.Ny +
                             (int64_t)(h0 + q - i * cols) * a.sh) * 4);
#pragma unroll
        for (int mb = 0; mb < MB; ++mb)
#pragma unroll
          for (int j = 0; j < 16; ++j) acc[mb][nb][j] = 0.f;
      }
      constexpr int U = 2;
      struct Raw {
        u32x4_t a[U][MB];
        uint32_t b[U][4][NB];
      };
      auto fetch_raw = [&](Raw& o, int e0) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int e = e0 + 8 * u + 4 * half;  // (past the end: masked in the products)
#pragma unroll
          for (int mb = 0; mb < MB; ++mb)
            o.a[u][mb] = __builtin_bit_cast(
                u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                             kr, ko[mb] + (uint32_t)min(e, K - 1) * 4, 0, 0));
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int x = min(e + i, K - 1), c = fdiv(x, t.rsd), q = x - c * RS, r = fdiv(q, t.nsd);
            const uint32_t off = (uint32_t)c * plane + (uint32_t)(r * a.Ny + q - r * Ns) * 4;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
              o.b[u][i][nb] = __builtin_amdgcn_raw_buffer_load_b32(ir, io[nb] + off, 0, 0);
          }
        }
      };
      Raw cur, nxt;
      fetch_raw(cur, 0);
      for (int e0 = 0; e0 < K; e0 += 8 * U) {
        fetch_raw(nxt, e0 + 8 * U);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const bool in = e0 + 8 * u + 4 * half + i < K;
#pragma unroll
            for (int mb = 0; mb < MB; ++mb)
#pragma unroll
              for (int nb = 0; nb < NB; ++nb)
                acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(
                    in ? __uint_as_float(cur.a[u][mb][i]) : 0.f,
                    in ? __uint_as_float(cur.b[u][i][nb]) : 0.f, acc[mb][nb], 0, 0, 0);
          }
        cur = nxt;
      }
    }
  }
  __syncthreads();

  // ---- epilogue: register j of a 32x32 accumulator holds feature
  // 8 (j / 4) + 4 half + j % 4 of output l32.  Each wave turns its blocks
  // through LDS, 32 features at a time, so that a lane stores 16 bytes of
  // consecutive outputs of one feature (fp32), or of each of two (bf16).
  constexpr bool O16 = sizeof(TO) == 2;
  constexpr int OPC = O16 ? 8 : 4;           // outputs per lane's chunk
  constexpr int CPR = NB * 32 / OPC;         // chunks per feature (or pair)
  constexpr int RPI = 64 / CPR;              // features (pairs) per pass of the wave
  constexpr int NROW = O16 ? 16 : 32;        // features (pairs) of a block row
  uint32_t* xp = reinterpret_cast<uint32_t*>(smem) + wave * NROW * NB * 32;
  const __amdgpu_buffer_rsrc_t orr =
      rsrc_words(Out + (int64_t)b0 * a.Nk * a.hw,
             (a.out_total - (int64_t)b0 * a.Nk * a.hw) * (int64_t)sizeof(TO));
  const int ch = lane % CPR, frow = lane / CPR;
  // byte offsets of the chunk's outputs, feature k0; past every feature's end
  // (the store is dropped) for those that are not, or that the neighbouring band
  // stores
  constexpr uint32_t kNone = 0x80000000u;
  uint32_t oo[OPC];
  const int qlast = (wn * NB) * 32 + ch * OPC + OPC - 1;
#pragma unroll
  for (int e = 0; e < OPC; ++e) {
    const int q = min(qlast - (OPC - 1) + e, nout - 1);
    const int i = fdiv(q, t.ctd);
    const int orow = row0 + i;
    const int b = fdiv(orow, t.nw);
    oo[e] = (uint32_t)((((int64_t)(b - b0) * a.Nk + k0) * a.hw + (int64_t)(orow - b * a.Nw) * a.Nh +
                        h0 + q - i * cols) * (int64_t)sizeof(TO));
    if (qlast - (OPC - 1) + e >= nout || (F32 && q - i * cols < own)) oo[e] = kNone;
  }
  const bool whole = oo[OPC - 1] - oo[0] == (OPC - 1) * sizeof(TO);
  const bool some = oo[0] != kNone || oo[OPC - 1] != kNone;
  const uint32_t fbytes = (uint32_t)a.hw * (uint32_t)sizeof(TO);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if constexpr (O16) {
#pragma unroll
        for (int j = 0; j < 16; j += 2)
          xp[(4 * (j >> 2) + 2 * half + ((j & 3) >> 1)) * NB * 32 + nb * 32 + l32] =
              pk_bf16(acc[mb][nb][j], acc[mb][nb][j + 1]);
      } else {
#pragma unroll
        for (int j = 0; j < 16; ++j)
          xp[(8 * (j >> 2) + 4 * half + (j & 3)) * NB * 32 + nb * 32 + l32] =
              __float_as_uint(acc[mb][nb][j]);
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // wave-private: LDS keeps a wave's order
#pragma unroll
    for (int it = 0; it < NROW / RPI; ++it) {
      const int f = it * RPI + frow;
      const u32x4_t* rp = reinterpret_cast<const u32x4_t*>(xp + f * NB * 32 + ch * OPC);
      const int kl = (wm * MB + mb) * 32 + (O16 ? 2 * f : f);  // feature within the tile
      u32x4_t v[O16 ? 2 : 1];
      if constexpr (O16) {
        const u32x4_t x0 = rp[0], x1 = rp[1];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          v[0][i] = __builtin_amdgcn_perm(x0[2 * i + 1], x0[2 * i], 0x05040100u);
          v[1][i] = __builtin_amdgcn_perm(x0[2 * i + 1], x0[2 * i], 0x07060302u);
          v[0][2 + i] = __builtin_amdgcn_perm(x1[2 * i + 1], x1[2 * i], 0x05040100u);
          v[1][2 + i] = __builtin_amdgcn_perm(x1[2 * i + 1], x1[2 * i], 0x07060302u);
        }
      } else {
        v[0] = rp[0];
      }
#pragma unroll
      for (int u = 0; u < (O16 ? 2 : 1); ++u) {
        if (k0 + kl + u >= a.Nk) continue;
        const uint32_t fo = (uint32_t)(kl + u) * fbytes;
        if (whole) {
          __builtin_amdgcn_raw_buffer_store_b128(v[u], orr, oo[0] + fo, 0, 0);
        } else if (some) {
#pragma unroll
          for (int e = 0; e < OPC; ++e) {
            if constexpr (O16)
              __builtin_amdgcn_raw_buffer_store_b16((uint16_t)(v[u][e >> 1] >> (16 * (e & 1))), orr,
                                                    oo[e] + fo, 0, 0);
            else
              __builtin_amdgcn_raw_buffer_store_b32(v[u][e], orr, oo[e] + fo, 0, 0);
          }
        }
      }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

// ---- instantiation table, in groups that compile separately ------------------
// (id, dtype, WM, WN, MB, NB, KS, NR, NS, MAXP, KCH, OCC)
#define CNN_TILE_F32(X)                              \
  X(3000, CNN_F32, 2, 4, 1, 2, 1, 3, 3, 1, 0, 1)     \
  X(3001, CNN_F32, 1, 4, 1, 2, 1, 3, 3, 1, 0, 1)     \
  X(3002, CNN_F32, 2, 4, 1, 2, 2, 1, 1, 1, 1, 1)     \
  X(3003, CNN_F32, 1, 4, 1, 2, 1, 0, 0, 2, 4, 1)     \
  X(3004, CNN_F32, 1, 8, 1, 1, 1, 0, 0, 1, 7, 1)
#define CNN_TILE_3X3(X, base, dt)                    \
  X(base + 0, dt, 1, 4, 2, 4, 1, 3, 3, 1, 0, 2)      \
  X(base + 1, dt, 1, 4, 2, 2, 1, 3, 3, 1, 0, 2)      \
  X(base + 2, dt, 2, 2, 2, 2, 1, 3, 3, 1, 0, 2)      \
  X(base + 3, dt, 2, 4, 2, 4, 1, 3, 3, 1, 0, 1)      \
  X(base + 4, dt, 1, 4, 1, 2, 1, 3, 3, 2, 0, 2)      \
  X(base + 5, dt, 1, 8, 2, 4, 1, 3, 3, 1, 0, 1)
#define CNN_TILE_ANY(X, base, dt)                    \
  X(base + 0, dt, 1, 4, 2, 2, 4, 1, 1, 1, 2, 2)      \
  X(base + 1, dt, 2, 2, 2, 2, 4, 1, 1, 1, 4, 2)      \
  X(base + 2, dt, 2, 4, 2, 2, 4, 1, 1, 1, 2, 1)      \
  X(base + 3, dt, 1, 4, 2, 2, 1, 0, 0, 1, 2, 2)      \
  X(base + 4, dt, 1, 4, 1, 2, 1, 0, 0, 1, 4, 2)      \
  X(base + 5, dt, 1, 4, 1, 2, 1, 0, 0, 2, 7, 1)      \
  X(base + 6, dt, 2, 4, 2, 2, 1, 0, 0, 1, 4, 1)
#define CNN_TILE_VARIANTS(X)         \
  CNN_TILE_F32(X)                    \
  CNN_TILE_3X3(X, 3100, CNN_BF16)    \
  CNN_TILE_ANY(X, 3120, CNN_BF16)    \
  CNN_TILE_3X3(X, 3200, CNN_BF16_OBF16) \
  CNN_TILE_ANY(X, 3220, CNN_BF16_OBF16)

template <int DT, int WM, int WN, int MB, int NB, int KS, int NR, int NS, int MAXP, int KCH, int OCC>
static hipError_t launch_t(const void* In, const void* Ker, void* Out, const ConvArgs& a,
                           const TileGeo& t, int form, int64_t lds, int64_t grid,
                           hipStream_t stream) {
  typedef typename std::conditional<DT == CNN_F32, float, bf16_t>::type TI;
  typedef typename std::conditional<DT == CNN_BF16_OBF16, bf16_t, float>::type TO;
  void (*kern)(const TI*, const TI*, TO*, ConvArgs, TileGeo) = nullptr;
  if (form == kPairs) kern = conv_tile<TI, TO, WM, WN, MB, NB, KS, NR, NS, MAXP, KCH, OCC, kPairs>;
  if (form == kWide1) kern = conv_tile<TI, TO, WM, WN, MB, NB, KS, NR, NS, MAXP, KCH, OCC, kWide1>;
  if constexpr (NS != 1)
    if (form == kWide2) kern = conv_tile<TI, TO, WM, WN, MB, NB, KS, NR, NS, MAXP, KCH, OCC, kWide2>;
  // 1 wide, or any; not with 128 features on four waves (tile_geometry)
  if constexpr (NS <= 1 && !(NR == 1 && WM * MB == 4 && WM * WN == 4))
    if (form == kGather2)
      kern = conv_tile<TI, TO, WM, WN, MB, NB, KS, NR, NS, MAXP, KCH, OCC, kGather2>;
  if (!kern) return hipErrorInvalidValue;
  const hipError_t e = allow_max_lds((const void*)kern);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * WM * WN), (unsigned)lds, stream,
                     (const TI*)In, (const TI*)Ker, (TO*)Out, a, t);
  return hipGetLastError();
}

// One group's launcher: hipErrorInvalidValue if `id` is not one of it.
typedef hipError_t (*TileLaunch)(int id, const void* In, const void* Ker, void* Out,
                                 const ConvArgs& a, const TileGeo& t, int form, int64_t lds,
                                 int64_t grid, hipStream_t stream);
hipError_t launch_tile_f32(int, const void*, const void*, void*, const ConvArgs&, const TileGeo&,
                           int, int64_t, int64_t, hipStream_t);
hipError_t launch_tile_3x3_bf16(int, const void*, const void*, void*, const ConvArgs&,
                                const TileGeo&, int, int64_t, int64_t, hipStream_t);
hipError_t launch_tile_3x3_obf16(int, const void*, const void*, void*, const ConvArgs&,
                                 const TileGeo&, int, int64_t, int64_t, hipStream_t);
hipError_t launch_tile_any_bf16(int, const void*, const void*, void*, const ConvArgs&,
                                const TileGeo&, int, int64_t, int64_t, hipStream_t);
hipError_t launch_tile_any_obf16(int, const void*, const void*, void*, const ConvArgs&,
                                 const TileGeo&, int, int64_t, int64_t, hipStream_t);

#define CNN_CASET(id_, dt, wm, wn, mb, nb, ks, nr, ns, maxp, kch, occ)                      \
  case id_:                                                                                 \
    return launch_t<dt, wm, wn, mb, nb, ks, nr, ns, maxp, kch, occ>(In, Ker, Out, a, t, form, \
                                                                   lds, grid, stream);
#define CNN_TILE_LAUNCHER(name, ...)                                                        \
  hipError_t name(int id, const void* In, const void* Ker, void* Out, const ConvArgs& a,    \
                  const TileGeo& t, int form, int64_t lds, int64_t grid,                    \
                  hipStream_t stream) {                                                     \
    switch (id) {                                                                           \
      __VA_ARGS__                                                                           \
      default:                                                                              \
        return hipErrorInvalidValue;                                                        \
    }                                                                                       \
  }

}  // namespace cnnlib
