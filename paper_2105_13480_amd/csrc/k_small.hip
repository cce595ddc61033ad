// Convolution of layers with few outputs (gfx950): any dtype, stencil,
// strides and feature counts, no workspace, one launch, a fixed summation
// order.
//
// Such layers (a batch-1 network's last stages, tiny inputs) have too few
// tiles of the usual size to fill the GPU, so their time is latency and the
// bytes one CU can have outstanding.  Here a workgroup owns 16 features by
// TP = 16 PB outputs of one image and up to 16 waves share its contraction
// (the paper's Case 2, W_c < N_c, inside a workgroup): the K dimension is the
// flattened (c, r, s) index, K-step i of 32 (fp32: 16) elements belongs to
// wave i mod W, and the waves' partial tiles are added in wave order in LDS.
//
// * Ker (A operand): a feature's K run is contiguous in memory, so a lane's
//   operand is one 16-byte load, straight into registers, at any alignment;
//   the waves of a workgroup read neighbouring steps of the same 16 runs.  The
//   first U steps' loads go out behind the first of In's and land while that is
//   written to LDS.
// * In (B operand): the input rows of the tile's outputs, all channels (or a
//   chunk of them), staged once in their natural layout by 16-byte loads; a
//   lane gathers its output's 8 (fp32: 4) elements of a step at offsets read
//   from a table over the K index.
// * What bounds it: one memory latency, the workgroup's bytes and the gathers
//   (batch-1 3x3 512 -> 512 at 7x7, bf16 Out: 147 KB of Ker and 55 KB of In on
//   each of 128 CUs, 10.8 us, where 16 workgroups that walk all channels took
//   23.2; eight features a workgroup on 256 CUs 10.9, so not the bytes).
//   16-feature fp32 3x3 at 16x16: 3.9 us against 9.2 of the staging tiles.
#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "common.h"

namespace cnnlib {

struct SmallGeo {
  int32_t LP;      // LDS pitch of a channel (elements, whole 16-byte chunks)
  int32_t chk;     // channels per chunk
  int32_t nti;     // tiles per image
  int32_t kpad;    // K elements of a full chunk, whole steps
  FastDiv ti, pt, nh, cpc, rs, ns;
};

template <typename TI, typename TO, int PB, int KF>
__global__ __launch_bounds__(1024) void conv_small(const TI* __restrict__ In,
                                                   const TI* __restrict__ Ker,
                                                   TO* __restrict__ Out, ConvArgs a, SmallGeo t) {
  constexpr bool F32 = std::is_same<TI, float>::value;
  constexpr int ES = (int)sizeof(TI), EPC = 16 / ES;
  constexpr int KS = 4 * EPC;  // K elements per step
  constexpr int TP = 16 * PB;
  constexpr int U = 4;         // steps whose Ker loads are in flight
  constexpr int US = 4;        // 16-byte In loads in flight per thread
  extern __shared__ __attribute__((aligned(16))) char smem[];
  TI* slab = reinterpret_cast<TI*>(smem);  // [channel][LP]
  uint32_t* tab = reinterpret_cast<uint32_t*>(slab + (int64_t)t.chk * t.LP);  // [kpad] byte offsets

  const int tid = threadIdx.x, nt = blockDim.x;
  const int lane = tid & 63, W = nt >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g = lane >> 4;
  const int RS = a.Nr * a.Ns;

  // tile: feature tile major, so that the tiles sharing Ker rows share an L2
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int kt = fdiv(tile, t.pt);
  const int pt = tile - kt * a.n_ptiles;
  const int b = fdiv(pt, t.ti);
  const int p0 = (pt - b * t.nti) * TP, k0 = kt * KF;
  const int pl = min(p0 + TP, a.hw) - 1;  // last output
  const int x0 = a.sw * fdiv(p0, t.nh);   // first input row

  const __amdgpu_buffer_rsrc_t kr = rsrc_words(Ker, (int64_t)a.Nk * a.Nc * RS * ES);
  const uint32_t krow = (uint32_t)(a.Nc * RS * ES);
  const int kf = min(k0 + l16 % KF, a.Nk - 1);
  const uint32_t kbase = (uint32_t)kf * krow + 16u * g;
  const int64_t in0 = (int64_t)b * a.in_img + (int64_t)x0 * a.Ny;
  const __amdgpu_buffer_rsrc_t ir = rsrc_words(In + in0, (a.in_total - in0) * ES);
  // the tensors' last bf16 elements, which the range check drops with a dword
  // that straddles the tensor's end
  uint32_t ker_last = 0u, in_last = 0u;
  if constexpr (!F32) {
    ker_last = Ker[(int64_t)a.Nk * a.Nc * RS - 1];
    in_last = In[a.in_total - 1];
  }
  const uint32_t in_end = last_index(a.in_total - in0);  // its index from in0

  u32x4_t av[U];
  auto load_a = [&](int c0, int s, int steps) -> u32x4_t {  // (past the end: not used)
    return __builtin_bit_cast(
        u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(
                     kr, kbase + (uint32_t)(c0 * RS + min(s, steps - 1) * KS) * ES, 0, 0));
  };

  int pix[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) {
    const int p = min(p0 + 16 * pb + l16, pl);
    const int w = fdiv(p, t.nh);
    pix[pb] = ((a.sw * w - x0) * a.Ny + a.sh * (p - w * a.Nh)) * ES;
  }
  f32x4_t acc[PB];
#pragma unroll
  for (int pb = 0; pb < PB; ++pb) acc[pb] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int cpc = t.LP / EPC;  // 16-byte chunks per channel
  for (int c0 = 0; c0 < a.Nc; c0 += t.chk) {
    const int nch = min(t.chk, a.Nc - c0);
    const int Kc = nch * RS, steps = (Kc + KS - 1) / KS;
    // In: chunk j of channel c; the first round's loads go out before Ker's,
    // which then land while the slab is written and the products begin
    const int n = nch * cpc;
    u32x4_t v[US];
    uint32_t off[US];
    auto load_in = [&](int e0) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < US; ++u) {
        const int e = min(e0 + u * nt, n - 1);
        const int c = fdiv(e, t.cpc);
        off[u] = (uint32_t)((c0 + c) * a.nxny + (e - c * cpc) * EPC);
        v[u] = __builtin_bit_cast(u32x4_t,
                                  __builtin_amdgcn_raw_buffer_load_b128(ir, off[u] * ES, 0, 0));
      }
    };
    load_in(tid);
#pragma unroll
    for (int u = 0; u < U; ++u) av[u] = load_a(c0, wave + W * u, steps);
    if (c0 > 0) __syncthreads();  // the previous chunk's gathers are done
    for (int e0 = tid; e0 < n; e0 += US * nt) {
      if (e0 != tid) load_in(e0);
#pragma unroll
      for (int u = 0; u < US; ++u) {
        if constexpr (!F32) {
          const uint32_t d = in_end - off[u];  // the last element's place in the chunk
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (d == (uint32_t)i)
              v[u][i >> 1] = i & 1 ? (v[u][i >> 1] & 0xffffu) | (in_last << 16)
                                   : (v[u][i >> 1] & 0xffff0000u) | in_last;
        }
        if (e0 + u * nt < n) *reinterpret_cast<u32x4_t*>(slab + (int64_t)(e0 + u * nt) * EPC) = v[u];
      }
    }
    if (c0 == 0)
      for (int k = tid; k < t.kpad; k += nt) {
        // (padding of the last step: any staged element, masked when used)
        const int c = fdiv(k, t.rs), q = k - c * RS, r = fdiv(q, t.ns);
        tab[k] = c < t.chk ? (uint32_t)(c * t.LP + r * a.Ny + q - r * a.Ns) * ES : 0u;
      }
    __syncthreads();
    // one step: the lane's eight (four) elements of Ker in aw; in the chunk's
    // last step, ke of them exist
    auto product = [&](int s, u32x4_t aw, auto tail_c, int ke) __attribute__((always_inline)) {
      constexpr bool TAIL = decltype(tail_c)::value;
      if constexpr (TAIL) {
#pragma unroll
        for (int i = 0; i < EPC; ++i) {
          if constexpr (F32) {
            if (i >= ke) aw[i] = 0u;
          } else {
            const uint32_t sh = 16 * (i & 1), m = 0xffffu << sh;
            if (i == ke - 1 && kf == a.Nk - 1 && c0 + nch == a.Nc)
              aw[i >> 1] = (aw[i >> 1] & ~m) | (ker_last << sh);
            if (i >= ke) aw[i >> 1] &= ~m;
          }
        }
      }
      const u32x4_t o0 = *reinterpret_cast<const u32x4_t*>(tab + s * KS + EPC * g);
      uint32_t off[EPC];
#pragma unroll
      for (int i = 0; i < 4; ++i) off[i] = o0[i];
      if constexpr (!F32) {
        const u32x4_t o1 = *reinterpret_cast<const u32x4_t*>(tab + s * KS + EPC * g + 4);
#pragma unroll
        for (int i = 0; i < 4; ++i) off[4 + i] = o1[i];
      }
#pragma unroll
      for (int pb = 0; pb < PB; ++pb) {
        if constexpr (F32) {
          float bv[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            bv[i] = *reinterpret_cast<const float*>(smem + off[i] + pix[pb]);
            if (TAIL && i >= ke) bv[i] = 0.f;
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
            acc[pb] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(aw[i]), bv[i], acc[pb],
                                                           0, 0, 0);
        } else {
          u32x4_t bv;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            uint32_t lo = *reinterpret_cast<const uint16_t*>(smem + off[2 * i] + pix[pb]);
            uint32_t hi = *reinterpret_cast<const uint16_t*>(smem + off[2 * i + 1] + pix[pb]);
            if (TAIL && 2 * i >= ke) lo = 0u;
            if (TAIL && 2 * i + 1 >= ke) hi = 0u;
            bv[i] = lo | (hi << 16);
          }
          acc[pb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, aw),
                                                            __builtin_bit_cast(bf16x8_t, bv),
                                                            acc[pb], 0, 0, 0);
        }
      }
    };
    const int full = Kc / KS;  // whole steps
    int s = wave;
    for (; s + (U - 1) * W < full; s += U * W) {
      u32x4_t cur[U];
#pragma unroll
      for (int u = 0; u < U; ++u) cur[u] = av[u];
#pragma unroll
      for (int u = 0; u < U; ++u) av[u] = load_a(c0, s + (U + u) * W, steps);
#pragma unroll
      for (int u = 0; u < U; ++u) product(s + u * W, cur[u], std::false_type(), 0);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {  // fewer than U steps are left
      const int q = s + u * W;
      if (q < full)
        product(q, av[u], std::false_type(), 0);
      else if (q < steps)
        product(q, av[u], std::true_type(), Kc - q * KS - EPC * g);
    }
  }

  // ---- the waves' tiles, added in wave order.  Register j of a 16x16
  // accumulator holds feature 4 g + j of output l16: [wave][pb][feature][16].
  __syncthreads();
  float* part = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int pb = 0; pb < PB; ++pb)
#pragma unroll
    for (int j = 0; j < 4; ++j) part[(wave * PB + pb) * 256 + (4 * g + j) * 16 + l16] = acc[pb][j];
  __syncthreads();
  for (int o = tid; o < 256 * PB; o += nt) {
    if (KF < 16 && ((o >> 4) & 15) >= KF) continue;  // (copies of the others)
    const int pb = o >> 8, k = k0 + ((o >> 4) & 15), p = p0 + 16 * pb + (o & 15);
    float sum = part[o];
    for (int w = 1; w < W; ++w) sum += part[w * PB * 256 + o];
    if (k < a.Nk && p <= pl) Out[((int64_t)b * a.Nk + k) * a.hw + p] = from_f32<TO>(sum);
  }
}

// ---- instantiation table ----------------------------------------------------
// (id, dtype, PB, KF, waves on a SIMD as its registers allow): tk = KF, tp = 16 PB.
#define CNN_SMALL_VARIANTS(X)       \
  X(3300, CNN_F32, 1, 16, 7)        \
  X(3301, CNN_F32, 2, 16, 6)        \
  X(3302, CNN_F32, 1, 8, 7)         \
  X(3310, CNN_BF16, 1, 16, 5)       \
  X(3311, CNN_BF16, 2, 16, 4)       \
  X(3312, CNN_BF16, 4, 16, 4)       \
  X(3313, CNN_BF16, 1, 8, 5)        \
  X(3320, CNN_BF16_OBF16, 1, 16, 5) \
  X(3321, CNN_BF16_OBF16, 2, 16, 4) \
  X(3322, CNN_BF16_OBF16, 4, 16, 4) \
  X(3323, CNN_BF16_OBF16, 1, 8, 5)

static const VariantM kVariantsM[] = {
#define CNN_ROWM(id, dt, pb, kf, simd) {id, dt, kf, 16 * (pb), 4 * (pb), simd},
    CNN_SMALL_VARIANTS(CNN_ROWM)
#undef CNN_ROWM
};

const VariantM* variants_small(int* count) {
  *count = (int)(sizeof(kVariantsM) / sizeof(kVariantsM[0]));
  return kVariantsM;
}

// The geometry of instantiation v in chunks of chk channels (0: as many as fit
// lds_max bytes); false if it does not fit.
bool small_geometry(const VariantM& v, const cnn_problem& p, int dtype, int64_t lds_max,
                    int64_t chk, SmallShape* s) {
  const int64_t es = in_bytes(dtype), epc = 16 / es, ks = 4 * epc, RS = p.Nr * p.Ns;
  const int64_t Nx = p.sw * (p.Nw - 1) + p.Nr, Ny = p.sh * (p.Nh - 1) + p.Ns, hw = p.Nw * p.Nh;
  // 32-bit byte offsets from an image's rows, and into Ker
  const int64_t lim = 1LL << 31;
  if (p.Nc * Nx * Ny >= lim / (2 * es) || (p.Nk + 16) * p.Nc * RS >= lim / es) return false;
  // a tile's outputs touch at most this many output rows, so this many input rows
  const int64_t tp = std::min(v.tp, hw);
  const int64_t wr = std::min(p.Nw, (tp - 1 + p.Nh - 1) / p.Nh + 1);
  s->S = std::min(Nx, p.sw * (wr - 1) + p.Nr);
  const int64_t LP = (s->S * Ny + epc - 1) / epc * epc;
  // a chunk is whole 32-channel groups, or all channels; its slab and offset
  // table fit LDS
  lds_max = std::min<int64_t>(lds_max, 160 * 1024);
  auto bytes = [&](int64_t c) {
    return c * LP * es + (c * RS + ks - 1) / ks * ks * 4;
  };
  auto fits = [&](int64_t c) { return bytes(c) <= lds_max; };
  if (chk == 0) chk = p.Nc;
  else if (chk < 1 || chk > p.Nc || (chk < p.Nc && chk % 32)) return false;
  else if (!fits(chk)) return false;
  if (!fits(chk)) {
    const int64_t n = lds_max / (LP * es + RS * 4) / 32;
    if (n < 1) return false;
    // chunks of equal size
    const int64_t parts = (p.Nc + 32 * n - 1) / (32 * n);
    chk = ((p.Nc + parts - 1) / parts + 31) / 32 * 32;
    if (!fits(chk)) return false;
  }
  const int64_t steps = (chk * RS + ks - 1) / ks;
  s->LP = LP;
  s->chk = chk;
  s->kpad = steps * ks;
  s->nti = (hw + v.tp - 1) / v.tp;
  // waves: four steps each where there are as many (16 at most, 4 at least)
  s->waves = steps >= 48 ? 16 : steps >= 16 ? 8 : 4;
  s->lds = std::max(bytes(chk), s->waves * (v.tp / 16) * 1024);
  s->lds = (s->lds + 15) / 16 * 16;
  s->grid = p.Nb * s->nti * ((p.Nk + v.tk - 1) / v.tk);
  return s->lds <= lds_max && s->grid <= 0x7fffffffLL;
}

template <int DT, int PB, int KF>
static hipError_t launch_m(const void* In, const void* Ker, void* Out, const ConvArgs& a,
                           const SmallGeo& t, const SmallShape& s, hipStream_t stream) {
  typedef typename std::conditional<DT == CNN_F32, float, bf16_t>::type TI;
  typedef typename std::conditional<DT == CNN_BF16_OBF16, bf16_t, float>::type TO;
  auto kern = conv_small<TI, TO, PB, KF>;
  const hipError_t e = allow_max_lds((const void*)kern);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, dim3((unsigned)s.grid), dim3(64 * (unsigned)s.waves), (unsigned)s.lds,
                     stream, (const TI*)In, (const TI*)Ker, (TO*)Out, a, t);
  return hipGetLastError();
}

hipError_t launch_small(const VariantM& v, const void* In, const void* Ker, void* Out,
                        const ConvArgs& a0, const SmallShape& s, hipStream_t stream) {
  ConvArgs a = a0;
  a.n_ptiles = (int32_t)(a.Nb * s.nti);
  SmallGeo t;
  t.LP = (int32_t)s.LP;
  t.chk = (int32_t)s.chk;
  t.nti = (int32_t)s.nti;
  t.kpad = (int32_t)s.kpad;
  t.ti = make_fastdiv((uint32_t)s.nti);
  t.pt = make_fastdiv((uint32_t)a.n_ptiles);
  t.nh = make_fastdiv((uint32_t)a.Nh);
  t.cpc = make_fastdiv((uint32_t)(s.LP * in_bytes(v.dtype) / 16));
  t.rs = make_fastdiv((uint32_t)(a.Nr * a.Ns));
  t.ns = make_fastdiv((uint32_t)a.Ns);
  switch (v.id) {
#define CNN_CASEM(id, dt, pb, kf, simd) \
  case id:                              \
    return launch_m<dt, pb, kf>(In, Ker, Out, a, t, s, stream);
    CNN_SMALL_VARIANTS(CNN_CASEM)
#undef CNN_CASEM
    default:
      return hipErrorInvalidValue;
  }
}

}  // namespace cnnlib
