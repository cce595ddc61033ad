// C ABI entry points (include/cnn.h): argument validation, plan cache,
// dispatch to the kernels.  Every argument check happens before the first
// HIP call, so error returns never leave work queued.
#include <hip/hip_runtime.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <chrono>
#include <map>
#include <set>
#include <mutex>
#include <string>
#include <tuple>
#include <vector>

#include "internal.h"

namespace cnnlib {
int select_plan(const cnn_problem& p, int dtype, const cnn_budget& bud, int kernel,
                int64_t tk, int64_t tp, int64_t tc, cnn_plan_t* out);
void eq1_terms(const cnn_problem& p, const cnn_tiles& t, int exact, double terms[3],
               double* footprint);
void slab_terms(const cnn_problem& p, int64_t tk, int64_t tp, double terms[3]);
int enumerate_plans(const cnn_problem& p, int dtype, const cnn_budget& bud, cnn_plan_t* out,
                    int cap);
int list_variants(cnn_variant_t* out, int cap);
}  // namespace cnnlib

using namespace cnnlib;

namespace {

thread_local std::string g_last_error;

int fail(int status, const char* fmt, ...) __attribute__((format(printf, 2, 3)));
int fail(int status, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return status;
}

bool mul_ok(int64_t a, int64_t b, int64_t* r) { return !__builtin_mul_overflow(a, b, r); }

// Shape validation and the element counts the kernels index with.
int check_problem(const cnn_problem& p) {
  const int64_t v[9] = {p.Nb, p.Nc, p.Nk, p.Nw, p.Nh, p.Nr, p.Ns, p.sw, p.sh};
  static const char* names[9] = {"Nb", "Nc", "Nk", "Nw", "Nh", "Nr", "Ns", "sw", "sh"};
  for (int i = 0; i < 9; ++i)
    if (v[i] < 1) return fail(CNN_E_SHAPE, "%s = %lld must be >= 1", names[i], (long long)v[i]);
  for (int i = 0; i < 9; ++i)
    if (v[i] > 0x7fffffffLL) return fail(CNN_E_OVERFLOW, "%s = %lld exceeds 2^31-1", names[i], (long long)v[i]);
  int64_t Nx, Ny, t;
  if (!mul_ok(p.sw, p.Nw - 1, &t) || (Nx = t + p.Nr) > 0x7fffffffLL ||
      !mul_ok(p.sh, p.Nh - 1, &t) || (Ny = t + p.Ns) > 0x7fffffffLL)
    return fail(CNN_E_OVERFLOW, "input extent exceeds 2^31-1");
  // Counts the kernels keep in 32-bit: outputs per image plane, flattened
  // (b, w, h) outputs, input plane, flattened (b, x, y) input positions,
  // Ker elements per feature.
  int64_t hw = 0, npix = 0, nxny = 0, bxy = 0, kel = 0;
  if (!mul_ok(p.Nw, p.Nh, &hw) || !mul_ok(hw, p.Nb, &npix) || npix > 0x7fffffffLL ||
      !mul_ok(Nx, Ny, &nxny) || !mul_ok(nxny, p.Nb, &bxy) || bxy > 0x7fffffffLL ||
      !mul_ok(p.Nc, p.Nr * p.Ns, &kel) || kel > 0x7fffffffLL || p.Nr * p.Ns > 0x7fffffffLL)
    return fail(CNN_E_OVERFLOW, "problem exceeds 32-bit kernel indexing (outputs %lld, positions %lld)",
                (long long)npix, (long long)bxy);
  // Whole-tensor element counts below 2^62.
  int64_t in_n, ker_n, out_n;
  if (!mul_ok(bxy, p.Nc, &in_n) || in_n >= (1LL << 62) || !mul_ok(kel, p.Nk, &ker_n) ||
      ker_n >= (1LL << 62) || !mul_ok(npix, p.Nk, &out_n) || out_n >= (1LL << 62))
    return fail(CNN_E_OVERFLOW, "tensor element count exceeds 2^62");
  return CNN_OK;
}

int check_dtype(int dtype) {
  if (dtype != CNN_F32 && dtype != CNN_BF16 && dtype != CNN_BF16_OBF16)
    return fail(CNN_E_DTYPE, "unknown dtype %d", dtype);
  return CNN_OK;
}

void tensor_bytes(const cnn_problem& p, int dtype, int64_t* in_b, int64_t* ker_b, int64_t* out_b) {
  const int64_t Nx = p.sw * (p.Nw - 1) + p.Nr, Ny = p.sh * (p.Nh - 1) + p.Ns;
  *in_b = p.Nb * p.Nc * Nx * Ny * in_bytes(dtype);
  *ker_b = p.Nk * p.Nc * p.Nr * p.Ns * in_bytes(dtype);
  *out_b = p.Nb * p.Nk * p.Nw * p.Nh * out_bytes(dtype);
}

bool overlap(const void* a, int64_t na, const void* b, int64_t nb) {
  const uintptr_t x = (uintptr_t)a, y = (uintptr_t)b;
  return x < y + (uintptr_t)nb && y < x + (uintptr_t)na;
}

int check_buffers(const void* In, const void* Ker, const void* Out, const cnn_problem& p, int dtype) {
  if (!In || !Ker || !Out) return fail(CNN_E_NULL, "In, Ker and Out must be non-NULL");
  int64_t ib, kb, ob;
  tensor_bytes(p, dtype, &ib, &kb, &ob);
  if (overlap(Out, ob, In, ib) || overlap(Out, ob, Ker, kb))
    return fail(CNN_E_ALIAS, "Out overlaps In or Ker");
  return CNN_OK;
}

ConvArgs make_args(const cnn_plan_t& pl) {
  const cnn_problem& p = pl.prob;
  ConvArgs a;
  memset(&a, 0, sizeof(a));
  a.Nb = (int32_t)p.Nb; a.Nc = (int32_t)p.Nc; a.Nk = (int32_t)p.Nk;
  a.Nw = (int32_t)p.Nw; a.Nh = (int32_t)p.Nh; a.Nr = (int32_t)p.Nr; a.Ns = (int32_t)p.Ns;
  a.sw = (int32_t)p.sw; a.sh = (int32_t)p.sh;
  a.Nx = (int32_t)(p.sw * (p.Nw - 1) + p.Nr);
  a.Ny = (int32_t)(p.sh * (p.Nh - 1) + p.Ns);
  a.hw = (int32_t)(p.Nw * p.Nh);
  a.npix = (int32_t)(p.Nb * p.Nw * p.Nh);
  a.nxny = a.Nx * a.Ny;
  a.in_img = (int64_t)p.Nc * a.nxny;
  a.in_total = a.in_img * p.Nb;
  a.out_total = (int64_t)a.npix * p.Nk;
  a.tp = (int32_t)pl.tp;
  a.tk = (int32_t)pl.tk;
  a.tc = (int32_t)pl.tc;
  a.n_ptiles = (int32_t)((a.npix + pl.tp - 1) / pl.tp);
  a.n_ktiles = (int32_t)((p.Nk + pl.tk - 1) / pl.tk);
  a.slab_max = (int32_t)pl.slab_rows;
  a.grid = (int32_t)pl.grid;
  return a;
}

bool same_problem(const cnn_problem& a, const cnn_problem& b) {
  return a.Nb == b.Nb && a.Nc == b.Nc && a.Nk == b.Nk && a.Nw == b.Nw && a.Nh == b.Nh &&
         a.Nr == b.Nr && a.Ns == b.Ns && a.sw == b.sw && a.sh == b.sh;
}

const VariantS* find_variant_s(int id) {
  int n = 0;
  const VariantS* vs = variants_smallc(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

// Geometry a few-channel plan must carry (the kernel sizes LDS from it).
// turn: its LDS is that of the 16-byte stores' turn.
bool smallc_geometry_ok(const VariantS& v, const cnn_plan_t& pl, bool* turn) {
  const cnn_problem& p = pl.prob;
  if (p.Ns > 8 || (p.Nc * p.Nr + 1) / 2 > v.ks || pl.tp < 1 || pl.tp > v.tp ||
      !smallc_stencil_ok(v, p) || !ranges_ok_smallc(v, p, pl.dtype))
    return false;
  const int64_t S = slab_rows_max(p, pl.tp);
  const int64_t grid = ((p.Nb * p.Nw * p.Nh + pl.tp - 1) / pl.tp) * ((p.Nk + v.tk - 1) / v.tk);
  *turn = pl.dtype == CNN_BF16_OBF16 && pl.lds_bytes == smallc_lds_bytes(v, p, S, true);
  return pl.slab_rows == S && pl.grid == grid &&
         (*turn || pl.lds_bytes == smallc_lds_bytes(v, p, S, false)) && pl.lds_bytes <= 160 * 1024;
}

const VariantR* find_variant_r(int id) {
  int n = 0;
  const VariantR* vs = variants_rows(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

// Geometry a row-streaming plan must carry: whole output rows of one image
// per tile (the kernel derives its band from tp), its LDS size and grid.
bool rows_geometry_ok(const VariantR& v, const cnn_plan_t& pl) {
  const cnn_problem& p = pl.prob;
  if (!rows_fits(v, p) || !ranges_ok_whole(p, pl.dtype, 1LL << 31) || pl.tc != p.Nc ||
      pl.tp < p.Nh || pl.tp % p.Nh)
    return false;
  const int64_t L = pl.tp / p.Nh;
  if (p.Nw % L) return false;
  const int64_t grid = p.Nb * (p.Nw / L) * ((p.Nk + v.tk - 1) / v.tk);
  return pl.slab_rows == L + p.Nr - 1 && pl.grid == grid &&
         pl.lds_bytes == rows_lds_bytes(v, p) && pl.lds_bytes <= 160 * 1024;
}

const VariantG* find_variant_g(int id) {
  int n = 0;
  const VariantG* vs = variants_gemm1(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

// Geometry a 1x1 GEMM plan must carry: its tile within the instantiation's,
// the grid its tiles imply, its LDS size.
bool gemm1_geometry_ok(const VariantG& v, const cnn_plan_t& pl) {
  const cnn_problem& p = pl.prob;
  if (pl.tp < 1 || pl.tp > v.tp || !gemm1_fits(v, p, pl.tp) ||
      !ranges_ok_whole(p, pl.dtype, 1LL << 30))
    return false;
  const int64_t grid = ((p.Nb * p.Nw * p.Nh + pl.tp - 1) / pl.tp) * ((p.Nk + v.tk - 1) / v.tk);
  return pl.grid == grid && pl.lds_bytes == gemm1_lds_bytes(v) && pl.lds_bytes <= 160 * 1024;
}

const VariantQ* find_variant_q(int id) {
  int n = 0;
  const VariantQ* vs = variants_srows(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

// Geometry a stride-2 row-band plan must carry: bands of the instantiation's
// L whole rows of one image, 16 channels per chunk, its grid, LDS and
// workspace sizes.
bool srows_geometry_ok(const VariantQ& v, const cnn_plan_t& pl) {
  const cnn_problem& p = pl.prob;
  if (!srows_fits(v, p) || !ranges_ok_srows(v, p, pl.dtype) || pl.tc != 16 ||
      pl.tp != v.L * p.Nh)
    return false;
  const int64_t grid = p.Nb * (p.Nw / v.L) * ((p.Nk + v.tk - 1) / v.tk);
  return pl.slab_rows == srows_slab_rows(v) && pl.grid == grid &&
         pl.lds_bytes == srows_lds_bytes(v) && pl.lds_bytes <= 160 * 1024 &&
         pl.ws_bytes == srows_ws_bytes(v, p);
}

const Variant4* find_variant4(int id) {
  int n = 0;
  const Variant4* vs = variants4(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

const Variant3* find_variant3(int id) {
  int n = 0;
  const Variant3* vs = variants3(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

const Variant2* find_variant2(int id) {
  int n = 0;
  const Variant2* vs = variants2(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

const Variant* find_variant(int id) {
  int n = 0;
  const Variant* vs = variants(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

const VariantC* find_variant_c(int id) {
  int n = 0;
  const VariantC* vs = variants_cslice(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

// Geometry a channel-slice plan must carry: the slab, grid and LDS size its
// tile implies, on a problem the instantiation serves.
bool cslice_geometry_ok(const VariantC& v, const cnn_plan_t& pl) {
  const cnn_problem& p = pl.prob;
  const int64_t Ny = p.sh * (p.Nh - 1) + p.Ns;
  const int64_t S = slab_rows_max(p, pl.tp);
  const int64_t grid = ((p.Nb * p.Nw * p.Nh + pl.tp - 1) / pl.tp) * ((p.Nk + v.tk - 1) / v.tk);
  return cslice_fits(v, p) && pl.slab_rows == S && pl.grid == grid &&
         pl.lds_bytes == cslice_lds_bytes(v, S, Ny) && pl.lds_bytes <= 160 * 1024;
}

const VariantT* find_variant_t(int id) {
  int n = 0;
  const VariantT* vs = variants_tile(&n);
  for (int i = 0; i < n; ++i)
    if (vs[i].id == id) return &vs[i];
  return nullptr;
}

// Geometry a two-dimensional-tile plan must carry: runs of whole output rows,
// the workgroups, slab and LDS size they imply.
bool tile_plan_ok(const VariantT& v, const cnn_plan_t& pl, TileShape* s) {
  const cnn_problem& p = pl.prob;
  if (!tile_geometry(v, p, pl.dtype, pl.kc, s) || pl.tp != s->tr * s->ct) return false;
  const int64_t grid = s->n_rt * s->ncol * ((p.Nk + v.tk - 1) / v.tk);
  return pl.slab_rows == s->S && pl.grid == grid && pl.lds_bytes == s->lds && pl.ws_bytes == 0;
}

// Geometry a few-outputs plan must carry.
bool small_plan_ok(const VariantM& v, const cnn_plan_t& pl, SmallShape* s) {
  return v.dtype == pl.dtype && v.tk == pl.tk && v.tp == pl.tp && small_geometry(v, pl, s) &&
         pl.slab_rows == s->S && pl.grid == s->grid && pl.lds_bytes == s->lds && pl.ws_bytes == 0;
}

// Geometry a plain staging plan (and its split form) must carry: the slab,
// grid and LDS size its tile implies.
bool igemm_geometry_ok(const Variant& v, const cnn_plan_t& pl) {
  const cnn_problem& p = pl.prob;
  const int64_t Ny = p.sh * (p.Nh - 1) + p.Ns;
  const int64_t S = slab_rows_max(p, pl.tp);
  const int64_t grid = ((p.Nb * p.Nw * p.Nh + pl.tp - 1) / pl.tp) * ((p.Nk + v.tk - 1) / v.tk);
  return pl.slab_rows == S && pl.grid == grid &&
         pl.lds_bytes == igemm_lds_bytes(v, S, Ny, p.Nr * p.Ns) && pl.lds_bytes <= 160 * 1024;
}

// The launch geometry a pipelined-kernel plan carries must be the one its
// tile size implies: the kernel sizes LDS and its tile loop from it.
bool v2_geometry_ok(const Variant2& v, const cnn_plan_t& pl) {
  const cnn_problem& p = pl.prob;
  const int64_t Ny = p.sh * (p.Nh - 1) + p.Ns;
  const int64_t S = slab_rows_max(p, pl.tp);
  const int64_t grid = ((p.Nb * p.Nw * p.Nh + pl.tp - 1) / pl.tp) * ((p.Nk + v.tk - 1) / v.tk);
  if (v.nr > 0 && (v.nr != p.Nr || v.ns != p.Ns)) return false;
  if (v.rawk && (p.Nc % 8 != 0 || !ranges_ok_rawk(p))) return false;
  if (!ranges_ok_tile(p, pl.dtype, v.tp, 0)) return false;
  const int64_t pairs = v.pw ? (pl.tp + 1) / 2 : (S * Ny + 1) / 2;
  if (v.pw && (p.Nr != 1 || p.Ns != 1)) return false;
  return pl.slab_rows == S && pairs <= 256LL * v.maxp && pl.grid == grid &&
         pl.lds_bytes == igemm2_lds_bytes(v, S, Ny, p.Nr * p.Ns, pl.tp) &&
         pl.lds_bytes <= 160 * 1024;
}

// ws: the caller's workspace (at least pl.ws_bytes), or nullptr when the
// plan needs none.  The library itself never allocates device memory here.
// dry: check the plan only (no HIP call), return the status a run would.
int run_plan(const void* In, const void* Ker, void* Out, const cnn_plan_t& pl, hipStream_t st,
             void* ws = nullptr, bool dry = false) {
  if (pl.ws_bytes < 0) return fail(CNN_E_PLAN, "negative ws_bytes");
  if (pl.ws_bytes > 0 && !ws && !dry)
    return fail(CNN_E_UNSUPPORTED,
                "plan needs a %lld-byte device workspace: use cnn_fwd_plan_ws",
                (long long)pl.ws_bytes);
  const ConvArgs a = make_args(pl);
  hipError_t e;
  if (pl.kernel == CNN_K_DIRECT) {
    if (dry) return CNN_OK;
    e = launch_direct(In, Ker, Out, a, pl.dtype, st);
  } else if (pl.kernel == CNN_K_GEMM1) {
    const VariantG* vg = find_variant_g(pl.variant);
    if (!vg || vg->dtype != pl.dtype || vg->tk != pl.tk || vg->tc != pl.tc ||
        !gemm1_geometry_ok(*vg, pl))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_gemm1(*vg, In, Ker, Out, a, pl.lds_bytes, st);
  } else if (pl.kernel == CNN_K_ROWS) {
    const VariantR* vr = find_variant_r(pl.variant);
    if (!vr || vr->dtype != pl.dtype || vr->tk != pl.tk || !rows_geometry_ok(*vr, pl))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_rows(*vr, In, Ker, Out, a, pl.lds_bytes, st);
  } else if (pl.kernel == CNN_K_SROWS) {
    const VariantQ* vq = find_variant_q(pl.variant);
    if (!vq || vq->dtype != pl.dtype || vq->tk != pl.tk || !srows_geometry_ok(*vq, pl))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_srows(*vq, In, Ker, Out, ws, a, pl.lds_bytes, st);
  } else if (pl.kernel == CNN_K_SPLITC) {
    // the CNN_K_IGEMM tiles split over slices, or the channel-slice kernel
    const VariantC* vc = find_variant_c(pl.variant);
    const Variant* v = vc ? nullptr : find_variant(pl.variant);
    const cnn_problem& p = pl.prob;
    const int64_t stages = (p.Nc + pl.tc - 1) / (pl.tc > 0 ? pl.tc : 1);
    // a direct plan is one of the few-outputs kernel
    SmallShape ms;
    const VariantM* vm = vc && vc->mode == 2 ? small_variant(pl) : nullptr;
    const bool match =
        vm ? vc->dtype == pl.dtype && cslice_fits(*vc, p) && small_plan_ok(*vm, pl, &ms)
        : vc ? vc->dtype == pl.dtype && vc->tk == pl.tk && vc->tp == pl.tp && vc->tc == pl.tc &&
                 cslice_geometry_ok(*vc, pl)
           : v && v->kernel == CNN_K_IGEMM && v->dtype == pl.dtype && v->tk == pl.tk &&
                 v->tp == pl.tp && v->tc == pl.tc && igemm_geometry_ok(*v, pl);
    if (!match)
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    const int64_t ws_want = vc && vc->mode ? 0 : 4LL * pl.kc * p.Nb * p.Nk * p.Nw * p.Nh;
    if (pl.kc < 1 || pl.kc > stages || pl.kc > 65535 || pl.ws_bytes != ws_want ||
        (vc && vc->mode == 2 && pl.kc != 1))
      return fail(CNN_E_PLAN,
                  "split plan needs 1 <= kc <= %lld and ws_bytes = 4*kc*|Out| "
                  "(0 for the atomic-sum and direct instantiations; kc = 1 for the direct ones)",
                  (long long)stages);
    if (dry) return CNN_OK;
    // (direct plans that carry the 32 x 64 tile, as earlier versions made them,
    // run that kernel too, in the LDS they name; images and Ker beyond its
    // 32-bit offsets the one that takes any shape)
    const bool direct = vc && vc->mode == 2;
    if (direct && !vm) vm = small_direct(p, pl.dtype, {256, pl.lds_bytes, 128, 2}, &ms);
    e = vm       ? launch_small(*vm, In, Ker, Out, a, ms, st)
        : direct ? launch_direct(In, Ker, Out, a, pl.dtype, st)
        : vc     ? launch_cslice(*vc, In, Ker, Out, ws, a, pl.lds_bytes, pl.kc, pl.dtype, st)
                 : launch_splitc(*v, In, Ker, Out, ws, a, pl.lds_bytes, pl.kc, pl.dtype, st);
  } else if (pl.kernel == CNN_K_SMALLC) {
    const VariantS* vs = find_variant_s(pl.variant);
    bool turn = false;
    if (!vs || vs->dtype != pl.dtype || vs->tk != pl.tk || !smallc_geometry_ok(*vs, pl, &turn))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_smallc(*vs, In, Ker, Out, a, pl.lds_bytes, turn, st);
  } else if (const Variant4* v4 = find_variant4(pl.variant)) {
    if (pl.kernel != CNN_K_IGEMM_WIDE || v4->dtype != pl.dtype || v4->tk != pl.tk ||
        v4->tp != pl.tp || v4->tc != pl.tc || pl.ws_bytes != igemm4_ws_bytes(*v4, pl.prob))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_igemm4(*v4, In, Ker, Out, ws, a, pl.lds_bytes, st);
  } else if (const Variant3* v3 = find_variant3(pl.variant)) {
    if (pl.kernel != CNN_K_IGEMM_DMA || v3->dtype != pl.dtype || v3->tk != pl.tk ||
        v3->tp != pl.tp || v3->tc != pl.tc || pl.ws_bytes != igemm3_ws_bytes(*v3, pl.prob))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_igemm3(*v3, In, Ker, Out, ws, a, pl.lds_bytes, st);
  } else if (const Variant2* v2 = find_variant2(pl.variant)) {
    if (pl.kernel != v2_family(*v2) || v2->dtype != pl.dtype ||
        v2->tk != pl.tk ||
        pl.tp < 1 || pl.tp > v2->tp || v2->tc != pl.tc ||
        pl.ws_bytes != igemm2_ws_bytes(*v2, pl.prob) || !v2_geometry_ok(*v2, pl))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_igemm2(*v2, In, Ker, Out, ws, a, pl.lds_bytes, st);
  } else if (const VariantM* vm = small_variant(pl)) {
    SmallShape ms;
    if (pl.tc != pl.prob.Nc || !small_plan_ok(*vm, pl, &ms))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_small(*vm, In, Ker, Out, a, ms, st);
  } else if (const VariantT* vt = find_variant_t(pl.variant)) {
    TileShape ts;
    if (pl.kernel != CNN_K_IGEMM || vt->dtype != pl.dtype || vt->tk != pl.tk || vt->tc != pl.tc ||
        !tile_plan_ok(*vt, pl, &ts))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_tile(*vt, In, Ker, Out, a, ts, pl.grid, st);
  } else {
    const Variant* v = find_variant(pl.variant);
    if (!v || v->kernel != pl.kernel || v->dtype != pl.dtype || v->tk != pl.tk ||
        v->tp != pl.tp || v->tc != pl.tc || !igemm_geometry_ok(*v, pl))
      return fail(CNN_E_PLAN, "plan names no matching kernel instantiation (variant %d)", pl.variant);
    if (dry) return CNN_OK;
    e = launch_igemm(*v, In, Ker, Out, a, pl.lds_bytes, st);
  }
  if (e != hipSuccess) return fail(CNN_E_HIP, "kernel launch failed: %s", hipGetErrorString(e));
  return CNN_OK;
}

// Kernels whose dynamic-LDS limit was raised, per device.
std::mutex g_lds_mu;
std::set<std::pair<const void*, int>> g_lds_done;

// Plan cache keyed by (problem, dtype, device).
typedef std::tuple<int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int, int> Key;
std::mutex g_cache_mu;
std::map<Key, cnn_plan_t> g_cache;

}  // namespace

namespace cnnlib {

int device_cus() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 256;
  std::lock_guard<std::mutex> g(g_lds_mu);
  static std::map<int, int> cus;
  auto it = cus.find(dev);
  if (it != cus.end()) return it->second;
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1)
    n = 256;
  cus.emplace(dev, n);
  return n;
}

hipError_t allow_max_lds(const void* kernel) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  std::lock_guard<std::mutex> g(g_lds_mu);
  if (g_lds_done.count(std::make_pair(kernel, dev))) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  if (e == hipSuccess) g_lds_done.insert(std::make_pair(kernel, dev));
  return e;
}

}  // namespace cnnlib

extern "C" {

int cnn_abi_version(void) { return CNN_ABI_VERSION; }

const char* cnn_last_error(void) { return g_last_error.c_str(); }

const char* cnn_strerror(int status) {
  switch (status) {
    case CNN_OK: return "success";
    case CNN_E_NULL: return "NULL pointer argument";
    case CNN_E_SHAPE: return "size or stride below 1";
    case CNN_E_DTYPE: return "unknown dtype";
    case CNN_E_OVERFLOW: return "problem too large for the kernels' indexing";
    case CNN_E_ALIAS: return "Out overlaps In or Ker";
    case CNN_E_UNSUPPORTED: return "kernel or tiling not available for this problem";
    case CNN_E_HIP: return "HIP runtime error";
    case CNN_E_PLAN: return "plan does not match the problem";
    default: return "unknown status";
  }
}

int cnn_device_budget(int device, cnn_budget* budget) {
  if (!budget) return fail(CNN_E_NULL, "budget must be non-NULL");
  hipDeviceProp_t prop;
  hipError_t e = hipGetDeviceProperties(&prop, device);
  if (e != hipSuccess) return fail(CNN_E_HIP, "hipGetDeviceProperties: %s", hipGetErrorString(e));
  budget->cus = prop.multiProcessorCount;
  budget->lds_bytes = (int64_t)prop.maxSharedMemoryPerMultiProcessor;
  if (budget->lds_bytes <= 0) budget->lds_bytes = (int64_t)prop.sharedMemPerBlock;
  budget->acc_regs = 128;
  budget->wg_per_cu = 2;
  return CNN_OK;
}

static int resolve_budget(const cnn_budget* in, cnn_budget* out) {
  if (in) {
    if (in->cus < 1 || in->lds_bytes < 1 || in->acc_regs < 1 || in->wg_per_cu < 1)
      return fail(CNN_E_SHAPE, "budget fields must be >= 1");
    *out = *in;
    return CNN_OK;
  }
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(CNN_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  return cnn_device_budget(dev, out);
}

int cnn_plan_tiles(const cnn_problem* prob, int dtype, int kernel, int64_t tk, int64_t tp,
                   int64_t tc, const cnn_budget* budget, cnn_plan_t* plan) {
  if (!prob || !plan) return fail(CNN_E_NULL, "prob and plan must be non-NULL");
  int st;
  if ((st = check_problem(*prob)) || (st = check_dtype(dtype))) return st;
  if (kernel < CNN_K_AUTO || kernel > CNN_K_AUTO_NO_WORKSPACE || kernel == 9)
    return fail(CNN_E_UNSUPPORTED, "unknown kernel %d", kernel);
  cnn_budget bud;
  if ((st = resolve_budget(budget, &bud))) return st;
  st = select_plan(*prob, dtype, bud, kernel, tk, tp, tc, plan);
  if (st) return fail(st, "no kernel instantiation for kernel %d tk %lld tp %lld tc %lld dtype %d",
                      kernel, (long long)tk, (long long)tp, (long long)tc, dtype);
  return CNN_OK;
}

int cnn_plan(const cnn_problem* prob, int dtype, const cnn_budget* budget, cnn_plan_t* plan) {
  return cnn_plan_tiles(prob, dtype, CNN_K_AUTO, 0, 0, 0, budget, plan);
}

int cnn_plan_candidates(const cnn_problem* prob, int dtype, const cnn_budget* budget,
                        cnn_plan_t* out, int cap, int* count) {
  if (!prob || !count || (cap > 0 && !out))
    return fail(CNN_E_NULL, "prob, count (and out when cap > 0) must be non-NULL");
  int st;
  if ((st = check_problem(*prob)) || (st = check_dtype(dtype))) return st;
  cnn_budget bud;
  if ((st = resolve_budget(budget, &bud))) return st;
  *count = enumerate_plans(*prob, dtype, bud, out, cap < 0 ? 0 : cap);
  return CNN_OK;
}

int cnn_variants(cnn_variant_t* out, int cap, int* count) {
  if (!count || (cap > 0 && !out)) return fail(CNN_E_NULL, "count (and out when cap > 0) must be non-NULL");
  *count = list_variants(out, cap < 0 ? 0 : cap);
  return CNN_OK;
}

int cnn_fwd_plan(const void* In, const void* Ker, void* Out, const cnn_problem* prob, int dtype,
                 const cnn_plan_t* plan, void* stream) {
  if (!prob || !plan) return fail(CNN_E_NULL, "prob and plan must be non-NULL");
  int st;
  if ((st = check_problem(*prob)) || (st = check_dtype(dtype))) return st;
  if ((st = check_buffers(In, Ker, Out, *prob, dtype))) return st;
  if (!same_problem(plan->prob, *prob) || plan->dtype != dtype)
    return fail(CNN_E_PLAN, "plan was made for another problem or dtype");
  return run_plan(In, Ker, Out, *plan, (hipStream_t)stream);
}

int cnn_fwd_plan_ws(const void* In, const void* Ker, void* Out, const cnn_problem* prob,
                    int dtype, const cnn_plan_t* plan, void* workspace, int64_t ws_bytes,
                    void* stream) {
  return cnnlib::fwd_plan_checked(In, Ker, Out, prob, dtype, plan, workspace, ws_bytes, stream,
                                  false);
}

}  // extern "C"

namespace cnnlib {

int set_error(int status, const char* msg) { return fail(status, "%s", msg); }

int fwd_plan_checked(const void* In, const void* Ker, void* Out, const cnn_problem* prob,
                     int dtype, const cnn_plan_t* plan, void* workspace, int64_t ws_bytes,
                     void* stream, bool dry) {
  if (!prob || !plan) return fail(CNN_E_NULL, "prob and plan must be non-NULL");
  int st;
  if ((st = check_problem(*prob)) || (st = check_dtype(dtype))) return st;
  if ((st = check_buffers(In, Ker, Out, *prob, dtype))) return st;
  if (!same_problem(plan->prob, *prob) || plan->dtype != dtype)
    return fail(CNN_E_PLAN, "plan was made for another problem or dtype");
  if (plan->ws_bytes > 0) {
    if (!workspace && !dry)
      return fail(CNN_E_NULL, "plan needs a %lld-byte workspace", (long long)plan->ws_bytes);
    if (ws_bytes < plan->ws_bytes || ((uintptr_t)workspace & 15))
      return fail(CNN_E_SHAPE, "workspace must be >= %lld bytes and 16-byte aligned",
                  (long long)plan->ws_bytes);
  }
  return run_plan(In, Ker, Out, *plan, (hipStream_t)stream, workspace, dry);
}

}  // namespace cnnlib

extern "C" {

// The plan cnn_fwd uses on the current device: the cached one (the model's
// choice, or the winner of cnn_plan_find), else the model's choice, cached.
static int current_plan(const cnn_problem& p, int dtype, cnn_plan_t* plan) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail(CNN_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  const Key key(p.Nb, p.Nc, p.Nk, p.Nw, p.Nh, p.Nr, p.Ns, p.sw, p.sh, dtype, dev);
  {
    std::lock_guard<std::mutex> g(g_cache_mu);
    auto it = g_cache.find(key);
    if (it != g_cache.end()) {
      *plan = it->second;
      return CNN_OK;
    }
  }
  cnn_budget bud;
  int st;
  if ((st = cnn_device_budget(dev, &bud))) return st;
  if ((st = select_plan(p, dtype, bud, CNN_K_AUTO_NO_WORKSPACE, 0, 0, 0, plan)))
    return fail(st, "tile selection failed");
  std::lock_guard<std::mutex> g(g_cache_mu);
  g_cache.emplace(key, *plan);  // keeps a plan another thread stored first
  *plan = g_cache[key];
  return CNN_OK;
}

int cnn_plan_lookup(const cnn_problem* prob, int dtype, cnn_plan_t* plan) {
  if (!prob || !plan) return fail(CNN_E_NULL, "prob and plan must be non-NULL");
  int st;
  if ((st = check_problem(*prob)) || (st = check_dtype(dtype))) return st;
  return current_plan(*prob, dtype, plan);
}

int cnn_plan_find(const void* In, const void* Ker, void* Out, const cnn_problem* prob, int dtype,
                  void* stream, cnn_plan_t* plan, double* best_ms) {
  if (!prob || !plan) return fail(CNN_E_NULL, "prob and plan must be non-NULL");
  int st;
  if ((st = check_problem(*prob)) || (st = check_dtype(dtype))) return st;
  if ((st = check_buffers(In, Ker, Out, *prob, dtype))) return st;
  hipStream_t hs = (hipStream_t)stream;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  hipError_t e = hipStreamIsCapturing(hs, &cap);
  if (e != hipSuccess) return fail(CNN_E_HIP, "hipStreamIsCapturing: %s", hipGetErrorString(e));
  if (cap != hipStreamCaptureStatusNone)
    return fail(CNN_E_UNSUPPORTED, "cnn_plan_find times kernels and cannot run under capture");
  int dev = 0;
  if ((e = hipGetDevice(&dev)) != hipSuccess)
    return fail(CNN_E_HIP, "hipGetDevice: %s", hipGetErrorString(e));
  cnn_budget bud;
  if ((st = cnn_device_budget(dev, &bud))) return st;
  std::vector<cnn_plan_t> cands(256);
  int n = enumerate_plans(*prob, dtype, bud, cands.data(), (int)cands.size());
  if (n > (int)cands.size()) {
    cands.resize(n);
    n = enumerate_plans(*prob, dtype, bud, cands.data(), n);
  }
  // One workspace for the candidates that need one, freed before returning.
  int64_t ws_need = 0;
  for (int i = 0; i < n; ++i) ws_need = std::max(ws_need, cands[i].ws_bytes);
  void* ws = nullptr;
  if (ws_need > 0 && (e = hipMalloc(&ws, (size_t)ws_need)) != hipSuccess)
    return fail(CNN_E_HIP, "workspace of %lld bytes for timing: %s", (long long)ws_need,
                hipGetErrorString(e));
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if ((e = hipEventCreate(&e0)) != hipSuccess || (e = hipEventCreate(&e1)) != hipSuccess) {
    if (e0) (void)hipEventDestroy(e0);
    if (ws) (void)hipFree(ws);
    return fail(CNN_E_HIP, "hipEventCreate: %s", hipGetErrorString(e));
  }
  // Times `reps` back-to-back runs of candidate i: launched one by one, or
  // (graph) captured on a private stream into a HIP graph replayed on the
  // caller's stream.  Eager launches of kernels shorter than a few
  // microseconds time the host's launch rate rather than the kernels; a
  // graph replay times the kernels, as a captured caller runs them.
  auto time_it = [&](int i, int reps, float* ms, bool graph) -> int {
    int s2;
    hipGraphExec_t exec = nullptr;
    if (graph) {
      hipStream_t cs = nullptr;
      hipGraph_t g = nullptr;
      if ((e = hipStreamCreateWithFlags(&cs, hipStreamNonBlocking)) != hipSuccess)
        return fail(CNN_E_HIP, "hipStreamCreate: %s", hipGetErrorString(e));
      s2 = CNN_OK;
      if ((e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal)) == hipSuccess) {
        for (int r = 0; r < reps && s2 == CNN_OK; ++r) s2 = run_plan(In, Ker, Out, cands[i], cs, ws);
        const hipError_t e2 = hipStreamEndCapture(cs, &g);
        if (e == hipSuccess) e = e2;
      }
      if (e == hipSuccess && s2 == CNN_OK) e = hipGraphInstantiate(&exec, g, nullptr, nullptr, 0);
      if (g) (void)hipGraphDestroy(g);
      (void)hipStreamDestroy(cs);
      if (s2 != CNN_OK) return s2;
      if (e != hipSuccess) return fail(CNN_E_HIP, "graph capture: %s", hipGetErrorString(e));
      if ((e = hipGraphLaunch(exec, hs)) != hipSuccess) {  // first replay: untimed
        (void)hipGraphExecDestroy(exec);
        return fail(CNN_E_HIP, "hipGraphLaunch: %s", hipGetErrorString(e));
      }
    }
    if ((e = hipEventRecord(e0, hs)) != hipSuccess) {
      if (exec) (void)hipGraphExecDestroy(exec);
      return fail(CNN_E_HIP, "hipEventRecord: %s", hipGetErrorString(e));
    }
    if (exec) {
      e = hipGraphLaunch(exec, hs);
      if (e != hipSuccess) {
        (void)hipGraphExecDestroy(exec);
        return fail(CNN_E_HIP, "hipGraphLaunch: %s", hipGetErrorString(e));
      }
    } else {
      for (int r = 0; r < reps; ++r)
        if ((s2 = run_plan(In, Ker, Out, cands[i], hs, ws))) return s2;
    }
    if ((e = hipEventRecord(e1, hs)) != hipSuccess || (e = hipEventSynchronize(e1)) != hipSuccess ||
        (e = hipEventElapsedTime(ms, e0, e1)) != hipSuccess) {
      if (exec) (void)hipGraphExecDestroy(exec);
      return fail(CNN_E_HIP, "timing: %s", hipGetErrorString(e));
    }
    if (exec) (void)hipGraphExecDestroy(exec);
    *ms /= (float)reps;
    return CNN_OK;
  };
  const float kGraphBelowMs = 0.05f;  // candidates faster than this are timed by graph replay
  st = CNN_OK;
  // Warm-up: about 0.2 s of the first candidate, so that the first pass does
  // not time kernels while the clocks are still rising from idle.
  if (n > 0) {
    const auto t_start = std::chrono::steady_clock::now();
    for (int round = 0; round < 100000 && st == CNN_OK; ++round) {
      for (int r = 0; r < 8 && st == CNN_OK; ++r) st = run_plan(In, Ker, Out, cands[0], hs, ws);
      if (st == CNN_OK && (e = hipStreamSynchronize(hs)) != hipSuccess)
        st = fail(CNN_E_HIP, "warm-up: %s", hipGetErrorString(e));
      if (std::chrono::steady_clock::now() - t_start > std::chrono::milliseconds(200)) break;
    }
  }
  std::vector<float> first(n, 0.f), final_t(n, 0.f);
  for (int i = 0; i < n && st == CNN_OK; ++i) {
    float t1 = 0.f, t = 0.f;
    if ((st = time_it(i, 1, &t1, false))) break;  // first run: caches
    const int reps = t1 <= 0.f ? 20 : std::max(3, std::min(20, (int)(2.0f / t1)));
    if ((st = time_it(i, reps, &t, false))) break;
    if (t < kGraphBelowMs && (st = time_it(i, reps, &t, true))) break;
    first[i] = final_t[i] = t;
  }
  // The fastest candidates (overall, and among those that need no
  // workspace) and those within 25 % of them (at most six of each) are
  // timed again, interleaved over three rounds of longer runs, and ranked
  // by their fastest round: one short run per candidate differs by a few
  // per cent from run to run.
  auto argmin = [&](const std::vector<float>& t, bool ws_free) {
    int b = -1;
    for (int i = 0; i < n; ++i)
      if ((!ws_free || cands[i].ws_bytes == 0) && (b < 0 || t[i] < t[b])) b = i;
    return b;
  };
  if (st == CNN_OK && n > 0) {
    std::vector<int> fin;
    for (int pass = 0; pass < 2; ++pass) {
      const int b = argmin(first, pass == 1);
      if (b < 0) continue;
      std::vector<int> near;
      for (int i = 0; i < n; ++i)
        if ((pass == 0 || cands[i].ws_bytes == 0) && first[i] <= 1.25f * first[b]) near.push_back(i);
      std::sort(near.begin(), near.end(), [&](int x, int y) { return first[x] < first[y]; });
      if (near.size() > 6) near.resize(6);
      for (int i : near)
        if (std::find(fin.begin(), fin.end(), i) == fin.end()) fin.push_back(i);
    }
    if (fin.size() > 1) {
      for (int round = 0; round < 3 && st == CNN_OK; ++round)
        for (size_t f = 0; f < fin.size() && st == CNN_OK; ++f) {
          const float t0 = first[fin[f]];
          const int reps = t0 <= 0.f ? 50 : std::max(10, std::min(100, (int)(0.5f / t0)));
          float t = 0.f;
          if ((st = time_it(fin[f], reps, &t, t0 < kGraphBelowMs))) break;
          if (round == 0 || t < final_t[fin[f]]) final_t[fin[f]] = t;
        }
    }
  }
  const int best = st == CNN_OK ? argmin(final_t, false) : -1;
  const int best_free = st == CNN_OK ? argmin(final_t, true) : -1;
  if (best >= 0) {
    // Leave Out holding the returned plan's result, like a cnn_fwd call would.
    st = run_plan(In, Ker, Out, cands[best], hs, ws);
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (ws) {
    e = hipStreamSynchronize(hs);
    const hipError_t e2 = hipFree(ws);
    if (st == CNN_OK && (e != hipSuccess || e2 != hipSuccess))
      st = fail(CNN_E_HIP, "workspace release: %s", hipGetErrorString(e != hipSuccess ? e : e2));
  }
  if (st == CNN_OK && best < 0) st = fail(CNN_E_UNSUPPORTED, "no candidate plan");
  if (st == CNN_OK) {
    *plan = cands[best];
    if (best_ms) *best_ms = final_t[best];
    if (best_free >= 0) {
      const cnn_problem& p = *prob;
      std::lock_guard<std::mutex> g(g_cache_mu);
      g_cache[Key(p.Nb, p.Nc, p.Nk, p.Nw, p.Nh, p.Nr, p.Ns, p.sw, p.sh, dtype, dev)] =
          cands[best_free];
    }
  }
  return st;
}

int cnn_fwd(const void* In, const void* Ker, void* Out, int64_t Nb, int64_t Nc, int64_t Nk,
            int64_t Nw, int64_t Nh, int64_t Nr, int64_t Ns, int64_t sw, int64_t sh, int dtype,
            void* stream) {
  const cnn_problem p = {Nb, Nc, Nk, Nw, Nh, Nr, Ns, sw, sh};
  int st;
  if ((st = check_problem(p)) || (st = check_dtype(dtype))) return st;
  if ((st = check_buffers(In, Ker, Out, p, dtype))) return st;
  cnn_plan_t plan;
  if ((st = current_plan(p, dtype, &plan))) return st;
  return run_plan(In, Ker, Out, plan, (hipStream_t)stream);
}

int cnn_eq1_cost(const cnn_problem* prob, const cnn_tiles* tiles, int halo_mode, double terms[3],
                 double* footprint) {
  if (!prob || !tiles || !terms) return fail(CNN_E_NULL, "prob, tiles and terms must be non-NULL");
  int st;
  if ((st = check_problem(*prob))) return st;
  if (tiles->Tb < 1 || tiles->Tk < 1 || tiles->Tc < 1 || tiles->Tw < 1 || tiles->Th < 1)
    return fail(CNN_E_SHAPE, "tile sizes must be >= 1");
  if (halo_mode != 0 && halo_mode != 1) return fail(CNN_E_SHAPE, "halo_mode must be 0 or 1");
  eq1_terms(*prob, *tiles, halo_mode, terms, footprint);
  return CNN_OK;
}

int cnn_hbm_bytes(const cnn_plan_t* plan, int64_t xcds, int64_t l2_bytes, double terms[3]) {
  if (!plan || !terms) return fail(CNN_E_NULL, "plan and terms must be non-NULL");
  int st;
  if ((st = check_problem(plan->prob)) || (st = check_dtype(plan->dtype))) return st;
  if (xcds < 1 || l2_bytes < 1) return fail(CNN_E_SHAPE, "xcds and l2_bytes must be >= 1");
  if (plan->kernel == CNN_K_DIRECT || plan->kernel <= CNN_K_AUTO || plan->kernel > CNN_K_SPLITC ||
      plan->kernel == 9 ||
      plan->tk < 1 || plan->tp < 1)
    return fail(CNN_E_PLAN, "needs a tiled plan (not the direct kernel)");
  hbm_terms(*plan, xcds, l2_bytes, terms);
  return CNN_OK;
}

int cnn_closed_form(const cnn_problem* prob, double P, double M, int capacity_mode,
                    cnn_closed_form_t* out) {
  if (!prob || !out) return fail(CNN_E_NULL, "prob and out must be non-NULL");
  int st;
  if ((st = check_problem(*prob))) return st;
  if (!(P >= 1.0) || !(M > 0.0) || (capacity_mode != 0 && capacity_mode != 1))
    return fail(CNN_E_SHAPE, "need P >= 1, M > 0 and capacity_mode 0 or 1");
  closed_form(*prob, P, M, capacity_mode, out);
  if (!(out->M_L > 0.0)) return fail(CNN_E_SHAPE, "M leaves no relaxed capacity");
  return CNN_OK;
}

int cnn_slab_cost(const cnn_problem* prob, int64_t tk, int64_t tp, double terms[3]) {
  if (!prob || !terms) return fail(CNN_E_NULL, "prob and terms must be non-NULL");
  int st;
  if ((st = check_problem(*prob))) return st;
  if (tk < 1 || tp < 1) return fail(CNN_E_SHAPE, "tk and tp must be >= 1");
  slab_terms(*prob, tk, tp, terms);
  return CNN_OK;
}

}  // extern "C"
