// Host side of the two-dimensional-tile kernel (conv_tile): its instantiation
// table, the geometry of a tile on a problem, the launch.
#include "tile_kernel.h"

namespace cnnlib {

static const VariantT kVariantsT[] = {
#define CNN_ROWT(id, dt, wm, wn, mb, nb, ks, nr, ns, maxp, kch, occ)                       \
  {id, dt, 32 * (wm) * (mb), 32 * (wn) * (nb), 16 * (ks), 16 * (mb) * (nb), nr, ns, maxp, \
   kch, occ, nb, (wm) * (wn)},
    CNN_TILE_VARIANTS(CNN_ROWT)
#undef CNN_ROWT
};

const VariantT* variants_tile(int* count) {
  *count = (int)(sizeof(kVariantsT) / sizeof(kVariantsT[0]));
  return kVariantsT;
}

// The geometry of instantiation v with tiles of tr whole output rows; false
// if it does not fit.
bool tile_geometry(const VariantT& v, const cnn_problem& p, int dtype, int64_t tr, TileShape* s) {
  const int64_t es = in_bytes(dtype), RS = p.Nr * p.Ns;
  const int64_t Nx = p.sw * (p.Nw - 1) + p.Nr, Ny = p.sh * (p.Nh - 1) + p.Ns;
  if ((v.nr && (v.nr != p.Nr || v.ns != p.Ns)) || tr < 1 || tr > v.tp) return false;
  // the fewest bands whose columns fit the accumulators, of equal width; of
  // whole 32 columns where that makes no more bands, else of whole 8, so that a
  // lane's 16 bytes of Out never straddle two rows of a band (64 -> 32 features
  // at 196x196, batch 5, bf16 Out: bands of 49 columns 37.7 us, of 40 21.1);
  // the last band then overlaps its neighbour
  const int64_t ctmax = v.tp / tr;
  const int64_t bands = (p.Nh + ctmax - 1) / ctmax;
  int64_t ct = (p.Nh + bands - 1) / bands;
  if (bands > 1) {
    const int64_t up32 = (ct + 31) / 32 * 32, up8 = (ct + 7) / 8 * 8;
    if (ctmax < 8) return false;
    ct = up32 <= ctmax && (p.Nh + up32 - 1) / up32 == bands ? up32
         : up8 <= ctmax                                     ? up8
                                                            : ctmax / 8 * 8;
    if (ct > p.Nh) ct = p.Nh;
  }
  s->tr = tr;
  s->ct = ct;
  s->ncol = (p.Nh + ct - 1) / ct;
  s->gather = p.Ns == 1 && p.sh > 1;
  s->squeeze = p.sw >= p.Nr;
  s->cw = s->gather ? ct : p.sh * (ct - 1) + p.Ns;
  s->hp = s->gather ? ct : (s->cw + p.sh - 1) / p.sh;
  s->pitch = s->gather ? ct : s->hp * p.sh;
  // 16-byte items where a band is that wide; pairs need two columns
  const int64_t epc = 16 / es;
  s->form = s->cw < epc || p.sh > 2 ? kPairs : p.sh == 1 ? kWide1 : s->gather ? kGather2 : kWide2;
  s->pw = s->form == kPairs ? 2 : epc;
  // (two loads per item and 128 features on four waves: the registers spill,
  // 20 us where the model says 12 -- 240 -> 221 features, 1x1 stride 2 at 22x13,
  // batch 5, 14 us by other plans)
  if (s->gather && v.nr == 1 && v.tk == 128 && v.waves == 4) return false;
  if (s->cw < 2) return false;
  const int64_t rows_total = p.Nb * p.Nw;
  const int64_t rows = tr < rows_total ? tr : rows_total;
  // a run of rows crosses at most this many image boundaries (none where runs
  // divide images, one less where images divide runs)
  int64_t cross = p.Nw % tr == 0   ? 0
                  : tr % p.Nw == 0 ? rows / p.Nw - 1
                                   : (rows - 1 + p.Nw - 1) / p.Nw;
  if (cross > p.Nb - 1) cross = p.Nb - 1;
  s->S = s->squeeze ? rows * p.Nr : p.sw * (rows - 1) + p.Nr + cross * (p.Nr - p.sw);
  // 16-bit vector positions, an odd count of them per channel group; 8-bit taps
  s->SP = (s->S * s->pitch) | 1;
  if (s->SP > 65535 || RS > 255) return false;
  const int64_t groups = v.tc / 8, planes = dtype == CNN_F32 ? 3 : 1;
  // Ker items per feature: 16 bytes of channels (1x1), or runs of 16 bytes of
  // taps of a channel (pair)
  s->njt = (RS + epc - 1) / epc;
  s->nch = v.nr == 1 ? v.tc / epc : v.tc / (dtype == CNN_F32 ? 1 : 2) * s->njt;
  const int64_t nt = 64 * v.waves;
  const int64_t pt = groups < v.waves ? nt / groups : 64;
  if (s->S * ((s->cw + s->pw - 1) / s->pw) > pt * v.maxp ||
      (v.nr != 3 && v.tk * s->nch > nt * v.kch))
    return false;
  s->lds = 2 * (planes * groups * s->SP * 16 +
                tile_ker_bytes((int)v.tk, (int)es, v.nr * v.ns, (int)groups, (int)RS));
  // the epilogue's transposition: 32 features of every wave's outputs
  const int64_t xp = v.waves * 32 * 32 * v.nb * (dtype == CNN_BF16_OBF16 ? 2 : 4);
  if (s->lds < xp) s->lds = xp;
  if (s->lds > 160 * 1024) return false;
  s->n_rt = (rows_total + tr - 1) / tr;
  // 32-bit byte offsets from a tile's first image, and into Ker
  const int64_t imgs = cross + 1;
  const int64_t lim = 1LL << 31;
  return imgs * p.Nc * Nx * Ny < lim / es && p.Nk * p.Nc * RS < lim / es &&
         imgs * (p.Nk + 288) * p.Nw * p.Nh < lim / out_bytes(dtype);
}

hipError_t launch_tile(const VariantT& v, const void* In, const void* Ker, void* Out,
                       const ConvArgs& a, const TileShape& s, int64_t grid, hipStream_t stream) {
  TileGeo t;
  t.tr = (int32_t)s.tr;
  t.ct = (int32_t)s.ct;
  t.ncol = (int32_t)s.ncol;
  t.rows_total = a.Nb * a.Nw;
  t.pitch = (int32_t)s.pitch;
  t.hp = (int32_t)s.hp;
  t.SP = (int32_t)s.SP;
  t.squeeze = s.squeeze;
  t.nch = (int32_t)s.nch;
  t.njt = (int32_t)s.njt;
  t.njd = make_fastdiv((uint32_t)s.njt);
  t.nst = (a.Nc + (int32_t)v.tc - 1) / (int32_t)v.tc;
  t.units = v.dtype == CNN_F32 && (int64_t)a.Nc * a.Nr * a.Ns < 8;
  t.kt = make_fastdiv((uint32_t)a.n_ktiles);
  t.ncold = make_fastdiv((uint32_t)s.ncol);
  t.nw = make_fastdiv((uint32_t)a.Nw);
  t.nx = make_fastdiv((uint32_t)a.Nx);
  t.ipr = make_fastdiv((uint32_t)((s.cw + s.pw - 1) / s.pw));
  t.ctd = make_fastdiv((uint32_t)s.ct);
  t.shd = make_fastdiv((uint32_t)a.sh);
  t.nr = make_fastdiv((uint32_t)a.Nr);
  t.rsd = make_fastdiv((uint32_t)(a.Nr * a.Ns));
  t.nsd = make_fastdiv((uint32_t)a.Ns);
  t.nchd = make_fastdiv((uint32_t)s.nch);
  for (TileLaunch f : {launch_tile_f32, launch_tile_3x3_bf16, launch_tile_3x3_obf16,
                       launch_tile_any_bf16, launch_tile_any_obf16}) {
    const hipError_t e = f(v.id, In, Ker, Out, a, t, s.form, s.lds, grid, stream);
    if (e != hipErrorInvalidValue) return e;
  }
  return hipErrorInvalidValue;
}

}  // namespace cnnlib
