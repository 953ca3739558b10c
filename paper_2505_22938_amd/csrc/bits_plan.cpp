// Host side of the bit-plane path (bitplane.h): which windows take it, which
// variant, and the launch.

#include <algorithm>
#include <atomic>

#include "mf_internal.h"

namespace mf {

namespace {

struct Variant {
  int g, p, threads, sx, sy, tw, th;
};

template <int G, int P>
constexpr Variant variant() {
  using B = BitsGeo<G>;
  return {G, P, B::NT, B::SX, B::SY, B::TW, B::TH};
}

constexpr Variant kVariants[] = {
#define MF_BITS_ROW(I, G, P) variant<G, P>(),
    MF_BITS_TABLE(MF_BITS_ROW)
#undef MF_BITS_ROW
};
static_assert(sizeof(kVariants) / sizeof(kVariants[0]) == kBitsVariants, "variant table");

std::atomic<int> g_variant{MF_BITS_AUTO};   // mf_set_bits_override

// LDS: eight planes of the words, the box, the tap table
int lds_bytes(const Variant& v, int W, int H, int es) {
  const BitsLayout l = bits_layout(v.sx, v.sy, W, H);
  return 32 * l.nw + es * l.rp * l.rh + 4 * v.g * v.p;
}

// Estimated time in microseconds of variant v on a w x h image: instructions
// of a wave times the cycles each takes, plus launch, box load and output.
// A SIMD issues one vector instruction in about nine cycles with one wave on
// it and one in about four with two or more (measured with chains of single
// instructions: 9.4 and 4.8, 4.5 with four waves); the largest boxes leave
// room in the LDS for one workgroup, one wave per SIMD.  Estimated / measured
// us: uint16 disc 1 / 5 / 8 / 12 at 4096 x 4096 45 / 132 / 396 / 957 against
// 35 / 138 / 369 / 902; uint8 disc 4 / 16 at 256 x 256 15 / 23 against 10 / 17.
double bits_us(const Variant& v, int W, int H, int es, int lds_max, long long w, long long h) {
  const BitsLayout l = bits_layout(v.sx, v.sy, W, H);
  int lg = 0;
  while ((1 << lg) < v.g) ++lg;
  const double build = 350.0 * ((l.nw / 4 + v.threads - 1) / v.threads) + 120.0;
  const double n = es * (8.0 * (9.3 * v.p + 40.0 + 24.0 * lg) + build) + 600.0;
  const double waves = (double)((w + v.tw - 1) / v.tw) * (double)((h + v.th - 1) / v.th) *
                       (v.threads / 64);
  const double cycles = 2 * lds_bytes(v, W, H, es) <= lds_max ? 4.2 : 9.0;
  return 6.0 + std::max(9.0, cycles * waves / 1024.0) * n / 2400.0;
}

// The tile engine on the same image, near the line where the two paths meet:
// what it takes at least, by the pixel (4096 x 4096, disc 8 to 16: uint8 1.21
// ms, uint16 1.00, float32 1.35 before its first rows were halved, about 0.87
// times that since) and for one round of the smallest tiles.  At 4096 x 4096,
// smooth content, the bit planes win up to disc 12 for uint16 (0.87 ms against
// 0.95), disc 18 for uint8 (1.13 against 1.29) and disc 10 for float32 (0.98
// against 1.29).
double tile_us(int dtype, long long w, long long h) {
  const double ns = dtype == MF_U8 ? 0.063 : dtype == MF_U16 ? 0.052 : 0.072;
  return std::max(25.0, 1e-3 * ns * (double)w * (double)h);
}

}  // namespace

int bits_threads(int v) { return kVariants[v].threads; }

int bits_plan(int dtype, const mf_footprint* fp, int lds_max, int w, int h, int cus, ImageDesc* d,
              double* us, ImageDesc* tile_plan) {
  int tw = 0, th = 0;
  get_override(&tw, &th);
  // a tile shape asks for the tile engine, and the work counters count its work
  if (tw > 0 || work_counters_ptr()) return MF_ERR_UNSUPPORTED;
  const int forced = g_variant.load();
  if (forced == MF_BITS_OFF) return MF_ERR_UNSUPPORTED;
  const int H = (int)fp->row_lo.size(), W = (int)fp->col_lo.size(), es = elem_size(dtype);
  if (H > 64) return MF_ERR_UNSUPPORTED;   // the tap table is built by one wave, a row per lane
  // the filter's limit on windows is the tile engine's, whichever path runs:
  // the smallest tile's box, 8 x 8 pixels grown by the window, is at most 255
  // wide (and 256 tall, which 64 rows are)
  if (W + 7 > 255) return MF_ERR_UNSUPPORTED;
  int pairs = 0;
  for (int i = 0; i < H; ++i) {
    if (fp->row_hi[i] < fp->row_lo[i]) return MF_ERR_UNSUPPORTED;
    pairs += (fp->row_hi[i] - fp->row_lo[i] + 2) / 2;
  }
  const bool huge = ((double)w + 128.0) * ((double)h + 64.0) > 4e9;   // (tiles are at most 128 x 64)
  int best = -1;
  double best_us = 1e30;
  for (int i = 0; i < kBitsVariants; ++i) {
    const Variant& v = kVariants[i];
    if (forced >= 0 && i != forced) continue;
    if (v.g * v.p < pairs || lds_bytes(v, W, H, es) > lds_max) continue;
    // a launch holds fewer than 2^32 threads (half a thread to a pixel for 16
    // lanes a window; the tiles of the tile engine take a quarter)
    if (huge && (long long)((w + v.tw - 1) / v.tw) * ((h + v.th - 1) / v.th) * v.threads > 0xffffffffLL)
      continue;
    const double t = bits_us(v, W, H, es, lds_max, w, h);
    if (t < best_us) {
      best = i;
      best_us = t;
    }
  }
  if (best < 0) return MF_ERR_UNSUPPORTED;
  const double floor_us = tile_us(dtype, w, h);
  // Not clearly faster: against the tile plan, whose estimate is for smooth
  // content, whole rounds and walks as under large windows.  Noise takes up to a
  // quarter less, and many rounds drift apart, so over more than two the line
  // lies a tenth lower and part of a round counts as that (uint8 2048 x 2048
  // disc 20: 327 us here, tiles 345 on smooth content and 258 on noise; disc 14:
  // 162 here, the tiles more than 264).  Images of two values take the tiles two
  // to twelve times as long as smooth ones and no longer here (uint8 2077 x 1741
  // disc 20 309 us against 654, a checkerboard of 2465 x 2738 disc 19 535 against
  // 6440), so the line is not moved to where noise alone would put it.
  if (forced < 0 && best_us > floor_us) {
    constexpr int kManyTaps = 1 << 20;
    ImageDesc t{};
    if (choose_plan(dtype, fp, lds_max, 33, &t, w, h, cus) == MF_OK) {
      const long long tiles = (long long)((w + t.tw - 1) / t.tw) * ((h + t.th - 1) / t.th);
      const double tus = plan_us(t, kManyTaps, w, h, cus) *
                         (tiles > 2LL * cus ? 0.9 * (double)tiles / (double)((tiles + cus - 1) / cus * cus)
                                            : 1.0);
      if (best_us > std::max(floor_us, tus)) {
        if (tile_plan) *tile_plan = t;
        return MF_ERR_UNSUPPORTED;
      }
    }
  }
  if (us) *us = best_us;
  const Variant& v = kVariants[best];
  *d = ImageDesc{};
  d->bits = 1 + best;
  d->kt = dtype;
  d->shape = fp->kind == 0 ? SHAPE_DISC : SHAPE_SPANS;
  d->tw = v.tw;
  d->th = v.th;
  d->bw = v.tw + W - 1;
  d->bh = v.th + H - 1;
  d->T = d->bw * d->bh;
  d->dx_min = fp->dx_min;
  d->dy_min = fp->dy_min;
  d->nrows = H;
  d->ncols = W;
  d->limit = (int)fp->limit;
  d->lds_bytes = lds_bytes(v, W, H, es);
  return MF_OK;
}

int call_plan(int dtype, const mf_footprint* fp, const DeviceInfo& di, int w, int h, ImageDesc* d) {
  ImageDesc t;
  t.tw = 0;   // (set with the rest of it if tiles are the faster)
  if (bits_plan(dtype, fp, di.lds_max, w, h, di.cus, d, nullptr, &t) == MF_OK) return MF_OK;
  if (t.tw) {
    *d = t;
    return MF_OK;
  }
  return choose_plan(dtype, fp, di.lds_max, 33, d, w, h, di.cus);
}

int launch_bits(const ImageDesc& a, hipStream_t stream) {
  const int v = a.bits - 1;
  PlainKernelFn k = a.kt == MF_U8 ? pick_bits_u8(v) : a.kt == MF_U16 ? pick_bits_u16(v)
                                                                     : pick_bits_f32(v);
  const long long ntiles = (long long)a.tiles_x * a.tiles_y;
  if (ntiles > 0x7fffffffLL) return MF_ERR_UNSUPPORTED;
  (void)hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize,
                            a.lds_bytes);
  void* args[] = {const_cast<ImageDesc*>(&a)};
  if (hipLaunchKernel((const void*)k, dim3((unsigned)ntiles), dim3((unsigned)bits_threads(v)), args,
                      (size_t)a.lds_bytes, stream) != hipSuccess)
    return MF_ERR_HIP;
  return MF_OK;
}

}  // namespace mf

extern "C" int mf_set_bits_override(int variant) {
  if (variant < MF_BITS_OFF || variant >= MF_BITS_VARIANTS) return MF_ERR_INVALID_ARG;
  mf::g_variant.store(variant);
  return MF_OK;
}
