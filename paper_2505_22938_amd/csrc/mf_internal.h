// Internal declarations shared by the library's host sources.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/median_filter.h"

struct mf_footprint {
  // kind: 0 = disc given by an integer squared limit; 1 = general convex
  // shape given only by its spans.  Both carry the spans.
  int kind = 1;
  long long limit = 0;
  int dx_min = 0, dx_max = 0, dy_min = 0, dy_max = 0;
  int taps = 0;
  std::vector<int> row_lo, row_hi;  // index dy - dy_min: dx range of that row
  std::vector<int> col_lo, col_hi;  // index dx - dx_min: dy range of that column

  // Per-device copies of the span tables (int16 pairs: rows then columns).
  struct DevCopy {
    int device;
    void* ptr;
  };
  mutable std::mutex mu;
  mutable std::vector<DevCopy> dev;
};

namespace mf {

constexpr int kThreads = 1024;            // threads per tile workgroup
constexpr int kWaves = kThreads / 64;     // wave64
constexpr int kDigits = 16;               // 4-bit radix digits
constexpr int kCounterBytes = kDigits * kThreads * 2;
constexpr int kHistWords = 256;           // seed histogram bins per wave (32-bit)
constexpr int kHistBytes = kWaves * kHistWords * 4;

enum { KEY_U8 = 0, KEY_U16 = 1, KEY_F32 = 2 };
enum { SHAPE_DISC = 0, SHAPE_SPANS = 1 };

// Bit-plane variants (bitplane.h): index, lanes per window, tap pairs per
// lane.  A window of n pairs fits where n <= lanes * pairs.
#define MF_BITS_TABLE(X) \
  X(0, 1, 4) X(1, 1, 9) X(2, 1, 18) X(3, 1, 29) X(4, 1, 46) \
  X(5, 2, 32) X(6, 2, 41) X(7, 2, 50) \
  X(8, 4, 8) X(9, 4, 12) X(10, 4, 18) X(11, 4, 27) X(12, 4, 34) X(13, 4, 43) X(14, 4, 50) \
  X(15, 8, 22) X(16, 8, 30) X(17, 8, 36) X(18, 8, 42) X(19, 8, 47) \
  X(20, 16, 22) X(21, 16, 27) X(22, 16, 33) X(23, 16, 41) X(24, 16, 50)
constexpr int kBitsVariants = MF_BITS_VARIANTS;

// Their workgroup and tile: G lanes share a window; GX x GY sub-tiles of SX x
// SY pixels, one word of 32 pixels (one of each sub-tile) per G threads.
template <int G>
struct BitsGeo {
  static constexpr int NT = 256;   // threads
  static constexpr int WD = NT / G;               // words = pixels of a sub-tile
  static constexpr int SX = G <= 2 ? 32 : G == 16 ? 8 : 16;
  static constexpr int SY = WD / SX;
  static constexpr int GX = 4, GY = 8;
  static constexpr int TW = GX * SX, TH = GY * SY;
};

// LDS layout for a window of W x H: rows of `pitch` words (a multiple of
// four), nw words a plane; box rows of rp pixels, rh of them.
struct BitsLayout {
  int pitch, nw, rp, rh;
};
__host__ __device__ inline BitsLayout bits_layout(int sx, int sy, int W, int H) {
  BitsLayout l;
  l.pitch = (sx + W - 1 + 3) & ~3;
  l.nw = l.pitch * (sy + H - 1);
  l.rp = (3 * sx + l.pitch + 15) & ~15;
  l.rh = 8 * sy + H - 1;
  return l;
}

// Everything one tile needs to know about its image and plan.  Passed by
// value to the plain kernels and stored in the batched descriptor table.
constexpr int kMaxRankOutputs = MF_MAX_RANK_OUTPUTS;   // planes of one general-rank call

// Window of one output plane when the planes of a general-rank call use
// different footprints (all inside the plan's box): its device span table
// (rows then columns, as ImageDesc::spans), geometry, disc limit and the
// largest valid rank (taps - 1).
struct PlaneFp {
  const short2* spans;
  int dx_min, dy_min, nrows, ncols, limit, rank_hi;
};

struct ImageDesc {
  const void* img;
  void* out;
  long long stride;  // elements (image and output)
  int w, h, boundary;
  int tw, th, tiles_x, tiles_y;
  int bw, bh, T, pitch;
  int dx_min, dy_min, nrows, ncols;
  int rank, limit;
  int segs, band_rows, hist_shift;
  const short2* spans;  // nrows row spans (index dy - dy_min) then ncols column spans
  // LDS layout, bytes (off_I: the ordinal image)
  int off_p, off_C, off_B, off_I, off_hist, off_tab, lds_bytes;
  unsigned long long* counters;  // optional work counters (null: off)
  // global-scratch variant: per-workgroup slot of slot_bytes at scratch;
  // claim: the persistent grid's tile-claim words (zero between launches)
  unsigned char* scratch;
  long long slot_bytes;
  unsigned int* claim;
  // off_sort: LDS offset of the digit counters of float keys sorted in LDS
  int off_x1, off_sort, ipt;
  // kernel selection: key type, shape, 1 = global-scratch variant, and the
  // register capacity (elements per thread) of the LDS variant
  int kt, shape, gs, imax;
  int bits;   // 0, or 1 + the bit-plane variant (tw x th then its tile)
  int default_gs;   // choose_plan: 1 = the default shape (before fitting) takes scratch
  // bracketed tiles (learned path): per-tile [lo, hi] keys, the number of
  // in-bracket pixels region A can hold, and the list (y * w + x) and count
  // of output pixels whose median fell outside their tile's bracket
  const uint2* brackets;
  int br_cap;
  unsigned int* miss;
  unsigned int* miss_count;
  // general ranks (kernels instantiated for them only): nq output planes
  // from one ordinal transform per tile; plane q is written to outs[q] at
  // rank ranks[q], or at the per-pixel rank rmaps[q][y * rmap_strides[q] +
  // x] (int32, clamped to [0, rank_hi]) where rmaps[q] is set.  nq = 0: the
  // single plane `out` at `rank`.
  int nq, rank_hi;
  void* outs[kMaxRankOutputs];
  const int* rmaps[kMaxRankOutputs];
  long long rmap_strides[kMaxRankOutputs];  // elements
  int ranks[kMaxRankOutputs];
  // multi_fp = 1: plane q uses the window pfp[q] instead of the plan's
  // (whose box, tables and kernel shape cover all of them)
  int multi_fp;
  PlaneFp pfp[kMaxRankOutputs];
  // chained tiles: LDS offset of the forwarded last-row locations (64 u16)
  int off_fwd;
};

// Vertical slide of a window by one row over the ordinal image: the entering
// pixel (low half) and the leaving one (high half) of window column j, whose
// pixels are rows lo .. hi of the window's offset rectangle, as 16-bit
// elements from the rectangle's top left before the slide (going up: from one
// row above that).  Either way the two lie on rows lo and hi + 1 from there,
// so the largest is nrows * pitch + ncols - 1, and the plan's pitch keeps that
// below 2^16.
__host__ __device__ inline uint32_t slide_offsets(int lo, int hi, int pitch, int j, bool up) {
  const uint32_t top = (uint32_t)(lo * pitch + j), below = (uint32_t)((hi + 1) * pitch + j);
  return up ? top | (below << 16) : below | (top << 16);
}
// A column that counts nothing: the leaving pixel of `o` twice, a pixel of the
// window before the slide and so in the box (the place the offsets count from
// may lie above it: chained tiles slide from the row above the tile).
__host__ __device__ inline uint32_t slide_padding(uint32_t o) { return (o & 0xffff0000u) | (o >> 16); }

struct DeviceInfo {
  int lds_max = 0;
  int cus = 0;
};
int device_info(int dev, DeviceInfo* out);

// Tile plans.  make_plan: everything in LDS; make_plan_gs: the omnigram in
// a global scratch slot.  choose_plan picks the tuned shape
// for this (dtype, footprint) if one is recorded, else the widest layout
// that fits, LDS first; imax_cap bounds the register capacity of LDS plans.
int make_plan(int dtype, const mf_footprint* fp, int lds_max, int tw, int th, ImageDesc* d);
int make_plan_gs(int dtype, const mf_footprint* fp, int lds_max, int tw, int th, ImageDesc* d);
// w, h, cus (image size and compute units, 0 = unknown) let the default
// choice keep enough tiles per CU; with `spread` it is fitted to the call
// (fit_plan, and for small images by plan_us, a shape's estimated time).
// Without cus the image is one of a batch, whose other tiles fill the chip.
// choose_plan_tall: the override or the tallest default shape, ignoring the
// tuned table (bracketed tiles).
int choose_plan(int dtype, const mf_footprint* fp, int lds_max, int imax_cap, ImageDesc* d,
                int w = 0, int h = 0, int cus = 0, bool spread = true);
// choose_plan without the override and the tuned table.
int untuned_plan(int dtype, const mf_footprint* fp, int lds_max, int imax_cap, ImageDesc* d,
                 int w, int h, int cus, bool spread);
double plan_us(const ImageDesc& c, int taps, int w, int h, int cus);
int choose_plan_tall(int dtype, const mf_footprint* fp, int lds_max, int imax_cap,
                     ImageDesc* d);
// Bracketed-tile plan (8/16-bit keys) for a given shape: region A holds only
// the in-bracket pixels (up to br_cap of them), region B the ordinal image
// of the whole box.  MF_ERR_UNSUPPORTED if fewer than 1024 fit.
int make_plan_br(int dtype, const mf_footprint* fp, int lds_max, int tw, int th, ImageDesc* d);
// Enumerate every valid plan (for the autotuner).
std::vector<ImageDesc> candidate_plans(int dtype, const mf_footprint* fp, int lds_max,
                                       int imax_cap);
// The slot of float keys sorted in LDS holds the omnigram only, a quarter of the
// plan's layout with the words of the stable passes (done by bind_image).
void trim_slot(ImageDesc* d);
// Fill the per-image fields of a plan.
void bind_image(ImageDesc* d, const void* img, int w, int h, size_t stride_bytes, int dtype,
                const mf_footprint* fp, int boundary, int rank, const void* spans);

int validate_image(const void* img, int w, int h, size_t stride_bytes, int dtype,
                   const mf_footprint* fp, int boundary, const void* out);

// Global scratch cached per (device, stream); never allocates while the
// stream is capturing (MF_ERR_UNSUPPORTED instead).  release_scratch frees
// every cached buffer (mf_release_scratch).  *out points to `bytes` of slot
// space; the kClaimBytes before it hold the tile-claim words (nine used),
// zeroed when the buffer is allocated and left zero by every launch that
// uses them.  Outside capture the buffer is grown to keep_bytes if that is more
// and there is memory for it.  The caller keeps `hold` until its kernel is queued.
constexpr int kClaimBytes = 256;
int get_scratch(int dev, hipStream_t stream, size_t bytes, void** out,
                std::unique_lock<std::mutex>* hold, size_t keep_bytes = 0);
int release_scratch();

// Tuned tile shapes, keyed by dtype and footprint.
std::string tune_key(int dtype, const mf_footprint* fp);
bool tuned_shape(int dtype, const mf_footprint* fp, int* tw, int* th);
void record_tuned_shape(int dtype, const mf_footprint* fp, int tw, int th, double ms);
void erase_tuned_shape(int dtype, const mf_footprint* fp);
int tune_cache_load(const char* path);
int tune_cache_save(const char* path);

// Device work counters of the plain engine (null when counting is off).
unsigned long long* work_counters_ptr();

// Plain-filter launch with a complete plan (median_plain.hip); a.nq > 0
// runs the general-rank kernels (median_general.hip).
// ext_scratch (non-null): a global-scratch plan takes its slots from this
// buffer of ext_bytes bytes instead of the cached per-stream scratch, its
// persistent grid shrunk to the slots that fit (MF_ERR_SCRATCH_LIMIT if not
// even one does); nothing is allocated.  keep_bytes: cached scratch that is
// allocated holds at least that much where there is memory for it.
using PlainKernelFn = void (*)(ImageDesc);
int launch_with_plan(ImageDesc a, int dev, const DeviceInfo& di, hipStream_t stream,
                     unsigned char* ext_scratch = nullptr, size_t ext_bytes = 0,
                     size_t keep_bytes = 0);
PlainKernelFn pick_general_kernel(const ImageDesc& d);
// Workgroups of a global-scratch plan bound to its image, a slot each.
long long scratch_slots(const ImageDesc& a, const DeviceInfo& di);
// The LDS shape of least estimated time (MF_ERR_UNSUPPORTED: no box fits).
int lds_plan(int dtype, const mf_footprint* fp, int lds_max, int imax_cap, int w, int h, int cus,
             ImageDesc* d);
// What an uncaptured call's default plan would have taken of its stream's
// scratch where the fitted one takes none (forgotten by release_scratch).
void note_scratch(int dev, hipStream_t stream, size_t bytes);
bool scratch_noted(int dev, hipStream_t stream, size_t bytes);
// The same for the plan of choose_plan(.., spread), completed by `bind`.  Scratch
// belongs to the stream: graphs captured on one stream bake in the same buffer
// and tile claims, and hipStreamPerThread names a stream of each thread.  So a
// window whose default plan is an LDS one runs on that there, and the fitted
// global-scratch plan is for calls that the stream orders.  Where scratch is not
// to be had (a capturing stream with too little, no memory) the default plan is
// tried.  A captured call is to run wherever an uncaptured one on an image as
// large came before it on the stream: that one leaves the scratch of its default
// plan, or a note of it where its tiles sort in LDS (the captured call's may
// then, too).
template <typename Bind>
int launch_fitted(ImageDesc a, int dtype, const mf_footprint* fp, int w, int h, int dev,
                  const DeviceInfo& di, hipStream_t stream, Bind&& bind) {
  bind(&a);
  if (!a.gs && !a.default_gs) return launch_with_plan(a, dev, di, stream);
  ImageDesc d{};
  int rc = choose_plan(dtype, fp, di.lds_max, 33, &d, w, h, di.cus, false);
  if (rc) return rc;
  bind(&d);
  const size_t need = d.gs ? (size_t)scratch_slots(d, di) * (size_t)d.slot_bytes : 0;
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  const bool known = hipStreamIsCapturing(stream, &cap) == hipSuccess;
  const bool capturing = cap != hipStreamCaptureStatusNone;
  if (!a.gs) {
    if (!known) (void)hipGetLastError();
    else if (!capturing) note_scratch(dev, stream, need);
    return launch_with_plan(a, dev, di, stream);
  }
  if (!known) return MF_ERR_HIP;
  if (!d.gs && (capturing || stream == hipStreamPerThread))
    return launch_with_plan(d, dev, di, stream);
  rc = launch_with_plan(a, dev, di, stream, nullptr, 0, need);
  if (rc != MF_ERR_UNSUPPORTED && rc != MF_ERR_NOMEM) return rc;
  (void)hipGetLastError();
  rc = launch_with_plan(d, dev, di, stream);
  if (rc != MF_ERR_UNSUPPORTED || !scratch_noted(dev, stream, need)) return rc;
  ImageDesc l{};
  if (lds_plan(dtype, fp, di.lds_max, 33, w, h, di.cus, &l) != MF_OK) return rc;
  bind(&l);
  return launch_with_plan(l, dev, di, stream);
}
// The plan of a plain call: bit planes, or tiles fitted to the image.
int call_plan(int dtype, const mf_footprint* fp, const DeviceInfo& di, int w, int h, ImageDesc* d);
// Bit-plane path: plan for a window it takes (MF_ERR_UNSUPPORTED otherwise),
// kernel, and launch with a complete plan.
// us (optional): the estimated time of the image.  tile_plan (optional): set to
// choose_plan's where that was found the faster.
int bits_plan(int dtype, const mf_footprint* fp, int lds_max, int w, int h, int cus, ImageDesc* d,
              double* us = nullptr, ImageDesc* tile_plan = nullptr);
PlainKernelFn pick_bits_u8(int v);
PlainKernelFn pick_bits_u16(int v);
PlainKernelFn pick_bits_f32(int v);
int bits_threads(int v);
// Kernels of batch plans: descriptors (read through the constant address
// space, so that each field is a scalar load where it is used instead of a
// copy in registers), tile queue, slice [begin, end), counters and scratch.
using ConstDesc = const __attribute__((address_space(4))) ImageDesc;
using BatchKernelFn = void (*)(ConstDesc*, const int2*, int, int, int*, unsigned char*, long long);
BatchKernelFn pick_bits_batched_u8(int v);
BatchKernelFn pick_bits_batched_u16(int v);
BatchKernelFn pick_bits_batched_f32(int v);
int launch_bits(const ImageDesc& a, hipStream_t stream);
// median_filter_windows: one pass for all windows (set by
// mf_set_window_fusion) instead of grouping them by box size.
bool window_fusion_all();
void set_window_fusion_all(int all);
int launch_window_pass(const void* img, int w, int h, size_t stride_bytes, int dtype,
                       int boundary, const mf_window_output* outs, const int* idx, int n,
                       int dev, const DeviceInfo& di, hipStream_t stream);

// Tile-shape override (measurement): 0 = off.
void get_override(int* tw, int* th);

// Upload (once per device) and return the device span table of `fp`:
// [row (lo,hi) pairs as int16][column (lo,hi) pairs as int16].
// MF_ERR_UNSUPPORTED if the table is not there yet and `stream` is capturing.
int footprint_device_table(const mf_footprint* fp, int device, const void** table,
                           hipStream_t stream);
// The same footprint with one empty row added above its first row (cached,
// owned by the library): a box planned for it has one extra row on top, the
// row whose windows chained tiles forward.
const mf_footprint* footprint_with_top_row(const mf_footprint* fp);
// The same table on the host: 2 * (rows + columns) int16 values written to
// `dst` (which holds at least that many); returns the count.
size_t footprint_span_table(const mf_footprint* fp, int16_t* dst);
size_t footprint_span_table_len(const mf_footprint* fp);

inline int elem_size(int dtype) { return dtype == MF_U8 ? 1 : dtype == MF_U16 ? 2 : 4; }

}  // namespace mf
