// Vertical-slide offsets of the tile engine, on the host: for every plan of
// many windows and of low tiles (whose boxes are the tallest), the two 16-bit
// offsets of each column hold the exact positions of the entering and leaving
// pixels, and those lie in the ordinal image whatever row the slide goes to.
// So do the padding columns' two, in chained tiles too, which slide from the
// row above the tile.
#include <cstdio>
#include <vector>

#include "mf_internal.h"

namespace {

long long checked = 0;
int failures = 0;

void check(const mf::ImageDesc& d, const mf_footprint* fp) {
  ++checked;
  const int nc = (int)fp->col_lo.size();
  for (int j = 0; j < nc && failures < 20; ++j) {
    const int lo = fp->col_lo[j] - fp->dy_min, hi = fp->col_hi[j] - fp->dy_min;
    for (const bool up : {false, true}) {
      const uint32_t o = mf::slide_offsets(lo, hi, d.pitch, j, up);
      const int enter = (int)(o & 0xffffu), leave = (int)(o >> 16);
      // rows of the box, from the row the offsets count from
      const int er = up ? lo : hi + 1, lr = up ? hi + 1 : lo;
      bool ok = enter == er * d.pitch + j && leave == lr * d.pitch + j;
      // first and last tile row a slide starts from
      for (const int row : {up ? 1 : 0, up ? d.th - 1 : d.th - 2})
        for (const int col : {0, d.tw - 1}) {
          const int base = (row - (up ? 1 : 0)) * d.pitch + col;
          ok = ok && base + enter >= 0 && base + enter < d.pitch * d.bh && base + leave >= 0 &&
               base + leave < d.pitch * d.bh;
        }
      if (!ok) {
        std::printf("tile %dx%d box %dx%d pitch %d window %zux%d column %d up %d: %d %d\n", d.tw,
                    d.th, d.bw, d.bh, d.pitch, fp->row_lo.size(), nc, j, up, enter, leave);
        ++failures;
      }
    }
  }
}

// Padding columns of d's tables, for slides that start from tile rows r0 on.
void check_padding(const mf::ImageDesc& d, const mf_footprint* fp, int r0) {
  ++checked;
  const int lo = fp->col_lo[0] - fp->dy_min, hi = fp->col_hi[0] - fp->dy_min;
  for (const bool up : {false, true}) {
    if (up && r0 < 0) continue;   // (chained tiles slide down only)
    const uint32_t o = mf::slide_padding(mf::slide_offsets(lo, hi, d.pitch, 0, up));
    bool ok = (o & 0xffffu) == o >> 16;
    for (const int row : {up ? 1 : r0, up ? d.th - 1 : d.th - 2})
      for (const int col : {0, d.tw - 1}) {
        const int at = (row - (up ? 1 : 0)) * d.pitch + col + (int)(o >> 16);
        ok = ok && at >= 0 && at < d.pitch * d.bh;
      }
    if (!ok && failures++ < 20)
      std::printf("padding: tile %dx%d box %dx%d window %zux%zu up %d from row %d: %u\n", d.tw, d.th,
                  d.bw, d.bh, fp->row_lo.size(), fp->col_lo.size(), up, r0, o);
  }
}

void walk(const mf_footprint* fp) {
  const int lds_max = 160 * 1024;
  for (int dtype : {MF_U8, MF_U16, MF_F32})
    for (int tw : {1, 2, 3, 7, 8, 16, 31, 32, 56, 62, 63, 64})
      for (int th : {2, 3, 4, 5, 6, 7, 8, 11, 16, 48, 128}) {   // (one row does not slide)
        mf::ImageDesc d{};
        if (mf::make_plan(dtype, fp, lds_max, tw, th, &d) == MF_OK) check(d, fp);
        if (mf::make_plan_gs(dtype, fp, lds_max, tw, th, &d) == MF_OK) {
          check(d, fp);
          check_padding(d, fp, 0);
        }
        const mf_footprint* fx = mf::footprint_with_top_row(fp);
        if (mf::make_plan(dtype, fx, lds_max - 128, tw, th, &d) == MF_OK) check_padding(d, fx, -1);
      }
}

}  // namespace

int main() {
  for (int r : {0, 1, 2, 16, 60, 95, 100, 120, 123, 124, 125, 126, 127}) {
    mf_footprint* fp = nullptr;
    if (mf_footprint_disc(r, &fp) != MF_OK) return 2;
    walk(fp);
    mf_footprint_destroy(fp);
  }
  for (int w : {1, 3, 64, 191, 192, 193, 239, 252, 253, 254})
    for (int h : {1, 2, 100, 192, 240, 247, 248, 249, 250, 251, 252, 253, 254, 255}) {
      const double x0 = -(w / 2), x1 = x0 + w - 1, y0 = -(h / 2), y1 = y0 + h - 1, e = 0.25;
      const double xy[] = {x0 - e, y0 - e, x1 + e, y0 - e, x1 + e, y1 + e, x0 - e, y1 + e};
      mf_footprint* fp = nullptr;
      if (mf_footprint_polygon(xy, 4, &fp) != MF_OK) return 2;
      if ((int)fp->col_lo.size() != w || (int)fp->row_lo.size() != h) return 3;
      walk(fp);
      mf_footprint_destroy(fp);
    }
  std::printf("slide_check: %lld plans checked, %d failures\n", checked, failures);
  return failures ? 1 : 0;
}
