// Relationship matrix on the int8 matrix cores (grm_int.hip): plan and launch.
#pragma once

#include "tiles.h"

namespace pg {

// Where the int8 kernels are the path; elsewhere their fixed cost (the digit
// tables and the operand, 120 us a call) is not earned back.  Measured, us
// per call, int8 / fp64 (samples x variants), frequencies from 0.01 to 0.5, and in
// brackets panels of rare alleles alone (0.0005 to 0.004, all on low places):
//   work (samples^2 x variants) from 8e9 on: 2,000 x 2,000 244 / 337 (302), 1,500
//   x 4,000 259 / 265 (317), 800 x 16,000 267 / 315 (326), 1,000 x 8,000 256 / 244
//   (313), 1,500 x 8,000 319 / 464 (390); below: 1,200 x 4,000 223 / 196, 1,700 x
//   2,000 227 / 208;
//   long panels: 64 x 64,000 235 / 620, 300 x 64,000 295 / 638 (368);
//   small cohorts on 800 to 8,192 variants, where the fp64 kernel's ranges of
//   1,024 variants leave the chip idle: 100 x 1,000 128 / 176 (160), 400 x 8,000
//   181 / 191 (225), 800 x 4,000 187 / 195 (234); shorter: 100 x 500 122 / 100.
// From 4 million calls on the small cohorts lose a little (600 x 8,000 210 / 198,
// 1,000 x 4,000 224 / 203) and keep the smaller error.
constexpr double kGrmIntMinWork = 8e9;
constexpr int64_t kGrmIntLong = 32768;
constexpr int64_t kGrmIntSmall = 1024, kGrmIntShortMin = 800, kGrmIntShortMax = 8192;
// Its scratch beyond T: at most a ninth of the card, and the whole call (panel,
// T, scratch, full results) at most 224 GiB of 268; the fp64 kernel, which
// needs next to nothing beyond T, takes larger ones (100,000 samples x 3,000,000
// variants: 270 GB there, 355 GB here).
constexpr int64_t kGrmIntMaxBytes = (int64_t)32 << 30, kGrmIntMaxCall = (int64_t)224 << 30;

struct GrmIntPlan {
  int64_t nch;              // chunks of 64 variants
  int64_t tiles, nj;        // tiles, column strips
  int64_t blocks32;         // 32-sample blocks of G
  int64_t head;             // tiles run whole; the others in n_split ranges
  int64_t n_split, cps;     //   of cps chunks
  int64_t off_G, off_tab, off_cnt, off_stat, off_marks, off_panel, off_fine, off_part_s,
      off_part_n;
  int64_t bytes;
};
// Plans the int8 path for m samples and nv variants over the sample-major
// operand T (rows_pad x wp words), scratch from workspace offset `base` on;
// false where the fp64 kernel is the path.
bool grm_int_plan(int64_t m, int64_t nv, int64_t rows_pad, int64_t wp, int64_t base,
                  GrmIntPlan& p);
int launch_grm_int(const GrmIntPlan& p, char* ws, const uint32_t* T, int64_t m, int64_t rows_pad,
                   int64_t wp, double* grm, uint32_t* n_used, int full, hipStream_t st);

}  // namespace pg
