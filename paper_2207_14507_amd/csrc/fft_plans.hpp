// Radix plans of the transform lengths the library is built for.
//
// Row plans run on pairs of real rows packed into one complex row (length N = frame
// width), one transform per workgroup of 64 threads (128 for widths 1280 and 1920, 192 for
// 2160, 256 for 3840); the first radix is chosen so that the first pass maps one butterfly
// onto each thread, since a second, nearly empty round of it gathers almost as long as the
// first.  1080 = 18 x 6 x 10 has 60, 180 and 108 butterflies for 64 lanes and runs the row
// kernel in 2.9 us per candidate of 1920 x 1080 and the band kernel in 0.23, against 4.1
// and 0.29 as 15 x 8 x 9 (72 butterflies: two rounds); 2160 = 12 x 15 x 12 has 180, 144
// and 180 for 192 lanes: 3.95 and 0.40 us per candidate of 1280 x 2160 against 5.75 and
// 0.55 as 15 x 12 x 12 on 128 (18 x 10 x 12 on 128: 4.05 and 0.45).  3840 stays at three
// passes: 15 x 4 x 8 x 8 runs the 4K bf16 row kernel alone in 11.3 against 11.8 us, but a
// whole search 1% slower (the clock falls).  Widths of 256 and less take three small
// radices instead of two large ones, because a first radix of 8 to 16 leaves a wave 8 to
// 16 butterflies, each with all its samples to gather: 256 = 4 x 8 x 8 (64 butterflies)
// runs the row kernel in 0.117 instead of 0.186 us per candidate of 256 x 256 (16 x 16),
// the band kernel in 0.064 instead of 0.082.
//
// Column plans run on strips of 8 interleaved columns of the packed half spectrum (length
// M = frame height) with 256 threads (512 from 720 rows on; from 1280 rows on each
// 4-column half of a strip); their radices keep most lanes busy with few butterflies per
// thread (1920 = 8 x 16 x 15 has 960, 480 and 512 butterflies in a half strip: 3.9 to 4.0
// us per candidate of 1920 x 1080 against 4.1 as 16 x 12 x 10; 1280 = 16 x 8 x 10 has 320,
// 640 and 512: 1.77 us per candidate of 1280 x 720 on 512 threads against 1.92 on 256 and
// 2.30 on 320; heights of 256 and less: three small radices keep all four waves busy, 256
// = 8 x 4 x 8 0.123 us per candidate against 0.135 as 16 x 16, 160 = 5 x 8 x 4 0.067
// against 0.079, 120 = 5 x 6 x 4 0.056 against 0.071 on 256-wide frames).  At 1080 and
// 2160 rows the plans were picked by timing the alternatives on the device: an odd last
// radix (the inverse transform's first, whose stores a radix apart then fall on distinct
// LDS banks; at 1080 rows an odd first radix too) with a large middle radix beats the
// plans that keep every pass fullest (9 x 24 x 5 is 7% faster than 18 x 6 x 10, 12 x 20 x
// 9 is 12% faster than 18 x 6 x 20).  As prime-factor plans (no twiddle loads or
// multiplies; the column kernel reads the rows of dimension 0 in the Ruritanian order),
// 1080 = 27 x 8 x 5 is 8% faster again than 9 x 24 x 5 and 720 = 16 x 9 x 5 10% faster
// than 12 x 12 x 5 (9 x 16 x 5 and 5 x 16 x 9 lie between); at 2160 rows the prime-factor
// plans 27 x 16 x 5 and 16 x 27 x 5 lose to 12 x 20 x 9.  The inverse column transform
// uses the reversed column plan, so that its first pass consumes the forward transform's
// last-pass registers directly.
#pragma once

#include "fft_device.hpp"

namespace prnu {

template <int L>
struct RowPlan;
template <int L>
struct ColPlan;

#define PRNU_PLAN(KIND, L, ...)                              \
  template <>                                                \
  struct KIND<L> {                                           \
    using RS = Radices<__VA_ARGS__>;                         \
    static_assert(RS::product() == L, "plan must factor L"); \
    static_assert(RS::count >= 2, "at least two passes");    \
  };

// A prime-factor plan: pairwise coprime dimensions, no twiddles (Coprime above).
#define PRNU_PLAN_PFA(KIND, L, ...)                          \
  template <>                                                \
  struct KIND<L> {                                           \
    using RS = Coprime<__VA_ARGS__>;                         \
    static_assert(RS::product() == L, "plan must factor L"); \
    static_assert(RS::count >= 2, "at least two passes");    \
  };

PRNU_PLAN(RowPlan, 64, 2, 4, 8)
PRNU_PLAN(RowPlan, 96, 3, 4, 8)
PRNU_PLAN(RowPlan, 120, 3, 5, 8)
PRNU_PLAN(RowPlan, 160, 4, 5, 8)
PRNU_PLAN(RowPlan, 256, 4, 8, 8)
PRNU_PLAN(RowPlan, 720, 12, 6, 10)
PRNU_PLAN(RowPlan, 1080, 18, 6, 10)
PRNU_PLAN(RowPlan, 1280, 10, 16, 8)
PRNU_PLAN(RowPlan, 1920, 15, 8, 16)
PRNU_PLAN(RowPlan, 2160, 12, 15, 12)
PRNU_PLAN(RowPlan, 3840, 15, 16, 16)

PRNU_PLAN(ColPlan, 64, 4, 4, 4)
PRNU_PLAN(ColPlan, 96, 4, 6, 4)
PRNU_PLAN(ColPlan, 120, 5, 6, 4)
PRNU_PLAN(ColPlan, 160, 5, 8, 4)
PRNU_PLAN(ColPlan, 256, 8, 4, 8)
PRNU_PLAN_PFA(ColPlan, 720, 16, 9, 5)
PRNU_PLAN_PFA(ColPlan, 1080, 27, 8, 5)
PRNU_PLAN(ColPlan, 1280, 16, 8, 10)
PRNU_PLAN(ColPlan, 1920, 8, 16, 15)
PRNU_PLAN(ColPlan, 2160, 12, 20, 9)

#undef PRNU_PLAN
#undef PRNU_PLAN_PFA

// X-macro lists of supported lengths: every planned length can be a row length (frame
// width N); column lengths (frame height M) are limited by the LDS of one column strip.
#define PRNU_FOR_EACH_LENGTH(X) \
  X(64) X(96) X(120) X(160) X(256) X(720) X(1080) X(1280) X(1920) X(2160) X(3840)
#define PRNU_FOR_EACH_COL_LENGTH(X) \
  X(64) X(96) X(120) X(160) X(256) X(720) X(1080) X(1280) X(1920) X(2160)

// Which twiddle table: the row plan, the column plan, or the reversed column plan.
enum PlanKind { kRowPlan = 0, kColPlan = 1, kColPlanRev = 2 };

}  // namespace prnu
