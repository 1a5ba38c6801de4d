// Rules by which the host layer shapes the edge path's launches: plain
// functions of the views' sizes, with no HIP calls, so that they can be
// exercised on a machine without a GPU.
#pragma once

#include <stdint.h>

#include "../../include/igsp.h"

namespace igsp {

// Strip geometry of the fused stencil kernel: a wavefront owns 64 lanes x 4
// adjacent columns = 256 input columns, of which the 4 outermost on each
// side are halo (2 blur + 1 Sobel + 1 suppression), leaving 248 outputs.
constexpr int kLanePx = 4;
constexpr int kWaveCols = 64 * kLanePx;       // 256
constexpr int kHalo = 4;
constexpr int kStripCols = kWaveCols - 2 * kHalo;  // 248

// Wavefronts of a call's stencil launch at a segment height: all views' together
// or, in the plain form, which launches each view on its own, one view's (the
// mean).
inline int64_t stencil_waves(const igsp_view* views, int32_t n, int seg, int form) {
  int64_t waves = 0;
  for (int i = 0; i < n; ++i)
    waves += (int64_t)((views[i].width + kStripCols - 1) / kStripCols) * ((views[i].height + seg - 1) / seg);
  return form == IGSP_PLAIN && n > 0 ? waves / n : waves;
}

// Segment height when none is given or tuned: the tallest of a few heights
// that still gives a stencil launch 16 wavefronts per CU (four per SIMD),
// else the shortest. A wavefront's march is a chain of dependent rows, so a
// launch with fewer wavefronts than the chip holds lasts about one segment:
// shorter segments then save more time than their extra halo rows cost.
constexpr int kShortestSeg = 10;

inline int default_seg_rows(const igsp_view* views, int32_t n, int form, int cus) {
  const int heights[] = {64, 40, 28, 22, 16, kShortestSeg};
  const int64_t target = 16 * (int64_t)cus;
  for (int seg : heights)
    if (stencil_waves(views, n, seg, form) >= target) return seg;
  return kShortestSeg;
}

// Rows per segment as a plan marches a given, tuned or default height: whole
// rounds of the stencil loop's six rows (the rows past a segment's end would be
// computed all the same; 150 views BF16, 100 rows marched as 102: 864 -> 855 us
// of edge maps). Plans are told apart by this height. A plan
// of the shortest segments whose wavefronts would leave most SIMDs with one
// or none splits them once more, to one round: a lone wavefront takes about
// 0.5 us a row, and shorter segments save more than their window-filling rows
// (2.7 rows' work) and histogram flushes cost. At 10 rows marched as 12 / 6, us,
// with the launch's wavefronts at 6 rows (256 CUs): one FP32 256x192 view (64)
// 22.8 / 19.9, 1297x840 (840) 27.0 / 26.1, 1736x1098 (1281) 30.4 / 29.1, 2232x1020
// (1530) 32.3 / 31.8, BF16 23.9 / 24.4, two 1297x840 (1680) 37.4 / 37.6: the line is
// at 1.5 wavefronts per SIMD. A plain call's launches follow one another, so that
// each fills gaps of the last: three FP32 1297x840 views 78.0 / 74.3, 1500x1000
// (1169) 83.1 / 84.5, 1600x1067 (1246) 84.7 / 87.5, BF16 63.1 / 61.0, 66.6 / 66.7,
// 66.8 / 68.6: the line is at one wavefront per SIMD. (So also where 10 rows are
// asked for: igsp_edge_resolve names the default by that height.)
constexpr int kRound = 6;

inline int marched_rows(const igsp_view* views, int32_t n, int seg, int form, int cus) {
  const int per_cu = form == IGSP_PLAIN && n > 1 ? 4 : 6;
  if (seg == kShortestSeg && stencil_waves(views, n, kRound, form) <= per_cu * (int64_t)cus) return kRound;
  return (seg + kRound - 1) / kRound * kRound;
}

// Slots (one strip's stored row each, 248 pixels) per work-group of the
// normalisation and of the short median chains' median_gather, about 4 Ki pixels
// (measured best for normalisation).
constexpr int kChunkSlots = 16;

inline int64_t view_chunks(const igsp_view& d) {
  const int64_t slots = (int64_t)d.height * ((d.width + kStripCols - 1) / kStripCols);
  return (slots + kChunkSlots - 1) / kChunkSlots;
}

// The launches between the stencil and the normalisation of some views.
enum : int {
  kChainLong = 0,    // median_select, then FP16's refinement pass or FP32's two
  kChainShort = 1,   // median_gather
  kChainGuarded = 2  // FP32: median_gather, then a refinement pass, for views whose bucket holds many values
};

// Which of them the stages of some views take together. The short chain saves
// FP32 two launches of 4 us and FP16 half of that, but every one of its
// work-groups (one per chunk) selects from its view's whole first histogram, and
// FP32 adds every different value of the median's bucket to the view's counts:
// few in photographs, hundreds a chunk where all edges are alike but for the
// sensor's noise. The guarded chain leaves such views' last digit to a refinement
// launch, which otherwise ends at once (2 us). Additions to one address follow one
// another, hence a line on the chunks of the largest view besides that on all.
// us, photographs / 6-pixel stripes with noise, chunks of a view in brackets.
// FP32, short, guarded, long, and the five launches of all sizes before them:
//   1 view (315)  25.4 28.5 35.2 42.2 / 39.4 36.2 36.0 42.9
//   1 (413)       28.1 30.7 38.2 43.6 / 46.4 40.8 39.5 44.8
//   1 (688)       32.8 34.5 42.1 50.9 / 61.0 51.3 45.3 54.8
//   1 (816)       36.1 38.0 44.9 52.4 / 69.5 57.7 49.2 55.2
//   3 (250)       32.5  -   41.6 51.6 / 54.1  -   49.2 59.2
//   3 (315)       35.3  -   44.0 51.8 / 61.4  -   53.3 59.7
//   8 (315)       54.9 56.4 60.3 71.0 / 110  70.8 78.0 81.0
//   10 (315)      67.2 69.1 67.2 80.8 / 134  85.9 86.6 93.5
//   12 (90)       37.5  -   45.9 53.2 / 59.2  -   55.6 61.4
//   24 (90)       48.5 50.4 53.8 68.1 / 88.3 58.3 63.0 78.0
//   40 (65)       56.6 58.3 57.3 75.6 / 97.3 65.0 75.3 84.4
//   64 (24)       42.4 45.0 46.4 70   / 64.9 50.3 54.6 70
// The short chain's lines keep stripes with noise no slower than the five launches
// and the guarded one's also photographs no slower than the long chain.
// FP16, short and long:
//   1 (438)       27.3 27.7 / 27.6 28.7     1 (504)  29.2 29.4 / 29.4 30.2
//   1 (550)       31.8 30.9 / 31.8 31.6     1 (688)  34.0 32.4 / 34.2 33.4
//   4 (315)       35.7 38.0 / 35.5 38.6     5 (315)  44.0 43.2 / 44.3 44.2
//   3 (404)       36.8 37.9 / 36.4 38.4     4 (404)  45.4 43.4 / 45.3 44.2
//   20 (90)       43.5 44.3 / 43.5 44.8     70 (24)  42.5 44.5 / 42.0 45.0
//   95 (24)       44.8 46.6 / 44.9 47.1    120 (24)  52.9 51.1 / 53.4 52.1
constexpr int kFineViews = 64;  // most views of an FP32 launch that counts values: 16 MiB of counts to clear, 3 us

inline int median_chain(int precision, const igsp_view* views, int32_t n) {
  if (precision == IGSP_BF16 || (precision == IGSP_FP32 && n > kFineViews)) return kChainLong;
  const bool fp32 = precision == IGSP_FP32;
  const int64_t each = fp32 ? 470 : 385, most_short = fp32 ? 360 : 510, room = fp32 ? 670000 : 1000000;
  int64_t most = 0, total = 0, cost = 0;
  for (int i = 0; i < n && cost <= 3000000; ++i) {  // (2550 chunks of the largest allowed views cost less)
    const int64_t c = view_chunks(views[i]);
    most = c > most ? c : most;
    total += c;
    cost += c * (each + c);
  }
  if (most <= most_short && cost <= room) return kChainShort;
  return fp32 && most <= 700 && total <= 2550 ? kChainGuarded : kChainLong;
}

}  // namespace igsp
