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

}  // namespace igsp
