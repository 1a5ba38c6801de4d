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

// Wavefronts of a stencil launch over the views at a segment height.
inline int64_t stencil_waves(const igsp_view* views, int32_t n, int seg) {
  int64_t waves = 0;
  for (int i = 0; i < n; ++i)
    waves += (int64_t)((views[i].width + kStripCols - 1) / kStripCols) * ((views[i].height + seg - 1) / seg);
  return waves;
}

// Segment height when none is given or tuned: the tallest of a few heights
// that still gives a stencil launch 16 wavefronts per CU (four per SIMD),
// else the shortest. A wavefront's march is a chain of dependent rows, so a
// launch with fewer wavefronts than the chip holds lasts about one segment:
// shorter segments then save more time than their extra halo rows cost. The
// plain form launches each view on its own, so it counts per view.
constexpr int kShortestSeg = 10;

inline int default_seg_rows(const igsp_view* views, int32_t n, int form, int cus) {
  const int heights[] = {64, 40, 28, 22, 16, kShortestSeg};
  const int64_t target = 16 * (int64_t)cus;
  for (int seg : heights) {
    int64_t waves = stencil_waves(views, n, seg);
    if (form == IGSP_PLAIN && n > 0) waves /= n;
    if (waves >= target) return seg;
  }
  return kShortestSeg;
}

// Rows per segment as a plan marches a given, tuned or default height: whole
// rounds of the stencil loop's six rows (the rows past a segment's end would be
// computed all the same; 150 views BF16, 100 rows marched as 102: 864 -> 855 us
// of edge maps). Plans are told apart by this height. A plan
// of the shortest segments whose wavefronts would leave most SIMDs with one
// or none splits them once more, to one round: a lone wavefront takes about
// 0.5 us a row, and shorter segments save more than their window-filling rows
// (2.7 rows' work) and histogram flushes cost. At 10 rows marched as 12 / 6:
// one FP32 256x192 view (64 wavefronts at 6 rows) 22.8 / 19.9 us, 1297x840
// (840) 29.4 / 28.1, 1600x1067 (1246) 34.7 / 34.4, two 1297x840 (1680) 37.4 /
// 37.6: the line is at 1.5 wavefronts per SIMD. (So also where 10 rows are
// asked for: igsp_edge_resolve names the default by that height.)
constexpr int kRound = 6;

inline int marched_rows(const igsp_view* views, int32_t n, int seg, int cus) {
  if (seg == kShortestSeg && stencil_waves(views, n, kRound) <= 6 * (int64_t)cus) return kRound;
  return (seg + kRound - 1) / kRound * kRound;
}

}  // namespace igsp
