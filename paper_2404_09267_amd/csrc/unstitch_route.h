// How one tg_unstitch call runs, by its sizes (host code without HIP, so that the rules can be
// tested on their own).
#ifndef TG_UNSTITCH_ROUTE_H
#define TG_UNSTITCH_ROUTE_H

#include <algorithm>
#include <cstdint>

namespace tg_detail {

// One workgroup, one launch: up to this many boxes, on a plan of up to this many RoIs, which one
// canvas may hold (us, 256 boxes on one canvas, overlap rule, in one launch and in two: 20
// patches 5.1 and 7.8, 64 6.7 and 7.9, 100 9.0 and 8.0, 128 10.0 and 8.0; centre rule 4.4 and
// 7.8, 5.3 and 7.8, 6.7 and 7.8, 7.2 and 8.0).
constexpr int32_t kSmallBoxes = 256, kSmallRois = 96;

// Gathering the plan costs a box about as much as its canvas has patches, but never less than
// eight, once the boxes fill the chip; fewer wait for the latency of the gathers alone. Laying
// the plan out costs a launch and some time per canvas, after which patches hardly count. So the
// line lies lower past kManyBoxes. Gathered and laid out (us, whole calls): canvases of 31
// patches, 10,000 boxes 8.9 and 11.3, 40,000 14.4 and 13.7, 65,000 17.8 and 13.5; 60 of 300, 5,000
// boxes 13.7 and 15.1, 8,000 19.0 and 15.0; eight of 533, 2,000 boxes 11.3 and 17.4, 4,000 13.9
// and 17.0, 8,000 21.3 and 16.8; of 4, 100,000 boxes 11.1 and 12.8, 200,000 16.9 and 16.4;
// 100,000 canvases of 4, 200,000 boxes 39 and 46, 400,000 69 and 57; 500,000 canvases of 2,
// 400,000 boxes 52 and 143, 2,000,000 230 and 225.
constexpr int32_t kManyBoxes = 32768;
constexpr int64_t kLaidOutTests = 1 << 21, kLaidOutTestsMany = 3 << 18;
constexpr int64_t kLaidOutPerCanvas = 24;
constexpr int64_t kLeastTests = 8;

// An emit workgroup counts the kept boxes before its own by itself up to here when the plan was
// gathered (us, canvases of 29 patches: 16,384 boxes 13.0, with counts from the assign 13.0;
// 32,768 20.6 and 13.7; 65,536 34.4 and 20.0), ...
constexpr int32_t kOwnCountBoxes = 16384;
// ... sums the counts of kCountBlock boxes each up to here, and past it finds its sum in the
// scanned counts: what all workgroups sum together grows with the square of the boxes
// (us: 2^20 boxes 52.5, scanned 54.4; 2^21 91.3 and 92.0; 2^22 170 and 164; 2^24 933 and 763;
// 2^25 2,267 and 1,521).
constexpr int32_t kSumBoxes = 1 << 21;
constexpr int32_t kCountBlock = 128;  // boxes per count (a byte of workspace each)

struct UnstitchRoute {
  bool small;     // small_kernel alone
  bool laid_out;  // prep, and the assign over its layout; else the assign gathers the plan
  int lanes;      // per box in the assign
  // Where an emit workgroup finds the kept boxes before its own: in roi_of_box (neither), in
  // the counts (counted), or in the scanned counts (scanned as well).
  bool counted, scanned;
};

// `room`: there is scratch for the layout.
inline UnstitchRoute unstitch_route(int32_t n_boxes, int32_t n_rois, int32_t n_canvases,
                                    bool room) {
  UnstitchRoute r = {};
  const int64_t per_canvas =
      n_canvases > 0 ? (int64_t(n_rois) + n_canvases - 1) / n_canvases : 1;
  r.small = n_boxes <= kSmallBoxes && n_rois <= kSmallRois;
  if (r.small) return r;
  r.laid_out = room && n_rois > 0 && n_canvases > 0 &&
               n_boxes * std::max(per_canvas, kLeastTests) >=
                   (n_boxes > kManyBoxes ? kLaidOutTestsMany : kLaidOutTests) +
                       kLaidOutPerCanvas * n_canvases;
  r.counted = r.laid_out || n_boxes > kOwnCountBoxes;
  r.scanned = r.counted && n_boxes > kSumBoxes;
  // Laid out: a 32-patch word per lane (of 1, 2 and 4 lanes per box on canvases of about 30
  // patches 2 are fastest, of 4 and 8 on canvases of hundreds 8). Gathered: a round is two
  // dependent gathers, so 64 lanes, for one round to settle a box, unless canvases hold at most
  // 16 patches (10,000 boxes on canvases of 32: 11.6 us with 64 lanes, 12.0 with 32, 14.9 with
  // 16); many boxes fill the chip with 8, which can count them too (400,000 boxes on canvases of
  // 30: 113 us with 8 lanes, 161 with 64 and a pass that counts; of 300, 100,000 boxes: 227 and
  // 211).
  if (r.laid_out)
    r.lanes = per_canvas <= 64 ? 2 : 8;
  else if (r.counted && per_canvas <= 64)
    r.lanes = 8;
  else
    r.lanes = per_canvas <= 16 ? 16 : 64;
  return r;
}

}  // namespace tg_detail

#endif  // TG_UNSTITCH_ROUTE_H
