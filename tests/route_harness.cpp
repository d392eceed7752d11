// CPU driver for the rules by which tg_unstitch picks its passes (csrc/unstitch_route.h), run by
// test_unstitch_route.py: a line "n_boxes n_rois n_canvases room" in, "small laid_out lanes
// counted scanned" out.
#include <cstdio>

#include "unstitch_route.h"

int main() {
  int boxes, rois, canvases, room;
  while (std::scanf("%d %d %d %d", &boxes, &rois, &canvases, &room) == 4) {
    const tg_detail::UnstitchRoute r =
        tg_detail::unstitch_route(boxes, rois, canvases, room != 0);
    std::printf("%d %d %d %d %d\n", r.small, r.laid_out, r.lanes, r.counted, r.scanned);
  }
  return 0;
}
