"""Which passes tg_unstitch takes by the sizes of a call (csrc/unstitch_route.h), on the CPU."""
import os
import shutil
import subprocess
from collections import namedtuple

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2404_09267_amd", "csrc")
Route = namedtuple("Route", "small laid_out lanes counted scanned")
I32 = 2 ** 31 - 1
OWN = 16384  # most boxes that emit workgroups count by themselves


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not found")
    exe = str(tmp_path_factory.mktemp("route") / "route")
    subprocess.run([gxx, "-std=c++17", "-Wall", "-Werror", "-fsanitize=undefined",
                    "-fno-sanitize-recover=undefined", "-I", CSRC,
                    os.path.join(HERE, "route_harness.cpp"), "-o", exe], check=True)

    def run(boxes, rois, canvases, room=True):
        out = subprocess.run([exe], input=f"{boxes} {rois} {canvases} {int(room)}\n",
                             capture_output=True, text=True, check=True).stdout
        return Route(*map(int, out.split()))

    return run


def test_no_layout_without_room(route):
    """Without scratch for the layout (or without a plan) the plan is gathered as in calls that
    never lay it out: where canvases hold hundreds of patches by 64 lanes per box."""
    for boxes in (10000, 100000, 1 << 24, I32):
        counted = boxes > OWN
        for rois, canvases, lanes in [(150000, 5000, 8 if counted else 64), (150000, 500, 64),
                                      (150000, 150000, 8 if counted else 16)]:
            r = route(boxes, rois, canvases, room=False)
            assert (r.laid_out, r.lanes, r.counted) == (0, lanes, counted)
    assert not route(I32, 0, 5).laid_out
    assert not route(I32, 0, 0).laid_out


def test_layout_pays_for_its_canvases(route):
    """Laying the plan out takes time per canvas, whether boxes meet it or not."""
    assert not route(300000, 1000000, 500000).laid_out
    assert not route(300000, 2000000, 2000000).laid_out
    assert not route(1 << 24, I32, I32).laid_out
    assert route(2000000, 400000, 100000).laid_out
    assert route(200000, 120000, 4000).laid_out


def test_counts_read_again_stay_linear(route):
    """What the emit workgroups (256 boxes each) read to find the kept boxes before their own
    -- 4 bytes per box, or a byte per 128 boxes -- is at most 16 KB each, half of it on average:
    it does not grow with the square of the boxes."""
    boxes = 1
    while boxes <= I32:
        for rois, canvases, room in [(120000, 4000, 1), (150000, 500, 0), (40, 2, 1)]:
            r = route(boxes, rois, canvases, room)
            if r.small or r.scanned:
                continue
            assert (boxes // 128 if r.counted else 4 * boxes) <= 1 << (14 if r.counted else 18)
        boxes = 2 * boxes + 1
    assert route(1 << 24, 120000, 4000).scanned


@pytest.mark.parametrize("boxes,rois,canvases,room,want", [
    (256, 96, 3, 1, Route(1, 0, 0, 0, 0)),
    (257, 96, 3, 1, Route(0, 0, 64, 0, 0)),
    (256, 97, 9, 1, Route(0, 0, 16, 0, 0)),
    (10000, 2000, 63, 1, Route(0, 0, 64, 0, 0)),      # canvases of 31 patches
    (20000, 15500, 500, 1, Route(0, 0, 8, 1, 0)),
    (40000, 15500, 500, 1, Route(0, 1, 2, 1, 0)),
    (5000, 18000, 60, 1, Route(0, 0, 64, 0, 0)),      # of 300
    (8000, 18000, 60, 1, Route(0, 1, 8, 1, 0)),
    (3000, 4264, 8, 1, Route(0, 0, 64, 0, 0)),        # of 533
    (8000, 4264, 8, 1, Route(0, 1, 8, 1, 0)),
    (16384, 8000, 2000, 1, Route(0, 0, 16, 0, 0)),    # of 4
    (16385, 8000, 2000, 1, Route(0, 0, 8, 1, 0)),
    (100000, 8000, 2000, 1, Route(0, 0, 8, 1, 0)),
    (200000, 8000, 2000, 1, Route(0, 1, 2, 1, 0)),
    (300000, 1000000, 500000, 1, Route(0, 0, 8, 1, 0)),
    (2000000, 1000000, 500000, 1, Route(0, 1, 2, 1, 0)),
    (1 << 21, 120000, 4000, 1, Route(0, 1, 2, 1, 0)),
    ((1 << 21) + 1, 120000, 4000, 1, Route(0, 1, 2, 1, 1)),
    ((1 << 21) + 1, 150000, 500, 0, Route(0, 0, 64, 1, 1)),
])
def test_measured_lines(route, boxes, rois, canvases, room, want):
    """The sides on which the measured sizes lie."""
    assert route(boxes, rois, canvases, room) == want
