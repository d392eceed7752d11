"""The mask scan of tg_mask_rois on the CPU: the kernel's text is taken from csrc/rois.hip and
run as 256 lanes whose waves go one after the other between barriers (scan_harness.cpp), in
every order of the four waves. The tile bitmap and the row masks must be those of the mask
whatever the order: nothing a wave writes may depend on another one's having started."""
import itertools
import os
import re
import subprocess

import numpy as np
import pytest

from paper_2404_09267_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))


def _definition(src, head):
    """The definition that starts at the line holding `head`, up to its closing brace."""
    at = src.index(head)
    start = src.rindex("\n", 0, at) + 1
    end = src.index("\n}", at)
    return src[start:end + 2] + (";" if src[end + 2] == ";" else "") + "\n"


@pytest.fixture(scope="module")
def scan(tmp_path_factory):
    clang = os.path.join(os.path.dirname(B.hipcc()), "..", "llvm", "bin", "clang++")
    if not os.path.exists(clang):
        pytest.skip("clang++ not found")
    with open(os.path.join(B.CSRC, "rois.hip")) as f:
        src = f.read()
    parts = [re.search(rf"^constexpr int {n} = .*$", src, re.M).group(0) + "\n"
             for n in ("kTile", "kScanTiles", "kScanThreads")]
    parts += [_definition(src, h) for h in ("struct Tiles {", "uint32_t nonzero_bytes(",
                                            "void scan_kernel(")]
    d = tmp_path_factory.mktemp("scan")
    (d / "scan_extract.inc").write_text("\n".join(parts))
    exe = str(d / "scan")
    subprocess.run([clang, "-std=c++17", "-O1", "-g", "-fsanitize=address", "-I", str(d),
                    os.path.join(HERE, "scan_harness.cpp"), "-o", exe], check=True)

    def run(mask, offset, orders):
        F, H, W = mask.shape
        text = "".join(map(str, mask.reshape(-1).tolist()))
        lines = [f"{o} {F} {W} {H} {offset} {text}" for o in orders]
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True,
                             timeout=120, check=True).stdout
        return [list(map(int, ln.split())) for ln in out.strip().splitlines()]

    return run


def _expected(mask):
    F, H, W = mask.shape
    tx, ty = (W + 31) // 32, (H + 31) // 32
    wpb = (tx + 31) // 32
    full = np.zeros((F, ty * 32, tx * 32), np.uint64)
    full[:, :H, :W] = mask != 0
    rows = (full.reshape(F, ty, 32, tx, 32) << np.arange(32, dtype=np.uint64)).sum(-1)
    rows = rows.transpose(0, 1, 3, 2).reshape(F * ty, tx, 32)  # [band, tile, row]
    bits = np.zeros((F * ty, wpb * 32), np.uint64)
    bits[:, :tx] = rows.any(-1)
    words = (bits.reshape(-1, 32) << np.arange(32, dtype=np.uint64)).sum(-1)
    want = [wpb] + words.tolist()
    for t, r in enumerate(rows.reshape(-1, 32).tolist()):
        if any(r):
            want += [t] + r
    return [int(v) for v in want]


@pytest.mark.parametrize("F,H,W,offset,density", [
    (1, 32, 1024, 0, 0.02),    # one workgroup, whole tiles
    (1, 33, 1025, 0, 0.003),   # a second band of one row, a second word of one column
    (2, 40, 77, 3, 0.01),      # rows and mask at any byte
    (1, 70, 16, 1, 0.05),      # the narrowest row read in 16-byte chunks
    (1, 9, 15, 5, 0.2),        # narrower still: byte by byte
    (1, 64, 1040, 0, 0.0),     # nothing
    (1, 31, 40, 7, 1.0),       # everything
])
def test_scan_in_every_wave_order(scan, F, H, W, offset, density):
    rng = np.random.default_rng(F * 1000 + H + W)
    mask = (rng.random((F, H, W)) < density).astype(np.uint8)
    orders = ["".join(map(str, p)) for p in itertools.permutations(range(4))]
    want = _expected(mask)
    for order, got in zip(orders, scan(mask, offset, orders)):
        assert got == want, order
