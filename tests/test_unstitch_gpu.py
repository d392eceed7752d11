"""tg_unstitch on the GPU against the oracle: bit-exact roi_of_box, dets and n_out."""
import numpy as np
import pytest

import oracle
from conftest import load_golden
from gpu_helpers import oracle_plan, say
from paper_2404_09267_amd import tg
from paper_2404_09267_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a visible MI355X"
    tg.lib()
    return torch


def run_unstitch(torch, boxes, box_canvas, rois, plan, clip, dplan=None, rule=0):
    dplan = dplan or tg.DevicePlan(rois, plan)
    n = boxes.shape[0]
    b_d = torch.from_numpy(np.ascontiguousarray(boxes, np.float32).reshape(n, 4)).cuda()
    c_d = torch.from_numpy(np.ascontiguousarray(box_canvas, np.int32)).cuda()
    bufs = tg.UnstitchBuffers(n, dplan.n_rois)
    bufs.roi_of_box.fill_(-7)
    bufs.n_out.fill_(-7)
    tg.unstitch(b_d, c_d, dplan, clip, bufs, rule=rule)
    torch.cuda.synchronize()
    return bufs.roi_of_box.cpu().numpy(), bufs.dets_numpy(), int(bufs.n_out.item())


def check(torch, boxes, box_canvas, rois, plan, clip, dplan=None, rule=0):
    rob, dets, n_out = run_unstitch(torch, boxes, box_canvas, rois, plan, clip, dplan, rule)
    rob_o, dets_o = oracle.unstitch(boxes, box_canvas, rois, oracle_plan(plan), clip, rule)
    np.testing.assert_array_equal(rob, rob_o)
    assert n_out == len(dets_o)
    # compare bit patterns (NaN-free by construction: kept boxes have finite sums)
    np.testing.assert_array_equal(dets.view(np.int32).reshape(-1, 7),
                                  dets_o.view(np.int32).reshape(-1, 7))
    return rob, dets


def test_golden_example(torch):
    g = load_golden("unstitch_example.json")
    ex = load_golden("pack_examples.json")["examples"][0]
    cw, ch = ex["canvas"]
    fw, fh, nf = ex["frame"]
    rois = np.array(ex["rois"])
    plan = tg.plan_pack(rois, cw, ch, fw, fh, nf, tg.GUILLOTINE_BSSF)
    boxes = np.array(g["boxes"], dtype=np.float32)
    boxes[g["box_nan_index"], 0] = np.nan
    for clip, key in ((1, "dets_clip"), (0, "dets_noclip")):
        say("golden clip", clip)
        rob, dets, n_out = run_unstitch(torch, boxes, np.array(g["box_canvas"]), rois, plan, clip)
        assert rob.tolist() == g["roi_of_box"]
        assert n_out == len(g[key])
        got = [tuple(d) for d in dets.tolist()]
        assert got == [tuple(r[:3]) + tuple(np.float32(v) for v in r[3:]) for r in g[key]]


@pytest.mark.parametrize("per_canvas", [4, 24, 60, 300])
def test_random_plans(torch, per_canvas):
    """Patches per canvas around 16, 32 and 64+ select the three lane widths."""
    rng = np.random.default_rng(per_canvas)
    side = int(np.sqrt(200 * 200 / per_canvas))
    for policy in (0, 1, 2):
        rois = W.random_rois(rng, 30 * per_canvas, 4, 800, 600, max(1, side // 2), side, side)
        plan = tg.plan_pack(rois, 200, 200, 800, 600, 4, policy)
        n = 20000
        cx, cy = rng.uniform(-8, 208, n), rng.uniform(-8, 208, n)
        bw, bh = rng.uniform(0, 60, n), rng.uniform(0, 60, n)
        boxes = np.stack([cx - bw / 2, cy - bh / 2, cx + bw / 2, cy + bh / 2], 1).astype(np.float32)
        boxes[:3000] = np.round(boxes[:3000])          # centres on patch edges
        boxes[3000:3100, 0] = np.nan
        boxes[3100:3200, 3] = np.inf
        canv = rng.integers(-2, plan.n_canvases + 2, n).astype(np.int32)
        boxes[3200:3400] = np.round(boxes[3200:3400])  # integer corners: overlap ties
        for clip, rule in ((0, 0), (1, 0), (1, 1), (0, 1)):
            say("random", per_canvas, "policy", policy, "clip", clip, "rule", rule)
            check(torch, boxes, canv, rois, plan, clip, rule=rule)


@pytest.mark.parametrize("name", W.ORDERED)
def test_workload_boxes(torch, name):
    wl = W.WORKLOADS[name]
    say("workload", name)
    rois = W.make_rois(wl)
    plan = tg.plan_pack(rois, wl.canvas, wl.canvas, wl.frame_w, wl.frame_h, wl.n_frames, 0)
    boxes, canv = W.make_boxes(wl, plan.n_canvases)
    rob, dets = check(torch, boxes, canv, rois, plan, 1)
    assert (rob >= 0).sum() > 0.1 * len(rob)  # sanity: boxes do land on patches


def test_own_box_identity(torch):
    """Stitch then unstitch of each patch's own placed rect gives back its source rect."""
    wl = W.WORKLOADS["cam20_4k"]
    rois = W.make_rois(wl)
    plan = tg.plan_pack(rois, wl.canvas, wl.canvas, wl.frame_w, wl.frame_h, wl.n_frames, 0)
    pl = plan.place
    boxes = np.stack([pl[:, 1], pl[:, 2], pl[:, 1] + rois[:, 3], pl[:, 2] + rois[:, 4]],
                     1).astype(np.float32)
    say("identity")
    rob, dets, n_out = run_unstitch(torch, boxes, pl[:, 0], rois, plan, 1)
    assert rob.tolist() == list(range(len(rois))) and n_out == len(rois)
    got = np.stack([dets["x1"], dets["y1"], dets["x2"], dets["y2"]], 1)
    want = np.stack([rois[:, 1], rois[:, 2], rois[:, 1] + rois[:, 3], rois[:, 2] + rois[:, 4]], 1)
    np.testing.assert_array_equal(got, want.astype(np.float32))
    assert dets["frame"].tolist() == rois[:, 0].tolist()


def test_zero_boxes_and_no_canvases(torch):
    rois = np.array([[0, 0, 0, 4, 4]])
    plan = tg.plan_pack(rois, 8, 8, 8, 8, 1, 0)
    say("zero boxes")
    bufs = tg.UnstitchBuffers(0, 1)
    bufs.n_out.fill_(-5)
    dplan = tg.DevicePlan(rois, plan)
    tg.unstitch(torch.empty((0, 4), dtype=torch.float32, device="cuda"),
                torch.empty(0, dtype=torch.int32, device="cuda"), dplan, 1, bufs)
    torch.cuda.synchronize()
    assert bufs.n_out.item() == 0
    say("empty plan")
    empty = tg.plan_pack(np.zeros((0, 5)), 8, 8, 8, 8, 1, 0)
    boxes = np.array([[0, 0, 1, 1]], np.float32)
    rob, dets, n_out = run_unstitch(torch, boxes, np.array([0]), np.zeros((0, 5)), empty, 1)
    assert rob.tolist() == [-1] and n_out == 0


def test_deterministic(torch):
    wl = W.WORKLOADS["window_64x30"]
    rois = W.make_rois(wl)
    plan = tg.plan_pack(rois, wl.canvas, wl.canvas, wl.frame_w, wl.frame_h, wl.n_frames, 0)
    boxes, canv = W.make_boxes(wl, plan.n_canvases)
    dplan = tg.DevicePlan(rois, plan)
    say("determinism")
    a = run_unstitch(torch, boxes, canv, rois, plan, 1, dplan)
    b = run_unstitch(torch, boxes, canv, rois, plan, 1, dplan)
    np.testing.assert_array_equal(a[0], b[0])
    np.testing.assert_array_equal(a[1], b[1])


def test_overlap_rule_example(torch):
    """The hand-worked overlap example of the oracle tests, through the C ABI."""
    rois = np.array([[0, 100, 50, 10, 10], [1, 200, 0, 10, 10], [0, 0, 0, 10, 10]], np.int32)
    plan = tg.Plan(np.array([[0, 0, 0], [0, 10, 0], [0, 0, 10]], np.int32),
                   np.array([0, 1, 2], np.int32), np.array([0, 3], np.int32), 1)
    boxes = np.array([[4, 2, 16, 8], [8, 0, 13, 5], [-5, -5, 2, 2], [30, 30, 40, 40],
                      [np.nan, 0, 5, 5], [2, 8, 8, 14]], np.float32)
    rob, dets, n_out = run_unstitch(torch, boxes, np.zeros(6, np.int32), rois, plan, 1, rule=1)
    assert rob.tolist() == [0, 1, 0, -1, -1, 2]
    assert tuple(dets[0])[:3] == (0, 0, 0) and tuple(dets[0])[3:] == (104, 52, 110, 58)


@pytest.mark.parametrize("name", ["cam5_4k", "cam20_4k", "small_roi_8cam"])
def test_workload_boxes_overlap_rule(torch, name):
    wl = W.WORKLOADS[name]
    rois = W.make_rois(wl)
    plan = tg.plan_pack(rois, wl.canvas, wl.canvas, wl.frame_w, wl.frame_h, wl.n_frames, 0)
    boxes, canv = W.make_boxes(wl, plan.n_canvases)
    say("workload overlap rule", name)
    check(torch, boxes, canv, rois, plan, 1, rule=1)


def test_patch_records_switch(torch):
    """The calls on either side of the switch to a laid out plan (more than 32,768 boxes:
    786,432 box-patch tests, n_boxes times the mean patches per canvas, and 24 for each
    canvas), and a larger one, agree with the oracle and with each other on their common boxes:
    gathering and the layout give one result."""
    rng = np.random.default_rng(91)
    rois = W.random_rois(rng, 900, 4, 800, 600, 24, 60, 60)
    plan = tg.plan_pack(rois, 200, 200, 800, 600, 4, tg.SHELF_FFDH)
    per_canvas = -(-len(rois) // plan.n_canvases)
    n_switch = -(-((3 << 18) + 24 * plan.n_canvases) // per_canvas)
    assert n_switch > 32768
    n = -(-(1 << 21) // per_canvas) + 100
    cx, cy = rng.uniform(-4, 204, n), rng.uniform(-4, 204, n)
    bw, bh = rng.uniform(0, 20, n), rng.uniform(0, 20, n)
    boxes = np.stack([cx - bw / 2, cy - bh / 2, cx + bw / 2, cy + bh / 2], 1).astype(np.float32)
    boxes[:500] = np.round(boxes[:500])
    canv = rng.integers(-1, plan.n_canvases + 1, n).astype(np.int32)
    dplan = tg.DevicePlan(rois, plan)
    for rule in (0, 1):
        say("layout switch", per_canvas, n_switch, "rule", rule)
        lo = check(torch, boxes[:n_switch - 1], canv[:n_switch - 1], rois, plan, 1, dplan, rule)
        at = check(torch, boxes[:n_switch], canv[:n_switch], rois, plan, 1, dplan, rule)
        hi = check(torch, boxes, canv, rois, plan, 1, dplan, rule)
        np.testing.assert_array_equal(lo[0], hi[0][:n_switch - 1])
        np.testing.assert_array_equal(at[0], hi[0][:n_switch])


@pytest.mark.parametrize("rule", [0, 1])
def test_layout_switch_of_few_boxes(torch, rule):
    """The same with at most 32,768 boxes, where the switch is at 2^21 tests."""
    rng = np.random.default_rng(93)
    rois = W.random_rois(rng, 9000, 4, 800, 600, 5, 11, 11)
    plan = tg.plan_pack(rois, 200, 200, 800, 600, 4, tg.SHELF_FFDH)
    n = -(-((1 << 21) + 24 * plan.n_canvases) // -(-len(rois) // plan.n_canvases))
    assert n <= 32768
    c, s = rng.uniform(-4, 204, (n, 2)), rng.uniform(0, 20, (n, 2))
    boxes = np.concatenate([c - s / 2, c + s / 2], 1).astype(np.float32)
    canv = rng.integers(-1, plan.n_canvases + 1, n).astype(np.int32)
    dplan = tg.DevicePlan(rois, plan)
    say("layout switch, few boxes", n, rule)
    lo = check(torch, boxes[:n - 1], canv[:n - 1], rois, plan, 1, dplan, rule)
    at = check(torch, boxes, canv, rois, plan, 1, dplan, rule)
    np.testing.assert_array_equal(lo[0], at[0][:n - 1])


@pytest.mark.parametrize("rule", [0, 1])
def test_patch_records_with_small_canvases(torch, rule):
    """The layout of canvases of about 24 patches (one word of band bits each): 120,000
    boxes, centres on edges, NaN and infinite corners, bad canvases."""
    rng = np.random.default_rng(95 + rule)
    rois = W.random_rois(rng, 720, 4, 800, 600, 28, 48, 48)
    plan = tg.plan_pack(rois, 200, 200, 800, 600, 4, tg.SHELF_FFDH)
    n = 120_000
    cx, cy = rng.uniform(-8, 208, n), rng.uniform(-8, 208, n)
    bw, bh = rng.uniform(0, 60, n), rng.uniform(0, 60, n)
    boxes = np.stack([cx - bw / 2, cy - bh / 2, cx + bw / 2, cy + bh / 2], 1).astype(np.float32)
    boxes[:20000] = np.round(boxes[:20000])
    boxes[20000:20500, 1] = np.nan
    boxes[20500:21000, 2] = np.inf
    canv = rng.integers(-2, plan.n_canvases + 2, n).astype(np.int32)
    per_canvas = -(-len(rois) // plan.n_canvases)
    assert per_canvas <= 32 and n * per_canvas >= 1 << 21
    for clip in (0, 1):
        say("records, small canvases", per_canvas, "rule", rule, "clip", clip)
        check(torch, boxes, canv, rois, plan, clip, rule=rule)


def _grid_plan(sizes, cell, cw):
    """A plan of one canvas per entry of `sizes`, that many cell x cell patches in rows."""
    per = cw // cell
    place, rois, begin = [], [], [0]
    for c, n in enumerate(sizes):
        for j in range(n):
            place.append((c, cell * (j % per), cell * (j // per)))
            rois.append((0, (7 * len(rois)) % 300, (3 * len(rois)) % 200, cell, cell))
        begin.append(len(rois))
    order = np.arange(len(rois), dtype=np.int32)
    return (np.array(rois, np.int32),
            tg.Plan(np.array(place, np.int32), order, np.array(begin, np.int32), len(sizes)))


@pytest.mark.parametrize("sizes", [[16, 17, 32, 33, 64, 65, 0, 1], [300, 257, 256, 129],
                                   [1000, 5, 96, 97], [15, 16, 17, 18]])
@pytest.mark.parametrize("rule", [0, 1])
def test_band_layout_sizes(torch, sizes, rule):
    """Canvases around the smallest count with band words and around whole 32-patch words,
    in calls of both lanes-per-box widths over the layout and on either side of the most boxes
    that a gathering call counts in its emit (16,384); boxes on patch edges,
    with NaN and infinite corners and inverted, whole-canvas boxes, bad canvases."""
    rois, plan = _grid_plan(sizes, 9, 300)
    rng = np.random.default_rng(len(rois))
    most = -(-(1 << 21) * len(sizes) // len(rois)) + 7  # enough boxes for the laid out path
    for n in (min(most, 140000), 16384, 16385):
        c, s = rng.uniform(-5, 305, (n, 2)), rng.uniform(0, 30, (n, 2))
        boxes = np.concatenate([c - s / 2, c + s / 2], 1).astype(np.float32)
        boxes[:4000] = np.round(boxes[:4000])
        boxes[4000:4050, 0] = np.nan
        boxes[4050:4100, 2] = np.inf
        boxes[4100:4150, 1] = -np.inf
        boxes[4150:4200] = boxes[4150:4200][:, [2, 3, 0, 1]]
        boxes[4200:4250] = [-10, -10, 400, 400]
        canv = rng.integers(-1, plan.n_canvases + 1, n).astype(np.int32)
        say("bands", sizes, rule, n)
        check(torch, boxes, canv, rois, plan, 1, rule=rule)


def test_laid_out_path_with_corrupt_plans(torch):
    """Positions holding no RoI, RoIs placed on another canvas, and canvas_begin that does not
    cut the plan into consecutive segments: the same boxes in calls that lay the plan out
    and in calls that gather it."""
    rois, plan = _grid_plan([100, 200, 300, 40], 9, 300)
    rng = np.random.default_rng(3)
    n = 20000
    c = rng.uniform(-5, 305, (n, 2))
    boxes = np.concatenate([c - 6, c + 6], 1).astype(np.float32)
    canv = rng.integers(0, 4, n).astype(np.int32)
    for what in ("ids", "begin"):
        place, order, begin = plan.place.copy(), plan.order.copy(), plan.canvas_begin.copy()
        if what == "ids":
            order[::7], order[3::31] = 100000, -4
            place[5::11, 0] = 3
        else:
            begin[:] = [50, 310, 250, 700, 600]  # overlapping, empty, past the end
        dplan = tg.DevicePlan(rois, tg.Plan(place, order, begin, 4))
        for rule in (0, 1):
            say("corrupt", what, rule)
            whole = run_unstitch(torch, boxes, canv, rois, plan, 1, dplan, rule)
            parts = [run_unstitch(torch, boxes[k:k + 2500], canv[k:k + 2500], rois, plan, 1, dplan,
                                  rule)[0] for k in range(0, n, 2500)]
            assert (whole[0] >= 0).any()
            np.testing.assert_array_equal(whole[0], np.concatenate(parts))
            assert whole[2] == (whole[0] >= 0).sum()
            np.testing.assert_array_equal(whole[1]["box"], np.flatnonzero(whole[0] >= 0))


@pytest.mark.parametrize("n", [1, 63, 64, 255, 256, 257])
def test_few_boxes(torch, n):
    """The one-workgroup path and the first size past it, by boxes and by RoIs."""
    rng = np.random.default_rng(n)
    for n_rois in (1, 96, 97, 128, 129):
        rois = W.random_rois(rng, n_rois, 2, 400, 300, 4, 60, 60)
        plan = tg.plan_pack(rois, 160, 160, 400, 300, 2, 0)
        c, s = rng.uniform(0, 160, (n, 2)), rng.uniform(0, 40, (n, 2))
        boxes = np.concatenate([c - s / 2, c + s / 2], 1).astype(np.float32)
        canv = rng.integers(-1, plan.n_canvases + 1, n).astype(np.int32)
        for rule in (0, 1):
            say("few", n, n_rois, rule)
            check(torch, boxes, canv, rois, plan, 1, rule=rule)


@pytest.mark.parametrize("n", [16384, 16385, 40000, 120000])
@pytest.mark.parametrize("rule", [0, 1])
def test_uneven_canvases(torch, n, rule):
    """Canvases of 257, 700 and 2,000 patches among thousands of one to four: the boxes of long
    ones are assigned by whole waves where the others take few lanes, and every path agrees."""
    sizes = [3, 2000, 1, 257, 256, 0, 700] + [1, 4, 2] * 1000
    rois, plan = _grid_plan(sizes, 6, 300)
    rng = np.random.default_rng(n + rule)
    c, s = rng.uniform(-5, 305, (n, 2)), rng.uniform(0, 12, (n, 2))
    boxes = np.concatenate([c - s / 2, c + s / 2], 1).astype(np.float32)
    canv = rng.integers(-1, len(sizes) + 1, n).astype(np.int32)
    canv[:n // 4] = rng.integers(0, 8, n // 4)
    boxes[:50, 0] = np.nan
    perm = rng.permutation(n)
    say("uneven canvases", n, rule)
    check(torch, boxes[perm], canv[perm], rois, plan, 1, rule=rule)


@pytest.mark.parametrize("at", [1, 2047, 2048, 9000, 16383, 16384, 19999, 20000])
def test_broken_begin_among_many_canvases(torch, at):
    """One entry of canvas_begin out of order among 20,001: found wherever it is, so that calls
    that lay the plan out give what calls that gather it give."""
    C = 20000
    rois, plan = _grid_plan([20] * C, 9, 60)
    begin = plan.canvas_begin.copy()
    begin[at] += 30 if at < C else -len(rois)
    dplan = tg.DevicePlan(rois, tg.Plan(plan.place, plan.order, begin, C))
    rng = np.random.default_rng(at)
    n = 150000
    c = rng.uniform(-5, 65, (n, 2))
    boxes = np.concatenate([c - 6, c + 6], 1).astype(np.float32)
    canv = rng.integers(0, C, n).astype(np.int32)
    canv[:2000] = rng.integers(at - 3, at + 3, 2000)  # canvases beside the broken entry
    for rule in (0, 1):
        say("broken begin", at, rule)
        whole = run_unstitch(torch, boxes, canv, rois, plan, 1, dplan, rule)
        parts = [run_unstitch(torch, boxes[k:k + 10000], canv[k:k + 10000], rois, plan, 1, dplan,
                              rule)[0] for k in range(0, n, 10000)]
        assert (whole[0] >= 0).any()
        np.testing.assert_array_equal(whole[0], np.concatenate(parts))


@pytest.mark.parametrize("n", [1 << 21, (1 << 21) + 1, (1 << 21) + 1279, (1 << 22) + 4096 * 1024 + 77])
def test_scanned_counts(torch, n):
    """Calls on both sides of the scan of the counts, with a last word that is not full and
    more words than one step of the scan takes."""
    rois, plan = _grid_plan([25, 30, 0, 31], 9, 60)
    rng = np.random.default_rng(n)
    c = rng.uniform(-5, 65, (n, 2)).astype(np.float32)
    boxes = np.concatenate([c - 6, c + 6], 1)
    canv = rng.integers(-1, 5, n).astype(np.int32)
    canv[5000:9000] = -1  # whole counts of nothing, and of everything
    c[9000:13000] = 15
    boxes[9000:13000] = [10, 10, 20, 20]
    canv[9000:13000] = 1
    say("scanned counts", n)
    check(torch, boxes, canv, rois, plan, 1)


@pytest.mark.parametrize("n", [1, 64, 256])
@pytest.mark.parametrize("rule", [0, 1])
def test_few_boxes_corrupt_plans(torch, n, rule):
    """The one-workgroup path on plans with positions that hold no RoI, RoIs placed on another
    canvas and segments that overlap or leave the plan: as the passes that gather (the same
    boxes among 300)."""
    rois, plan = _grid_plan([30, 1, 40, 0, 20], 9, 90)
    rng = np.random.default_rng(n)
    c, s = rng.uniform(-5, 95, (300, 2)), rng.uniform(0, 25, (300, 2))
    boxes = np.concatenate([c - s / 2, c + s / 2], 1).astype(np.float32)
    boxes[::37, 1] = np.nan
    canv = rng.integers(-1, 6, 300).astype(np.int32)
    for what in ("ids", "begin"):
        place, order, begin = plan.place.copy(), plan.order.copy(), plan.canvas_begin.copy()
        if what == "ids":
            order[::7], order[3::31] = 100000, -4
            place[5::11, 0] = 2
            place[6::13, 0] = -1
        else:
            begin[:] = [20, 95, 10, 70, 60, 88]
        dplan = tg.DevicePlan(rois, tg.Plan(place, order, begin, 5))
        say("few boxes, corrupt", what, n, rule)
        few = run_unstitch(torch, boxes[:n], canv[:n], rois, plan, 1, dplan, rule)
        all_ = run_unstitch(torch, boxes, canv, rois, plan, 1, dplan, rule)
        np.testing.assert_array_equal(few[0], all_[0][:n])
        assert few[2] == (few[0] >= 0).sum()
        np.testing.assert_array_equal(few[1].view(np.int32), all_[1][:few[2]].view(np.int32))


@pytest.mark.parametrize("rule", [0, 1])
def test_few_boxes_cost(torch, rule):
    """256 boxes on one canvas of 96 patches, one launch, cost no more than 1.75 times 300 boxes,
    two launches (0.8 to 1.5 times by rule and by how closely launches follow each other; 2.0 to
    2.8 when the one launch gathered the plan for every box)."""
    rois, plan = _grid_plan([96], 9, 90)
    dplan = tg.DevicePlan(rois, plan)
    rng = np.random.default_rng(5)
    c = rng.uniform(0, 90, (300, 2))
    boxes = torch.from_numpy(np.concatenate([c - 9, c + 9], 1).astype(np.float32)).cuda()
    canv = torch.zeros(300, dtype=torch.int32, device="cuda")

    def us(n):
        bufs = tg.UnstitchBuffers(n, dplan.n_rois)
        args = tg.unstitch_args(boxes[:n], canv[:n], dplan, 1, bufs, rule)
        best = float("inf")
        for _ in range(20):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            torch.cuda.synchronize()
            e0.record()
            for _ in range(50):
                tg.unstitch_raw(args)
            e1.record()
            torch.cuda.synchronize()
            best = min(best, 20 * e0.elapsed_time(e1))
        return best

    one, two = us(256), us(300)
    say("few boxes", one, two)
    assert one <= 1.75 * two
