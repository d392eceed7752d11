"""Timed cases of the patch-stitching path, through the C ABI of libtg.so.

A serving program holds its frames, RoI tables, detector boxes and argument blocks on the
device (as bench.py does) and calls the library once per batch of work; `prepare` makes
what such a program has in hand and `run` makes the calls. The listed cases are the
workloads of paper_2404_09267_amd/workload.py and bench.py, call by call and as whole
serving steps, plus odd frame and canvas sizes; `draw` spreads over the same calls with
camera counts, frame, RoI, canvas, box, zone and model sizes between the smallest and the
largest of them. The host-only calls (the planner inside the steps, the invoker replay of
Alg. 2) need no case of their own: the steps time the planner, and the invoker costs
0.02 us per arrival.

Kinds (`case["kind"]`):
  step       tg_plan_pack -> tg_plan_upload -> tg_stitch per batch -> tg_unstitch -> tg_merge
  stitch     tg_stitch of every batch of a plan
  unstitch   tg_unstitch of a detector's boxes
  merge      tg_merge of tg_unstitch's output
  partition  tg_partition of background-model RoIs
  gmm        tg_gmm_update of one frame per camera into a settled (or fresh) model
  mask       tg_mask_rois of a foreground mask, then tg_partition of its RoIs
"""
from __future__ import annotations

import ctypes
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2404_09267_amd import tg
from paper_2404_09267_amd import workload as W

# Normalisations a detector asks for: ImageNet statistics, plain scaling to [0, 1], mean
# subtraction with one scale; and statistics whose values tg_stitch takes from its byte
# table (no exact fp32 constants exist for them).
NORMS = {
    "imagenet": (W.MEAN, W.STD, W.PAD),
    "unit": ((0.0, 0.0, 0.0), (255.0, 255.0, 255.0), W.PAD),
    "mean": ((103.94, 116.78, 123.68), (58.824, 58.824, 58.824), (0, 114, 255)),
    "table": ((174.00369262695312, 189.9988250732422, 150.99696350097656),
              (0.031708136200904846, 1.5641870498657227, 1.5637657642364502), (3, 200, 90)),
}
GMM_T_BG, GMM_T_OWN, GMM_V_INIT, GMM_V_MIN, GMM_V_MAX = 16.0, 9.0, 15.0, 4.0, 75.0
GMM_RATIO, GMM_CT, GMM_ALPHA = 0.9, 0.05, 0.002
LIVE_FRAMES = 4  # frames a gmm case cycles through


# ------------------------------------------------------------------------------ the cases

def _plan_case(kind, wl, **more):
    """A case with a workload's plan: frames, RoIs, canvases and boxes."""
    w = W.WORKLOADS[wl]
    c = dict(kind=kind, frames=w.n_frames, frame_w=w.frame_w, frame_h=w.frame_h, rois=w.n_rois,
             dist=w.roi_dist, roi_lo=w.roi_lo, roi_hi=w.roi_hi, canvas_w=w.canvas,
             canvas_h=w.canvas, cap=w.batch_cap, policy=tg.SHELF_FFDH, norm="imagenet",
             boxes=w.n_boxes, box_lo=w.box_lo, box_hi=w.box_hi, rule=0, clip=True, iou=0.5,
             cross_only=True)
    c.update(more)
    return c


def listed():
    return [
        # one 1080p camera, one canvas: what a single small request costs, launches and all
        dict(_plan_case("step", "cam1_1080p"), name="step_cam1_1080p"),
        # the headline workload: 20 cameras at 4K, two batches, 10,000 boxes, end to end
        dict(_plan_case("step", "cam20_4k"), name="step_cam20_4k"),
        # five cameras at 4K: an ordinary batch of nine canvases in one launch
        dict(_plan_case("stitch", "cam5_4k"), name="stitch_cam5_4k"),
        # 16,000 crops of 8-64 pixels: short source rows, hundreds of patches per canvas
        dict(_plan_case("stitch", "small_roi_8cam"), name="stitch_small_roi_8cam"),
        # cropped streams and a detector input of odd sides: nothing is aligned
        dict(_plan_case("stitch", "cam5_4k", frames=6, frame_w=2047, frame_h=1151, rois=400,
                        roi_lo=24, roi_hi=400, canvas_w=999, canvas_h=667, norm="mean"),
             name="stitch_odd_sizes"),
        # 50,000 boxes on canvases of 300 patches, the largest-overlap rule
        dict(_plan_case("unstitch", "small_roi_8cam", rule=1), name="unstitch_overlap_small_roi"),
        # a window of 64 cameras x 30 frames: 200,000 boxes over 4,010 canvases
        dict(_plan_case("unstitch", "window_64x30"), name="unstitch_window_64x30"),
        # few frames with thousands of detections each
        dict(_plan_case("merge", "small_roi_8cam"), name="merge_small_roi_8cam"),
        # many frames with about a hundred detections each
        dict(_plan_case("merge", "window_64x30"), name="merge_window_64x30"),
        # Alg. 1 over the window's 1,920 frames, 4 x 4 zones
        dict(kind="partition", frames=1920, frame_w=3840, frame_h=2160, per_frame=30, zones_x=4,
             zones_y=4, name="partition_window_64x30"),
        # one frame from each of 20 cameras into five-component models
        dict(kind="gmm", frames=20, frame_w=3840, frame_h=2160, n_mix=5, busy=0.08, fresh=False,
             name="gmm_cam20_4k"),
        # that model's mask: 40 moving objects per camera and a little sensor speckle
        dict(kind="mask", frames=20, frame_w=3840, frame_h=2160, objects=40, obj_lo=16,
             obj_hi=256, speckle=1e-5, min_area=16, zones_x=4, zones_y=4,
             name="mask_rois_cam20_4k"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _frame_size(rng):
    """Common camera sizes, or any size between 640x360 and 3840x2160, odd ones among them."""
    if rng.random() < 0.5:
        return rng.choice([(1280, 720), (1920, 1080), (2560, 1440), (3840, 2160)])
    return _log_int(rng, 640, 3840), _log_int(rng, 360, 2160)


def draw(rng):
    kind = rng.choice(["step", "stitch", "stitch", "unstitch", "merge", "partition", "gmm",
                       "mask"])
    fw, fh = _frame_size(rng)
    if kind == "partition":
        return dict(kind=kind, frames=_log_int(rng, 1, 1920), frame_w=fw, frame_h=fh,
                    per_frame=_log_int(rng, 2, 60), zones_x=rng.choice([2, 4, 6, 7, 16]),
                    zones_y=rng.choice([2, 4, 6, 9, 16]))
    if kind == "gmm":
        return dict(kind=kind, frames=_log_int(rng, 1, 16), frame_w=fw, frame_h=fh,
                    n_mix=rng.choice([1, 2, 3, 4, 5, 5, 5]), busy=round(rng.uniform(0.0, 0.25), 3),
                    fresh=rng.random() < 0.15)
    if kind == "mask":
        hi = _log_int(rng, 32, min(fw, fh, 400))
        return dict(kind=kind, frames=_log_int(rng, 1, 20), frame_w=fw, frame_h=fh,
                    objects=_log_int(rng, 2, 80), obj_lo=rng.randint(4, 16), obj_hi=hi,
                    speckle=rng.choice([0.0, 1e-6, 1e-5, 1e-4]), min_area=rng.choice([1, 16, 64]),
                    zones_x=rng.choice([2, 4, 6]), zones_y=rng.choice([2, 4, 6]))
    frames = _log_int(rng, 1, 20)
    canvas = rng.choice([320, 512, 640, 1024, 1280])
    cw, ch = canvas, canvas
    if rng.random() < 0.4:  # a detector input that is not square, of any size
        cw, ch = rng.randint(300, 1300), rng.randint(300, 1300)
    lo = _log_int(rng, 8, 40)
    hi = _log_int(rng, 48, min(640, cw, ch, fw, fh))
    dist = rng.choice(["uniform", "loguniform"])
    # RoIs: up to 2,000 per frame where they are small, fewer where they are large, and at
    # most about 90 million pixels in all
    mean_side = (lo + hi) / 2 if dist == "uniform" else (hi - lo) / math.log(hi / lo)
    most = max(8, min(16000, int(9e7 / mean_side ** 2)))
    if kind in ("unstitch", "merge"):  # no pixels: only the plan
        frames = _log_int(rng, 1, 1920)
        most = max(8, min(100000, 60 * frames + 2000, int(2e9 / mean_side ** 2)))
    rois = _log_int(rng, 8, most)
    boxes = _log_int(rng, 50, min(200000, 12 * rois + 200))
    policy = rng.choice([tg.SHELF_FFDH, tg.SHELF_FFDH, tg.SHELF_ARRIVAL, tg.GUILLOTINE_BSSF])
    if rois > 4000:
        policy = tg.SHELF_FFDH
    return dict(kind=kind, frames=frames, frame_w=fw, frame_h=fh, rois=rois, dist=dist, roi_lo=lo,
                roi_hi=hi, canvas_w=cw, canvas_h=ch, cap=rng.choice([0, 8, 32, 64]),
                policy=policy, norm=rng.choice(["imagenet"] * 4 + ["unit", "unit", "mean", "table"]),
                boxes=boxes, box_lo=4.0, box_hi=float(max(12, min(256, hi))),
                rule=rng.choice([0, 0, 1]), clip=rng.random() < 0.8,
                iou=rng.choice([0.3, 0.5, 0.7]), cross_only=rng.random() < 0.7)


# ------------------------------------------------------------------------------ the inputs

def _rois(case, rng):
    """int32 [n, 5], arrival order: the frames in turn, an even share of the RoIs each."""
    n, lo, hi = case["rois"], case["roi_lo"], case["roi_hi"]
    if case["dist"] == "uniform":
        w, h = rng.integers(lo, hi + 1, n), rng.integers(lo, hi + 1, n)
    else:
        w = np.rint(np.exp(rng.uniform(np.log(lo), np.log(hi), 4 * n))).astype(np.int64)
        h = np.rint(np.exp(rng.uniform(np.log(lo), np.log(hi), 4 * n))).astype(np.int64)
        if case["dist"] == "loguniform_aspect":
            ok = np.flatnonzero((h <= 2 * w) & (w <= 2 * h))
            ok = np.resize(ok, n)
        else:
            ok = np.arange(n)
        w, h = w[ok], h[ok]
    x = rng.integers(0, case["frame_w"] - w + 1)
    y = rng.integers(0, case["frame_h"] - h + 1)
    f = np.arange(n) * case["frames"] // n
    return np.stack([f, x, y, w, h], 1).astype(np.int32)


def _canvas_cap(case):
    """Canvases a program sizes its output for: what a plan of such RoIs takes, and some."""
    rois = _rois(case, np.random.default_rng(0))
    J = int(_pack(rois, case["canvas_w"], case["canvas_h"], case["policy"])[0][:, 0].max()) + 1
    return J + 4 + J // 4


def _boxes(case, rng, n_canvases):
    n = case["boxes"]
    bw, bh = (rng.uniform(case["box_lo"], case["box_hi"], n) for _ in range(2))
    cx, cy = rng.uniform(0, case["canvas_w"], n), rng.uniform(0, case["canvas_h"], n)
    b = np.stack([cx - bw / 2, cy - bh / 2, cx + bw / 2, cy + bh / 2], 1).astype(np.float32)
    return b, rng.integers(0, n_canvases, n).astype(np.int32)


def _pixels(shape, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randint(0, 256, shape, dtype=torch.uint8, device="cuda", generator=g)


def _plan(case, rois):
    return tg.plan_pack(rois, case["canvas_w"], case["canvas_h"], case["frame_w"],
                        case["frame_h"], case["frames"], case["policy"])


def _zeroed(bufs):
    """Output buffers start zeroed, so that what a call leaves unwritten is the same twice."""
    for v in vars(bufs).values():
        if isinstance(v, torch.Tensor):
            v.zero_()
    return bufs


def _call(name, args, stream=None):
    h = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream if stream is None else stream)
    rc = getattr(tg.lib(), name)(ctypes.byref(args), h)
    if rc != tg.OK:
        raise tg.TgError(name, rc)


def _prepare_plan_case(case, seed):
    """step, stitch, unstitch and merge: a plan and what its calls read and write."""
    kind, rng = case["kind"], np.random.default_rng([seed, 1])
    s = SimpleNamespace(kind=kind, turn=0)
    rois = _rois(case, rng)
    plan = _plan(case, rois)
    n, J = len(rois), plan.n_canvases
    mean, std, pad = NORMS[case["norm"]]
    s.rois, s.n, s.J = rois, n, J
    s.stream = torch.cuda.current_stream().cuda_stream
    s.lib, s.h = tg.lib(), ctypes.c_void_p(s.stream)
    s.dplan = tg.DevicePlan(rois, plan)
    if kind == "step":
        # the plan arrives anew in every step, through double-buffered pinned staging
        words = 5 * n + 1
        s.staging = [torch.zeros(words, dtype=torch.int32, pin_memory=True) for _ in range(2)]
        s.upload = [torch.cuda.Event() for _ in range(2)]
        s.plan_d = torch.zeros(words, dtype=torch.int32, device="cuda")
        s.dplan = tg.DevicePlan.from_tensors(
            s.dplan.rois, s.plan_d[:3 * n].view(n, 3), s.plan_d[3 * n:4 * n],
            s.plan_d[4 * n:4 * n + J + 1], J)
        s.params = tg.PackParams(case["canvas_w"], case["canvas_h"], case["frame_w"],
                                 case["frame_h"], case["frames"], case["policy"])
        s.counts = np.zeros(2, np.int32)  # canvases, bad index
        s.rois_p = rois.ctypes.data
        s.count_p = [s.counts.ctypes.data, s.counts.ctypes.data + 4]
        s.staging_p = [[t.data_ptr(), t.data_ptr() + 12 * n, t.data_ptr() + 16 * n]
                       for t in s.staging]
    if kind in ("step", "stitch"):
        s.frames = _pixels((case["frames"], case["frame_h"], case["frame_w"], 3), seed)
        s.out = torch.zeros((_canvas_cap(case), 3, case["canvas_h"], case["canvas_w"]),
                            dtype=torch.float16, device="cuda")
        batches = [tg.batch_range(J, case["cap"], k)
                   for k in range(tg.batch_count(J, case["cap"]))]
        s.stitch = [tg.stitch_args(s.frames, s.dplan, first, count, case["canvas_w"],
                                   case["canvas_h"], mean, std, pad, s.out[first:first + count])
                    for first, count in batches]
    if kind != "stitch":
        boxes, canvas = _boxes(case, rng, J)
        s.boxes, s.box_canvas = torch.from_numpy(boxes).cuda(), torch.from_numpy(canvas).cuda()
        s.ubufs = _zeroed(tg.UnstitchBuffers(len(boxes), n))
        s.uargs = tg.unstitch_args(s.boxes, s.box_canvas, s.dplan, case["clip"], s.ubufs,
                                   case["rule"])
        # a detection's ids and its box, as two views of the same rows
        s.det_ids = s.ubufs.dets[:, :3]
        s.det_boxes = s.ubufs.dets.view(torch.float32)[:, 3:]
    if kind in ("step", "merge"):
        s.scores = torch.from_numpy(rng.uniform(0, 1, case["boxes"]).astype(np.float32)).cuda()
        s.mbufs = _zeroed(tg.MergeBuffers(case["boxes"], case["frames"]))
        s.margs = tg.merge_args(s.ubufs.dets, s.ubufs.n_out, s.scores, case["frames"],
                                case["iou"], case["cross_only"], s.mbufs)
    if kind == "merge":
        _call("tg_unstitch", s.uargs, s.stream)
    return s


def _gmm_scene(case, seed):
    """What a fixed camera has seen: per pixel the mean colour of each component, the
    components in use (rectangles of busy pixels where things come and go, one component
    elsewhere), weights heaviest first, variances; and a generator of live frames. All
    from the seed, per camera, so that one camera can be made alone."""
    fw, fh, K = case["frame_w"], case["frame_h"], case["n_mix"]
    n = fw * fh

    def camera(f):
        g = torch.Generator(device="cuda")
        g.manual_seed(seed * 1000 + f)
        rng = np.random.default_rng([seed, f])
        cell = torch.randint(40, 200, ((fh + 15) // 16, (fw + 15) // 16, 3), device="cuda",
                             generator=g).float()
        bg = cell.repeat_interleave(16, 0).repeat_interleave(16, 1)[:fh, :fw].reshape(n, 3)
        used = torch.ones((fh, fw), dtype=torch.uint8, device="cuda")
        area, k = 0, 0
        while area < case["busy"] * n and k < 4000:
            w, h = (min(int(v), s) for v, s in zip(np.exp(rng.uniform(np.log(24), np.log(300), 2)),
                                                   (fw, fh)))
            x, y = rng.integers(0, fw - w + 1), rng.integers(0, fh - h + 1)
            m = rng.choice([2, 3, 4, 5], p=[0.7, 0.2, 0.07, 0.03])
            used[y:y + h, x:x + w] = min(int(m), K)
            area, k = area + w * h, k + 1
        used = used.reshape(n)
        state = torch.zeros((K, 5, n), device="cuda")
        total = torch.zeros(n, device="cuda")
        for m in range(K):
            on = used > m
            wm = torch.rand(n, device="cuda", generator=g) * 0.3 + 0.85
            state[m, 0] = torch.where(on, wm * 4.0 ** -m, 0.0)
            total += state[m, 0]
            if m == 0:
                mu = bg + torch.randn((n, 3), device="cuda", generator=g) * 0.3
            else:
                mu = torch.rand((n, 3), device="cuda", generator=g) * 255.0
            state[m, 1:4] = torch.where(on, mu.T, 0.0)
            state[m, 4] = torch.where(on, torch.rand(n, device="cuda", generator=g) * 8 + 4.0, 0.0)
        state[:, 0] /= total
        objs = [(int(w), int(h), rng.uniform(0, 1, 2), rng.uniform(-8, 8, 2),
                 rng.integers(0, 256, 3).tolist())
                for w, h in np.exp(rng.uniform(np.log(16), np.log(256), (40, 2)))]
        live = []
        for t in range(LIVE_FRAMES):
            px = bg + torch.randint(-3, 4, (n, 3), device="cuda", generator=g)
            # in busy places the second component's colour shows in a fifth of the pixels
            if K > 1:
                swap = (used > 1) & (torch.rand(n, device="cuda", generator=g) < 0.2)
                px = torch.where(swap[:, None], state[1, 1:4].T, px)
            img = px.clamp_(0, 255).round_().to(torch.uint8).view(fh, fw, 3)
            for w, h, p, v, rgb in objs:
                w, h = min(w, fw), min(h, fh)
                x = int(np.clip(p[0] * (fw - w) + v[0] * t, 0, fw - w))
                y = int(np.clip(p[1] * (fh - h) + v[1] * t, 0, fh - h))
                img[y:y + h, x:x + w] = torch.tensor(rgb, dtype=torch.uint8, device="cuda")
            live.append(img)
        if case["fresh"]:
            used = torch.zeros_like(used)
            state.zero_()
        return state, used, live

    return camera


def _prepare_gmm(case, seed):
    F, fw, fh, K = case["frames"], case["frame_w"], case["frame_h"], case["n_mix"]
    s = SimpleNamespace(kind="gmm", turn=0)
    s.stream = torch.cuda.current_stream().cuda_stream
    s.model = tg.GmmModel(F, fw, fh, K)
    planes, n = s.model.planes(), fw * fh
    s.live = [torch.empty((F, fh, fw, 3), dtype=torch.uint8, device="cuda")
              for _ in range(LIVE_FRAMES)]
    camera = _gmm_scene(case, seed)
    for f in range(F):
        state, used, live = camera(f)
        planes[:, :, f * n:(f + 1) * n] = state
        s.model.modes[f * n:(f + 1) * n] = used
        for t in range(LIVE_FRAMES):
            s.live[t][f] = live[t]
    params = tg.gmm_params(n_mix=K, alpha=GMM_ALPHA, var_threshold=GMM_T_BG,
                           var_threshold_gen=GMM_T_OWN, var_init=GMM_V_INIT, var_min=GMM_V_MIN,
                           var_max=GMM_V_MAX, background_ratio=GMM_RATIO,
                           complexity_reduction=GMM_CT)
    s.args = [tg.gmm_args(fr, s.model, params) for fr in s.live]
    return s


def _prepare_partition(case, seed):
    found, fb = W.make_gmm_boxes(case["frames"], case["per_frame"], case["frame_w"],
                                 case["frame_h"], seed)
    # buffers for the most RoIs there can be; frame_begin says how many there are
    boxes = np.zeros((2 * case["frames"] * case["per_frame"], 5), np.int32)
    boxes[:len(found)] = found
    s = SimpleNamespace(kind="partition")
    s.stream = torch.cuda.current_stream().cuda_stream
    s.boxes, s.frame_begin = torch.from_numpy(boxes).cuda(), torch.from_numpy(fb).cuda()
    s.bufs = _zeroed(tg.PartitionBuffers(len(boxes), case["frames"]))
    s.args = tg.partition_args(s.boxes, s.frame_begin, case["frame_w"], case["frame_h"],
                               case["zones_x"], case["zones_y"], s.bufs)
    return s


def _prepare_mask(case, seed):
    F, fw, fh = case["frames"], case["frame_w"], case["frame_h"]
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    rng = np.random.default_rng([seed, 2])
    mask = torch.zeros((F, fh, fw), dtype=torch.uint8, device="cuda")
    for f in range(F):
        if case["speckle"]:
            mask[f] = torch.rand((fh, fw), device="cuda", generator=g) < case["speckle"]
        sides = np.exp(rng.uniform(np.log(case["obj_lo"]), np.log(case["obj_hi"]),
                                   (case["objects"], 2))).astype(int)
        for w, h in sides.tolist():
            x, y = int(rng.integers(0, fw - w + 1)), int(rng.integers(0, fh - h + 1))
            yy = torch.linspace(-1, 1, h, device="cuda")[:, None] if h > 1 else torch.zeros((1, 1), device="cuda")
            xx = torch.linspace(-1, 1, w, device="cuda")[None] if w > 1 else torch.zeros((1, 1), device="cuda")
            # a box, or an ellipse with a ragged rim: what moves is seldom a clean shape
            r = xx * xx + yy * yy if rng.random() < 0.5 else torch.zeros((h, w), device="cuda")
            on = r + 0.4 * torch.rand((h, w), device="cuda", generator=g) < 1.0
            mask[f, y:y + h, x:x + w] |= on.to(torch.uint8)
    s = SimpleNamespace(kind="mask", mask=mask.view(-1))
    s.stream = torch.cuda.current_stream().cuda_stream
    cap = 1 << 16
    s.bufs = _zeroed(tg.MaskRoisBuffers(F, fw, fh, cap, 1 << 20))
    s.args = tg.mask_rois_args(s.mask, s.bufs, case["min_area"])
    s.pbufs = _zeroed(tg.PartitionBuffers(cap, F))
    s.pargs = tg.partition_args(s.bufs.rois, s.bufs.frame_begin, fw, fh, case["zones_x"],
                                case["zones_y"], s.pbufs)
    return s


def prepare(case, seed):
    kind = case["kind"]
    if kind == "gmm":
        return _prepare_gmm(case, seed)
    if kind == "partition":
        return _prepare_partition(case, seed)
    if kind == "mask":
        return _prepare_mask(case, seed)
    return _prepare_plan_case(case, seed)


# ------------------------------------------------------------------------------ one pass

def run(s):
    kind = s.kind
    if kind == "step":
        k = s.turn & 1
        s.turn += 1
        s.upload[k].synchronize()  # the staging of two steps ago has been read
        place, order, begin = s.staging_p[k]
        rc = s.lib.tg_plan_pack(s.rois_p, s.n, ctypes.byref(s.params), place, order, begin,
                                s.count_p[0], s.count_p[1])
        if rc != tg.OK or s.counts[0] != s.J:
            raise tg.TgError("tg_plan_pack", rc)
        tg.plan_upload(s.staging[k], s.plan_d)
        s.upload[k].record()
        for a in s.stitch:
            _call("tg_stitch", a, s.stream)
        _call("tg_unstitch", s.uargs, s.stream)
        _call("tg_merge", s.margs, s.stream)
        return {"canvases": s.out, "roi_of_box": s.ubufs.roi_of_box, "n_dets": s.ubufs.n_out,
                "det_ids": s.det_ids, "det_boxes": s.det_boxes, "keep": s.mbufs.keep,
                "merged": s.mbufs.out, "n_kept": s.mbufs.n_kept}
    if kind == "stitch":
        for a in s.stitch:
            _call("tg_stitch", a, s.stream)
        return {"canvases": s.out}
    if kind == "unstitch":
        _call("tg_unstitch", s.uargs, s.stream)
        return {"roi_of_box": s.ubufs.roi_of_box, "n_dets": s.ubufs.n_out, "det_ids": s.det_ids,
                "det_boxes": s.det_boxes}
    if kind == "merge":
        _call("tg_merge", s.margs, s.stream)
        return {"keep": s.mbufs.keep, "merged": s.mbufs.out, "n_kept": s.mbufs.n_kept}
    if kind == "partition":
        _call("tg_partition", s.args, s.stream)
        return {"patches": s.bufs.patches, "zone_of_box": s.bufs.zone_of_box,
                "n_patches": s.bufs.n_patches}
    if kind == "gmm":
        a = s.args[s.turn % LIVE_FRAMES]
        s.turn += 1
        _call("tg_gmm_update", a, s.stream)
        return {"state": s.model.state, "modes": s.model.modes, "mask": s.model.mask}
    _call("tg_mask_rois", s.args, s.stream)
    _call("tg_partition", s.pargs, s.stream)
    return {"rois": s.bufs.rois, "areas": s.bufs.areas, "frame_begin": s.bufs.frame_begin,
            "counts": s.bufs.counts, "patches": s.pbufs.patches,
            "zone_of_box": s.pbufs.zone_of_box, "n_patches": s.pbufs.n_patches}


# ------------------------------------------------------------------------------ its work

def work(case):
    """Bytes: every input read once, every output written once. Expected values where the
    count depends on the seed (canvas fill, kept boxes)."""
    kind = case["kind"]
    n_px = case["frames"] * case["frame_w"] * case["frame_h"]
    if kind == "partition":
        n = case["frames"] * case["per_frame"]
        return {"bytes": 20 * n + 4 * n + 4 * case["frames"] + 20 * n // 3, "flops": 0}
    if kind == "gmm":
        # sample, count in and out, mask; 20 bytes of state per component in use, each way
        comps = 1.0 + 0.43 * case["busy"] * (case["n_mix"] > 1)
        read = 0.0 if case["fresh"] else comps
        return {"bytes": n_px * (6 + 20 * (read + max(comps, 1.0))), "flops": 60 * n_px}
    if kind == "mask":
        return {"bytes": n_px + 64 * case["frames"] * case["objects"], "flops": 0}
    lo, hi, n, b = case["roi_lo"], case["roi_hi"], case["rois"], case["boxes"]
    side = (lo + hi) / 2 if case["dist"] == "uniform" else (hi - lo) / math.log(max(hi / lo, 1.01))
    roi_px = n * side * side
    bytes_ = 0.0
    if kind in ("step", "stitch"):
        # 3 bytes read and 6 written per covered pixel, canvases about 82 % covered, the plan
        bytes_ += 3 * roi_px + 6 * roi_px / 0.82 + 36 * n
    if kind in ("step", "unstitch"):
        bytes_ += b * (16 + 4 + 4 + 0.8 * 28) + 36 * n
    if kind in ("step", "merge"):
        bytes_ += 0.8 * b * (28 + 4 + 4 + 28)
    return {"bytes": bytes_, "flops": 0}


def tolerance(case):
    """Every result is a correctly rounded value or an integer decided in binary32 with each
    operation rounded on its own, so two correct implementations agree in every bit."""
    return "exact"


# ------------------------------------------------------------------------------ in 64 bits

def _pack(rois, cw, ch, policy):
    """Placements (canvas, x, y) per RoI as the three policies define them (include/tg.h)."""
    n = len(rois)
    place = np.zeros((n, 3), np.int64)
    order = np.arange(n)
    if policy == tg.SHELF_FFDH:
        order = np.argsort(-rois[:, 4], kind="stable")
    canvas = -1
    if policy == tg.GUILLOTINE_BSSF:
        free = []
        for i in order:
            w, h = int(rois[i, 3]), int(rois[i, 4])
            fits = [(min(f[2] - w, f[3] - h), max(f[2] - w, f[3] - h), k)
                    for k, f in enumerate(free) if f[2] >= w and f[3] >= h]
            if not fits:
                canvas, free, pick = canvas + 1, [(0, 0, cw, ch)], 0
            else:
                pick = min(fits)[2]
            x, y, a, b = free.pop(pick)
            place[i] = canvas, x, y
            if a <= b:
                parts = [(x + w, y, a - w, h), (x, y + h, a, b - h)]
            else:
                parts = [(x + w, y, a - w, b), (x, y + h, w, b - h)]
            free += [p for p in parts if p[2] > 0 and p[3] > 0]
        return place, order
    shelves, depth = [], 0
    for i in order:
        w, h = int(rois[i, 3]), int(rois[i, 4])
        for s in shelves:
            if h <= s[1] and w <= cw - s[2]:
                break
        else:
            if canvas < 0 or h > ch - depth:
                canvas, shelves, depth = canvas + 1, [], 0
            s = [depth, h, 0]
            shelves.append(s)
            depth += h
        place[i] = canvas, s[2], s[0]
        s[2] += w
    return place, order


def _exact_canvases(case, seed, rois, place, J):
    mean, std, pad = (np.asarray(v, np.float32).astype(np.float64) for v in NORMS[case["norm"]])
    mean_d = torch.tensor(mean, device="cuda").view(3, 1, 1)
    std_d = torch.tensor(std, device="cuda").view(3, 1, 1)
    frames = _pixels((case["frames"], case["frame_h"], case["frame_w"], 3), seed)
    out = torch.zeros((_canvas_cap(case), 3, case["canvas_h"], case["canvas_w"]),
                      dtype=torch.float64, device="cuda")
    out[:J] = ((torch.tensor(pad, device="cuda").view(3, 1, 1) - mean_d) / std_d)
    for (f, x, y, w, h), (c, dx, dy) in zip(rois.tolist(), place.tolist()):
        crop = frames[f, y:y + h, x:x + w].permute(2, 0, 1).double()
        out[c, :, dy:dy + h, dx:dx + w] = (crop - mean_d) / std_d
    return out


def _exact_det_boxes(case, rois, place, J, boxes, canvas):
    """Boxes in frame pixels, kept ones first. The patch of a box is decided in binary32, as
    declared; its coordinates are exact sums."""
    dev = "cuda"
    by = np.lexsort((np.arange(len(rois)), place[:, 0]))
    first = np.searchsorted(place[by, 0], np.arange(J + 1))
    most = int(np.diff(first).max())
    ids = np.full((J, most), -1, np.int64)
    for c in range(J):
        ids[c, :first[c + 1] - first[c]] = by[first[c]:first[c + 1]]
    ids = torch.from_numpy(ids).to(dev)
    r, p = torch.from_numpy(rois.astype(np.int64)).to(dev), torch.from_numpy(place).to(dev)
    rect = torch.stack([p[:, 1], p[:, 2], p[:, 1] + r[:, 3], p[:, 2] + r[:, 4]], 1)
    b_all, c_all = torch.from_numpy(boxes).to(dev), torch.from_numpy(canvas).to(dev).long()
    got = []
    for k in range(0, len(boxes), 20000):
        b, cand = b_all[k:k + 20000], ids[c_all[k:k + 20000]]
        q = rect[cand.clamp(min=0)].float()
        if case["rule"] == 0:
            cx, cy = ((b[:, 0] + b[:, 2]) * 0.5)[:, None], ((b[:, 1] + b[:, 3]) * 0.5)[:, None]
            hit = (cand >= 0) & (q[..., 0] <= cx) & (cx < q[..., 2]) & (q[..., 1] <= cy) & (cy < q[..., 3])
            got.append(torch.where(hit, cand, -1).amax(1))
        else:
            ow = (torch.minimum(b[:, None, 2], q[..., 2]) - torch.maximum(b[:, None, 0], q[..., 0])).clamp(min=0)
            oh = (torch.minimum(b[:, None, 3], q[..., 3]) - torch.maximum(b[:, None, 1], q[..., 1])).clamp(min=0)
            area = torch.where(cand >= 0, ow * oh, 0.0)
            top = area.amax(1, keepdim=True)
            low = torch.where((area == top) & (area > 0), cand, len(rois)).amin(1)
            got.append(torch.where(low < len(rois), low, -1))
    roi = torch.cat(got)
    keep = (roi >= 0).nonzero()[:, 0]
    v, i = b_all[keep].double(), roi[keep]
    if case["clip"]:
        lo, hi = rect[i][:, [0, 1, 0, 1]].double(), rect[i][:, [2, 3, 2, 3]].double()
        v = torch.minimum(torch.maximum(v, lo), hi)
    off = (r[i][:, 1:3] - p[i][:, 1:3]).double()
    out = torch.zeros((len(boxes), 4), dtype=torch.float64, device=dev)
    out[:len(keep)] = v + off.repeat(1, 2)
    return out


def _exact_gmm(case, seed):
    F, n, K = case["frames"], case["frame_w"] * case["frame_h"], case["n_mix"]
    stride = (F * n + 63) // 64 * 64
    out = torch.zeros((K, 5, stride), dtype=torch.float64, device="cuda")
    camera = _gmm_scene(case, seed)
    alpha = float(np.float32(GMM_ALPHA))
    decay = float(np.float32(GMM_ALPHA) * np.float32(GMM_CT))
    for f in range(F):
        state, used, live = camera(f)
        c, M = state.double(), used.long()  # c: [K, 5, n]
        x = live[0].reshape(n, 3).T.double()
        ks = torch.arange(K, device="cuda")[:, None]
        on = ks < M
        d2 = ((x - c[:, 1:4]) ** 2).sum(1)
        close = on & (d2 < GMM_T_OWN * c[:, 4])
        owner = torch.where(close, ks, K).amin(0)
        w = torch.where(on, c[:, 0] + alpha * ((ks == owner).double() - c[:, 0]) - decay, 0.0)
        own = ks == owner
        rho = (alpha / torch.where(own, w, 1.0))[:, None]
        mu = torch.where(own[:, None], c[:, 1:4] + rho * (x - c[:, 1:4]), c[:, 1:4])
        v = torch.where(own, (c[:, 4] + rho[:, 0] * (d2 - c[:, 4])).clamp(GMM_V_MIN, GMM_V_MAX),
                        c[:, 4])
        c = torch.cat([w[:, None], mu, v[:, None]], 1)
        del w, mu, v, d2, own, rho

        def swaps(wrong):
            for p in range(K - 1):
                for j in range(K - 1 - p):
                    s = wrong(j)
                    a, b = c[j].clone(), c[j + 1].clone()
                    c[j], c[j + 1] = torch.where(s, b, a), torch.where(s, a, b)

        swaps(lambda j: (j + 1 < M) & (c[j, 0] < 0) & ~(c[j + 1, 0] < 0))
        M = (on & ~(c[:, 0] < 0)).sum(0)
        new = owner == K
        at = torch.where(M < K, M, K - 1)
        put = (ks == at) & new
        c[:, 0] = torch.where(put, alpha, c[:, 0])
        c[:, 1:4] = torch.where(put[:, None], x, c[:, 1:4])
        c[:, 4] = torch.where(put, GMM_V_INIT, c[:, 4])
        M = torch.where(new, at + 1, M)
        on = ks < M
        c[:, 0] = torch.where(on, c[:, 0] / torch.where(on, c[:, 0], 0.0).sum(0), c[:, 0])
        swaps(lambda j: (j + 1 < M) & (c[j + 1, 0] > c[j, 0]))
        out[:, :, f * n:(f + 1) * n] = torch.where((ks < M)[:, None], c, 0.0)
        del c, state, live
    return out.view(-1)


def exact(case, seed):
    """What run returns for these inputs in 64 bits; None for ids, counts and flags (and for
    all of partition, merge and mask, whose outputs are integers or copies)."""
    kind = case["kind"]
    if kind in ("partition", "mask", "merge"):
        return None
    if kind == "gmm":
        return {"state": _exact_gmm(case, seed), "modes": None, "mask": None}
    rng = np.random.default_rng([seed, 1])
    rois = _rois(case, rng)
    place, order = _pack(rois, case["canvas_w"], case["canvas_h"], case["policy"])
    J = int(place[:, 0].max()) + 1
    got = {}
    if kind in ("step", "stitch"):
        got["canvases"] = _exact_canvases(case, seed, rois, place, J)
    if kind in ("step", "unstitch"):
        boxes, canvas = _boxes(case, rng, J)
        got.update(roi_of_box=None, n_dets=None, det_ids=None,
                   det_boxes=_exact_det_boxes(case, rois, place, J, boxes, canvas))
    if kind == "step":
        got.update(keep=None, merged=None, n_kept=None)
    return got
