// tg_unstitch: map detector boxes from canvas pixels back to frame pixels.
//
// The paper scores detections per source frame (Sec. V-D) after inferring stitched
// canvases (Sec. III-C) but does not say how a detection finds its patch. This
// library's rule: a box belongs to the patch holding its centre (half-open on the
// right and bottom edges); it is optionally clipped to that patch and shifted by the
// patch's frame offset minus its canvas offset.
//
// Every size is bound by latency (launches and chains of dependent loads), not by bytes:
// 24 bytes in and up to 32 out per box. Launches on the caller's stream, by size
// (the rules and where their lines lie: unstitch_route.h):
//  - few boxes on a small plan: one workgroup, one launch (small_kernel; cam1_1080p, 200
//    boxes: 6.2 us in two launches, 4.4 in one).
//  - boxes that test few patches in all, or no room for a layout: assign (LPB lanes per box test
//    the box canvas's patches, gathered from the plan) and emit, whose workgroups count the
//    kept boxes before their own by reading roi_of_box; many boxes are counted by a pass in
//    between.
//  - more: prep, assign, emit. prep lays out each canvas's patches: one rectangle per plan
//    position and, for canvases of at least kBandPatches patches, a bit per patch and band
//    -- the canvas's extent cut into kBands columns and kBands rows, band i's bits naming
//    the patches that touch it. A box's candidates are the AND of its columns' and its
//    rows' bits, a few patches instead of the canvas's hundreds. assign (L lanes per box, a
//    32-patch word each) tests those and counts the kept boxes of each kCountBlock boxes;
//    emit sums the counts before its own, or reads them scanned.
// No pass takes tickets or waits for another workgroup.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cstdint>

#include "bands.h"
#include "tg.h"
#include "unstitch_route.h"

// Built with -ffp-contract=off: every binary32 operation here is rounded on its own (no
// multiply-add fusion), so decisions taken in floating point match any plain IEEE
// implementation of the same steps.

namespace {

using tg_detail::band_axis;
using tg_detail::band_of;
using tg_detail::BandAxis;
using tg_detail::kCountBlock;
using tg_detail::kSmallBoxes;
using tg_detail::kSmallRois;
using tg_detail::transpose32;
using tg_detail::unstitch_route;
using tg_detail::UnstitchRoute;
using tg_detail::wave_min;

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / 64;
constexpr int kBandThreads = 1024;  // assign over prep's layout
constexpr int kScanThreads = 1024;
constexpr int kSmallLanes = 4;      // lanes per box in small_kernel
constexpr int kSmallThreads = kSmallBoxes * kSmallLanes;
constexpr int kCheckGroups = 8;     // workgroups of prep that check canvas_begin, a byte each
constexpr int kBands = 15;          // per axis: 30 bits of a patch's mask
constexpr int kBandWords = 4;       // a canvas's header: band origin and scale per axis
// Fewest patches whose bands fit their canvas's 8 bytes per patch:
// kBandWords + 2 kBands ceil(n / 32) <= 2 n for every n >= 17.
constexpr int kBandPatches = 17;

struct UnstitchParams {
  const tg_box *boxes;
  const int32_t *box_canvas;
  int32_t n_boxes;
  const tg_roi *rois;
  const tg_place *place;
  const int32_t *order;
  const int32_t *canvas_begin;
  int32_t n_rois, n_canvases, clip, rule;
  int32_t *roi_of_box;
  tg_det *dets;
  int32_t *n_out;
  uint8_t *gather;  // kCheckGroups verdicts of prep: any set, and the assign gathers the plan
  uint8_t *counts;  // 4-byte aligned: kept boxes of each kCountBlock boxes
  float4 *rect;    // per plan position k: the placed rectangle of RoI order[k] (prep) ...
  int32_t *bands;  // ... and the canvas's header and band words, from word 2 k_lo on
};

// Neighbouring words read with one load.
typedef int32_t i32x2 __attribute__((ext_vector_type(2), aligned(4)));
typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(8)));

// The plan segment of canvas c, clamped so that a corrupt plan cannot index outside it
// (empty for a canvas out of range).
__device__ __forceinline__ void segment_of(const UnstitchParams &P, int c, int &k_lo, int &k_hi) {
  k_lo = k_hi = 0;
  if (c >= 0 && c < P.n_canvases) {
    const i32x2 v = *reinterpret_cast<const i32x2 *>(P.canvas_begin + c);
    k_lo = min(max(v.x, 0), P.n_rois);
    k_hi = min(max(v.y, k_lo), P.n_rois);
  }
}

// The placed rectangle of the RoI at plan position k for a box of canvas c, and order[k]; a
// position that holds no RoI of that canvas gets a rectangle no box meets.
__device__ __forceinline__ float4 patch_at(const UnstitchParams &P, int k, int c, int &id) {
  const float inf = __builtin_inff();
  float4 r = make_float4(inf, inf, -inf, -inf);
  id = P.order[k];
  if (id >= 0 && id < P.n_rois) {
    const tg_place pl = P.place[id];
    const tg_roi ro = P.rois[id];
    const bool here = pl.canvas == c;  // (a branch would load the RoI only after the placement)
    r.x = here ? float(pl.x) : inf;
    r.y = here ? float(pl.y) : inf;
    r.z = here ? float(pl.x + ro.w) : -inf;
    r.w = here ? float(pl.y + ro.h) : -inf;
  }
  return r;
}

__device__ __forceinline__ bool holds(float4 r, float cx, float cy) {
  return r.x <= cx && cx < r.z && r.y <= cy && cy < r.w;
}

__device__ __forceinline__ float overlap(float4 r, const tg_box &b) {
  const float ow = fmaxf(0.0f, __fsub_rn(fminf(b.x2, r.z), fmaxf(b.x1, r.x)));
  const float oh = fmaxf(0.0f, __fsub_rn(fminf(b.y2, r.w), fmaxf(b.y1, r.y)));
  return __fmul_rn(ow, oh);
}

__device__ __forceinline__ bool any_nan(const tg_box &b) {
  return b.x1 != b.x1 || b.y1 != b.y1 || b.x2 != b.x2 || b.y2 != b.y2;
}

// The patch of a box among plan positions [k_lo, k_hi) of canvas c, gathered from the plan
// by LPB lanes (lane sl of the box; the segment is the LPB-aligned run of lanes holding
// them, all active): the RoI id, or -1, in every lane. Rule 0: the lowest position whose
// patch holds the centre. Rule 1: the largest overlap area above 0, ties to the lower RoI
// id; each lane keeps the best of its patches and the lanes' bests are compared once at the
// end (comparing them after every LPB patches was 5 shuffle reductions per box on canvases
// of 300 patches).
template <int LPB>
__device__ __forceinline__ int find_direct(const UnstitchParams &P, const tg_box &box, int c,
                                           int k_lo, int k_hi, int sl) {
  if (P.rule == 1) {
    if (any_nan(box)) k_hi = k_lo;  // matches nothing
    float best = 0.0f;
    int best_id = -1;
    for (int k = k_lo + sl; k < k_hi; k += LPB) {
      int id;
      const float a = overlap(patch_at(P, k, c, id), box);
      if (a > best || (a == best && a > 0.0f && id < best_id)) {
        best = a;
        best_id = id;
      }
    }
#pragma unroll
    for (int o = 1; o < LPB; o <<= 1) {
      const float a2 = __shfl_xor(best, o);
      const int i2 = __shfl_xor(best_id, o);
      if (a2 > best || (a2 == best && a2 > 0.0f && i2 < best_id)) {
        best = a2;
        best_id = i2;
      }
    }
    return best > 0.0f ? best_id : -1;
  }
  const float cx = (box.x1 + box.x2) * 0.5f, cy = (box.y1 + box.y2) * 0.5f;
  const int seg = (threadIdx.x & 63) - sl;  // the box's first lane
  const uint64_t seg_mask = LPB == 64 ? ~uint64_t(0) : ((uint64_t(1) << (LPB & 63)) - 1);
  for (int base = k_lo; base < k_hi; base += LPB) {
    const int k = base + sl;
    int id = -1;
    const bool hit = k < k_hi && holds(patch_at(P, k, c, id), cx, cy);
    const uint64_t m = (__ballot(hit) >> seg) & seg_mask;
    if (m) return __shfl(id, seg + __builtin_ctzll(m));  // lowest k wins
  }
  return -1;
}

template <int LPB>
__global__ __launch_bounds__(kThreads) void assign_kernel(const UnstitchParams P) {
  const int sl = threadIdx.x % LPB;
  const uint32_t b = blockIdx.x * (kThreads / LPB) + threadIdx.x / LPB;
  if (b >= static_cast<uint32_t>(P.n_boxes)) return;  // whole segments
  const tg_box box = P.boxes[b];
  const int c = P.box_canvas[b];
  int k_lo, k_hi;
  segment_of(P, c, k_lo, k_hi);
  const int roi = find_direct<LPB>(P, box, c, k_lo, k_hi, sl);
  if (sl == 0) P.roi_of_box[b] = roi;
}

// Lays out every canvas's patches (kWavesPer waves a canvas): its rectangles (positions
// that hold no RoI of the canvas: one that no box meets) and, from kBandPatches patches on,
// its header and band words. The first kCheckGroups workgroups check that canvas_begin cuts the
// plan into consecutive segments; where it does not, two canvases may share positions, whose
// rectangles are then not those of one canvas, and the assign gathers from the plan instead.
// (One workgroup alone for the check took 1,000 us for 2,000,000 canvases.)
template <int kWavesPer>
__global__ __launch_bounds__(kThreads) void prep_kernel(const UnstitchParams P) {
  __shared__ float s_ext[4][kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (blockIdx.x < kCheckGroups) {
    int bad = 0;
    constexpr int kPer = 8;  // canvases per thread and step, their words loaded together
    for (int64_t c0 = kPer * (int64_t(blockIdx.x) * kThreads + tid); c0 < P.n_canvases;
         c0 += kPer * kThreads * kCheckGroups) {
      int v[kPer + 1];
#pragma unroll
      for (int j = 0; j <= kPer; ++j)
        v[j] = P.canvas_begin[min(c0 + j, static_cast<int64_t>(P.n_canvases))];
#pragma unroll
      for (int j = 0; j < kPer; ++j) bad |= v[j] < 0 || v[j + 1] < v[j] || v[j + 1] > P.n_rois;
    }
    bad = __syncthreads_or(bad);
    if (tid == 0) P.gather[blockIdx.x] = static_cast<uint8_t>(bad != 0);
    return;
  }
  const int64_t c64 =
      (int64_t(blockIdx.x) - kCheckGroups) * (kWaves / kWavesPer) + wave / kWavesPer;
  if (kWavesPer == 1 && c64 >= P.n_canvases) return;
  const int c = static_cast<int>(c64);
  const int wv = wave % kWavesPer;
  int k_lo, k_hi;
  segment_of(P, c, k_lo, k_hi);
  const int n = k_hi - k_lo;
  const float inf = __builtin_inff();
  float x0 = inf, y0 = inf, x1 = -inf, y1 = -inf;
  float4 first = make_float4(inf, inf, -inf, -inf);  // this lane's patch of the first round
  for (int k = k_lo + 64 * wv + lane; k < k_hi; k += 64 * kWavesPer) {
    int id;
    const float4 r = patch_at(P, k, c, id);
    P.rect[k] = r;
    if (k < k_lo + 64 * kWavesPer) first = r;
    x0 = fminf(x0, r.x);
    y0 = fminf(y0, r.y);
    x1 = fmaxf(x1, r.z);
    y1 = fmaxf(y1, r.w);
  }
  if (n < kBandPatches) return;  // the canvas's waves leave together
  x0 = wave_min(x0);
  y0 = wave_min(y0);
  x1 = -wave_min(-x1);
  y1 = -wave_min(-y1);
  if (kWavesPer > 1) {
    if (lane == 0) {
      s_ext[0][wave] = x0;
      s_ext[1][wave] = y0;
      s_ext[2][wave] = x1;
      s_ext[3][wave] = y1;
    }
    __syncthreads();
    for (int w = 0; w < kWaves; ++w) {
      x0 = fminf(x0, s_ext[0][w]);
      y0 = fminf(y0, s_ext[1][w]);
      x1 = fmaxf(x1, s_ext[2][w]);
      y1 = fmaxf(y1, s_ext[3][w]);
    }
  }
  const BandAxis ax = band_axis(x0, x1, kBands), ay = band_axis(y0, y1, kBands);
  int32_t *at = P.bands + 2 * static_cast<int64_t>(k_lo);
  if (wv == 0 && lane == 0) {
    reinterpret_cast<float2 *>(at)[0] = make_float2(ax.origin, ax.scale);
    reinterpret_cast<float2 *>(at)[1] = make_float2(ay.origin, ay.scale);
  }
  at += kBandWords;
  const int words = (n + 31) / 32;
  for (int base = 64 * wv; base < n; base += 64 * kWavesPer) {
    float4 r = first;
    if (base >= 64 * kWavesPer)
      r = base + lane < n ? P.rect[k_lo + base + lane] : make_float4(inf, inf, -inf, -inf);
    uint32_t mask = 0;  // columns in bits 0 .. kBands - 1, rows above them
    if (r.x <= r.z && r.y <= r.w)
      mask = (((2u << band_of(r.z, ax, kBands)) - (1u << band_of(r.x, ax, kBands))) |
              ((2u << band_of(r.w, ay, kBands)) - (1u << band_of(r.y, ay, kBands))) << kBands);
    // lane i of each half-wave: the half's patches in band i
    mask = transpose32(mask, lane);
    const int band = lane & 31, w = base / 32 + (lane >> 5);
    if (band < 2 * kBands && w < words) at[band * words + w] = static_cast<int32_t>(mask);
  }
}

// Counts the kept boxes of a workgroup of kBandThreads threads, L lanes per box, by kCountBlock
// boxes and stores the counts, with no atomic: adding them to shared words queued at 9 ns an
// add (50,000 boxes in 3,125 workgroups: 28 us). `kept`: a kept box's first lane.
template <int L>
__device__ __forceinline__ void store_counts(const UnstitchParams &P, bool kept) {
  constexpr int kBlocks = kBandThreads / L / kCountBlock;  // counted blocks per workgroup
  static_assert(kBlocks >= 1, "a workgroup holds whole counted blocks");
  __shared__ int s_kept[kBandThreads / 64];
  const int tid = threadIdx.x;
  const uint64_t m = __ballot(kept);
  if ((tid & 63) == 0) s_kept[tid >> 6] = __popcll(m);
  __syncthreads();
  if (tid < kBlocks) {
    int sum = 0;
#pragma unroll
    for (int w = 0; w < 2 * L; ++w) sum += s_kept[2 * L * tid + w];  // kCountBlock boxes' waves
    const uint32_t blk = blockIdx.x * kBlocks + tid;
    if (blk * kCountBlock < static_cast<uint32_t>(P.n_boxes))
      P.counts[blk] = static_cast<uint8_t>(sum);
  }
}

// assign_kernel with few lanes per box and the counts (many boxes). A plan's canvases may hold
// many more patches than they do on average (the last ones of a plan packed by height): a box
// whose canvas would take more than kLongRounds rounds is left to the whole wave.
template <int L>
__global__ __launch_bounds__(kBandThreads) void assign_count_kernel(const UnstitchParams P) {
  constexpr int kLongRounds = 32;
  const int lane = threadIdx.x & 63, sl = threadIdx.x % L;
  const uint32_t b = blockIdx.x * (kBandThreads / L) + threadIdx.x / L;
  const bool in = b < static_cast<uint32_t>(P.n_boxes);  // whole segments
  tg_box box = {};
  int c = -1, k_lo = 0, k_hi = 0, roi = -1;
  if (in) {
    box = P.boxes[b];
    c = P.box_canvas[b];
    segment_of(P, c, k_lo, k_hi);
  }
  const bool is_long = k_hi - k_lo > kLongRounds * L;
  if (!is_long) roi = find_direct<L>(P, box, c, k_lo, k_hi, sl);
  for (uint64_t m = __ballot(is_long && sl == 0); m != 0; m &= m - 1) {
    const int from = __builtin_ctzll(m);
    const tg_box long_box = {__shfl(box.x1, from), __shfl(box.y1, from), __shfl(box.x2, from),
                             __shfl(box.y2, from)};
    const int r = find_direct<64>(P, long_box, __shfl(c, from), __shfl(k_lo, from),
                                  __shfl(k_hi, from), lane);
    if (lane / L == from / L) roi = r;
  }
  if (in && sl == 0) P.roi_of_box[b] = roi;
  store_counts<L>(P, in && sl == 0 && roi >= 0);
}

// The assign over prep's layout: L lanes per box, each taking every L-th word of 32 patches
// (every L-th patch of canvases without bands). The pass is a chain of dependent loads
// (canvas, segment, header, bands, rectangles), each of which meets a line per box, so
// neighbouring words share a load and a patch's RoI id is read only when it decides.
template <int L>
__global__ __launch_bounds__(kBandThreads) void assign_bands_kernel(const UnstitchParams P) {
  const int tid = threadIdx.x, sl = tid % L;
  const uint32_t b = blockIdx.x * (kBandThreads / L) + tid / L;
  const bool gather = *reinterpret_cast<const uint64_t *>(P.gather) != 0;  // uniform
  int roi = -1;
  if (b < static_cast<uint32_t>(P.n_boxes)) {  // whole segments
    const tg_box box = P.boxes[b];
    const int c = P.box_canvas[b];
    int k_lo, k_hi;
    segment_of(P, c, k_lo, k_hi);
    if (gather) {
      roi = find_direct<L>(P, box, c, k_lo, k_hi, sl);
    } else {
      const bool area = P.rule == 1;
      const int n = area && any_nan(box) ? 0 : k_hi - k_lo;
      const float cx = (box.x1 + box.x2) * 0.5f, cy = (box.y1 + box.y2) * 0.5f;
      // The best patch so far. Rule 0: the lowest position holding the centre; rule 1: the
      // largest area, ties to the lower RoI id (roi: best_k's id once a tie asked for it).
      constexpr int kNone = 0x7FFFFFFF;
      float best = 0.0f;
      int best_k = kNone;
      auto test = [&](int k, float4 r) {
        if (!area) {
          if (holds(r, cx, cy)) best_k = min(best_k, k);
          return;
        }
        const float a = overlap(r, box);
        if (a > best) {
          best = a;
          best_k = k;
          roi = -1;
        } else if (a == best && a > 0.0f && k != best_k) {
          if (roi < 0) roi = P.order[best_k];
          const int id = P.order[k];
          if (id < roi) {
            best_k = k;
            roi = id;
          }
        }
      };
      if (n < kBandPatches) {
        for (int j = sl; j < n; j += 2 * L) {
          const int j1 = min(j + L, n - 1);
          const float4 r0 = P.rect[k_lo + j], r1 = P.rect[k_lo + j1];
          test(k_lo + j, r0);
          test(k_lo + j1, r1);  // the last patch again changes nothing
        }
      } else {
        const int32_t *at = P.bands + 2 * static_cast<int64_t>(k_lo);
        const f32x4 head = *reinterpret_cast<const f32x4 *>(at);
        const BandAxis ax = {head.x, head.y}, ay = {head.z, head.w};
        const int words = (n + 31) / 32;
        const int32_t *cols = at + kBandWords, *rows = cols + kBands * words;
        const int x0 = band_of(area ? box.x1 : cx, ax, kBands);
        const int x1 = area ? band_of(box.x2, ax, kBands) : x0;
        const int y0 = band_of(area ? box.y1 : cy, ay, kBands);
        const int y1 = area ? band_of(box.y2, ay, kBands) : y0;
        for (int w = sl; w < words; w += L) {
          uint32_t mc = 0, mr = 0;
          if (!area) {
            mc = cols[x0 * words + w];
            mr = rows[y0 * words + w];
          } else if (x0 <= x1 && y0 <= y1) {  // (an inverted box overlaps nothing)
            for (int i = 0; i <= max(x1 - x0, y1 - y0); i += 2) {
              const uint32_t c0 = cols[min(x0 + i, x1) * words + w];
              const uint32_t c1 = cols[min(x0 + i + 1, x1) * words + w];
              const uint32_t r0 = rows[min(y0 + i, y1) * words + w];
              const uint32_t r1 = rows[min(y0 + i + 1, y1) * words + w];
              mc |= c0 | c1;
              mr |= r0 | r1;
            }
          }
          for (uint32_t m = mc & mr; m != 0;) {  // two candidates' loads together
            const int k0 = k_lo + 32 * w + __builtin_ctz(m);
            m &= m - 1;
            const int k1 = m ? k_lo + 32 * w + __builtin_ctz(m) : k0;
            m &= m - 1;
            const float4 r0 = P.rect[k0], r1 = P.rect[k1];
            test(k0, r0);
            test(k1, r1);  // the same patch again changes nothing
          }
        }
      }
      if (!area) {
#pragma unroll
        for (int o = 1; o < L; o <<= 1) best_k = min(best_k, __shfl_xor(best_k, o));
        if (best_k != kNone) roi = P.order[best_k];
      } else {
        if (best_k != kNone && roi < 0) roi = P.order[best_k];
#pragma unroll
        for (int o = 1; o < L; o <<= 1) {
          const float a2 = __shfl_xor(best, o);
          const int i2 = __shfl_xor(roi, o);
          if (a2 > best || (a2 == best && a2 > 0.0f && i2 < roi)) {
            best = a2;
            roi = i2;
          }
        }
      }
    }
    if (sl == 0) P.roi_of_box[b] = roi;
  }
  store_counts<L>(P, sl == 0 && roi >= 0);
}

// The detection of kept box b (patch roi).
__device__ __forceinline__ tg_det make_det(const UnstitchParams &P, int32_t b, int roi) {
  const tg_roi r = P.rois[roi];
  const tg_place pl = P.place[roi];
  const tg_box box = P.boxes[b];
  float v[4] = {box.x1, box.y1, box.x2, box.y2};
  if (P.clip) {
    const float lo[2] = {float(pl.x), float(pl.y)};
    const float hi[2] = {float(pl.x + r.w), float(pl.y + r.h)};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (v[q] < lo[q & 1]) v[q] = lo[q & 1];
      if (v[q] > hi[q & 1]) v[q] = hi[q & 1];
    }
  }
  const float ox = float(r.x - pl.x), oy = float(r.y - pl.y);
  tg_det d;
  d.box = b;
  d.roi = roi;
  d.frame = r.frame;
  d.x1 = v[0] + ox;
  d.y1 = v[1] + oy;
  d.x2 = v[2] + ox;
  d.y2 = v[3] + oy;
  return d;
}

// The kept boxes of each kCountBlock boxes, for an assign that gathers and does not count: a
// wave per kCountBlock boxes.
__global__ __launch_bounds__(kThreads) void count_kernel(const UnstitchParams P) {
  static_assert(kCountBlock == 128, "two boxes per lane");
  const uint32_t blk = blockIdx.x * kWaves + (threadIdx.x >> 6), n = P.n_boxes;
  const uint32_t b = blk * kCountBlock + (threadIdx.x & 63);
  const uint64_t m0 = __ballot(b < n && P.roi_of_box[b] >= 0);
  const uint64_t m1 = __ballot(b + 64 < n && P.roi_of_box[b + 64] >= 0);
  if ((threadIdx.x & 63) == 0 && blk * kCountBlock < n)
    P.counts[blk] = static_cast<uint8_t>(__popcll(m0) + __popcll(m1));
}

// The counts scanned in place by one workgroup, so that an emit workgroup reads one word
// instead of summing all counts before its own: each 8 counts (1,024 boxes) become the kept
// boxes before them, and in the upper word those of their first 2, 4 and 6 counts in 10 bits
// each.
__global__ __launch_bounds__(kScanThreads) void scan_counts_kernel(const UnstitchParams P) {
  __shared__ int s_wave[kScanThreads / 64];
  constexpr int kPer = 4;  // words per thread and step
  uint64_t *words = reinterpret_cast<uint64_t *>(P.counts);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_counts = static_cast<int>((uint32_t(P.n_boxes) + kCountBlock - 1) / kCountBlock);
  const int n_words = (n_counts + 7) / 8;
  int carry = 0;
  for (int w0 = 0; w0 < n_words; w0 += kPer * kScanThreads) {
    const int first = w0 + kPer * tid;
    int pair[kPer][4], sum = 0;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const int w = first + k, left = n_counts - 8 * w;  // counts of this word and later ones
      uint64_t v = left > 0 ? words[w] : 0;
      if (left > 0 && left < 8) v &= (uint64_t(1) << (8 * left)) - 1;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        pair[k][j] = static_cast<int>((v >> (16 * j) & 0xFFu) + (v >> (16 * j + 8) & 0xFFu));
        sum += pair[k][j];
      }
    }
    int incl = sum;
    for (int o = 1; o < 64; o <<= 1) {
      const int t = __shfl_up(incl, o);
      if (lane >= o) incl += t;
    }
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int at = carry + incl - sum;
#pragma unroll
    for (int w = 0; w < kScanThreads / 64; ++w) {
      if (w < wave) at += s_wave[w];
      carry += s_wave[w];
    }
    __syncthreads();  // s_wave is written again by the next step
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      if (first + k >= n_words) break;
      const int p1 = pair[k][0], p2 = p1 + pair[k][1], p3 = p2 + pair[k][2];
      words[first + k] = static_cast<uint32_t>(at) |
                         static_cast<uint64_t>(p1 | p2 << 10 | p3 << 20) << 32;
      at += p3 + pair[k][3];
    }
  }
}

// Writes the kept boxes of 256 consecutive boxes, one per thread, in increasing box order: a
// stable compaction. The workgroup's first position is the kept boxes before its own:
// kOwnCounts all earlier box ids, read again by every workgroup; kSumCounts the sum of the
// earlier counts; kScanned its own word of the scanned counts.
enum EmitCounts { kOwnCounts, kSumCounts, kScanned };
template <EmitCounts kMode>
__global__ __launch_bounds__(kThreads) void emit_kernel(const UnstitchParams P) {
  __shared__ int s_before[kWaves], s_wave[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint32_t b0 = blockIdx.x * kThreads, b = b0 + tid;
  const int roi = b < static_cast<uint32_t>(P.n_boxes) ? P.roi_of_box[b] : -1;
  int before = 0;
  if (kMode == kScanned) {
    if (tid == 0) {
      const uint64_t v = reinterpret_cast<const uint64_t *>(P.counts)[b0 / (8 * kCountBlock)];
      const uint32_t part = b0 / kThreads % 4;
      before = static_cast<int>(static_cast<uint32_t>(v));
      if (part > 0) before += static_cast<int>(v >> (32 + 10 * (part - 1)) & 1023u);
    }
  } else if (kMode == kSumCounts) {  // the counts before b0 (an even number), four at a time
    const uint32_t n = b0 / kCountBlock;
#pragma unroll 4
    for (uint32_t i = 4 * tid; i < n; i += 4 * kThreads) {
      const uint32_t v = *reinterpret_cast<const uint32_t *>(P.counts + i);
      before += (v & 0xFFu) + (v >> 8 & 0xFFu);
      if (i + 2 < n) before += (v >> 16 & 0xFFu) + (v >> 24);
    }
  } else {
#pragma unroll 4
    for (uint32_t i = 4 * tid; i < b0; i += 4 * kThreads) {  // b0 is a multiple of 4
      const i32x4 v = *reinterpret_cast<const i32x4 *>(P.roi_of_box + i);
      before += (v.x >= 0) + (v.y >= 0) + (v.z >= 0) + (v.w >= 0);
    }
  }
  tg_det d;
  if (roi >= 0) d = make_det(P, b, roi);
  const uint64_t kept = __ballot(roi >= 0);
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  if (lane == 0) {
    s_before[wave] = before;
    s_wave[wave] = __popcll(kept);
  }
  __syncthreads();
  int pos = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    pos += s_before[w];
    if (w < wave) pos += s_wave[w];
    total += s_before[w] + s_wave[w];
  }
  if (roi >= 0) P.dets[pos + __popcll(kept & ((uint64_t(1) << lane) - 1))] = d;
  if (tid == 0 && blockIdx.x == gridDim.x - 1) *P.n_out = total;
}

// Up to kSmallBoxes boxes: assign and emit in one workgroup, every box at once (kSmallLanes
// lanes each) against the plan's rectangles, gathered once into LDS. (Gathered again for every
// box, canvases of more than 40 patches cost more than a second launch: 256 boxes on one canvas
// of 64 patches 10.5 us, of 20 6.5; as built 6.7 and 5.1.)
__global__ __launch_bounds__(kSmallThreads) void small_kernel(const UnstitchParams P) {
  __shared__ float4 s_rect[kSmallRois];
  __shared__ int s_canvas[kSmallRois], s_id[kSmallRois];
  __shared__ int s_roi[kSmallBoxes];
  __shared__ int s_wave[kSmallBoxes / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int sl = tid % kSmallLanes, own = tid / kSmallLanes;
  const bool area = P.rule == 1;
  int c = -1, k_lo = 0, k_hi = 0;
  tg_box box = {};
  if (own < P.n_boxes) {
    box = P.boxes[own];
    c = P.box_canvas[own];
    segment_of(P, c, k_lo, k_hi);
  }
  if (tid < P.n_rois) {  // position tid of the plan
    const int id = P.order[tid];
    s_id[tid] = id;
    s_canvas[tid] = -1;  // no box's, unless it holds a RoI
    if (id >= 0 && id < P.n_rois) {
      const tg_place pl = P.place[id];
      const tg_roi ro = P.rois[id];
      s_canvas[tid] = pl.canvas;
      s_rect[tid] = make_float4(float(pl.x), float(pl.y), float(pl.x + ro.w), float(pl.y + ro.h));
    }
  }
  __syncthreads();
  int best_k = 0x7FFFFFFF, best_id = -1;
  if (own < P.n_boxes) {
    if (area && any_nan(box)) k_hi = k_lo;
    const float cx = (box.x1 + box.x2) * 0.5f, cy = (box.y1 + box.y2) * 0.5f;
    float best = 0.0f;
    constexpr int kBatch = 4;  // patches whose LDS reads are issued together
    for (int k0 = k_lo + sl; k0 < k_hi; k0 += kSmallLanes * kBatch) {
      float4 r[kBatch];
      int id[kBatch], canvas[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {  // the last patch again past the end: no change
        const int k = min(k0 + u * kSmallLanes, k_hi - 1);
        r[u] = s_rect[k];
        id[u] = s_id[k];
        canvas[u] = s_canvas[k];
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int k = min(k0 + u * kSmallLanes, k_hi - 1);
        const bool here = canvas[u] == c;
        if (area) {
          const float a = here ? overlap(r[u], box) : 0.0f;
          if (a > best || (a == best && a > 0.0f && id[u] < best_id)) {
            best = a;
            best_id = id[u];
          }
        } else if (here && k < best_k && holds(r[u], cx, cy)) {
          best_k = k;
          best_id = id[u];
        }
      }
    }
#pragma unroll
    for (int o = 1; o < kSmallLanes; o <<= 1) {
      const int i2 = __shfl_xor(best_id, o), k2 = __shfl_xor(best_k, o);
      const float a2 = __shfl_xor(best, o);
      if (area ? a2 > best || (a2 == best && a2 > 0.0f && i2 < best_id) : k2 < best_k) {
        best = a2;
        best_k = k2;
        best_id = i2;
      }
    }
    if (sl == 0) {
      s_roi[own] = best_id;
      P.roi_of_box[own] = best_id;
    }
  }
  __syncthreads();
  int roi = -1;
  tg_det d;
  uint64_t kept = 0;
  if (tid < kSmallBoxes) {  // whole waves
    if (tid < P.n_boxes) roi = s_roi[tid];
    if (roi >= 0) d = make_det(P, tid, roi);
    kept = __ballot(roi >= 0);
    if (lane == 0) s_wave[wave] = __popcll(kept);
  }
  __syncthreads();
  if (tid >= kSmallBoxes) return;
  int pos = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kSmallBoxes / 64; ++w) {
    if (w < wave) pos += s_wave[w];
    total += s_wave[w];
  }
  if (roi >= 0) P.dets[pos + __popcll(kept & ((uint64_t(1) << lane) - 1))] = d;
  if (tid == 0) *P.n_out = total;
}

__global__ void zero_count_kernel(int32_t *n_out) { *n_out = 0; }

// Bytes of the flag (8) and the counts (8 per 1024 boxes) for n boxes, rounded up to 16 so
// that the rectangles after them are aligned.
size_t word_bytes(int32_t n) {
  constexpr size_t kEight = 8 * kCountBlock;
  return (8 * (1 + (static_cast<size_t>(n) + kEight - 1) / kEight) + 15) & ~size_t(15);
}

// Bytes of the layout of a plan of n_rois RoIs: a rectangle and 8 bytes of bands each.
size_t record_bytes(int32_t n_rois) {
  return n_rois > 0 ? 24 * static_cast<size_t>(n_rois) : 0;
}

// Workspace of the allocation-free entry point: the flag and count words for up
// to TG_UNSTITCH_NOALLOC_MAX_BOXES boxes, then the layout of plans of up to
// TG_UNSTITCH_NOALLOC_MAX_ROIS RoIs (3.3 MB in all). Each GPU the library runs on holds
// its own copy until the process ends; host code reaches it only through the address
// hipGetSymbolAddress returns for the current device.
constexpr size_t kScratchWords =
    (8 * (1 + size_t(TG_UNSTITCH_NOALLOC_MAX_BOXES) / (8 * kCountBlock)) + 15) & ~size_t(15);
constexpr size_t kScratchBytes = kScratchWords + 24 * size_t(TG_UNSTITCH_NOALLOC_MAX_ROIS);
__device__ __align__(256) uint64_t scratch[kScratchBytes / 8];

// Device address of `scratch` on the current device, looked up once per device id (null
// when the lookup fails).
void *scratch_address() {
  static std::atomic<void *> cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return nullptr;
  void *p = cached[dev].load(std::memory_order_acquire);
  if (p) return p;
  if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
  cached[dev].store(p, std::memory_order_release);
  return p;
}

// Argument checks shared by both entry points (the workspace aside).
int check_args(const tg_unstitch_args *a) {
  if (!a || a->n_boxes < 0 || a->n_rois < 0 || a->n_canvases < 0) return TG_E_INVAL;
  if (a->rule != 0 && a->rule != 1) return TG_E_INVAL;
  if (!a->n_out) return TG_E_INVAL;
  if (a->n_boxes == 0) return TG_OK;
  if (!a->boxes || !a->box_canvas || !a->roi_of_box || !a->dets) return TG_E_INVAL;
  if (a->n_canvases > 0 && !a->canvas_begin) return TG_E_INVAL;
  if (a->n_rois > 0 && (!a->rois || !a->place || !a->order)) return TG_E_INVAL;
  return TG_OK;
}

template <int L>
void launch_bands(int32_t n_boxes, hipStream_t s, const UnstitchParams &P) {
  const int64_t per_block = kBandThreads / L;
  hipLaunchKernelGGL(assign_bands_kernel<L>,
                     dim3(static_cast<uint32_t>((int64_t(n_boxes) + per_block - 1) / per_block)),
                     dim3(kBandThreads), 0, s, P);
}

// Enqueues the launches with `words` (device, 8-byte aligned, word_bytes(n_boxes) bytes)
// and `records` (16-byte aligned, record_bytes(n_rois) bytes, or null when the plan is to be
// gathered) as scratch.
int launch(const tg_unstitch_args *a, void *words, void *records, hipStream_t s) {
  if (a->n_boxes == 0) {
    hipLaunchKernelGGL(zero_count_kernel, dim3(1), dim3(1), 0, s, a->n_out);
    return hipGetLastError() == hipSuccess ? TG_OK : TG_E_HIP;
  }
  UnstitchParams P;
  P.boxes = a->boxes;
  P.box_canvas = a->box_canvas;
  P.n_boxes = a->n_boxes;
  P.rois = a->rois;
  P.place = a->place;
  P.order = a->order;
  P.canvas_begin = a->canvas_begin;
  P.n_rois = a->n_rois;
  P.n_canvases = a->n_canvases;
  P.clip = a->clip;
  P.rule = a->rule;
  P.roi_of_box = a->roi_of_box;
  P.dets = a->dets;
  P.n_out = a->n_out;
  P.gather = static_cast<uint8_t *>(words);
  P.counts = static_cast<uint8_t *>(words) + 8;
  const UnstitchRoute R =
      unstitch_route(a->n_boxes, a->n_rois, a->n_canvases, records != nullptr);
  const auto groups = [](int64_t work, int64_t per) {
    return dim3(static_cast<uint32_t>((work + per - 1) / per));
  };
  if (R.small) {
    hipLaunchKernelGGL(small_kernel, dim3(1), dim3(kSmallThreads), 0, s, P);
    return hipGetLastError() == hipSuccess ? TG_OK : TG_E_HIP;
  }
  if (R.laid_out) {
    P.rect = static_cast<float4 *>(records);
    P.bands = reinterpret_cast<int32_t *>(P.rect + a->n_rois);
    const int64_t per_canvas = (int64_t(a->n_rois) + a->n_canvases - 1) / a->n_canvases;
    if (per_canvas > 64)
      hipLaunchKernelGGL(prep_kernel<kWaves>, groups(int64_t(a->n_canvases) + kCheckGroups, 1),
                         dim3(kThreads), 0, s, P);
    else
      hipLaunchKernelGGL(prep_kernel<1>,
                         groups(int64_t(a->n_canvases) + kCheckGroups * kWaves, kWaves),
                         dim3(kThreads), 0, s, P);
    if (hipGetLastError() != hipSuccess) return TG_E_HIP;
    if (R.lanes == 2)
      launch_bands<2>(a->n_boxes, s, P);
    else
      launch_bands<8>(a->n_boxes, s, P);
  } else if (R.lanes == 8) {
    hipLaunchKernelGGL(assign_count_kernel<8>, groups(a->n_boxes, kBandThreads / 8),
                       dim3(kBandThreads), 0, s, P);
  } else {
    const dim3 grid = groups(a->n_boxes, kThreads / R.lanes);
    if (R.lanes == 16)
      hipLaunchKernelGGL(assign_kernel<16>, grid, dim3(kThreads), 0, s, P);
    else
      hipLaunchKernelGGL(assign_kernel<64>, grid, dim3(kThreads), 0, s, P);
    if (hipGetLastError() != hipSuccess) return TG_E_HIP;
    if (R.counted)
      hipLaunchKernelGGL(count_kernel, groups(a->n_boxes, kCountBlock * kWaves), dim3(kThreads), 0,
                         s, P);
  }
  if (hipGetLastError() != hipSuccess) return TG_E_HIP;
  if (R.scanned) hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(kScanThreads), 0, s, P);
  if (hipGetLastError() != hipSuccess) return TG_E_HIP;
  const dim3 grid = groups(a->n_boxes, kThreads);
  if (R.scanned)
    hipLaunchKernelGGL(emit_kernel<kScanned>, grid, dim3(kThreads), 0, s, P);
  else if (R.counted)
    hipLaunchKernelGGL(emit_kernel<kSumCounts>, grid, dim3(kThreads), 0, s, P);
  else
    hipLaunchKernelGGL(emit_kernel<kOwnCounts>, grid, dim3(kThreads), 0, s, P);
  return hipGetLastError() == hipSuccess ? TG_OK : TG_E_HIP;
}

}  // namespace

extern "C" size_t tg_unstitch_workspace_bytes(int32_t n_boxes, int32_t n_rois) {
  if (n_boxes <= 0) return 0;
  return word_bytes(n_boxes) + record_bytes(n_rois);
}

extern "C" int tg_unstitch(const tg_unstitch_args *a, void *stream) {
  const int rc = check_args(a);
  if (rc != TG_OK) return rc;
  if (a->n_boxes == 0) return launch(a, nullptr, nullptr, static_cast<hipStream_t>(stream));
  const size_t need = tg_unstitch_workspace_bytes(a->n_boxes, a->n_rois);
  if (!a->workspace || a->workspace_bytes < need ||
      reinterpret_cast<uintptr_t>(a->workspace) % 16 != 0)
    return TG_E_WORKSPACE;
  char *ws = static_cast<char *>(a->workspace);
  return launch(a, ws, ws + word_bytes(a->n_boxes), static_cast<hipStream_t>(stream));
}

extern "C" int tg_unstitch_noalloc(const tg_unstitch_args *a, void *stream) {
  const int rc = check_args(a);
  if (rc != TG_OK) return rc;
  if (a->n_boxes > TG_UNSTITCH_NOALLOC_MAX_BOXES) return TG_E_WORKSPACE;
  if (a->n_boxes == 0) return launch(a, nullptr, nullptr, static_cast<hipStream_t>(stream));
  char *ws = static_cast<char *>(scratch_address());
  if (!ws) return TG_E_HIP;
  // plans larger than the records area are gathered directly (same results)
  void *records = a->n_rois <= TG_UNSTITCH_NOALLOC_MAX_ROIS ? ws + kScratchWords : nullptr;
  return launch(a, ws, records, static_cast<hipStream_t>(stream));
}
