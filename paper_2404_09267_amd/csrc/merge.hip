// tg_merge: per-frame suppression of duplicate detections after tg_unstitch.
//
// When a frame is cut into zone patches (Sec. III-A, Alg. 1), neighbouring patches can
// overlap, so one object can come back from two patches once detections are mapped to
// their frame (Sec. V-D scores per frame). The paper does not spell out the merge; this
// library's reading: a frame's detections are ranked by score (higher first, equal scores
// by box index, a NaN score last), and walking that ranking a detection is kept unless one
// kept before it in the same frame (with cross_only: from another patch) overlaps it by
// IoU > threshold, decided as inter > threshold * union in binary32 with every operation
// rounded on its own. Kept detections are written in input order.
//
// The greedy walk keeps a detection exactly when no detection ranked above it that
// suppresses it is kept (by induction over the ranking). So no sorted ranking is needed:
// given each detection's suppressors ranked above it, rounds decide the frame -- a
// detection is suppressed once one of them is kept, kept once all of them are suppressed.
// The best-ranked undecided detection of a round has only decided suppressors, so every
// round decides at least one: a frame of n detections needs at most n rounds (two to four
// in practice, where chains of boxes suppressing each other are short).
//
// The call is bound by latency -- launches, and chains of dependent loads inside them --
// not by its bytes, so it takes few launches and no global atomics on shared counters:
//  1. hist:    each workgroup counts its chunk of detections per bin (a frame, or a run of
//              frames when there are more than kBinsMax) into its row of a small table.
//  2. scatter: each workgroup sums the table's columns for its positions and writes its
//              detections' ranking keys, boxes, patches and indices into bin order.
//  3. local:   one workgroup per bin orders a bin of several frames by frame in LDS and
//              decides every frame of at most kLocal detections there: band bits (bands.h)
//              name the few boxes that can meet each box, those pairs are listed and tested,
//              and the rounds run on the suppressing ones; where boxes crowd, rows of
//              suppressor bits take the place of the list. Larger frames, and a frame that
//              alone is too crowded for the rows, are put on a list.
//  4. tile:    the listed frames cut into tiles of about kTileDets detections (by their
//              top-left corners), a workgroup each: its detections' suppressors among the
//              frame's boxes that meet the rectangle around its own.
//  5. resolve: the rounds of each listed frame, over its detections that have suppressors.
//  6. compact: the kept detections in input order.
// Measured (unstitched detections, IoU 0.5 across patches), with the eight launches of a
// grid index per frame before: 8,249 in 20 frames 45.6 -> 27 us; 47,939 in 8 frames
// 111 -> 48; 164,685 in 1,920 frames 62.7 -> 45.4; 20,000 in one frame 317 -> 108, crowded
// into 300 x 300 pixels 619 ms (its pairs overran the lists) -> 1.7 ms.
// Tile and resolve return at once when no frame is listed. Inputs of at most kTiny
// detections (by capacity) take one launch instead (tiny_kernel).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "bands.h"
#include "lookback.h"
#include "tg.h"

// Built with -ffp-contract=off: every binary32 operation here is rounded on its own (no
// multiply-add fusion), so decisions taken in floating point match any plain IEEE
// implementation of the same steps.

namespace {

using tg_detail::band_axis;
using tg_detail::band_of;
using tg_detail::BandAxis;
using tg_detail::transpose32;
using tg_detail::wave_min;

constexpr int kThreads = 256;
constexpr int kPerThread = 4;  // look-back compaction: consecutive detections per thread
constexpr int kCompactBlock = kThreads * kPerThread;
constexpr int kCountThreads = 1024;   // counting compaction: a detection per thread
constexpr int kCountDets = 65536;     // largest capacity it takes
constexpr int kBinThreads = 1024;     // hist and scatter
constexpr int kBinsMax = 256;
constexpr int kChunksMax = 128;       // workgroups of hist and scatter: rows of the table
constexpr int kLocal = 1024;          // detections decided in LDS by one workgroup
constexpr int kLocalWords = kLocal / 32;
constexpr int kFrameHist = 4096;      // frames of a bin ordered in one pass
constexpr int kPairs = 4096;          // pairs that bands bring together, held in LDS
// and those that suppress; or words of suppressor rows, rows of 23 words for a frame of 712
// detections, of 15 for frames of up to 448 that fill kLocal
constexpr int kHits = 16384;
constexpr int kTileThreads = 1024;
// Detections per tile, about: kTileDets, or more where the call's would make more than four
// tiles for each of the kGridCap workgroups that run (every tile reads its whole frame, so
// fewer are then cheaper). With 256, 512 and 1,024 always: 8,000,000 in 256 frames 6.0, 3.7 and
// 3.3 ms; 1,000,000 in 8 1.20, 1.20 and 1.04; 20,000 in one 0.115, 0.120 and 0.153.
constexpr int kTileDets = 256, kTileDetsMax = 1024;
constexpr int kTilesMax = 256;        // tiles per frame, about
constexpr int kTilesPerAxis = 17;     // (a square root that may round up)
constexpr int kPredSlots = 16;        // suppressors kept in place per detection
// workgroups of tile and resolve, which step through their work: tile's LDS lets one run per
// CU (two small ones on one CU left others idle and ran one after the other: 37 -> 22 us)
constexpr int kGridCap = 256;
constexpr int kResolveThreads = 1024;
constexpr int32_t kUndecided = 0, kKept = 1, kSuppressed = 2;

// A frame of more than kLocal detections, or one too crowded to be decided in LDS:
// positions [lo, lo + n) of the frame order, cut into g x g tiles numbered from `start` among
// all listed frames' tiles: an even grid of dx x dy each from (x0, y0) on, or, g being
// negative, by samples (uneven_rect). open: how many of its detections have suppressors (their
// positions are listed in MergeParams::open from lo on).
struct LargeFrame {
  int32_t lo, n, g;
  uint32_t start;
  float x0, y0, dx, dy;
  int32_t open;
};

// A tile owns the detections of its frame whose top-left corner (a NaN coordinate taken as
// -infinity) is at or past (x0, y0) and not at or past (x1, y1). Tiles that share a cut hold
// the same value for it, and outer cuts are -infinity and NaN (which nothing is past), so each
// corner is in one tile of its frame.
struct TileRect {
  float x0, y0, x1, y1;
};

// What a detection has besides its box: ranking key, patch, index.
struct alignas(16) Aux {
  uint64_t key;
  int32_t roi, idx;
};

// A detection in bin or frame order. One 32-byte record, a whole memory sector, so that
// scattered writes replace sectors instead of merging into them (separate arrays of boxes,
// keys and the rest: the pass that read them waited 8-16 us for 165,000 detections in
// 1,920 frames, and the scatter itself took 18.8 us instead of 12).
struct alignas(16) Rec {
  float4 box;
  Aux aux;
};

struct MergeParams {
  const tg_det *dets;
  const int32_t *n_dets;
  int32_t n_max;
  const float *scores;
  int32_t n_scores, n_frames;
  float thr;
  int32_t cross_only;
  int32_t *keep;
  tg_det *out;
  int32_t *n_kept;
  int32_t chunk, n_chunks;  // detections per hist / scatter workgroup, and how many those are
  int32_t n_bins, per_bin;  // frames per bin (1 up to kBinsMax frames)
  int64_t n_words;          // 64-bit words from `ticket` on, zeroed by hist
  uint32_t *ticket;
  uint32_t *status;         // set when a frame's rounds overrun (cannot happen)
  unsigned long long *ovf_used;  // entries of ovf handed out
  unsigned long long *large_used;  // listed frames << 32 | their tiles
  uint64_t *state;          // look-back words of the compaction
  int32_t *table;           // [n_chunks][n_bins]
  int32_t *bin_begin;       // [n_bins + 1]
  LargeFrame *large;
  // Per detection, at its position in bin order ...
  Rec *crec;
  // ... and in frame order (the same arrays with one frame per bin; else only the bins that
  // do not fit one workgroup are written here).
  Rec *rec;
  int32_t *frame;
  // Listed frames, by position in frame order.
  int32_t *rstate;   // kUndecided, kKept or kSuppressed
  int32_t *rnpred;   // suppressors ranked above
  int32_t *rpred;    // [kPredSlots each] the first of them (positions)
  int32_t *rovf;     // a longer list's start in ovf, or -1: search again
  int32_t *open;     // positions of the frame's detections that have suppressors
  int32_t *ovf;      // whole lists of detections with more than kPredSlots
  int64_t ovf_cap;
};

__device__ __forceinline__ int count_of(const MergeParams &P) {
  return min(max(*P.n_dets, 0), P.n_max);
}

// Inclusive prefix sum over the 64 lanes of a wave (DPP row shifts, then row broadcasts).
__device__ __forceinline__ int wave_inclusive_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, false);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, false);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, false);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31
  return v;
}

// This lane's first place of `count` more in an LDS list of *n entries. Called by whole
// waves. (One atomic per wave: the compiler turns an atomic of many lanes on one address
// into a loop over the lanes.)
__device__ __forceinline__ int wave_places(int *n, int count) {
  const int incl = wave_inclusive_sum(count), total = __builtin_amdgcn_readlane(incl, 63);
  int base = 0;
  if ((threadIdx.x & 63) == 0 && total) base = atomicAdd(n, total);
  return __builtin_amdgcn_readfirstlane(base) + incl - count;
}

// One place for each active lane, which may be any lanes of the wave.
__device__ __forceinline__ int lane_place(int *n) {
  const uint64_t active = __ballot(1);
  const int lane = threadIdx.x & 63, leader = __builtin_ctzll(active);
  int base = 0;
  if (lane == leader) base = atomicAdd(n, __popcll(active));
  return __builtin_amdgcn_readlane(base, leader) + __popcll(active & ((uint64_t(1) << lane) - 1));
}

// Exclusive scan of v over a workgroup of kN threads (s: kN / 64 ints of LDS); *total gets the
// sum. Ends with a barrier.
template <int kN>
__device__ __forceinline__ int block_exclusive(int v, int *s, int *total) {
  const int incl = wave_inclusive_sum(v);
  if ((threadIdx.x & 63) == 63) s[threadIdx.x >> 6] = incl;
  __syncthreads();
  int before = 0, sum = 0;
#pragma unroll
  for (int w = 0; w < kN / 64; ++w) {
    if (w < static_cast<int>(threadIdx.x >> 6)) before += s[w];
    sum += s[w];
  }
  __syncthreads();
  *total = sum;
  return before + incl - v;
}

__device__ __forceinline__ int bin_of(const MergeParams &P, int f) {
  const uint32_t per = P.per_bin;
  return per == 1 ? f : static_cast<int>(static_cast<uint32_t>(f) / per);
}

// Detections of this workgroup's chunk per bin. (Counting into global counters instead
// needs a launch to clear them and an atomic per frame and workgroup, and they queue:
// window_64x30, 1,920 frames, count and scatter 23 us together.)
__global__ __launch_bounds__(kBinThreads) void hist_kernel(const MergeParams P) {
  __shared__ int hist[kBinsMax];
  const int tid = threadIdx.x, g = blockIdx.x;
  for (int64_t i = static_cast<int64_t>(g) * kBinThreads + tid; i < P.n_words;
       i += static_cast<int64_t>(gridDim.x) * kBinThreads)
    reinterpret_cast<uint64_t *>(P.ticket)[i] = 0;
  if (tid < P.n_bins) hist[tid] = 0;
  __syncthreads();
  const int64_t lo = static_cast<int64_t>(g) * P.chunk;
  const int64_t hi = min(lo + P.chunk, static_cast<int64_t>(count_of(P)));
#pragma unroll 4
  for (int64_t i = lo + tid; i < hi; i += kBinThreads) {
    const int f = P.dets[i].frame;
    if (f >= 0 && f < P.n_frames)
      atomicAdd(&hist[bin_of(P, f)], 1);
    else
      P.keep[i] = 0;  // no frame to merge in: dropped
  }
  __syncthreads();
  if (tid < P.n_bins) P.table[static_cast<int64_t>(g) * P.n_bins + tid] = hist[tid];
}

// Ranking key, ascending = higher score first, then lower box index. NaN ranks as -inf;
// -0 and +0 are the same score.
__device__ __forceinline__ uint64_t rank_key(float s, int32_t box) {
  if (s != s) s = -__builtin_inff();
  if (s == 0.0f) s = 0.0f;
  uint32_t b = __float_as_uint(s);
  b ^= (b & 0x80000000u) ? 0xFFFFFFFFu : 0x80000000u;  // ascending order of floats
  return (static_cast<uint64_t>(~b) << 32) | static_cast<uint32_t>(box);
}

// The chunk's detections into bin order (the order inside a bin does not matter: the
// ranking key is a total order).
__global__ __launch_bounds__(kBinThreads) void scatter_kernel(const MergeParams P) {
  __shared__ int s_all[kBinThreads], s_before[kBinThreads], s_start[kBinsMax];
  __shared__ int s_wave[kBinThreads / 64];
  const int tid = threadIdx.x, g = blockIdx.x;
  // column sums of the table: `parts` threads per bin
  int width = 1;
  while (width < P.n_bins) width *= 2;
  const int b = tid & (width - 1), parts = kBinThreads / width;
  int all = 0, before = 0;
  if (b < P.n_bins) {
#pragma unroll 8
    for (int r = tid / width; r < P.n_chunks; r += parts) {
      const int v = P.table[static_cast<int64_t>(r) * P.n_bins + b];
      all += v;
      before += r < g ? v : 0;
    }
  }
  for (int o = 32; o >= width; o >>= 1) {  // the lanes of a wave on one bin
    all += __shfl_xor(all, o);
    before += __shfl_xor(before, o);
  }
  s_all[tid] = all;
  s_before[tid] = before;
  __syncthreads();
  all = before = 0;
  if (tid < width) {
    for (int k = tid; k < kBinThreads; k += max(width, 64)) {
      all += s_all[k];
      before += s_before[k];
    }
  }
  int total;
  const int begin = block_exclusive<kBinThreads>(all, s_wave, &total);
  if (tid < P.n_bins) {
    s_start[tid] = begin + before;
    if (g == 0) P.bin_begin[tid] = begin;
  }
  if (g == 0 && tid == 0) P.bin_begin[P.n_bins] = total;
  __syncthreads();
  const int64_t lo = static_cast<int64_t>(g) * P.chunk;
  const int64_t hi = min(lo + P.chunk, static_cast<int64_t>(count_of(P)));
  for (int64_t i = lo + tid; i < hi; i += kBinThreads) {
    const tg_det d = P.dets[i];
    if (d.frame < 0 || d.frame >= P.n_frames) continue;
    const float s = (d.box >= 0 && d.box < P.n_scores) ? P.scores[d.box] : __builtin_nanf("");
    const int pos = atomicAdd(&s_start[bin_of(P, d.frame)], 1);
    P.crec[pos] = Rec{make_float4(d.x1, d.y1, d.x2, d.y2),
                      Aux{rank_key(s, d.box), d.roi, static_cast<int32_t>(i)}};
  }
}

// Area of a box (x1, y1, x2, y2 in .x .y .z .w), empty and inverted boxes 0.
__device__ __forceinline__ float box_area(float4 a) {
  return __fmul_rn(fmaxf(0.0f, __fsub_rn(a.z, a.x)), fmaxf(0.0f, __fsub_rn(a.w, a.y)));
}

// Whether boxes a and b, of areas area_a and area_b, overlap by more than thr of their
// union. The result does not depend on the order of a and b: the minima and maxima, the
// product and the sum are commutative, NaN operands included, and a difference of zeros
// differs in sign only, which no comparison sees.
__device__ __forceinline__ bool overlap_above(float4 a, float4 b, float area_a, float area_b,
                                              float thr) {
  const float w = fmaxf(0.0f, __fsub_rn(fminf(a.z, b.z), fmaxf(a.x, b.x)));
  const float h = fmaxf(0.0f, __fsub_rn(fminf(a.w, b.w), fmaxf(a.y, b.y)));
  const float inter = __fmul_rn(w, h);
  const float uni = __fsub_rn(__fadd_rn(area_a, area_b), inter);
  return inter > __fmul_rn(thr, uni);
}

// ---- frames decided by one workgroup in LDS --------------------------------------------
//
// Why the bands find every suppressor: with a threshold t >= 0, a suppresses b only if
// inter > t * union >= 0 (a union is never negative), so inter > 0 and both clipped widths
// are positive: min(x2a, x2b) > max(x1a, x1b) and likewise in y. The point
// (max(x1a, x1b), max(y1a, y1b)) then lies in both boxes, and since band_of is
// non-decreasing its column and row are among those of both. Boxes with a NaN coordinate
// (where min and max ignore the NaN operand), and every box when t < 0, are named in every
// band and look in every band. Boxes with x2 < x1 or y2 < y1 have no positive width with
// anything, so when t >= 0 they neither suppress nor are suppressed.
constexpr int kLocalBands = 32;  // per axis

// Up to kLocal boxes by band: per axis and band, the boxes that start at or before the band
// and those that end at or after it; the boxes meeting bands a .. b start at or before b
// and end at or after a.
struct BandTable {
  uint32_t starts[2][kLocalBands][kLocalWords + 1], ends[2][kLocalBands][kLocalWords + 1];
  float ext[4][kLocal / 64];
};

// The bands a box is named in and looks in: columns x0 .. x1, rows y0 .. y1.
struct BandSpan {
  int x0, x1, y0, y1;
  bool named;  // false: a box that meets nothing
};

__device__ __forceinline__ bool nan_corner(float4 b) {
  return b.x != b.x || b.y != b.y || b.z != b.z || b.w != b.w;
}

// `each`: boxes that do not meet count as well (a negative threshold).
__device__ __forceinline__ BandSpan span_of(float4 box, bool each, BandAxis ax, BandAxis ay) {
  BandSpan v = {0, kLocalBands - 1, 0, kLocalBands - 1, true};
  if (!each && !nan_corner(box)) {
    v.named = box.x <= box.z && box.y <= box.w;
    v.x0 = band_of(box.x, ax, kLocalBands);
    v.x1 = band_of(box.z, ax, kLocalBands);
    v.y0 = band_of(box.y, ay, kLocalBands);
    v.y1 = band_of(box.w, ay, kLocalBands);
  }
  return v;
}

// Builds the table of n <= kLocal boxes, box i held by thread i of a workgroup of kLocal
// (i >= n: any), and the axes. Ends with a barrier.
__device__ __forceinline__ void build_table(BandTable &T, float4 box, int n, bool each,
                                            BandAxis &ax, BandAxis &ay) {
  const int i = threadIdx.x, lane = i & 63, wave = i >> 6;
  const float inf = __builtin_inff();
  const bool plain = i < n && !nan_corner(box) && box.x <= box.z && box.y <= box.w;
  const float e0 = wave_min(plain && __builtin_isfinite(box.x) ? box.x : inf);
  const float e1 = wave_min(plain && __builtin_isfinite(box.y) ? box.y : inf);
  const float e2 = wave_min(plain && __builtin_isfinite(box.z) ? -box.z : inf);
  const float e3 = wave_min(plain && __builtin_isfinite(box.w) ? -box.w : inf);
  if (lane == 0) {
    T.ext[0][wave] = e0;
    T.ext[1][wave] = e1;
    T.ext[2][wave] = e2;
    T.ext[3][wave] = e3;
  }
  __syncthreads();
  // lane l of each row of 16 lanes reads wave l's extent: the waves' minima by DPP
  const int w16 = lane & (kLocal / 64 - 1);
  ax = band_axis(wave_min(T.ext[0][w16]), -wave_min(T.ext[2][w16]), kLocalBands);
  ay = band_axis(wave_min(T.ext[1][w16]), -wave_min(T.ext[3][w16]), kLocalBands);
  const int word = 2 * wave + (lane >> 5);
  if (64 * wave < n) {  // later words are not looked in
    const BandSpan v = span_of(box, each, ax, ay);
    const bool named = v.named && i < n;
    T.starts[0][lane & 31][word] = transpose32(named ? 0xFFFFFFFFu << v.x0 : 0u, lane);
    T.starts[1][lane & 31][word] = transpose32(named ? 0xFFFFFFFFu << v.y0 : 0u, lane);
    T.ends[0][lane & 31][word] = transpose32(named ? 0xFFFFFFFFu >> (31 - v.x1) : 0u, lane);
    T.ends[1][lane & 31][word] = transpose32(named ? 0xFFFFFFFFu >> (31 - v.y1) : 0u, lane);
  }
  __syncthreads();
}

// Boxes 32 w .. 32 w + 31 that share a column and a row with span v.
__device__ __forceinline__ uint32_t table_word(const BandTable &T, const BandSpan &v, int w) {
  return T.starts[0][v.x1][w] & T.ends[0][v.x0][w] & T.starts[1][v.y1][w] & T.ends[1][v.y0][w];
}

struct LocalLds {
  float4 box[kLocal];
  Aux aux[kLocal];
  uint16_t first[kLocal], end[kLocal];  // the positions of the detection's frame
  BandTable table;
  uint32_t pair[kPairs];  // position << 16 | a later position
  uint32_t hit[kHits];    // suppressed << 16 | suppressor; or suppressor rows (decide_rows)
  uint32_t kept[kLocalWords], open[kLocalWords];  // decide_rows: positions in that state
  uint8_t state[kLocal];
  uint8_t sees_kept[kLocal], sees_open[kLocal];  // this round, among its suppressors
  float ext[4][kLocal / 64];
  int n_pairs, n_hits, words;
};

// The words of 32 positions that hold o's frame.
__device__ __forceinline__ int frame_words(const LocalLds &S, int o) {
  return ((S.end[o] - 1) >> 5) - (S.first[o] >> 5) + 1;
}

// One pair of positions tested: listed as a hit when one suppresses the other.
__device__ __forceinline__ void test_pair(const MergeParams &P, LocalLds &S, int i, int j) {
  const float4 a = S.box[i], b = S.box[j];
  const Aux x = S.aux[i], y = S.aux[j];
  if (overlap_above(a, b, box_area(a), box_area(b), P.thr) && x.key != y.key &&
      !(P.cross_only && x.roi == y.roi)) {
    const int h = lane_place(&S.n_hits);
    if (h < kHits) S.hit[h] = x.key < y.key ? static_cast<uint32_t>(j) << 16 | static_cast<uint32_t>(i)
                                      : static_cast<uint32_t>(i) << 16 | static_cast<uint32_t>(j);
  }
}

// The bits of positions lo .. hi in the word of positions 32 w .. 32 w + 31.
__device__ __forceinline__ uint32_t range_bits(int w, int lo, int hi) {
  lo = max(lo - 32 * w, 0);
  hi = min(hi - 32 * w, 31);
  return lo <= hi ? (0xFFFFFFFFu << lo) & (0xFFFFFFFFu >> (31 - hi)) : 0u;
}

// Decides the detections at positions [a, b) of S, whole frames, whatever their suppressing
// pairs: each has a row of `stride` words (odd: rows in distinct banks) in which its
// suppressors' bits are set, from the word of its frame's first position on; the rounds test
// the rows against the kept and the undecided. Each pair is tested once: a detection takes
// those of the half of its frame that follows it, cyclically, so that the lanes of a wave have
// equally many (all later ones: 95 us instead of 84 below). The table of all boxes is built.
// Called after a barrier; ends without one.
// Pairs listed one by one overrun any list where boxes crowd, and frames sent to the tile pass
// instead wait there for few workgroups: 1,920 frames of 100 detections, a frame's all in one
// spot (4,700 pairs each), took 681 us so and take 84, around eight objects a frame 368 and 58;
// 256 frames of 250 in one spot 379 and 64.
__device__ void decide_rows(const MergeParams &P, LocalLds &S, int a, int b, int stride, bool each,
                            BandAxis ax, BandAxis ay) {
  const int i = threadIdx.x, lane = i & 63, wave = i >> 6, m = b - a;
  for (int k = i; k < m * stride; k += kLocal) S.hit[k] = 0;
  __syncthreads();
  int width = 64;
  while (width < m) width *= 2;
  const int o = a + (i & (width - 1)), part = i / width, parts = kLocal / width;
  if (o < b) {
    const float4 box = S.box[o];
    const Aux aux = S.aux[o];
    const float area = box_area(box);
    const BandSpan v = span_of(box, each, ax, ay);
    const int first = S.first[o], n = S.end[o] - first, w0 = first >> 5;
    const int last = o + (n % 2 == 0 && o - first < n / 2 ? n / 2 : (n - 1) / 2);
    for (int w = v.named ? w0 + part : kLocalWords; w < w0 + frame_words(S, o); w += parts) {
      uint32_t bits = table_word(S.table, v, w) & (range_bits(w, o + 1, min(last, first + n - 1)) |
                                                   range_bits(w, first, last - n));
      uint32_t own = 0;
      while (bits != 0) {  // two candidates' loads together
        const int k0 = __builtin_ctz(bits);
        bits &= bits - 1;
        const int k1 = bits ? __builtin_ctz(bits) : k0;
        bits &= bits - 1;
        const int j0 = 32 * w + k0, j1 = 32 * w + k1;
        const float4 q0 = S.box[j0], q1 = S.box[j1];
        const Aux y0 = S.aux[j0], y1 = S.aux[j1];
        auto test = [&](int k, float4 q, const Aux &y) {
          if (!overlap_above(box, q, area, box_area(q), P.thr) || y.key == aux.key ||
              (P.cross_only && y.roi == aux.roi))
            return;
          if (y.key < aux.key)
            own |= 1u << k;
          else
            atomicOr(&S.hit[(32 * w + k - a) * stride + (o >> 5) - w0], 1u << (o & 31));
        };
        test(k0, q0, y0);
        test(k1, q1, y1);  // the same one again changes nothing
      }
      if (own != 0) atomicOr(&S.hit[(o - a) * stride + w - w0], own);
    }
  }
  __syncthreads();
  const bool mine = i >= a && i < b;
  int st = mine ? kUndecided : kSuppressed;
  const int w0 = mine ? S.first[i] >> 5 : 0, words = mine ? frame_words(S, i) : 0;
  const uint32_t *row = S.hit + (mine ? (i - a) * stride : 0);
  for (int round = 0;; ++round) {
    const uint64_t kept = __ballot(st == kKept), open = __ballot(st == kUndecided);
    if (lane == 0) {
      S.kept[2 * wave] = static_cast<uint32_t>(kept);
      S.kept[2 * wave + 1] = static_cast<uint32_t>(kept >> 32);
      S.open[2 * wave] = static_cast<uint32_t>(open);
      S.open[2 * wave + 1] = static_cast<uint32_t>(open >> 32);
    }
    if (!__syncthreads_or(st == kUndecided)) break;
    if (round > m) {  // each round decides a frame's best-ranked undecided detection
      if (i == 0) *P.status = 1;
      break;
    }
    if (st == kUndecided) {
      uint32_t any_kept = 0, any_open = 0;
      for (int w = 0; w < words; ++w) {
        const uint32_t r = row[w];
        any_kept |= r & S.kept[w0 + w];
        any_open |= r & S.open[w0 + w];
      }
      st = any_kept ? kSuppressed : (any_open ? kUndecided : kKept);
    }
    __syncthreads();  // every row has been tested before the masks are rewritten
  }
  if (mine) P.keep[S.aux[i].idx] = st == kKept ? 1 : 0;
}

__device__ __forceinline__ int cell_of(float v, float origin, float scale, int g) {
  return static_cast<int>(
      fminf(fmaxf(__fmul_rn(__fsub_rn(v, origin), scale), 0.0f), static_cast<float>(g - 1)));
}

// The box that thread i of kLocal samples of the frame at positions [lo, lo + n).
__device__ __forceinline__ float4 sample_of(const MergeParams &P, int lo, int n, int i) {
  const uint64_t at = static_cast<uint64_t>(i) * static_cast<uint32_t>(n) / kLocal;
  return P.rec[lo + static_cast<int>(at)].box;
}

// Lists a frame for the tile and resolve passes, to be cut into g x g tiles. Called by the
// whole workgroup, after its boxes are in the workspace.
// A tile is one workgroup's work, so its share of the detections decides the pass's time. An
// even grid over the frame serves detections that are spread out (its tiles are then as
// alike as they come); where kLocal samples, whose extent the grid takes, show a cell with more
// than twice its share, the cuts go where the samples say (uneven_rect). (20,000 detections, half
// of them in 300 x 300 of 3840 x 2160 pixels: 13.8 ms over an even grid, 0.84 so; with one box a
// million pixels away 7.8 ms and 0.15; spread out 0.108 either way. Reading all boxes of a frame
// for its extent, and the samples among them, took 1.2 us more for eight frames of 6,000.)
__device__ void add_large(const MergeParams &P, LocalLds &S, int lo, int n) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float inf = __builtin_inff();
  // every tile reads the whole frame, so there are at most about kTilesMax of them
  const int per_tile = min(max(count_of(P) / (4 * kGridCap), kTileDets), kTileDetsMax);
  const float tiles = fminf(n * __builtin_amdgcn_rcpf(per_tile), static_cast<float>(kTilesMax));
  const int g = min(max(1, static_cast<int>(ceilf(__builtin_amdgcn_sqrtf(tiles)))), kTilesPerAxis);
  unsigned long long old = 0;  // (asked for here, waited for at the end)
  if (tid == 0)
    old = atomicAdd(P.large_used, (1ull << 32) | static_cast<unsigned long long>(g) * g);
  const float4 sample = sample_of(P, lo, n, tid);
  const bool fx = __builtin_isfinite(sample.x), fy = __builtin_isfinite(sample.y);
  float e[4] = {fx ? sample.x : inf, fy ? sample.y : inf, fx ? -sample.x : inf,
                fy ? -sample.y : inf};
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    e[k] = wave_min(e[k]);
    if (lane == 0) S.ext[k][wave] = e[k];
  }
  if (tid < g * g) S.hit[tid] = 0;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 4; ++k) e[k] = wave_min(S.ext[k][lane & (kLocal / 64 - 1)]);
  const float share = __builtin_amdgcn_rcpf(g);
  const float dx = (-e[2] - e[0]) * share, dy = (-e[3] - e[1]) * share;
  const int cell = cell_of(sample.y, e[1], __builtin_amdgcn_rcpf(dy), g) * g +
                   cell_of(sample.x, e[0], __builtin_amdgcn_rcpf(dx), g);
  const int before = atomicAdd(&S.hit[cell], 1);
  const bool even = !__syncthreads_or(before * g * g >= 2 * kLocal + 12 * g * g) &&
                    __builtin_isfinite(dx) && __builtin_isfinite(dy);
  if (tid == 0)
    P.large[old >> 32] =
        LargeFrame{lo, n, even ? g : -g, static_cast<uint32_t>(old), e[0], e[1], dx, dy, 0};
  __syncthreads();
}

// The detections at positions [a, b) of S, one frame, written to the workspace (at lo + a on)
// and listed.
__device__ void list_frame(const MergeParams &P, LocalLds &S, int lo, int a, int b) {
  const int tid = threadIdx.x;
  if (tid >= a && tid < b) P.rec[lo + tid] = Rec{S.box[tid], S.aux[tid]};
  __threadfence_block();
  __syncthreads();
  add_large(P, S, lo + a, b - a);
}

// Decides n <= kLocal detections, each frame's at consecutive positions of S, by a workgroup
// of kLocal threads, and writes their keep flags; a frame that alone is too crowded for the
// rows of decide_rows is listed for the tile and resolve passes (its positions in the
// workspace start at lo). Called after a barrier; ends without one.
// Testing only the pairs that bands bring together is what makes whole frames affordable
// here (a frame of 400 boxes of cam20_4k has 80,000 pairs, of which about 2,000 share bands),
// and listing them spreads the tests evenly: lanes that each step through their own
// candidates wait for the one in the most crowded place (9 us of 24, frames of 400; the whole
// pass takes 12 now). Code that runs once costs its instruction fetches, so loops stay loops.
__device__ void decide(const MergeParams &P, LocalLds &S, int lo, int n) {
  const int i = threadIdx.x;
  const bool mine = i < n, each = !(P.thr >= 0.0f);
  if (i == 0) S.n_pairs = S.n_hits = S.words = 0;
  S.state[i] = kKept;
  S.sees_kept[i] = S.sees_open[i] = 0;
  BandAxis ax, ay;
  build_table(S.table, S.box[i], n, each, ax, ay);
  // Each detection's pairs with later ones of its frame, in the words from its own on: `width`
  // threads take a detection each, `parts` of them share its words.
  int width = 64;
  while (width < n) width *= 2;
  const int o = i & (width - 1), part = i / width, parts = kLocal / width;
  BandSpan v = {0, 0, 0, 0, false};
  int w0 = 0, w1 = -1;
  if (o < n) v = span_of(S.box[o], each, ax, ay);
  if (v.named) {
    w0 = o >> 5;
    w1 = (S.end[o] - 1) >> 5;
  }
  const uint32_t tail = 0xFFFFFFFFu >> (31 - ((w1 >= 0 ? S.end[o] - 1 : 0) & 31));
  auto word_of = [&](int w) {
    uint32_t m = table_word(S.table, v, w);
    if (w == w0) m &= 0xFFFFFFFEu << (o & 31);
    return w == w1 ? m & tail : m;
  };
  int count = 0;
#pragma unroll 2
  for (int w = w0 + part; w <= w1; w += parts) count += __popc(word_of(w));
  int at = wave_places(&S.n_pairs, count);
  for (int w = w0 + part; w <= w1; w += parts)
    for (uint32_t m = word_of(w); m != 0 && at < kPairs; m &= m - 1)
      S.pair[at++] = static_cast<uint32_t>(o) << 16 | static_cast<uint32_t>(32 * w + __builtin_ctz(m));
  __syncthreads();
  const int n_pairs = S.n_pairs;
  if (n_pairs <= kPairs) {
    for (int p = i; p < n_pairs; p += kLocal) test_pair(P, S, S.pair[p] >> 16, S.pair[p] & 0xFFFFu);
  } else {  // crowded
    if (mine) atomicMax(&S.words, frame_words(S, i));
    __syncthreads();
    const int stride = S.words | 1;
    if (n * stride <= kHits) {
      decide_rows(P, S, 0, n, stride, each, ax, ay);
      return;
    }
    for (int w = w0 + part; w <= w1; w += parts)
      for (uint32_t m = word_of(w); m != 0; m &= m - 1) test_pair(P, S, o, 32 * w + __builtin_ctz(m));
  }
  __syncthreads();
  const int n_hits = S.n_hits;
  if (n_hits > kHits) {  // frame by frame
    for (int a = 0; a < n;) {  // uniform
      const int b = S.end[a], stride = frame_words(S, a) | 1;
      if ((b - a) * stride <= kHits)
        decide_rows(P, S, a, b, stride, each, ax, ay);
      else
        list_frame(P, S, lo, a, b);
      __syncthreads();
      a = b;
    }
    return;
  }
  for (int h = i; h < n_hits; h += kLocal) S.state[S.hit[h] >> 16] = kUndecided;
  bool overrun = false;
  if (n_hits > 0) {
    __syncthreads();
    for (int round = 0;; ++round) {
      for (int h = i; h < n_hits; h += kLocal) {
        const uint32_t v = S.hit[h];
        const int s = S.state[v & 0xFFFFu];
        if (s == kKept) S.sees_kept[v >> 16] = 1;
        if (s == kUndecided) S.sees_open[v >> 16] = 1;
      }
      __syncthreads();
      bool open = false;
      if (mine && S.state[i] == kUndecided) {
        if (S.sees_kept[i])
          S.state[i] = kSuppressed;
        else if (!S.sees_open[i])
          S.state[i] = kKept;
        else
          open = true;
        S.sees_open[i] = 0;
      }
      if (!__syncthreads_or(open)) break;
      if (round > n) {  // each round decides a frame's best-ranked undecided detection
        overrun = true;
        break;
      }
    }
  }
  if (mine) P.keep[S.aux[i].idx] = S.state[i] == kKept ? 1 : 0;
  if (overrun && i == 0) *P.status = 1;
}

// In-place exclusive scan of hist[0 .. nf) with hist[nf] = the sum, by the workgroup.
__device__ void scan_hist(int *hist, int nf, int *s_wave) {
  const int per = (nf + kLocal - 1) / kLocal, a = min(static_cast<int>(threadIdx.x) * per, nf);
  const int b = min(a + per, nf);
  int sum = 0, total;
  for (int k = a; k < b; ++k) sum += hist[k];
  int at = block_exclusive<kLocal>(sum, s_wave, &total);
  for (int k = a; k < b; ++k) {
    const int v = hist[k];
    hist[k] = at;
    at += v;
  }
  if (threadIdx.x == 0) hist[nf] = total;
  __syncthreads();
}

__global__ __launch_bounds__(kLocal) void local_kernel(const MergeParams P) {
  __shared__ LocalLds S;
  __shared__ int hist[kFrameHist + 1];
  __shared__ int s_wave[kLocal / 64];
  static_assert(kLocal == 1024, "sixteen waves: one per lane of a DPP row");
  const int tid = threadIdx.x;
  const int lo = P.bin_begin[blockIdx.x], n = P.bin_begin[blockIdx.x + 1] - lo;
  if (n <= 0) return;
  if (P.per_bin == 1) {
    if (n > kLocal) {
      add_large(P, S, lo, n);
      return;
    }
    if (tid < n) {
      const Rec r = P.rec[lo + tid];
      S.box[tid] = r.box;
      S.aux[tid] = r.aux;
      S.first[tid] = 0;
      S.end[tid] = static_cast<uint16_t>(n);
    }
    __syncthreads();
    decide(P, S, lo, n);
    return;
  }
  const int f0 = static_cast<int>(blockIdx.x) * P.per_bin;  // < n_frames
  const int nf_all = min(P.per_bin, P.n_frames - f0);
  if (n <= kLocal && nf_all <= kFrameHist) {  // the whole bin ordered and decided in LDS
    for (int k = tid; k < nf_all; k += kLocal) hist[k] = 0;
    __syncthreads();
    int f = 0, rank = 0, roi = 0, idx = 0;
    float4 box = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    uint64_t key = 0;
    if (tid < n) {
      const Rec *r = P.crec + lo + tid;
      box = r->box;
      key = r->aux.key;
      roi = r->aux.roi;
      idx = r->aux.idx;
      f = P.dets[idx].frame - f0;
      rank = atomicAdd(&hist[f], 1);
    }
    __syncthreads();
    scan_hist(hist, nf_all, s_wave);
    if (tid < n) {
      const int at = hist[f] + rank;
      S.box[at] = box;
      S.aux[at].key = key;
      S.aux[at].roi = roi;
      S.aux[at].idx = idx;
      S.first[at] = static_cast<uint16_t>(hist[f]);
      S.end[at] = static_cast<uint16_t>(hist[f + 1]);
    }
    __syncthreads();
    decide(P, S, lo, n);
    return;
  }
  // A bin that does not fit: ordered by frame in the workspace, kFrameHist frames at a time,
  // then decided in runs of whole frames of at most kLocal detections.
  int base = lo;
  for (int fw = 0; fw < nf_all; fw += kFrameHist) {
    const int nf = min(kFrameHist, nf_all - fw);
    for (int k = tid; k < nf; k += kLocal) hist[k] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += kLocal) {
      const int f = P.dets[P.crec[lo + i].aux.idx].frame - f0 - fw;
      if (f >= 0 && f < nf) atomicAdd(&hist[f], 1);
    }
    __syncthreads();
    scan_hist(hist, nf, s_wave);
    const int total = hist[nf];
    for (int i = tid; i < n; i += kLocal) {
      const Rec r = P.crec[lo + i];
      const int f = P.dets[r.aux.idx].frame - f0 - fw;
      if (f < 0 || f >= nf) continue;
      const int at = base + atomicAdd(&hist[f], 1);  // hist[f] ends as the end of frame f
      P.rec[at] = r;
      P.frame[at] = f;
    }
    __threadfence_block();
    __syncthreads();
    int f = 0, s = 0;  // the next frame and its first position (from base)
    while (f < nf && s < total) {
      int e = f, step = 1;  // the most frames from f on with at most kLocal detections
      while (step <= nf) step *= 2;
      for (; step > 0; step >>= 1)
        if (e + step <= nf && hist[e + step - 1] - s <= kLocal) e += step;
      if (e == f) {
        add_large(P, S, base + s, hist[f] - s);
        s = hist[f++];
        continue;
      }
      const int m = hist[e - 1] - s;
      if (m > 0) {
        if (tid < m) {
          const int at = base + s + tid, fr = P.frame[at];
          const Rec r = P.rec[at];
          S.box[tid] = r.box;
          S.aux[tid] = r.aux;
          S.first[tid] = static_cast<uint16_t>((fr > 0 ? hist[fr - 1] : 0) - s);
          S.end[tid] = static_cast<uint16_t>(hist[fr] - s);
        }
        __syncthreads();
        decide(P, S, base + s, m);
        __syncthreads();
      }
      s = hist[e - 1];
      f = e;
    }
    base += total;
    __syncthreads();
  }
}

// ---- larger frames ----------------------------------------------------------------------

constexpr int kTileRegs = 6;                          // boxes a thread loads at once
constexpr int kTileSpan = kTileRegs * kTileThreads;   // positions read at once: 6,144
constexpr int kTileCand = kTileThreads;               // candidates tested at once

struct TileLds {
  int32_t own[kTileSpan];      // positions of the tile's detections among kTileSpan
  float4 own_box[kTileThreads];// the detections being searched
  Aux own_aux[kTileThreads];
  int32_t count[kTileThreads]; // suppressors found of each
  int32_t at[kTileThreads];    // where their longer lists start in ovf, or -1
  float4 box[kTileCand];       // boxes that can meet them
  Aux aux[kTileCand];
  int32_t pos[kTileCand];
  BandTable table;
  uint32_t pair[kPairs];       // searched << 16 | candidate
  float ext[4][kTileThreads / 64];
  unsigned long long need[kTileThreads / 64], need_base;
  int n_own, n_cand, n_pairs, open_base;
};

// Positions p0 + kTileThreads u + tid of frame L: their boxes, all loads issued together.
__device__ __forceinline__ void load_span(const MergeParams &P, const LargeFrame &L, int p0,
                                          float4 q[kTileRegs]) {
#pragma unroll
  for (int u = 0; u < kTileRegs; ++u) {
    const int p = p0 + u * kTileThreads + static_cast<int>(threadIdx.x);
    q[u] = P.rec[L.lo + min(p, L.n - 1)].box;
  }
}

// Candidate c tested against searched detection o: a suppressor ranked above it goes to its
// place in rpred, or with `fill` to the longer list of a detection with more than
// kPredSlots; both count it.
__device__ __forceinline__ void test_owned(const MergeParams &P, TileLds &S, const int32_t *own,
                                           bool fill, int o, int c) {
  const float4 a = S.own_box[o], b = S.box[c];
  const Aux x = S.own_aux[o], y = S.aux[c];
  if (y.key < x.key && !(P.cross_only && x.roi == y.roi) &&
      overlap_above(b, a, box_area(b), box_area(a), P.thr) && (!fill || S.at[o] >= 0)) {
    const int slot = atomicAdd(&S.count[o], 1);
    if (fill)
      P.ovf[S.at[o] + slot] = S.pos[c];
    else if (slot < kPredSlots)
      P.rpred[kPredSlots * static_cast<int64_t>(own[o]) + slot] = S.pos[c];
  }
}

// The nc collected candidates tested against the m searched detections: the candidates' band
// table names each detection's among them, and those pairs are tested. Called by the whole
// workgroup; ends with a barrier.
__device__ void test_candidates(const MergeParams &P, TileLds &S, const int32_t *own, int m, int nc,
                                bool fill) {
  const int tid = threadIdx.x;
  const bool each = !(P.thr >= 0.0f);
  if (tid == 0) S.n_pairs = 0;
  __syncthreads();
  BandAxis ax, ay;
  build_table(S.table, S.box[tid], nc, each, ax, ay);
  int width = 64;
  while (width < m) width *= 2;
  const int o = tid & (width - 1), part = tid / width, parts = kTileThreads / width;
  BandSpan v = {0, 0, 0, 0, false};
  if (o < m) v = span_of(S.own_box[o], each, ax, ay);
  const int words = v.named ? (nc + 31) / 32 : 0;
  int count = 0;
#pragma unroll 2
  for (int w = part; w < words; w += parts) count += __popc(table_word(S.table, v, w));
  int at = wave_places(&S.n_pairs, count);
  for (int w = part; w < words; w += parts)
    for (uint32_t b = table_word(S.table, v, w); b != 0 && at < kPairs; b &= b - 1)
      S.pair[at++] = static_cast<uint32_t>(o) << 16 | static_cast<uint32_t>(32 * w + __builtin_ctz(b));
  __syncthreads();
  const int n_pairs = S.n_pairs;
  if (n_pairs <= kPairs) {
    for (int k = tid; k < n_pairs; k += kTileThreads)
      test_owned(P, S, own, fill, S.pair[k] >> 16, S.pair[k] & 0xFFFFu);
  } else {  // crowded: each lane its own
    for (int w = part; w < words; w += parts)
      for (uint32_t b = table_word(S.table, v, w); b != 0; b &= b - 1)
        test_owned(P, S, own, fill, o, 32 * w + __builtin_ctz(b));
  }
  __syncthreads();
}

// The suppressors ranked above each of m <= kTileThreads detections (positions own[]) of
// frame L, among the frame's boxes that can meet the rectangle around the m boxes. The point
// that two overlapping boxes share (see above) lies in the one and so in the rectangle, hence
// the comparisons; they let NaN corners through, and a NaN corner among the m, or a negative
// threshold, lets every box through. (Every detection against every candidate: 10-28 us a tile
// of 250 by 270.)
__device__ void search_owned(const MergeParams &P, TileLds &S, const LargeFrame &L,
                             const int32_t *own, int m, bool fill) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const float inf = __builtin_inff();
  const bool each = !(P.thr >= 0.0f);
  Rec r;
  if (tid < m) {
    r = P.rec[own[tid]];
    S.own_box[tid] = r.box;
    S.own_aux[tid] = r.aux;
    S.count[tid] = 0;
  }
  const float e0 = wave_min(tid < m ? r.box.x : inf), e1 = wave_min(tid < m ? r.box.y : inf);
  const float e2 = wave_min(tid < m ? -r.box.z : inf), e3 = wave_min(tid < m ? -r.box.w : inf);
  if (lane == 0) {
    S.ext[0][wave] = e0;
    S.ext[1][wave] = e1;
    S.ext[2][wave] = e2;
    S.ext[3][wave] = e3;
  }
  const bool all = __syncthreads_or(tid < m && nan_corner(r.box)) || each;
  const int w16 = lane & (kTileThreads / 64 - 1);
  const float bx0 = wave_min(S.ext[0][w16]), by0 = wave_min(S.ext[1][w16]);
  const float bx1 = -wave_min(S.ext[2][w16]), by1 = -wave_min(S.ext[3][w16]);
  // Candidates are collected until the next ones do not fit, then tested (one call, so that
  // its code is there once): `now` are the span's boxes to be placed next -- all that can
  // meet, or, when those alone are too many, one of each thread's at a time.
  int nc = 0, p0 = 0, u0 = -1;
  while (p0 < L.n || nc > 0) {
    bool full = p0 >= L.n;  // nothing more to collect
    if (!full) {
      float4 q[kTileRegs];
      load_span(P, L, p0, q);
      uint32_t now = 0;
#pragma unroll
      for (int u = 0; u < kTileRegs; ++u) {
        const bool in = p0 + u * kTileThreads + tid < L.n;
        const bool meets = all || !(q[u].x >= bx1 || q[u].z <= bx0 || q[u].y >= by1 || q[u].w <= by0);
        now |= (in && meets && (u0 < 0 || u == u0) ? 1u : 0u) << u;
      }
      if (tid == 0) S.n_cand = nc;
      __syncthreads();
      int slot = wave_places(&S.n_cand, __popc(now));
      __syncthreads();
      const int total = S.n_cand;
      __syncthreads();  // read by everyone before it is set again
      full = total > kTileCand;
      if (!full) {
        for (; now != 0; now &= now - 1, ++slot) {
          const int at = L.lo + p0 + __builtin_ctz(now) * kTileThreads + tid;
          const Rec x = P.rec[at];
          S.box[slot] = x.box;
          S.aux[slot] = x.aux;
          S.pos[slot] = at;
        }
        nc = total;
        if (u0 < 0 || ++u0 == kTileRegs) {
          p0 += kTileSpan;
          u0 = -1;
        }
      } else if (nc == 0) {
        u0 = 0;
      }
    }
    if (full && nc > 0) {
      test_candidates(P, S, own, m, nc, fill);
      nc = 0;
    }
  }
}

// The detections own[0 .. m) of frame L (entry k): their suppressors, then kept at once when
// there are none, else onto the frame's open list.
__device__ void search_part(const MergeParams &P, TileLds &S, const LargeFrame &L, int k,
                            const int32_t *own, int m) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int np = 0;
  for (int fill = 0;; ++fill) {
    search_owned(P, S, L, own, m, fill != 0);
    if (fill) break;
    np = tid < m ? S.count[tid] : 0;
    __syncthreads();
    if (tid < m) S.at[tid] = -1;
    if (!__syncthreads_or(np > kPredSlots)) break;
    // room for the longer lists, one atomic for all: this thread's place by a scan (64 bits,
    // as the lists of a very large frame may overrun the area by far)
    const unsigned long long need = np > kPredSlots ? np : 0;
    unsigned long long incl = need;
    for (int d = 1; d < 64; d <<= 1) {
      const unsigned long long t = __shfl_up(incl, d);
      if (lane >= d) incl += t;
    }
    if (lane == 63) S.need[wave] = incl;
    __syncthreads();
    if (tid == 0) {
      unsigned long long sum = 0;
      for (int w = 0; w < kTileThreads / 64; ++w) {
        const unsigned long long v = S.need[w];
        S.need[w] = sum;
        sum += v;
      }
      S.need_base = atomicAdd(P.ovf_used, sum);
    }
    __syncthreads();
    const unsigned long long at = S.need_base + S.need[wave] + incl - need;
    if (need > 0 && at + need <= static_cast<unsigned long long>(P.ovf_cap))
      S.at[tid] = static_cast<int>(at);
    __syncthreads();
  }
  if (tid == 0) S.n_cand = 0;
  __syncthreads();
  const int slot = wave_places(&S.n_cand, np > 0 ? 1 : 0);
  if (tid < m) {
    const int a = own[tid];
    P.rstate[a] = np > 0 ? kUndecided : kKept;
    if (np > 0) {
      P.rnpred[a] = np;
      P.rovf[a] = S.at[tid];
    } else {
      P.keep[P.rec[a].aux.idx] = 1;
    }
  }
  __syncthreads();
  if (tid == 0 && S.n_cand > 0) S.open_base = atomicAdd(&P.large[k].open, S.n_cand);
  __syncthreads();
  if (np > 0) P.open[L.lo + S.open_base + slot] = own[tid];
  __syncthreads();
}

// Floats as integers in the same order, NaN as -infinity; and back.
__device__ __forceinline__ uint32_t order_of(float v) {
  const uint32_t b = __float_as_uint(fmaxf(v, -__builtin_inff()));
  return b ^ ((b & 0x80000000u) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ float value_of(uint32_t o) {
  return __uint_as_float(o ^ ((o & 0x80000000u) ? 0x80000000u : 0xFFFFFFFFu));
}

// Sorts key[0 .. kLocal) upwards (bitonic), one element per thread. Called after a barrier,
// ends with one.
__device__ __forceinline__ void sort_keys(uint64_t *key) {
  const int i = threadIdx.x;
  for (int size = 2; size <= kLocal; size *= 2)
    for (int d = size / 2; d > 0; d /= 2) {
      const uint64_t a = key[i], b = key[i ^ d];
      const bool low = ((i & d) == 0) == ((i & size) == 0);  // this place takes the smaller
      __syncthreads();
      key[i] = (a < b) == low ? a : b;
      __syncthreads();
    }
}

// The rectangle of tile (tx, ty) of a frame whose tiles go by its samples: g columns of equally
// many samples, each cut into g rows of equally many. Called by the whole workgroup, ends with a
// barrier. (A tile computes its own rectangle, with the same cuts as its neighbours. With this
// in the pass that lists the frames, that pass was up to 1.5 us slower for all frames: its code
// no longer fitted its registers.)
__device__ TileRect uneven_rect(const MergeParams &P, TileLds &S, const LargeFrame &L, int tx,
                                int ty) {
  static_assert(kTileThreads == kLocal && sizeof(S.own) >= 12 * kLocal, "samples in own");
  const int tid = threadIdx.x, g = -L.g;
  uint64_t *key = reinterpret_cast<uint64_t *>(S.own);
  uint32_t *y_order = reinterpret_cast<uint32_t *>(key + kLocal);
  // the first of column c's samples (divisions by g, integer ones too, may expand to fused
  // multiply-adds: 1 / g in 16 bits)
  const int inv = static_cast<int>(65536.0f * __builtin_amdgcn_rcpf(g));
  auto first_of = [&](int c) { return c < g ? c * inv * kLocal >> 16 : kLocal; };
  const int a = first_of(tx), b = first_of(tx + 1);
  // (samples of one x in scrambled order, so that a column that takes part of them takes a fair
  // part)
  constexpr uint32_t kScramble = 0x9E3779B1u, kInverse = 0x0E8B2F51u;  // product 1 mod 2^32
  const float4 sample = sample_of(P, L.lo, L.n, tid);
  TileRect R = {-__builtin_inff(), -__builtin_inff(), __builtin_nanf(""), __builtin_nanf("")};
  y_order[tid] = order_of(sample.y);
  key[tid] = static_cast<uint64_t>(order_of(sample.x)) << 32 | tid * kScramble;
  __syncthreads();
  for (int axis = 0;; ++axis) {
    sort_keys(key);
    if (axis == 1) break;
    if (tx > 0) R.x0 = value_of(static_cast<uint32_t>(key[a] >> 32));
    if (tx < g - 1) R.x1 = value_of(static_cast<uint32_t>(key[b] >> 32));
    const uint32_t y = y_order[static_cast<uint32_t>(key[tid]) * kInverse];
    __syncthreads();
    key[tid] = tid >= a && tid < b ? y : ~uint64_t(0);  // the column's first
    __syncthreads();
  }
  if (ty > 0) R.y0 = value_of(static_cast<uint32_t>(key[(b - a) * ty * inv >> 16]));
  if (ty < g - 1) R.y1 = value_of(static_cast<uint32_t>(key[(b - a) * (ty + 1) * inv >> 16]));
  __syncthreads();
  return R;
}

__global__ __launch_bounds__(kTileThreads) void tile_kernel(const MergeParams P) {
  __shared__ TileLds S;
  const unsigned long long used = *P.large_used;
  const int n_large = static_cast<int>(used >> 32);
  const uint32_t n_tiles = static_cast<uint32_t>(used);
  const int tid = threadIdx.x, lane = tid & 63;
  const float inf = __builtin_inff();
  for (uint32_t v = blockIdx.x; v < n_tiles; v += gridDim.x) {
    int k = -1;  // the tile's frame: the last one whose tiles start at or before v
    for (int b = 0; b < n_large; b += 64) {
      const int hits = __popcll(__ballot(b + lane < n_large && P.large[b + lane].start <= v));
      k += hits;
      if (hits < 64) break;
    }
    const LargeFrame L = P.large[k];
    const int g = abs(L.g), t = static_cast<int>(v - L.start), ty = t / g, tx = t - ty * g;
    TileRect R = {-inf, -inf, __builtin_nanf(""), __builtin_nanf("")};
    if (L.g < 0) {
      R = uneven_rect(P, S, L, tx, ty);
    } else {
      if (tx > 0) R.x0 = L.x0 + tx * L.dx;
      if (ty > 0) R.y0 = L.y0 + ty * L.dy;
      if (tx < g - 1) R.x1 = L.x0 + (tx + 1) * L.dx;
      if (ty < g - 1) R.y1 = L.y0 + (ty + 1) * L.dy;
    }
    int n_own = 0, p0 = 0;  // collected until the next ones do not fit, then searched
    while (p0 < L.n || n_own > 0) {
      bool full = p0 >= L.n;
      if (!full) {
        float4 q[kTileRegs];
        load_span(P, L, p0, q);
        uint32_t own = 0;
#pragma unroll
        for (int u = 0; u < kTileRegs; ++u) {
          const bool in = p0 + u * kTileThreads + tid < L.n;
          const float x = fmaxf(q[u].x, -inf), y = fmaxf(q[u].y, -inf);
          own |= (in && x >= R.x0 && y >= R.y0 && !(x >= R.x1) && !(y >= R.y1) ? 1u : 0u) << u;
        }
        if (tid == 0) S.n_own = n_own;
        __syncthreads();
        int at = wave_places(&S.n_own, __popc(own));
        __syncthreads();
        const int total = S.n_own;
        __syncthreads();  // read by everyone before it is set again
        full = total > kTileSpan;  // (a span's detections fit alone)
        if (!full) {
          for (; own != 0; own &= own - 1)
            S.own[at++] = L.lo + p0 + __builtin_ctz(own) * kTileThreads + tid;
          n_own = total;
          p0 += kTileSpan;
        }
      }
      if (full) {
        __syncthreads();
        for (int o = 0; o < n_own; o += kTileThreads)
          search_part(P, S, L, k, S.own + o, min(kTileThreads, n_own - o));
        n_own = 0;
      }
    }
    __syncthreads();
  }
}

// This round's decision for an undecided detection a with more suppressors than its
// kPredSlots and no room for them in the overflow area (many boxes crowded on one spot):
// its frame searched again -- kSuppressed when one of its suppressors is kept, kUndecided
// when one is still undecided, else kKept.
__device__ __forceinline__ int32_t decide_searching(const MergeParams &P, const LargeFrame &L, int a) {
  const float4 box = P.rec[a].box;
  const Aux aux = P.rec[a].aux;
  const float area = box_area(box);
  bool pending = false;
  constexpr int kBatch = 8;
  for (int p0 = 0; p0 < L.n; p0 += kBatch) {
    float4 q[kBatch];
    Aux x[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int p = L.lo + min(p0 + u, L.n - 1);
      q[u] = P.rec[p].box;
      x[u] = P.rec[p].aux;
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int p = L.lo + min(p0 + u, L.n - 1);
      if (x[u].key < aux.key && overlap_above(q[u], box, box_area(q[u]), area, P.thr) &&
          !(P.cross_only && x[u].roi == aux.roi)) {
        const int32_t s = P.rstate[p];
        if (s == kKept) return kSuppressed;
        pending |= s == kUndecided;
      }
    }
  }
  return pending ? kUndecided : kKept;
}

// The rounds of each listed frame, then the keep flags of its open detections.
__global__ __launch_bounds__(kResolveThreads) void resolve_kernel(const MergeParams P) {
  const int n_large = static_cast<int>(*P.large_used >> 32);
  const int tid = threadIdx.x;
  for (int k = blockIdx.x; k < n_large; k += gridDim.x) {
    const LargeFrame L = P.large[k];
    for (int round = 0;; ++round) {
      int pending = 0;
      for (int j = tid; j < L.open; j += kResolveThreads) {
        const int a = P.open[L.lo + j];
        if (P.rstate[a] != kUndecided) continue;
        const int np = P.rnpred[a];
        const int32_t *list = P.rpred + kPredSlots * static_cast<int64_t>(a);
        int32_t st = kKept;
        const int at = np > kPredSlots ? P.rovf[a] : 0;
        if (at < 0) {
          st = decide_searching(P, L, a);
        } else {
          if (np > kPredSlots) list = P.ovf + at;
          constexpr int kFirst = 4;  // suppressors whose states are loaded together
          for (int j0 = 0; j0 < np && st != kSuppressed; j0 += kFirst) {
            int32_t s[kFirst];
#pragma unroll
            for (int u = 0; u < kFirst; ++u) s[u] = P.rstate[list[min(j0 + u, np - 1)]];
#pragma unroll
            for (int u = 0; u < kFirst; ++u) {
              if (s[u] == kKept)
                st = kSuppressed;
              else if (s[u] == kUndecided && st != kSuppressed)
                st = kUndecided;
            }
          }
        }
        if (st != kUndecided) {
          P.rstate[a] = st;
          P.keep[P.rec[a].aux.idx] = st == kKept ? 1 : 0;
        } else {
          pending = 1;
        }
      }
      __syncthreads();  // this round's decisions are visible to the next
      if (!__syncthreads_or(pending)) break;
      if (round >= L.n) {  // cannot happen (each round decides one); reported, not spun on
        if (tid == 0) *P.status = 1;
        break;
      }
    }
    __syncthreads();
  }
}

// ---- small inputs: one workgroup, one launch ------------------------------------------
//
// Up to kTiny detections (n_max <= kTiny) are merged by one workgroup: each thread holds
// one detection, its suppressors (ranked above it in the same frame, with cross_only from
// another patch, and suppressing it) are a kTiny-bit row in LDS found by testing each
// pair once, the rounds above run on those rows (suppressed once a suppressor is kept, kept
// once all are suppressed), and a workgroup prefix sum writes the kept detections in input
// order. On inputs this small the launches of the general path, not their work, are the
// cost.
constexpr int kTiny = 512;
constexpr int kTinyWords = kTiny / 32;

// A detection as the pair tests read it: one 32-byte LDS record.
struct alignas(16) TinyDet {
  float4 box;
  uint64_t key;
  int32_t frame, roi;
};

__global__ __launch_bounds__(kTiny) void tiny_kernel(const MergeParams P) {
  __shared__ TinyDet s_det[kTiny];
  __shared__ float s_area[kTiny];
  __shared__ uint32_t s_sup[kTiny][kTinyWords + 1];  // odd row stride: rows in distinct banks
  __shared__ uint32_t s_kept[kTinyWords], s_open[kTinyWords];
  __shared__ int32_t s_wave[kTiny / 64];
  const int i = threadIdx.x, lane = i & 63, wave = i >> 6;
  const int n = count_of(P);
  tg_det d = {0, 0, -1, 0.0f, 0.0f, 0.0f, 0.0f};
  int f = -1;
  uint64_t key = ~uint64_t(0);
  if (i < n) {
    d = P.dets[i];
    if (d.frame >= 0 && d.frame < P.n_frames) f = d.frame;
    const float s = (d.box >= 0 && d.box < P.n_scores) ? P.scores[d.box] : __builtin_nanf("");
    key = rank_key(s, d.box);
  }
  const float4 box = make_float4(d.x1, d.y1, d.x2, d.y2);
  const float area = box_area(box);
  s_det[i] = TinyDet{box, key, f, d.roi};
  s_area[i] = area;
#pragma unroll
  for (int w = 0; w < kTinyWords; ++w) s_sup[i][w] = 0;
  __syncthreads();

  // the suppressor rows, each pair tested once (as in decide_rows: thread i takes the
  // detections 1 .. n/2 places after it, cyclically, four records per step, and the bit goes
  // into the row of whichever of the two is ranked below); a pair with a detection outside the
  // frames sets no bit, so such a thread skips its share
  if (f >= 0) {
    const int last = (n % 2 == 0 && i < n / 2) ? n / 2 : (n - 1) / 2;
    for (int d0 = 1; d0 <= last; d0 += 4) {
      TinyDet q[4];
      float qa[4];
      int qj[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int j = i + min(d0 + u, last);  // < 2n
        qj[u] = j >= n ? j - n : j;
        q[u] = s_det[qj[u]];
        qa[u] = s_area[qj[u]];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        if (d0 + u <= last && q[u].frame == f && !(P.cross_only && q[u].roi == d.roi) &&
            overlap_above(q[u].box, box, qa[u], area, P.thr)) {
          const int j = qj[u];
          if (q[u].key < key)
            atomicOr(&s_sup[i][j >> 5], 1u << (j & 31));
          else if (key < q[u].key)
            atomicOr(&s_sup[j][i >> 5], 1u << (i & 31));
        }
      }
    }
  }
  __syncthreads();

  // rounds; a detection outside the frames is dropped (never kept, never a suppressor)
  int st = f >= 0 ? kUndecided : kSuppressed;
  bool overrun = false;
  for (int round = 0;; ++round) {
    const uint64_t kept = __ballot(st == kKept), open = __ballot(st == kUndecided);
    if (lane == 0) {
      s_kept[2 * wave] = static_cast<uint32_t>(kept);
      s_kept[2 * wave + 1] = static_cast<uint32_t>(kept >> 32);
      s_open[2 * wave] = static_cast<uint32_t>(open);
      s_open[2 * wave + 1] = static_cast<uint32_t>(open >> 32);
    }
    if (!__syncthreads_or(st == kUndecided)) break;
    if (round > n) {  // each round decides the best-ranked undecided detection
      overrun = true;
      break;
    }
    if (st == kUndecided) {
      bool any_kept = false, any_open = false;
#pragma unroll
      for (int w = 0; w < kTinyWords; ++w) {
        const uint32_t r = s_sup[i][w];
        any_kept = any_kept || (r & s_kept[w]) != 0;
        any_open = any_open || (r & s_open[w]) != 0;
      }
      st = any_kept ? kSuppressed : (any_open ? kUndecided : kKept);
    }
    __syncthreads();  // every row has been tested before the masks are rewritten
  }

  const int k = i < n && st == kKept ? 1 : 0;
  if (i < n) P.keep[i] = k;
  const int incl = wave_inclusive_sum(k);
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  int before = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kTiny / 64; ++w) {
    if (w < wave) before += s_wave[w];
    total += s_wave[w];
  }
  if (k) P.out[before + incl - 1] = d;
  if (i == 0) *P.n_kept = overrun ? TG_E_INTERNAL : total;
}

// Compaction of up to kCountDets detections: each workgroup counts the kept ones before its
// own by reading their flags, which costs less than a ticket and a look-back over the earlier
// workgroups.
__global__ __launch_bounds__(kCountThreads) void count_compact_kernel(const MergeParams P) {
  typedef int32_t i32x4 __attribute__((ext_vector_type(4), aligned(4)));
  __shared__ int s_before[kCountThreads / 64], s_wave[kCountThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = count_of(P);
  const int i0 = blockIdx.x * kCountThreads, i = i0 + tid;
  const bool kept = i < n && P.keep[i] != 0;
  int before = 0;
  if (i0 < n) {
#pragma unroll 4
    for (int j = 4 * tid; j < i0; j += 4 * kCountThreads) {  // i0 is a multiple of 4
      const i32x4 v = *reinterpret_cast<const i32x4 *>(P.keep + j);
      before += (v.x != 0) + (v.y != 0) + (v.z != 0) + (v.w != 0);
    }
  }
  tg_det d;
  if (kept) d = P.dets[i];
  const uint64_t b = __ballot(kept);
  for (int o = 32; o > 0; o >>= 1) before += __shfl_xor(before, o);
  if (lane == 0) {
    s_before[wave] = before;
    s_wave[wave] = __popcll(b);
  }
  __syncthreads();
  int pos = 0, total = 0;
#pragma unroll
  for (int w = 0; w < kCountThreads / 64; ++w) {
    pos += s_before[w];
    if (w < wave) pos += s_wave[w];
    total += s_before[w] + s_wave[w];
  }
  if (kept) P.out[pos + __popcll(b & ((uint64_t(1) << lane) - 1))] = d;
  // the workgroup with the last detection (the first one when there are none)
  if (tid == 0 && (n > 0 ? i0 < n && n <= i0 + kCountThreads : i0 == 0))
    *P.n_kept = *P.status != 0 ? TG_E_INTERNAL : total;
}

__global__ __launch_bounds__(kThreads) void compact_kernel(const MergeParams P) {
  __shared__ int s_blk, s_prefix;
  __shared__ int s_wave[kThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid == 0)
    s_blk = static_cast<int>(__hip_atomic_fetch_add(P.ticket, 1u, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT));
  __syncthreads();
  const int blk = s_blk;
  const int n = count_of(P);
  const int i0 = blk * kCompactBlock + kPerThread * tid;
  int flag[kPerThread];
  int cnt = 0;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j) {
    flag[j] = i0 + j < n ? P.keep[i0 + j] : 0;
    cnt += flag[j] != 0;
  }
  int incl = cnt;
  for (int o = 1; o < 64; o <<= 1) {
    const int t = __shfl_up(incl, o);
    if (lane >= o) incl += t;
  }
  if (lane == 63) s_wave[wave] = incl;
  __syncthreads();
  int before = 0, total = 0;
  for (int w = 0; w < kThreads / 64; ++w) {
    if (w < wave) before += s_wave[w];
    total += s_wave[w];
  }
  if (wave == 0) {
    bool failed;
    const int prefix = tg_detail::lookback_prefix(P.state, blk, total, &failed);
    if (lane == 0) {
      s_prefix = prefix;
      if (blk == static_cast<int>(gridDim.x) - 1)
        *P.n_kept = failed || __hip_atomic_load(P.status, __ATOMIC_RELAXED,
                                                __HIP_MEMORY_SCOPE_AGENT) != 0
                        ? TG_E_INTERNAL
                        : prefix + total;
    }
  }
  __syncthreads();
  int pos = s_prefix + before + incl - cnt;
#pragma unroll
  for (int j = 0; j < kPerThread; ++j)
    if (flag[j]) P.out[pos++] = P.dets[i0 + j];
}

__global__ void zero_kernel(int32_t *a) { *a = 0; }

int compact_blocks(int32_t n_max) { return (n_max + kCompactBlock - 1) / kCompactBlock; }

size_t round16(size_t v) { return (v + 15) / 16 * 16; }

// Bytes of the workspace: the look-back words and three more, per frame 516 bytes (12 past
// 16,384 frames) and per detection 344. The table of bins takes at most 128 KB of that, the
// passes' arrays 112 bytes per detection (148 with several frames per bin); the rest holds
// suppressor lists of more than kPredSlots.
size_t workspace_bytes(int32_t n_max, int32_t n_frames) {
  const size_t n = static_cast<size_t>(n_max), f = static_cast<size_t>(n_frames);
  const size_t head = sizeof(uint64_t) * (3 + static_cast<size_t>(compact_blocks(n_max))) +
                      8 * f * (n_frames <= 16384 ? 64 : 1) + 4 * (f + 1) + 4 * n;
  return round16(round16(head) + 212 * n) + 128 * n;
}

// Detections per workgroup of hist and scatter.
int32_t chunk_of(int32_t n_max) {
  const int64_t per = (int64_t(n_max) + kChunksMax - 1) / kChunksMax;
  return static_cast<int32_t>((per + kBinThreads - 1) / kBinThreads * kBinThreads);
}

// Lays the arrays out from `ws`; returns the bytes before ovf, which takes the rest.
size_t lay_out(uint8_t *ws, int32_t n_max, MergeParams &P) {
  const size_t n = static_cast<size_t>(n_max);
  size_t at = 0;
  auto take = [&](auto *&p, size_t count) {
    p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(ws + at);
    at = round16(at + sizeof(*p) * count);
  };
  uint64_t *words;
  P.n_words = 3 + compact_blocks(n_max);
  take(words, static_cast<size_t>(P.n_words));
  P.ticket = reinterpret_cast<uint32_t *>(words);
  P.status = P.ticket + 1;
  P.ovf_used = reinterpret_cast<unsigned long long *>(words + 1);
  P.large_used = reinterpret_cast<unsigned long long *>(words + 2);
  P.state = words + 3;
  take(P.table, static_cast<size_t>(P.n_chunks) * P.n_bins);
  take(P.bin_begin, static_cast<size_t>(P.n_bins) + 1);
  // Listed frames have more than 496 detections: fewer fit decide_rows wherever they start.
  take(P.large, n / 496 + 1);
  at = (at + sizeof(Rec) - 1) / sizeof(Rec) * sizeof(Rec);  // (if the workspace is so aligned)
  take(P.rec, n);
  P.crec = P.rec;
  P.frame = nullptr;
  if (P.per_bin > 1) {
    take(P.crec, n);
    take(P.frame, n);
  }
  take(P.rstate, n);
  take(P.rnpred, n);
  take(P.rovf, n);
  take(P.open, n);
  take(P.rpred, kPredSlots * n);
  P.ovf = reinterpret_cast<int32_t *>(ws + at);
  return at;
}

}  // namespace

extern "C" size_t tg_merge_workspace_bytes(int32_t n_max, int32_t n_frames) {
  if (n_max <= 0 || n_frames < 0) return 0;
  return workspace_bytes(n_max, n_frames);
}

extern "C" int tg_merge(const tg_merge_args *a, void *stream) {
  if (!a || a->n_max < 0 || a->n_scores < 0 || a->n_frames < 0 || !a->n_kept ||
      !(a->iou_threshold == a->iou_threshold))
    return TG_E_INVAL;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (a->n_max == 0) {
    hipLaunchKernelGGL(zero_kernel, dim3(1), dim3(1), 0, s, a->n_kept);
    return hipGetLastError() == hipSuccess ? TG_OK : TG_E_HIP;
  }
  if (!a->dets || !a->n_dets || !a->keep || !a->out || (a->n_scores > 0 && !a->scores))
    return TG_E_INVAL;
  if (int64_t(a->n_frames) + 1 > 0x7FFFFFFF / 2) return TG_E_INVAL;
  const size_t bytes = workspace_bytes(a->n_max, a->n_frames);
  if (!a->workspace || a->workspace_bytes < bytes ||
      reinterpret_cast<uintptr_t>(a->workspace) % 16 != 0)
    return TG_E_WORKSPACE;

  MergeParams P = {};
  P.dets = a->dets;
  P.n_dets = a->n_dets;
  P.n_max = a->n_max;
  P.scores = a->scores;
  P.n_scores = a->n_scores;
  P.n_frames = a->n_frames;
  P.thr = a->iou_threshold;
  P.cross_only = a->cross_only;
  P.keep = a->keep;
  P.out = a->out;
  P.n_kept = a->n_kept;
  if (a->n_max <= kTiny) {
    hipLaunchKernelGGL(tiny_kernel, dim3(1), dim3(kTiny), 0, s, P);
    return hipGetLastError() == hipSuccess ? TG_OK : TG_E_HIP;
  }
  P.chunk = chunk_of(a->n_max);
  P.n_chunks = static_cast<int32_t>((int64_t(a->n_max) + P.chunk - 1) / P.chunk);
  P.per_bin = std::max(1, (a->n_frames + kBinsMax - 1) / kBinsMax);
  P.n_bins = (a->n_frames + P.per_bin - 1) / P.per_bin;
  const size_t used = lay_out(static_cast<uint8_t *>(a->workspace), a->n_max, P);
  if (used > bytes) return TG_E_INTERNAL;  // never: workspace_bytes covers the arrays
  P.ovf_cap = std::min<int64_t>(static_cast<int64_t>((bytes - used) / sizeof(int32_t)), 0x7FFFFFFF);

  const dim3 chunks(static_cast<uint32_t>(P.n_chunks));
  hipLaunchKernelGGL(hist_kernel, chunks, dim3(kBinThreads), 0, s, P);
  if (P.n_bins > 0) {
    hipLaunchKernelGGL(scatter_kernel, chunks, dim3(kBinThreads), 0, s, P);
    hipLaunchKernelGGL(local_kernel, dim3(static_cast<uint32_t>(P.n_bins)), dim3(kLocal), 0, s, P);
    const int tiles = 2 * (a->n_max / kTileDets + 1);
    hipLaunchKernelGGL(tile_kernel, dim3(static_cast<uint32_t>(std::min(tiles, kGridCap))),
                       dim3(kTileThreads), 0, s, P);
    const int large = std::min(a->n_frames, a->n_max / 128 + 1);
    hipLaunchKernelGGL(resolve_kernel, dim3(static_cast<uint32_t>(std::min(large, kGridCap))),
                       dim3(kResolveThreads), 0, s, P);
  }
  if (a->n_max <= kCountDets)
    hipLaunchKernelGGL(count_compact_kernel,
                       dim3(static_cast<uint32_t>((a->n_max + kCountThreads - 1) / kCountThreads)),
                       dim3(kCountThreads), 0, s, P);
  else
    hipLaunchKernelGGL(compact_kernel, dim3(static_cast<uint32_t>(compact_blocks(a->n_max))),
                       dim3(kThreads), 0, s, P);
  return hipGetLastError() == hipSuccess ? TG_OK : TG_E_HIP;
}
