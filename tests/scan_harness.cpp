// CPU driver for the mask scan of tg_mask_rois, run by test_scan_waves.py, which copies the
// kernel's text from csrc/rois.hip into scan_extract.inc and compiles this file with clang (for
// its vector types). A workgroup runs as 256 lanes (ucontext fibers). Its waves run one after
// the other, in a given order, each up to the next barrier: every order is one that the
// hardware may take, so the result must not depend on it. LDS holds garbage at the start of
// each workgroup.
// stdin:  wave order (4 digits), frames, width, height, the mask's byte offset from a 16-byte
//         boundary, then the mask as text, a digit per pixel
// stdout: bitmap words per band, the bitmap, then per tile whose bit is set its id and 32 rows
#include <ucontext.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <vector>

namespace sim {

constexpr int kLanes = 256, kWave = 64;
enum State { kRun, kMeet, kBarrier, kDone };
struct Lane {
  ucontext_t ctx;
  std::unique_ptr<char[]> stack;
  State state;
  uint64_t put;
};
Lane lanes[kLanes];
uint64_t met[kLanes];  // what the lanes of a wave put at their last meeting
ucontext_t scheduler;
int now;  // the running lane
void (*body)();

void yield(State s) {
  Lane &l = lanes[now];
  const int me = now;
  l.state = s;
  swapcontext(&l.ctx, &scheduler);
  now = me;
}
// The values that the lanes of this wave put, once all of them are here.
const uint64_t *meet(uint64_t v) {
  lanes[now].put = v;
  const int first = now / kWave * kWave;
  yield(kMeet);
  return met + first;
}
void entry() {
  body();
  yield(kDone);
}

// Runs wave w until its lanes wait at a barrier (true) or are done (false).
bool run_wave(int w) {
  Lane *l = lanes + w * kWave;
  for (;;) {
    for (int i = 0; i < kWave; ++i) {
      now = w * kWave + i;
      swapcontext(&scheduler, &l[i].ctx);
    }
    for (int i = 1; i < kWave; ++i)
      if (l[i].state != l[0].state) std::abort();  // lanes of a wave wait at different places
    if (l[0].state != kMeet) return l[0].state == kBarrier;
    for (int i = 0; i < kWave; ++i) met[w * kWave + i] = l[i].put;
  }
}

// Runs a workgroup, its waves in the given order between barriers.
void run_group(void (*f)(), const int order[4]) {
  body = f;
  for (Lane &l : lanes) {
    constexpr size_t kStack = 64 * 1024;
    if (!l.stack) l.stack.reset(new char[kStack]);
    getcontext(&l.ctx);
    l.ctx.uc_stack.ss_sp = l.stack.get();
    l.ctx.uc_stack.ss_size = kStack;
    l.ctx.uc_link = &scheduler;
    makecontext(&l.ctx, entry, 0);
  }
  for (bool more = true; more;) {
    int waiting = 0;
    for (int k = 0; k < 4; ++k) waiting += run_wave(order[k]);
    if (waiting != 0 && waiting != 4) std::abort();  // a barrier that some waves never reach
    more = waiting == 4;
  }
}

}  // namespace sim

// What the kernel's text uses of the device.
#define __device__
#define __global__
#define __forceinline__ inline
#define __shared__ static __attribute__((section("lds")))
#define __launch_bounds__(n)
struct Dim {
  int x, y, z;
};
Dim blockIdx, gridDim;
struct {
  struct {
    operator int() const { return sim::now; }
  } x;
} threadIdx;
using std::max;
using std::min;
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
static void __syncthreads() { sim::yield(sim::kBarrier); }
static uint64_t __ballot(bool b) {
  const uint64_t *v = sim::meet(b);
  uint64_t m = 0;
  for (int i = 0; i < sim::kWave; ++i) m |= v[i] << i;
  return m;
}
// The one DPP control the kernel uses: quad permutation 1, 0, 3, 2.
#define __builtin_amdgcn_update_dpp dpp_lane_xor_1
static uint32_t dpp_lane_xor_1(uint32_t, uint32_t v, int ctrl, int, int, bool) {
  if (ctrl != 0xB1) std::abort();
  return static_cast<uint32_t>(sim::meet(v)[(sim::now ^ 1) % sim::kWave]);
}
#define __builtin_amdgcn_udot4 udot4
static uint32_t udot4(uint32_t a, uint32_t b, uint32_t c, bool) {
  for (int i = 0; i < 32; i += 8) c += (a >> i & 255u) * (b >> i & 255u);
  return c;
}

inline uint32_t atomicOr(uint32_t *p, uint32_t v) {
  const uint32_t old = *p;
  *p |= v;
  return old;
}

#include "scan_extract.inc"

extern "C" char __start_lds[], __stop_lds[];

namespace {

const uint8_t *mask;
int W, H;
int64_t frame_px, n_clear;
Tiles T;
std::vector<uint32_t> bits, rec;
std::vector<uint64_t> words;

void one_lane() {
  scan_kernel(mask, W, H, frame_px, T, bits.data(), rec.data(), words.data(), n_clear);
}

}  // namespace

int main() {
  int code, frames, offset;
  while (std::scanf("%d %d %d %d %d", &code, &frames, &W, &H, &offset) == 5) {
    const int order[4] = {code / 1000 % 10, code / 100 % 10, code / 10 % 10, code % 10};
    frame_px = static_cast<int64_t>(W) * H;
    // exactly the mask's bytes are allocated past the offset: a read outside them is reported
    std::unique_ptr<uint8_t[]> buf(new uint8_t[offset + frames * frame_px]);
    for (int64_t i = 0; i < frames * frame_px; ++i) {
      int d;
      if (std::scanf("%1d", &d) != 1) return 2;
      buf[offset + i] = static_cast<uint8_t>(d * 37);
    }
    mask = buf.get() + offset;
    T.tiles_x = (W + kTile - 1) / kTile;
    T.tiles_y = (H + kTile - 1) / kTile;
    T.wpb = (T.tiles_x + 31) / 32;
    T.n = static_cast<int64_t>(frames) * T.tiles_x * T.tiles_y;
    bits.assign(static_cast<size_t>(frames) * T.tiles_y * T.wpb, 0xA5A5A5A5u);
    rec.assign(32 * static_cast<size_t>(T.n), 0xA5A5A5A5u);
    words.assign(7, ~uint64_t(0));
    n_clear = static_cast<int64_t>(words.size());
    gridDim = {T.wpb, T.tiles_y, frames};
    for (blockIdx.z = 0; blockIdx.z < gridDim.z; ++blockIdx.z)
      for (blockIdx.y = 0; blockIdx.y < gridDim.y; ++blockIdx.y)
        for (blockIdx.x = 0; blockIdx.x < gridDim.x; ++blockIdx.x) {
          std::memset(__start_lds, 0x5A, __stop_lds - __start_lds);
          sim::run_group(one_lane, order);
        }
    for (uint64_t w : words)
      if (w != 0) return 3;  // a counter word that was not cleared
    std::printf("%d", T.wpb);
    for (uint32_t w : bits) std::printf(" %u", w);
    for (int64_t t = 0; t < T.n; ++t) {
      const int64_t band = t / T.tiles_x, tx = t - band * T.tiles_x;
      if (!(bits[band * T.wpb + tx / 32] >> (tx % 32) & 1u)) continue;
      std::printf(" %lld", static_cast<long long>(t));
      for (int r = 0; r < 32; ++r) std::printf(" %u", rec[32 * t + r]);
    }
    std::printf("\n");
  }
  return 0;
}
