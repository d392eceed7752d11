// CPU driver for the union-find walks of tg_mask_rois (csrc/unionfind.h), run by
// test_unionfind.py. Reads one case per line from stdin and prints one result line:
//   F n p_0 .. p_{n-1} i       -> "<root or -1> <parent() calls>"
//   U n p_0 .. p_{n-1} a b     -> "<1 or 0> <parent() calls> q_0 .. q_{n-1}" (array after)
//   X n p_0 .. p_{n-1} a b v   -> as U, but the first link() reports v as the link it
//                                 replaced, as if another thread had written v there
//   E n m a_0 b_0 .. a_m b_m   -> from the identity array, unite every edge in order;
//                                 "<all ok> r_0 .. r_{n-1} q_0 .. q_{n-1}" with r_i the
//                                 find of i after all edges and q the array
//   N n seed m a_0 b_0 .. a_m b_m -> as E, but at any access of a unite the next edges may be
//                                 united to their end first, nested up to 8 deep (the seed says
//                                 where), as a concurrent walk would do between two accesses;
//                                 "<all ok> <root links> r_0 .. r_{n-1} q_0 .. q_{n-1}"
//   A n seed m a_0 b_0 .. a_m b_m -> as N, but up to eight unites run at once, each stopped
//                                 before every access, and the seed says which goes on next:
//                                 the accesses of unfinished unites alternate in any order
// The accessor counts parent() reads so that the tests can bound the work of a walk over
// a broken array.
#include <ucontext.h>

#include <cstdint>
#include <cstdio>
#include <memory>
#include <utility>
#include <vector>

#include "unionfind.h"

namespace {

struct Plain {
  std::vector<int> a;
  long reads = 0;
  bool planted = false;
  int plant = 0;
  int parent(int i) {
    ++reads;
    return a[i];
  }
  int link(int i, int p) {
    const int old = a[i];
    if (p < old) a[i] = p;
    if (planted) {
      planted = false;
      return plant;
    }
    return old;
  }
};

bool read_array(int n, Plain &m) {
  m.a.resize(n);
  for (int k = 0; k < n; ++k)
    if (std::scanf("%d", &m.a[k]) != 1) return false;
  return true;
}

void print_array(const Plain &m) {
  for (int v : m.a) std::printf(" %d", v);
}

// An array whose accesses let other unites run first.
struct Nested {
  std::vector<int> a;
  std::vector<std::pair<int, int>> edges;
  size_t next = 0;
  int depth = 0, root_links = 0;
  uint32_t state = 1;
  bool ok = true;
  void others();
  int parent(int i) {
    others();
    return a[i];
  }
  int link(int i, int p) {
    others();
    const int old = a[i];
    if (p < old) a[i] = p;
    if (old == i && p < i) ++root_links;
    return old;
  }
  void relink(int i, int p) {
    others();
    if (a[i] == i) ok = false;  // only a node that is no root is relinked
    if (p < a[i]) a[i] = p;
  }
};

void Nested::others() {
  while (depth < 8 && next < edges.size()) {
    state = state * 1664525u + 1013904223u;
    if (state >> 30 != 0) return;
    const auto e = edges[next++];
    ++depth;
    ok = tg_detail::uf_unite(*this, e.first, e.second) && ok;
    --depth;
  }
}

// An array whose accesses each wait for their turn: every unite runs on a stack of its own and
// hands over to the scheduler before it reads or writes.
struct Turns {
  std::vector<int> a;
  int root_links = 0;
  bool ok = true;
  ucontext_t scheduler;
  ucontext_t *now = nullptr;
  void turn() {
    ucontext_t *me = now;
    swapcontext(me, &scheduler);
  }
  int parent(int i) {
    turn();
    return a[i];
  }
  int link(int i, int p) {
    turn();
    const int old = a[i];
    if (p < old) a[i] = p;
    if (old == i && p < i) ++root_links;
    return old;
  }
  void relink(int i, int p) {
    turn();
    if (a[i] == i) ok = false;  // only a node that is no root is relinked
    if (p < a[i]) a[i] = p;
  }
};

struct Walk {
  ucontext_t ctx;
  std::unique_ptr<char[]> stack;
  Turns *m;
  int x, y;
  bool running = false;
};

void run_walk(unsigned lo, unsigned hi) {
  Walk *w = reinterpret_cast<Walk *>(static_cast<uintptr_t>(hi) << 32 | lo);
  w->m->ok = tg_detail::uf_unite(*w->m, w->x, w->y) && w->m->ok;
  w->running = false;
  swapcontext(&w->ctx, &w->m->scheduler);
}

void alternate(Turns &m, const std::vector<std::pair<int, int>> &edges, uint32_t state) {
  constexpr int kWalks = 8;
  constexpr size_t kStack = 64 * 1024;
  Walk walks[kWalks];
  size_t next = 0;
  for (;;) {
    int running[kWalks], n = 0;
    for (int k = 0; k < kWalks; ++k) {
      Walk &w = walks[k];
      if (!w.running && next < edges.size()) {
        w.m = &m;
        w.x = edges[next].first;
        w.y = edges[next++].second;
        w.running = true;
        if (!w.stack) w.stack.reset(new char[kStack]);
        getcontext(&w.ctx);
        w.ctx.uc_stack.ss_sp = w.stack.get();
        w.ctx.uc_stack.ss_size = kStack;
        w.ctx.uc_link = nullptr;
        const uintptr_t p = reinterpret_cast<uintptr_t>(&w);
        makecontext(&w.ctx, reinterpret_cast<void (*)()>(run_walk), 2,
                    static_cast<unsigned>(p), static_cast<unsigned>(p >> 32));
      }
      if (w.running) running[n++] = k;
    }
    if (n == 0) return;
    state = state * 1664525u + 1013904223u;
    Walk &w = walks[running[(state >> 16) % n]];
    m.now = &w.ctx;
    swapcontext(&m.scheduler, &w.ctx);
  }
}

}  // namespace

int main() {
  char op;
  while (std::scanf(" %c", &op) == 1) {
    int n = 0;
    if (std::scanf("%d", &n) != 1 || n < 1) return 2;
    Plain m;
    if (op == 'F') {
      int i;
      if (!read_array(n, m) || std::scanf("%d", &i) != 1) return 2;
      const int r = tg_detail::uf_find(m, i);
      std::printf("%d %ld\n", r, m.reads);
    } else if (op == 'U') {
      int a, b;
      if (!read_array(n, m) || std::scanf("%d %d", &a, &b) != 2) return 2;
      const bool ok = tg_detail::uf_unite(m, a, b);
      std::printf("%d %ld", ok ? 1 : 0, m.reads);
      print_array(m);
      std::printf("\n");
    } else if (op == 'X') {
      int a, b;
      if (!read_array(n, m) || std::scanf("%d %d %d", &a, &b, &m.plant) != 3) return 2;
      m.planted = true;
      const bool ok = tg_detail::uf_unite(m, a, b);
      std::printf("%d %ld", ok ? 1 : 0, m.reads);
      print_array(m);
      std::printf("\n");
    } else if (op == 'E') {
      int e;
      if (std::scanf("%d", &e) != 1) return 2;
      m.a.resize(n);
      for (int k = 0; k < n; ++k) m.a[k] = k;
      bool ok = true;
      for (int k = 0; k < e; ++k) {
        int a, b;
        if (std::scanf("%d %d", &a, &b) != 2) return 2;
        ok = tg_detail::uf_unite(m, a, b) && ok;
      }
      std::printf("%d", ok ? 1 : 0);
      for (int k = 0; k < n; ++k) std::printf(" %d", tg_detail::uf_find(m, k));
      print_array(m);
      std::printf("\n");
    } else if (op == 'N') {
      int e;
      Nested q;
      if (std::scanf("%u %d", &q.state, &e) != 2) return 2;
      for (int k = 0; k < n; ++k) q.a.push_back(k);
      for (int k = 0; k < e; ++k) {
        int a, b;
        if (std::scanf("%d %d", &a, &b) != 2) return 2;
        q.edges.emplace_back(a, b);
      }
      while (q.next < q.edges.size()) {
        const auto x = q.edges[q.next++];
        q.ok = tg_detail::uf_unite(q, x.first, x.second) && q.ok;
      }
      std::printf("%d %d", q.ok ? 1 : 0, q.root_links);
      m.a = q.a;
      for (int k = 0; k < n; ++k) std::printf(" %d", tg_detail::uf_find(m, k));
      for (int v : q.a) std::printf(" %d", v);
      std::printf("\n");
    } else if (op == 'A') {
      int e;
      uint32_t seed;
      Turns t;
      std::vector<std::pair<int, int>> edges;
      if (std::scanf("%u %d", &seed, &e) != 2) return 2;
      for (int k = 0; k < n; ++k) t.a.push_back(k);
      for (int k = 0; k < e; ++k) {
        int a, b;
        if (std::scanf("%d %d", &a, &b) != 2) return 2;
        edges.emplace_back(a, b);
      }
      alternate(t, edges, seed);
      std::printf("%d %d", t.ok ? 1 : 0, t.root_links);
      m.a = t.a;
      for (int k = 0; k < n; ++k) std::printf(" %d", tg_detail::uf_find(m, k));
      print_array(m);
      std::printf("\n");
    } else {
      return 2;
    }
  }
  return 0;
}
