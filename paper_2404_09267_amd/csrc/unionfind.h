// Union-find walks with atomic-min linking, used by tg_mask_rois's connected-component
// labelling (the GPU union-find method of Playne and Hawick, 2018, with path halving).
//
// Invariant: a link never points to a larger index -- a root points to itself, and links
// only ever decrease (every write is an atomic min with a smaller index of the same set).
// Each step of a find therefore moves to a strictly smaller index, and each step of a unite
// lowers one of its two nodes, so both walks end; concurrent walks may see a link lowered
// under them but never raised. The walks also check the invariant as they
// go: a link that points upwards, or below zero, can only come from an inconsistent array
// (which the labelling never produces), and ends the walk with a failure instead of a
// loop.
//
// The walks are templates over an accessor M with
//   int parent(int i)        the link of i,
//   int link(int i, int p)   lowers the link of i to min(link, p) atomically and returns
//                            the link it replaced,
// so that the same code runs on LDS and global labels in the kernels and on a plain
// array in the CPU tests of these walks.
#ifndef TG_UNIONFIND_H
#define TG_UNIONFIND_H

#if defined(__HIPCC__)
#define TG_UF_FN __host__ __device__ inline
#else
#define TG_UF_FN inline
#endif

namespace tg_detail {

// Root of i's set, halving the path on the way (i relinked to its grandparent); -1 when
// the array breaks the invariant.
template <class M>
TG_UF_FN int uf_find(M &m, int i) {
  for (;;) {
    const int p = m.parent(i);
    if (p == i) return i;
    if (p < 0 || p > i) return -1;
    const int g = m.parent(p);
    if (g == p) return p;
    if (g < 0 || g > p) return -1;
    m.link(i, g);
    i = g;
  }
}

// Lowers the link of i, which is no root, to p: M's relink where it has one (a link whose
// replaced value nobody needs), else its link.
template <class M>
TG_UF_FN auto uf_relink(M &m, int i, int p, int) -> decltype(m.relink(i, p)) {
  m.relink(i, p);
}
template <class M>
TG_UF_FN void uf_relink(M &m, int i, int p, long) {
  m.link(i, p);
}

// Joins the sets of a and b (Rem's walk, with splicing): the node whose parent is larger
// gets the other's parent as its link, then continues from the parent it had. Two nodes with
// one parent are joined, however far their root is; a root that gets the link is joined too,
// unless it was linked meanwhile, when the walk goes on from what it then pointed to. Each
// step loads one link. False when the array breaks the invariant.
// A relink may replace a link that another walk lowered meanwhile: that walk, as this one,
// goes on to join what the node pointed to before with what it wrote, so no connection is
// lost.
template <class M>
TG_UF_FN bool uf_unite(M &m, int a, int b) {
  int pa = m.parent(a), pb = m.parent(b);
  if (pb < 0 || pb > b) return false;
  for (;;) {
    if (pa < 0 || pa > a) return false;
    if (pa == pb) return true;
    if (pa < pb) {
      int t = a;
      a = b;
      b = t;
      t = pa;
      pa = pb;
      pb = t;
    }
    if (pa == a) {
      const int old = m.link(a, pb);
      if (old == a) return true;
      if (old < 0 || old > a) return false;
      a = old;
    } else {
      uf_relink(m, a, pb, 0);
      a = pa;
    }
    pa = m.parent(a);
  }
}

}  // namespace tg_detail

#endif  // TG_UNIONFIND_H
