// Host-side forest topology: leaf table in key order, refinement with 2:1
// balance across faces, edges and corners, coarsening, and the remap lists
// (Sec. 2.2).  The paper delegates this to p4est on the CPU; here it is a
// small single-process implementation over the sorted leaf table and a hash
// index of it.
#include <algorithm>

#include "foap4_internal.h"
#include "morton.h"

namespace f4 {

void Topology::init_uniform(int ndim_, const int32_t nt_[3], int level) {
  ndim = ndim_;
  for (int d = 0; d < 3; d++) nt[d] = (d < ndim) ? nt_[d] : 1;
  leaves.clear();
  const int32_t ex = nt[0] << level, ey = nt[1] << level, ez = (ndim == 3) ? (nt[2] << level) : 1;
  leaves.reserve((size_t)ex * ey * ez);
  for (int32_t z = 0; z < ez; z++)
    for (int32_t y = 0; y < ey; y++)
      for (int32_t x = 0; x < ex; x++) leaves.push_back(Leaf{level, {x, y, z}});
  sort_and_index();
}

uint64_t Topology::key(const Leaf &l) const { return leaf_key(ndim, nt, l.level, l.g); }

int32_t Topology::tree_id(const Leaf &l) const {
  int32_t t[3] = {0, 0, 0};
  for (int d = 0; d < ndim; d++) t[d] = l.g[d] >> l.level;
  return t[0] + nt[0] * (t[1] + nt[1] * t[2]);
}

// (level, coordinates) in 64 bits: the row-major number of the region in its
// level's grid (below 2^58: fewer than 2^16 trees, levels up to 14), then the
// level
uint64_t Topology::pack(int32_t level, const int32_t g[3]) const {
  const uint64_t ex = (uint64_t)nt[0] << level, ey = (uint64_t)nt[1] << level;
  return (((uint64_t)(ndim == 3 ? g[2] : 0) * ey + (uint64_t)g[1]) * ex + (uint64_t)g[0]) << 4 | (uint64_t)level;
}

void Topology::sort_and_index() {
  std::vector<uint64_t> keys(leaves.size());
  for (size_t i = 0; i < leaves.size(); i++) keys[i] = key(leaves[i]);
  if (!std::is_sorted(keys.begin(), keys.end())) {
    std::vector<std::pair<uint64_t, Leaf>> tmp(leaves.size());
    for (size_t i = 0; i < leaves.size(); i++) tmp[i] = {keys[i], leaves[i]};
    std::sort(tmp.begin(), tmp.end(), [](const auto &a, const auto &b) { return a.first < b.first; });
    for (size_t i = 0; i < tmp.size(); i++) leaves[i] = tmp[i].second;
  }
  index_.reset(leaves.size());
  for (size_t i = 0; i < leaves.size(); i++) index_.insert(pack(leaves[i].level, leaves[i].g), (int32_t)i);
}

int64_t Topology::find(int32_t level, const int32_t g[3]) const { return index_.find(pack(level, g)); }

namespace {

// the 3^d - 1 neighbour directions
struct Directions {
  int n = 0;
  int o[26][3];
  explicit Directions(int ndim) {
    for (int dz = (ndim == 3 ? -1 : 0); dz <= (ndim == 3 ? 1 : 0); dz++)
      for (int dy = -1; dy <= 1; dy++)
        for (int dx = -1; dx <= 1; dx++)
          if (dx || dy || dz) {
            o[n][0] = dx;
            o[n][1] = dy;
            o[n][2] = dz;
            n++;
          }
  }
};

}  // namespace

// The old mesh is balanced (it is uniform, or the result of a regrid), so
// everything follows from the old leaf table and which of its leaves are
// refined: a refined leaf of level l makes leaves of level l + 1, which only a
// touching, unrefined leaf of level l - 1 unbalances, and no leaf is refined
// twice.  On one core, 216 leaves refined to 608 and coarsened again: 198 and
// 584 us with a node-based hash set of the new leaves, a fixpoint over all of
// them and a look-up of every cell along a parent's sides; 5 and 24 us now.
bool Topology::regrid(const int8_t *flags, int lmin, int lmax, std::vector<Leaf> &out, std::vector<int32_t> &op,
                      std::vector<int32_t> &src, std::vector<int32_t> &arg) const {
  const Directions D(ndim);
  const int nch = 1 << ndim;
  const size_t nb = leaves.size();
  // periodic wrap of region g at level l; false if g lies beyond the end of a
  // bounded axis (there is no region there)
  auto wrap = [&](int32_t l, int32_t g[3]) -> bool {
    for (int d = 0; d < ndim; d++) {
      const int32_t E = nt[d] << l;
      if (g[d] >= 0 && g[d] < E) continue;
      if (!periodic[d]) return false;
      g[d] = ((g[d] % E) + E) % E;
    }
    return true;
  };
  // old leaf that covers region (l, g), -1 if smaller leaves do
  auto covering = [&](int32_t l, const int32_t g[3]) -> int64_t {
    for (int32_t lc = l; lc >= 0; lc--) {
      const int32_t c[3] = {g[0] >> (l - lc), g[1] >> (l - lc), ndim == 3 ? g[2] >> (l - lc) : 0};
      const int64_t n = find(lc, c);
      if (n >= 0) return n;
    }
    return -1;
  };
  // 1. refine flagged leaves, and 2. to keep the 2:1 balance with corner
  //    connectivity, the touching leaves one level coarser, and so on
  std::vector<char> ref(nb, 0), gone(nb, 0);
  std::vector<int32_t> work;
  for (size_t n = 0; n < nb; n++)
    if (flags[n] > 0 && leaves[n].level < lmax) {
      ref[n] = 1;
      work.push_back((int32_t)n);
    }
  bool changed = !work.empty();
  while (!work.empty()) {
    const Leaf &L = leaves[work.back()];
    work.pop_back();
    if (L.level == 0) continue;
    for (int q = 0; q < D.n; q++) {
      int32_t h[3] = {L.g[0] + D.o[q][0], L.g[1] + D.o[q][1], ndim == 3 ? L.g[2] + D.o[q][2] : 0};
      if (!wrap(L.level, h)) continue;
      const int64_t m = covering(L.level, h);
      if (m >= 0 && leaves[m].level < L.level && !ref[m]) {
        ref[m] = 1;
        work.push_back((int32_t)m);
      }
    }
  }
  // 3. coarsen complete families of old leaves flagged -1 above lmin whose
  //    parent touches only leaves of level <= parent level + 1.  Siblings are
  //    neighbours in the leaf table; gone marks a merged family's first leaf (1)
  //    and the others (2).
  for (size_t n = 0; n + nch <= nb; n++) {
    const Leaf &L = leaves[n];
    if (flags[n] >= 0 || L.level <= lmin || L.level == 0) continue;
    if ((L.g[0] & 1) || (L.g[1] & 1) || (ndim == 3 && (L.g[2] & 1))) continue;
    bool ok = true;
    for (int c = 0; c < nch && ok; c++) {
      const Leaf &S = leaves[n + c];
      ok = flags[n + c] < 0 && !ref[n + c] && S.level == L.level && S.g[0] == L.g[0] + (c & 1) &&
           S.g[1] == L.g[1] + ((c >> 1) & 1) && (ndim == 2 || S.g[2] == L.g[2] + ((c >> 2) & 1));
    }
    const int32_t lp = L.level - 1, p[3] = {L.g[0] >> 1, L.g[1] >> 1, ndim == 3 ? L.g[2] >> 1 : 0};
    for (int q = 0; q < D.n && ok; q++) {
      int32_t r[3] = {p[0] + D.o[q][0], p[1] + D.o[q][1], ndim == 3 ? p[2] + D.o[q][2] : 0};
      if (!wrap(lp, r)) continue;
      if (covering(lp, r) >= 0) continue;  // a leaf of level <= lp, or its children
      // smaller leaves: the children of the region that touch the parent have
      // to be old leaves that stay
      int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
      for (int d = 0; d < ndim; d++) {
        lo[d] = D.o[q][d] == -1 ? 1 : 0;
        hi[d] = D.o[q][d] == 1 ? 0 : 1;
      }
      for (int z = lo[2]; z <= hi[2] && ok; z++)
        for (int y = lo[1]; y <= hi[1] && ok; y++)
          for (int x = lo[0]; x <= hi[0] && ok; x++) {
            const int32_t c[3] = {2 * r[0] + x, 2 * r[1] + y, ndim == 3 ? 2 * r[2] + z : 0};
            const int64_t m = find(lp + 1, c);
            ok = m >= 0 && !ref[m];
          }
    }
    if (!ok) continue;
    for (int c = 0; c < nch; c++) gone[n + c] = c ? 2 : 1;
    changed = true;
  }
  if (!changed) return false;
  // the new leaf table, in key order like the old one
  out.clear();
  op.clear();
  src.clear();
  arg.clear();
  for (size_t n = 0; n < nb; n++) {
    const Leaf &L = leaves[n];
    if (gone[n] == 2) continue;
    if (gone[n] == 1) {
      out.push_back(Leaf{L.level - 1, {L.g[0] >> 1, L.g[1] >> 1, ndim == 3 ? L.g[2] >> 1 : 0}});
      op.push_back(2);
      src.push_back((int32_t)n);
      arg.push_back(0);
    } else if (ref[n]) {
      for (int c = 0; c < nch; c++) {
        out.push_back(Leaf{L.level + 1,
                           {2 * L.g[0] + (c & 1), 2 * L.g[1] + ((c >> 1) & 1), ndim == 3 ? 2 * L.g[2] + ((c >> 2) & 1) : 0}});
        op.push_back(1);
        src.push_back((int32_t)n);
        arg.push_back(c);
      }
    } else {
      out.push_back(L);
      op.push_back(0);
      src.push_back((int32_t)n);
      arg.push_back(0);
    }
  }
  return true;
}

}  // namespace f4
