// Nested dissection of the nx x ny grid (host): the tree of separators, the
// index tables that carry Schur complements and updates from the halves of a
// block to the block, and the task lists of every launch.
//
// A block of grid nodes is split across its longer side by one line of nodes,
// the separator, which the five-point stencil makes independent halves of;
// blocks of at most kNdLeafNodes nodes are eliminated whole.  Unknowns are
// eliminated leaves first, the whole grid's separator last.  A block's border
// is the lines of nodes around it that later separators hold (the grid's own
// edge has none), side by side: left (i0 - 1), right (i1), low (j0 - 1), high
// (j1), each by its coordinate, the two unknowns of a node together.  So the
// separator is one run of either half's border, and the border of the block
// is made of runs of its halves' borders; the node at a separator's own end
// belongs to neither half's.
#include <algorithm>
#include <map>
#include <new>
#include <tuple>

#include "rr_internal.h"

namespace rr {
namespace {

struct Block {
  int i0, i1, j0, j1;
  bool leaf, across_x;  // across_x: the separator is the line i = mid
  int mid;
  int off[5];  // border offsets of left, right, low, high, and the total (unknowns)
};

void set_border(Block& b, int nx, int ny) {
  const int a = b.i1 - b.i0, c = b.j1 - b.j0;
  const int len[4] = {b.i0 > 0 ? c : 0, b.i1 < nx ? c : 0, b.j0 > 0 ? a : 0, b.j1 < ny ? a : 0};
  b.off[0] = 0;
  for (int s = 0; s < 4; s++) b.off[s + 1] = b.off[s] + 2 * len[s];
}

int64_t up16(int64_t v) { return (v + 15) & ~int64_t(15); }
int64_t tiles(int64_t v) { return (v + kNdTile - 1) / kNdTile; }
// Temporaries of a front past one tile: T12, the pivot block's row and column,
// two copies of the pivot inverse in either order.
int64_t temp_size(int64_t P, int64_t Q) {
  return P > kNdTile ? P * Q + 2 * kNdTile * P + 4 * kNdTile * kNdTile : 0;
}

}  // namespace

// Counted by distinct blocks: at one depth they differ by a node or so a side
// and by which sides border on a separator, a few dozen where a front each
// would be n / 32 (16384 x 8192: 4 s and 1.6 GB on the host).
void nd_sizes(int nx, int ny, NdPlan* plan) {
  NdPlan& pl = *plan;
  pl = NdPlan{};
  pl.nx = nx;
  pl.ny = ny;
  typedef std::tuple<int, int, bool, bool, bool, bool> Shape;  // nodes; left, right, low, high
  std::map<Shape, int64_t> level;
  level[Shape{nx, ny, false, false, false, false}] = 1;
  for (int d = 0; !level.empty(); d++) {
    std::map<Shape, int64_t> next;
    int64_t s = 0, u = 0, t = 0;
    for (const auto& [shape, count] : level) {
      const auto [a, c, left, right, low, high] = shape;
      const bool leaf = (int64_t)a * c <= kNdLeafNodes, across_x = a >= c;
      const int64_t P = up16(2 * (leaf ? (int64_t)a * c : across_x ? c : a));
      const int64_t Q = up16(2 * ((int64_t)c * (left + right) + (int64_t)a * (low + high)));
      pl.nfronts += count;
      pl.allrows += count * P;
      pl.border += count * Q;
      pl.factor += count * P * P;
      s += count * Q * Q;
      u += count * Q;
      t += count * temp_size(P, Q);
      if (leaf) {
        pl.ntasks += count;
        continue;
      }
      pl.rows += count * P;
      pl.factor += count * 2 * P * Q;
      const int64_t np = tiles(P), nq = tiles(Q);
      int64_t tasks = nq * nq;                      // schur
      tasks += P <= kNdDownP ? 1 : P / 16;          // down, rowsX
      if (P <= kNdTile)
        tasks++;
      else  // assemble, panel, update, border, gather, rowsP, rowsQ
        tasks += np * np + 2 * np * nq + 2 * np * (np - 1) + np * np * np + np * nq + np + P / 16 +
                 Q / 16;
      pl.ntasks += count * tasks;
      if (across_x) {
        next[Shape{(a - 1) / 2, c, left, true, low, high}] += count;
        next[Shape{a - 1 - (a - 1) / 2, c, true, right, low, high}] += count;
      } else {
        next[Shape{a, (c - 1) / 2, left, right, low, true}] += count;
        next[Shape{a, c - 1 - (c - 1) / 2, left, right, true, high}] += count;
      }
    }
    pl.schur[d & 1] = std::max(pl.schur[d & 1], s);
    pl.urows[d & 1] = std::max(pl.urows[d & 1], u);
    pl.temp = std::max(pl.temp, t);
    level.swap(next);
  }
}

void nd_make_plan(int nx, int ny, NdPlan* plan) {
  nd_sizes(nx, ny, plan);
  NdPlan& pl = *plan;
  std::vector<Block> blocks(1, Block{0, nx, 0, ny, false, false, 0, {}});
  std::vector<int> first(1, 0);  // first front of every depth
  for (size_t lo = 0; lo < blocks.size();) {
    const size_t hi = blocks.size();
    for (size_t f = lo; f < hi; f++) {
      Block b = blocks[f];
      set_border(b, nx, ny);
      const int a = b.i1 - b.i0, c = b.j1 - b.j0;
      b.leaf = (int64_t)a * c <= kNdLeafNodes;
      b.across_x = a >= c;
      b.mid = b.across_x ? b.i0 + (a - 1) / 2 : b.j0 + (c - 1) / 2;
      blocks[f] = b;
      NdFront fr{};
      fr.childA = fr.childB = -1;
      fr.p = 2 * (b.leaf ? a * c : b.across_x ? c : a);
      fr.q = b.off[4];
      fr.P = (int)up16(fr.p);
      fr.Q = (int)up16(fr.q);
      if (!b.leaf) {
        fr.childA = (int)blocks.size();
        fr.childB = fr.childA + 1;
        Block h = b;
        if (b.across_x) {
          h.i1 = b.mid;
          blocks.push_back(h);
          h = b;
          h.i0 = b.mid + 1;
        } else {
          h.j1 = b.mid;
          blocks.push_back(h);
          h = b;
          h.j0 = b.mid + 1;
        }
        blocks.push_back(h);
      }
      pl.fronts.push_back(fr);
    }
    lo = hi;
    first.push_back((int)hi);
  }
  const int depth = (int)first.size() - 1;
  pl.levels.resize(depth);
  // offsets: factors by front; Schur complements and updates in an arena per
  // parity of the depth (only the level above reads them); temporaries per level
  int64_t rows = 0, leaf_rows = pl.rows, border = 0, factor = 0;
  for (int d = 0; d < depth; d++) {
    int64_t s = 0, u = 0, t = 0;
    for (int f = first[d]; f < first[d + 1]; f++) {
      NdFront& fr = pl.fronts[f];
      const int64_t P = fr.P, Q = fr.Q;
      const bool leaf = fr.childA < 0;
      fr.row = (int)(leaf ? leaf_rows : rows);
      (leaf ? leaf_rows : rows) += P;
      fr.bor = (int)border;
      border += Q;
      fr.a = factor;
      fr.b12 = fr.a + P * P;
      fr.f21 = fr.b12 + (leaf ? 0 : P * Q);
      factor = fr.f21 + (leaf ? 0 : P * Q);
      fr.s = s;
      s += Q * Q;
      fr.urow = (int)u;
      u += Q;
      if (P > kNdTile) fr.t = t;
      t += temp_size(P, Q);
    }
  }

  std::vector<int> row_of((size_t)nx * ny);
  pl.pdof.assign(pl.allrows, -1);
  for (size_t f = 0; f < blocks.size(); f++) {
    const Block& b = blocks[f];
    const int i0 = !b.leaf && b.across_x ? b.mid : b.i0, i1 = !b.leaf && b.across_x ? b.mid + 1 : b.i1;
    const int j0 = !b.leaf && !b.across_x ? b.mid : b.j0;
    const int j1 = !b.leaf && !b.across_x ? b.mid + 1 : b.j1;
    int r = pl.fronts[f].row;
    for (int i = i0; i < i1; i++)
      for (int j = j0; j < j1; j++, r += 2) {
        const int node = i * ny + j;
        row_of[node] = r;
        pl.pdof[r] = 2 * node;
        pl.pdof[r + 1] = 2 * node + 1;
      }
  }
  pl.bmap.assign(pl.border, -1);
  pl.grow.assign(pl.border, (int)pl.rows);
  for (size_t f = 0; f < blocks.size(); f++) {
    const Block& b = blocks[f];
    NdFront& fr = pl.fronts[f];
    const Block* h[2] = {nullptr, nullptr};
    if (!b.leaf) {
      h[0] = &blocks[fr.childA];
      h[1] = &blocks[fr.childB];
      fr.baseA = h[0]->off[b.across_x ? 1 : 3];  // A's right / high side is the separator
      fr.baseB = h[1]->off[b.across_x ? 0 : 2];  // B's left / low side
    }
    if (!b.leaf) {
      const NdFront &ca = pl.fronts[fr.childA], &cb = pl.fronts[fr.childB];
      fr.QA = ca.Q;
      fr.QB = cb.Q;
      fr.uA = ca.urow;
      fr.uB = cb.urow;
      fr.sA = ca.s;
      fr.sB = cb.s;
    }
    std::copy(b.off, b.off + 5, fr.side);
    const int across = b.j1 - b.j0;  // a leaf's unknowns: i, then j, then u and v
    fr.across = b.leaf ? across : 0;
    for (int side = 0; side < 4; side++) {
      const bool along_y = side < 2;  // left and right run along y
      const int c0 = along_y ? b.j0 : b.i0;
      const int len = (b.off[side + 1] - b.off[side]) / 2;
      const int fixed = side == 0 ? b.i0 - 1 : side == 1 ? b.i1 : side == 2 ? b.j0 - 1 : b.j1;
      for (int e = 0; e < len; e++) {
        const int c = c0 + e;
        const int node = along_y ? fixed * ny + c : c * ny + fixed;
        int half = -1, pos = 0;
        if (!b.leaf) {
          if (along_y == b.across_x) {  // a side parallel to the separator: one half has all of it
            half = side & 1;
            pos = e;
          } else if (c != b.mid) {
            half = c > b.mid;
            pos = half ? c - b.mid - 1 : e;
          }
        }
        for (int u = 0; u < 2; u++) {
          const int at = fr.bor + b.off[side] + 2 * e + u;
          pl.grow[at] = row_of[node] + u;
          if (half >= 0) pl.bmap[at] = 2 * (h[half]->off[side] + 2 * pos + u) + half;
          if (b.leaf) {
            const int i = along_y ? (side == 0 ? 0 : b.i1 - b.i0 - 1) : e;
            const int j = along_y ? e : (side == 2 ? 0 : across - 1);
            pl.bmap[at] = 2 * (i * across + j) + u;
          }
        }
      }
    }
  }

  auto open = [&](NdSpan& sp) { sp.first = (int)pl.tasks.size(); };
  auto close = [&](NdSpan& sp) { sp.count = (int)pl.tasks.size() - sp.first; };
  for (int d = 0; d < depth; d++) {
    NdLevel& lv = pl.levels[d];
    const int f0 = first[d], f1 = first[d + 1];
    lv.front = f0;
    open(lv.leaf);
    for (int wide = 0; wide < 2; wide++) {
      open(lv.leafs[wide]);
      for (int f = f0; f < f1; f++)
        if (pl.fronts[f].childA < 0 && (pl.fronts[f].P > kNdLeafP) == (wide == 1)) {
          pl.tasks.push_back({f, 0, 0, 0});
          lv.leafP = std::max(lv.leafP, pl.fronts[f].P);
        }
      close(lv.leafs[wide]);
    }
    close(lv.leaf);
    // calls emit(front) for the fronts of one kind, collecting a span
    auto each = [&](NdSpan& sp, bool small, bool large, auto emit) {
      open(sp);
      for (int f = f0; f < f1; f++)
        if (pl.fronts[f].childA >= 0 && (pl.fronts[f].P <= kNdTile ? small : large))
          emit(f, pl.fronts[f]);
      close(sp);
    };
    each(lv.small, true, false, [&](int f, const NdFront& fr) {
      pl.tasks.push_back({f, 0, 0, 0});
      lv.maxP = std::max(lv.maxP, fr.P);
      lv.maxQ = std::max(lv.maxQ, fr.Q);
    });
    int steps = 0;
    each(lv.assemble, false, true, [&](int f, const NdFront& fr) {
      const int np = (int)tiles(fr.P), nq = (int)tiles(fr.Q);
      lv.largeP = std::max(lv.largeP, fr.P);
      steps = std::max(steps, np);
      for (int i = 0; i < np; i++)
        for (int j = 0; j < np; j++) pl.tasks.push_back({f, i, j, 0});
      for (int i = 0; i < np; i++)
        for (int j = 0; j < nq; j++) {
          pl.tasks.push_back({f, i, j, 1});
          pl.tasks.push_back({f, j, i, 2});
        }
    });
    lv.panel.resize(steps);
    lv.update.resize(steps);
    for (int k = 0; k < steps; k++) {
      each(lv.panel[k], false, true, [&](int f, const NdFront& fr) {
        const int np = (int)tiles(fr.P);
        for (int j = 0; j < np && k < np; j++)
          if (j != k) {
            pl.tasks.push_back({f, j, k, 0});
            pl.tasks.push_back({f, j, k, 1});
          }
      });
      each(lv.update[k], false, true, [&](int f, const NdFront& fr) {
        const int np = (int)tiles(fr.P);
        if (k >= np) return;
        if (k + 1 < np) pl.tasks.push_back({f, k + 1, k + 1, k});  // the next pivot tile first
        for (int i = 0; i < np; i++)
          for (int j = 0; j < np; j++)
            if (i != k + 1 || j != k + 1) pl.tasks.push_back({f, i, j, k});
      });
    }
    each(lv.border, false, true, [&](int f, const NdFront& fr) {
      for (int i = 0; i < tiles(fr.P); i++)
        for (int j = 0; j < tiles(fr.Q); j++) pl.tasks.push_back({f, i, j, 0});
    });
    each(lv.schur, true, true, [&](int f, const NdFront& fr) {
      for (int i = 0; i < tiles(fr.Q); i++)
        for (int j = 0; j < tiles(fr.Q); j++) pl.tasks.push_back({f, i, j, 0});
    });
    each(lv.gather, false, true, [&](int f, const NdFront& fr) {
      for (int i = 0; i < tiles(fr.P); i++) pl.tasks.push_back({f, i, 0, 0});
    });
    each(lv.rowsP, false, true, [&](int f, const NdFront& fr) {
      for (int i = 0; i < fr.P / 16; i++) pl.tasks.push_back({f, i, 0, 0});
    });
    each(lv.down, true, false, [&](int f, const NdFront& fr) {
      if (fr.P > kNdDownP) return;
      pl.tasks.push_back({f, 0, 0, 0});
      lv.downP = std::max(lv.downP, fr.P);
    });
    each(lv.rowsX, true, true, [&](int f, const NdFront& fr) {
      for (int i = 0; i < fr.P / 16 && fr.P > kNdDownP; i++) pl.tasks.push_back({f, i, 0, 0});
    });
    each(lv.rowsQ, false, true, [&](int f, const NdFront& fr) {
      for (int i = 0; i < fr.Q / 16; i++) pl.tasks.push_back({f, i, 0, 0});
    });
  }
}

}  // namespace rr

extern "C" int64_t rr_nd_plan(int32_t nx, int32_t ny, int32_t what, int64_t* out, int64_t cap) {
  if (nx < 1 || ny < 1 || 2 * (int64_t)nx * ny > (1ll << 30) || what < 0 || what > 5 ||
      (cap > 0 && !out))
    return -1;
  rr::NdPlan pl;
  try {
    if (what == 5) rr::nd_sizes(nx, ny, &pl);
    else rr::nd_make_plan(nx, ny, &pl);
  } catch (const std::bad_alloc&) {
    return -1;
  }
  int64_t count = 0;
  auto put = [&](int64_t v) {
    if (count < cap) out[count] = v;
    count++;
  };
  if (what == 0) {
    for (size_t f = 0; f < pl.fronts.size(); f++) {
      const rr::NdFront& x = pl.fronts[f];
      int depth = 0;
      for (size_t d = 0; d < pl.levels.size(); d++)
        if ((int)f >= pl.levels[d].front) depth = (int)d;
      for (int64_t v : {(int64_t)x.p, (int64_t)x.q, (int64_t)x.P, (int64_t)x.Q, (int64_t)x.row,
                        (int64_t)x.bor, (int64_t)x.childA, (int64_t)x.childB, (int64_t)x.baseA,
                        (int64_t)x.baseB, (int64_t)x.urow, x.a, x.b12, x.f21, x.s, x.t,
                        (int64_t)depth})
        put(v);
    }
  } else if (what == 4) {
    for (const rr::NdTask& t : pl.tasks)
      for (int v : {t.front, t.i, t.j, t.kind}) put(v);
  } else if (what == 5) {
    for (int64_t v : {pl.rows, pl.allrows, pl.border, pl.factor, pl.schur[0], pl.schur[1], pl.temp,
                      pl.urows[0], pl.urows[1], pl.ntasks})
      put(v);
  } else {
    for (int v : what == 1 ? pl.pdof : what == 2 ? pl.bmap : pl.grow) put(v);
  }
  return count;
}
