// Plans of the data-driven kernels (k_walk, k_hist_walk): walk programs for the
// units a block of output columns or a chunk of histogram bins needs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <map>
#include <memory>
#include <new>
#include <vector>

#include "wdf.h"
#include "wdf_dev.h"
#include "wdf_impl.h"
#include "wdf_internal.h"

namespace wdf {
namespace {

// A unit as the walk sees it: the tree node whose split completes its index (a
// quad: the node above its two pair nodes), the index's slot rule, and where
// the slot goes.
struct WalkUnit {
  int64_t node;
  int tree;
  bool quad;
  int fold_a, fold_b;
  uint32_t mask;
  int64_t group;  // whose path leads to the node
  int levels;     // path nodes up to and including `node`
};

// Writes the segments (one per tree, of at most `most` units) of the units
// [a, b) of `list`, which are in tree and depth-first order; unit list[k] hands
// its slot to out(k).  In that order a unit's path leaves the path of the one
// before it at some node and its last node is new, so the tests still to do are
// the path's from there on.
class Programs {
 public:
  explicit Programs(const wdf_model *M) : M_(M) {}

  std::vector<WalkOp> ops;
  std::vector<int2> segs;

  template <class Out>
  void add(const std::vector<WalkUnit> &units, const int32_t *list, int64_t a, int64_t b, Out out,
           int64_t most = INT64_MAX) {
    for (int64_t k = a; k < b;) {
      const int tree = units[(size_t)list[k]].tree;
      const size_t op0 = ops.size();
      const int64_t base = M_->node_offset[(size_t)tree], stop = b - k < most ? b : k + most;
      int64_t on[WDF_MAX_DEPTH + 2];  // the nodes whose splits are in P
      int have = 0;                   // splits in P
      for (; k < stop && units[(size_t)list[k]].tree == tree; ++k) {
        const WalkUnit &u = units[(size_t)list[k]];
        const int64_t *path = &M_->path_nodes[(size_t)M_->groups[(size_t)u.group].path_off];
        int at = 0;
        while (at < have && at < u.levels && on[at] == path[at]) ++at;
        for (; at < u.levels; ++at) {
          test(path[at], ops.size() == op0 ? kWalkDropAll : have - at);
          on[at] = path[at];
          have = at + 1;
        }
        if (u.quad) {  // the two pair nodes below; no other unit's path holds them
          test(base + M_->left[(size_t)u.node], 0);
          test(base + M_->right[(size_t)u.node], 0);
          on[have] = on[have + 1] = -1;
          have += 2;
        }
        WalkOp &o = ops.back();
        o.ctl |= kWalkEmit | (uint32_t)(u.fold_a ? u.fold_a : 31) << 8 | (uint32_t)(u.fold_b ? u.fold_b : 31) << 16;
        o.out = out(k) | u.mask << 20;
      }
      while ((ops.size() - op0) % 4) ops.push_back(WalkOp{0, 0u, 31u << 8 | 31u << 16, 0u});
      segs.push_back(int2{(int)op0, (int)ops.size()});
    }
  }

 private:
  void test(int64_t node, int drop) {
    const uint32_t bias = M_->default_left[(size_t)node] ? 0u : 1u;
    uint32_t b;
    std::memcpy(&b, &M_->threshold[(size_t)node], sizeof b);
    ops.push_back(WalkOp{M_->feature[(size_t)node], walk_key_bits(b) - bias,
                         (uint32_t)drop | (bias ? kWalkBias : 0u), 0u});
  }

  const wdf_model *M_;
};

// Arrays of one plan, copied into one device buffer: *ptr receives each one's
// address.  One allocation and one wait instead of one per array (a model of 10
// trees spent most of its load on them).
class Upload {
 public:
  template <class T>
  void add(const std::vector<T> &v, const T *&ptr) {
    parts_.push_back({v.data(), v.size() * sizeof(T), bytes_, (const void **)&ptr});
    bytes_ += (v.size() * sizeof(T) + 255) / 256 * 256;
  }
  int run(DevBuf &buf, hipStream_t s) {
    const int rc = buf.alloc(std::max<size_t>(bytes_, 256));
    if (rc) return rc;
    for (const Part &p : parts_) {
      *p.ptr = (const char *)buf.ptr + p.at;
      if (p.bytes) HIP_TRY(hipMemcpyAsync((char *)buf.ptr + p.at, p.src, p.bytes, hipMemcpyHostToDevice, s));
    }
    HIP_TRY(hipStreamSynchronize(s));
    return WDF_OK;
  }

 private:
  struct Part {
    const void *src;
    size_t bytes, at;
    const void **ptr;
  };
  std::vector<Part> parts_;
  size_t bytes_ = 0;
};

// unit of a group's own table (no quad)
WalkUnit group_unit(const wdf_model *M, int64_t g, uint32_t mask) {
  const Group &gr = M->groups[(size_t)g];
  return WalkUnit{M->path_nodes[(size_t)gr.path_off + (size_t)gr.depth - 1], gr.tree, false, 0, 0, mask, g, gr.depth};
}

// right turns of a group's path, root first (top bit)
uint32_t right_turns(const wdf_model *M, const Group &g) {
  uint32_t m = 0;
  for (int k = 0; k < g.depth; ++k) m = m << 1 | M->path[(size_t)g.path_off + (size_t)k].dir;
  return m;
}

// a value of a column: the unit and the entry's place in the tables
struct ColumnEntry {
  int32_t unit;
  int64_t tab;  // floats
};

// column lists of one group of output columns
struct ColumnGroup {
  int64_t col0;
  int32_t cols;
  std::vector<std::pair<int32_t, const std::vector<ColumnEntry> *>> lists;  // (column - col0, entries in unit order)
};

// no exception leaves a plan's construction (the callers are C entry points)
template <class Build>
int guarded(Build build) {
  try {
    return build();
  } catch (const std::bad_alloc &) {
    return set_error(WDF_E_OOM, "data-driven kernels: out of host memory");
  }
}

// units whose patterns a block of 64 rows holds
int chunk_units(bool wide) { return kWalkPatternBytes / 64 / (wide ? 2 : 1); }

constexpr int kZeroRun = 32;  // columns one wave clears at a time

int build_level(const wdf_model *M, const std::vector<WalkUnit> &units, const std::vector<ColumnGroup> &groups,
                bool wide, int entry_shift, int cap, WalkLevel &out) {
  Programs prog(M);
  std::vector<WalkGroup> gs;
  std::vector<WalkChunk> chunks;
  std::vector<WalkRun> runs;
  std::vector<WalkEntry> entries;
  std::vector<int32_t> slot(units.size(), -1);
  size_t total = 0;
  for (const ColumnGroup &cg : groups)
    for (const auto &l : cg.lists) total += l.second->size();
  entries.reserve(total);
  int most = 0;
  for (const ColumnGroup &cg : groups) {
    // the units of the group's columns, in order
    std::vector<int32_t> need;
    for (const auto &l : cg.lists)
      for (const ColumnEntry &e : *l.second)
        if (slot[(size_t)e.unit] != -2) slot[(size_t)e.unit] = -2, need.push_back(e.unit);
    if (need.size() < units.size() / 16) {
      std::sort(need.begin(), need.end());
    } else {
      need.clear();
      for (size_t u = 0; u < units.size(); ++u)
        if (slot[u] == -2) need.push_back((int32_t)u);
    }
    WalkGroup wg{cg.col0, (int32_t)chunks.size(), 0};
    std::vector<size_t> at(cg.lists.size(), 0);
    for (size_t a = 0; a == 0 || a < need.size(); a += (size_t)cap) {
      const size_t b = std::min(need.size(), a + (size_t)cap);
      WalkChunk ch{(int32_t)prog.segs.size(), 0, (int32_t)runs.size(), 0};
      prog.add(units, need.data(), (int64_t)a, (int64_t)b, [&](int64_t k) {
        slot[(size_t)need[(size_t)k]] = (int32_t)(k - (int64_t)a);
        return (uint32_t)(k - (int64_t)a);
      });
      most = std::max(most, (int)(b - a));
      int32_t zero = 0;  // columns from here on are not yet written (first chunk)
      auto zeros_to = [&](int32_t col) {
        for (; zero + kZeroRun < col; zero += kZeroRun)
          runs.push_back(WalkRun{zero, zero + kZeroRun, (int32_t)entries.size(), (int32_t)entries.size()});
      };
      for (size_t k = 0; k < cg.lists.size(); ++k) {
        const std::vector<ColumnEntry> &l = *cg.lists[k].second;
        const int32_t e0 = (int32_t)entries.size();
        for (; at[k] < l.size() && (b == need.size() || l[at[k]].unit < need[b]); ++at[k])
          entries.push_back(WalkEntry{(uint32_t)slot[(size_t)l[at[k]].unit] << 2 | (uint32_t)(l[at[k]].tab & 3),
                                      (uint32_t)(l[at[k]].tab >> 2)});
        if ((int32_t)entries.size() == e0) continue;
        const int32_t col = cg.lists[k].first;
        if (a == 0) zeros_to(col);
        runs.push_back(WalkRun{a == 0 ? zero : col, col, e0, (int32_t)entries.size()});
        zero = col + 1;
      }
      if (a == 0 && zero < cg.cols) {
        zeros_to(cg.cols);
        runs.push_back(WalkRun{zero, cg.cols, (int32_t)entries.size(), (int32_t)entries.size()});
      }
      ch.seg1 = (int32_t)prog.segs.size();
      ch.run1 = (int32_t)runs.size();
      chunks.push_back(ch);
    }
    wg.chunk1 = (int32_t)chunks.size();
    gs.push_back(wg);
  }
  if (prog.ops.size() > 0x7fffffff || entries.size() > 0x7fffffff || runs.size() > 0x7fffffff)
    return set_error(WDF_E_UNSUPPORTED, "model too large for the data-driven kernels");
  out.n_groups = (int)gs.size();
  out.max_slots = std::max(most, 1);
  out.wide = wide;
  out.entry_shift = entry_shift;
  out.max_column = 0;
  for (const ColumnGroup &cg : groups)
    for (const auto &l : cg.lists) out.max_column = std::max(out.max_column, (int64_t)l.second->size());
  Upload up;
  up.add(prog.ops, out.ops);
  up.add(prog.segs, out.segs);
  up.add(gs, out.groups);
  up.add(chunks, out.chunks);
  up.add(runs, out.runs);
  up.add(entries, out.entries);
  return up.run(out.buf, M->ctx->stream);
}

}  // namespace

// Levels of the explain walk, coarse to fine: columns (features) per block, 64,
// 16 and 4.  A coarse level computes a unit's slot for few blocks of columns, a
// fine one spreads few rows over more blocks; each is used for the row counts
// where its blocks just fill the device (walk_explain).  Small generic models
// have one more, of all columns, for blocks of 512 rows.
static int build_explain(wdf_model *M, bool tall) {
  JitPlan &P = M->jp;
  const int F = M->n_features;
  int rc;
  Upload up;
  up.add(P.xunits, P.d_xunits);
  up.add(P.unit_g0, P.d_unit_g0);
  if ((rc = up.run(P.d_units, M->ctx->stream))) return rc;
  std::vector<WalkUnit> units;
  std::vector<std::vector<ColumnEntry>> cols((size_t)F);
  bool wide = false;
  for (size_t u = 0; u < P.xunits.size(); ++u) {
    const XUnit &x = P.xunits[u];
    const int64_t g = P.unit_g0[u];
    const Group &gr = M->groups[(size_t)g];
    const int64_t E = (int64_t)1 << (x.depth + x.quad);
    wide = wide || E > 256;
    WalkUnit w = gr.depth ? group_unit(M, g, 0u) : WalkUnit{};
    if (x.quad) {
      w.node = M->path_nodes[(size_t)gr.path_off + (size_t)gr.depth - 2];
      w.quad = true;
      w.levels = gr.depth - 1;
    }
    w.fold_a = x.fold_a;
    w.fold_b = x.fold_b;
    units.push_back(w);
    for (int v = 0; v < x.nv; ++v) {
      const size_t pos = v < gr.depth ? (size_t)gr.path_off + (size_t)v
                                      : (size_t)M->groups[(size_t)g + 1].path_off + (size_t)gr.depth - 1;
      const PathNode &pn = M->path[pos];
      if (pn.first) cols[(size_t)pn.feat].push_back(ColumnEntry{(int32_t)u, x.dst + (v / 4) * 4 * E + v % 4});
    }
  }
  auto column_groups = [&](int per) {
    std::vector<ColumnGroup> groups;
    for (int c0 = 0; c0 < F; c0 += per) {
      ColumnGroup g{c0, std::min(per, F - c0), {}};
      for (int c = c0; c < c0 + g.cols; ++c)
        if (!cols[(size_t)c].empty()) g.lists.push_back({c - c0, &cols[(size_t)c]});
      groups.push_back(std::move(g));
    }
    return groups;
  };
  M->walk.clear();
  for (int per : {64, 16, 4}) {
    // finer levels repeat the programs in more groups: one level for the
    // largest models, and none finer than the first that splits nothing
    if (!M->walk.empty() && ((int64_t)P.xunits.size() > 100000 || F <= per)) continue;
    M->walk.emplace_back(new WalkLevel());
    rc = build_level(M, units, column_groups(per), wide, 4, chunk_units(wide), *M->walk.back());
    if (rc) return rc;
  }
  M->walk_tall.reset();
  if (tall && (int64_t)units.size() <= std::max<int64_t>(kWalkTallUnits, std::min<int64_t>(F, kWalkTallFeatures))) {
    M->walk_tall.reset(new WalkLevel());
    if ((rc = build_level(M, units, column_groups(F), wide, 4, kWalkTallUnits, *M->walk_tall))) return rc;
  }
  return WDF_OK;
}

// Interaction values: column (i, j) at i F + j, one group per feature i.  The
// units are the groups' patterns (the interaction tables are indexed by them).
static int build_iv(wdf_model *M) {
  const int F = M->n_features;
  M->walk_iv.reset();
  if (F > 4096) return WDF_OK;  // the runs that clear F x F columns would be most of the plan
  std::vector<WalkUnit> units(M->groups.size());
  std::vector<std::map<int32_t, std::vector<ColumnEntry>>> lists((size_t)F);
  for (size_t g = 0; g < M->groups.size(); ++g) {
    const Group &gr = M->groups[g];
    const int d = gr.depth;
    if (d < 2) continue;
    units[g] = group_unit(M, (int64_t)g, right_turns(M, gr));
    for (int k1 = 0; k1 < d; ++k1) {
      const PathNode &a = M->path[(size_t)gr.path_off + (size_t)k1];
      for (int k2 = 0; k2 < d && a.first; ++k2) {
        const PathNode &b = M->path[(size_t)gr.path_off + (size_t)k2];
        if (k2 == k1 || !b.first) continue;
        const int lo = std::min(k1, k2), hi = std::max(k1, k2), q = lo * (2 * d - lo - 1) / 2 + (hi - lo - 1);
        lists[(size_t)a.feat][b.feat].push_back(ColumnEntry{(int32_t)g, M->iv_off[g] + ((int64_t)q << d)});
      }
    }
  }
  std::vector<ColumnGroup> groups;
  for (int i = 0; i < F; ++i) {
    ColumnGroup g{(int64_t)i * F, F, {}};
    for (const auto &l : lists[(size_t)i]) g.lists.push_back({l.first, &l.second});
    groups.push_back(std::move(g));
  }
  std::unique_ptr<WalkLevel> L(new WalkLevel());
  const int rc = build_level(M, units, groups, false, 2, chunk_units(false), *L);
  if (rc == WDF_E_UNSUPPORTED) return WDF_OK;
  if (rc) return rc;
  M->walk_iv = std::move(L);
  return WDF_OK;
}

// Units of one segment of the histogram's programs: a chunk of the LDS bins
// holds few deep trees, and whole trees leave waves without work (500 trees of
// depth 3..8, 20k rows: 1.87 ms with whole trees, 1.40 ms with segments of
// eight, which repeat the paths down to them).
constexpr int64_t kHistSegmentUnits = 8;

static int build_hist(wdf_model *M) {
  const int64_t G = (int64_t)M->groups.size();
  Programs prog(M);
  std::vector<WalkUnit> units((size_t)G);
  std::vector<int32_t> list;
  std::vector<int64_t> roots;
  std::vector<WalkHistChunk> chunks;
  for (int64_t g = 0; g < G; ++g) {
    if (M->groups[(size_t)g].depth == 0) roots.push_back(M->groups[(size_t)g].hist_off);
    else units[(size_t)g] = group_unit(M, g, right_turns(M, M->groups[(size_t)g]));
  }
  const int64_t bins = hist_walk_bins(M->n_features);
  for (int64_t g = 0; g < G;) {
    const int64_t bin0 = M->groups[(size_t)g].hist_off;
    list.clear();
    int64_t end = bin0;
    for (; g < G && end - bin0 + ((int64_t)1 << M->groups[(size_t)g].depth) <= bins; ++g) {
      end += (int64_t)1 << M->groups[(size_t)g].depth;
      if (M->groups[(size_t)g].depth) list.push_back((int32_t)g);
    }
    WalkHistChunk ch{bin0, (int32_t)(end - bin0), (int32_t)prog.segs.size(), 0, 0};
    prog.add(units, list.data(), 0, (int64_t)list.size(),
             [&](int64_t k) { return (uint32_t)(M->groups[(size_t)list[(size_t)k]].hist_off - bin0); },
             kHistSegmentUnits);
    ch.seg1 = (int32_t)prog.segs.size();
    chunks.push_back(ch);
  }
  if (prog.ops.size() > 0x7fffffff || chunks.size() > 0x7fffffff)
    return set_error(WDF_E_UNSUPPORTED, "model too large for the data-driven histogram");
  WalkHist &W = M->walk_hist;
  W.n_chunks = (int)chunks.size();
  W.n_roots = (int)roots.size();
  Upload up;
  up.add(prog.ops, W.ops);
  up.add(prog.segs, W.segs);
  up.add(chunks, W.chunks);
  up.add(roots, W.roots);
  return up.run(W.buf, M->ctx->stream);
}

int walk_build_explain(wdf_model *M, bool tall) {
  return guarded([&] { return build_explain(M, tall); });
}
int walk_build_hist(wdf_model *M) {
  return guarded([&] { return build_hist(M); });
}
int walk_build_iv(wdf_model *M) {
  return guarded([&] { return build_iv(M); });
}

int walk_hist(const wdf_model *M, const float *B, int64_t m, int64_t ldb, uint32_t *hist, hipStream_t s) {
  const WalkHist &W = M->walk_hist;
  const int most = 65535;  // chunks of one launch (grid.y)
  for (int c0 = 0; c0 < W.n_chunks; c0 += most) {
    const HistWalkArgs a{B, ldb, m, hist, W.ops, W.segs, W.chunks + c0, W.roots, std::min(most, W.n_chunks - c0),
                         c0 ? 0 : W.n_roots, M->n_features, M->ctx->n_cu};
    HIP_TRY(launch_hist_walk(a, s));
  }
  return WDF_OK;
}

// level L's columns for n rows: the fewest rows per block that stay within two
// blocks per CU, else 64, or 512 (walk_tall)
static int walk_launch(const wdf_model *M, const WalkLevel &L, const float *tab, const float *X, int64_t n, int64_t ldx,
                       float *out, int64_t ldo, hipStream_t s) {
  const int64_t blocks = 2 * (int64_t)M->ctx->n_cu;
  int rows = 1;
  while (rows < 64 && (n + rows - 1) / rows * L.n_groups > blocks) rows *= 4;
  if (walk_tall(L, n)) rows = 512;
  const WalkArgs a{X, ldx, n, out, ldo, tab, L.ops, L.segs, L.groups, L.chunks, L.runs, L.entries, M->n_features, 0};
  HIP_TRY(launch_walk(a, L.n_groups, L.max_slots, L.wide, L.entry_shift, rows, s));
  return WDF_OK;
}

int walk_explain(const wdf_bg *bg, const float *X, int64_t n, int64_t ldx, float *phi, int64_t ldphi, hipStream_t s) {
  const wdf_model *M = bg->model;
  if (M->walk_tall && walk_tall(*M->walk_tall, n))
    return walk_launch(M, *M->walk_tall, bg->d_xtab.as<float>(), X, n, ldx, phi, ldphi, s);
  // the coarsest level whose 64-row blocks fill the device (two per CU), for
  // fewer rows the finest
  const int64_t blocks = 2 * (int64_t)M->ctx->n_cu, tiles = (n + 63) / 64;
  const WalkLevel *L = nullptr;
  for (const auto &l : M->walk) {
    L = l.get();
    if (tiles * L->n_groups >= blocks) break;
  }
  if (!L) return set_error(WDF_E_INVALID_ARG, "explain: no walk plan");
  return walk_launch(M, *L, bg->d_xtab.as<float>(), X, n, ldx, phi, ldphi, s);
}

int walk_explain_iv(const wdf_bg *bg, const float *X, int64_t n, int64_t ldx, float *iv, int64_t ldiv, hipStream_t s) {
  return walk_launch(bg->model, *bg->model->walk_iv, bg->d_tab.as<float>(), X, n, ldx, iv, ldiv, s);
}

}  // namespace wdf
