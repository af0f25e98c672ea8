// Plans of the data-driven kernels (k_walk, k_hist_walk): walk programs for the
// units a block of output columns or a chunk of histogram bins needs.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cstring>
#include <functional>
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
// its slot to out(k).
class Programs {
 public:
  explicit Programs(const wdf_model *M) : M_(M), mark_((size_t)M->n_nodes, -1), at_((size_t)M->n_nodes, -1) {}

  std::vector<WalkOp> ops;
  std::vector<int2> segs;

  void add(const std::vector<WalkUnit> &units, const int32_t *list, int64_t a, int64_t b,
           const std::function<uint32_t(int64_t)> &out, int64_t most = INT64_MAX) {
    for (int64_t k = a; k < b;) {
      const int tree = units[(size_t)list[k]].tree;
      int64_t e = k;
      while (e < b && e - k < most && units[(size_t)list[e]].tree == tree) ++e;
      ++stamp_;
      for (int64_t q = k; q < e; ++q) {
        const WalkUnit &u = units[(size_t)list[q]];
        const Group &g = M_->groups[(size_t)u.group];
        for (int i = 0; i < u.levels; ++i) mark_[(size_t)M_->path_nodes[(size_t)g.path_off + (size_t)i]] = stamp_;
        at_[(size_t)u.node] = q;
      }
      const int64_t op0 = (int64_t)ops.size();
      base_ = M_->node_offset[(size_t)tree];
      have_ = 0;
      visit(base_, 0, units, list, out);
      for (int64_t q = k; q < e; ++q) at_[(size_t)units[(size_t)list[q]].node] = -1;
      while ((ops.size() - (size_t)op0) % 4) ops.push_back(WalkOp{0, 0u, 31u << 8 | 31u << 16, 0u});
      segs.push_back(int2{(int)op0, (int)ops.size()});
      k = e;
    }
  }

 private:
  // test of `node` with `depth` path nodes above it
  void test(int64_t node, int depth) {
    const uint32_t bias = M_->default_left[(size_t)node] ? 0u : 1u;
    uint32_t b;
    std::memcpy(&b, &M_->threshold[(size_t)node], sizeof b);
    ops.push_back(WalkOp{M_->feature[(size_t)node], walk_key_bits(b) - bias,
                         (uint32_t)(have_ - depth) | (bias ? kWalkBias : 0u), 0u});
    have_ = depth + 1;
  }
  void emit(const WalkUnit &u, uint32_t out) {
    WalkOp &o = ops.back();
    o.ctl |= kWalkEmit | (uint32_t)(u.fold_a ? u.fold_a : 31) << 8 | (uint32_t)(u.fold_b ? u.fold_b : 31) << 16;
    o.out = out | u.mask << 20;
  }
  void visit(int64_t node, int depth, const std::vector<WalkUnit> &units, const int32_t *list,
             const std::function<uint32_t(int64_t)> &out) {
    if (mark_[(size_t)node] != stamp_) return;
    test(node, depth);
    const int64_t L = base_ + M_->left[(size_t)node], R = base_ + M_->right[(size_t)node];
    const int64_t k = at_[(size_t)node];
    if (k >= 0) {
      const WalkUnit &u = units[(size_t)list[k]];
      if (u.quad) {
        test(L, depth + 1);
        test(R, depth + 2);
      }
      emit(u, out(k));
      if (u.quad) return;
    }
    if (M_->feature[(size_t)L] >= 0) visit(L, depth + 1, units, list, out);
    if (M_->feature[(size_t)R] >= 0) visit(R, depth + 1, units, list, out);
  }

  const wdf_model *M_;
  std::vector<int64_t> mark_, at_;
  int64_t stamp_ = 0, base_ = 0;
  int have_ = 0;  // splits in P
};

template <class T>
int upload(DevBuf &buf, const std::vector<T> &v, hipStream_t s) {
  const int rc = buf.alloc(std::max<size_t>(v.size(), 1) * sizeof(T));
  if (rc || v.empty()) return rc;
  HIP_TRY(hipMemcpyAsync(buf.ptr, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice, s));
  HIP_TRY(hipStreamSynchronize(s));
  return WDF_OK;
}

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

constexpr int kZeroRun = 32;  // columns one wave clears at a time

int build_level(const wdf_model *M, const std::vector<WalkUnit> &units, const std::vector<ColumnGroup> &groups,
                bool wide, int entry_shift, WalkLevel &out) {
  const int cap = kWalkPatternBytes / 64 / (wide ? 2 : 1);
  Programs prog(M);
  std::vector<WalkGroup> gs;
  std::vector<WalkChunk> chunks;
  std::vector<WalkRun> runs;
  std::vector<WalkEntry> entries;
  std::vector<int32_t> slot(units.size(), -1);
  int most = 0;
  for (const ColumnGroup &cg : groups) {
    std::vector<int32_t> need;
    for (const auto &l : cg.lists)
      for (const ColumnEntry &e : *l.second) need.push_back(e.unit);
    std::sort(need.begin(), need.end());
    need.erase(std::unique(need.begin(), need.end()), need.end());
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
  hipStream_t s = M->ctx->stream;
  int rc;
  if ((rc = upload(out.ops, prog.ops, s)) || (rc = upload(out.segs, prog.segs, s)) ||
      (rc = upload(out.groups, gs, s)) || (rc = upload(out.chunks, chunks, s)) || (rc = upload(out.runs, runs, s)) ||
      (rc = upload(out.entries, entries, s)))
    return rc;
  return WDF_OK;
}

}  // namespace

// Levels of the explain walk, coarse to fine: columns (features) per block.  A
// coarse level computes a unit's slot for few blocks of columns, a fine one
// spreads few rows over more blocks; each is used for the row counts where its
// blocks just fill the device (launch).
static const int kWalkColumns[] = {64, 16, 4};

static int build_explain(wdf_model *M) {
  JitPlan &P = M->jp;
  const int F = M->n_features;
  int rc;
  if ((rc = upload(P.d_xunits, P.xunits, M->ctx->stream)) || (rc = upload(P.d_unit_g0, P.unit_g0, M->ctx->stream)))
    return rc;
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
  M->walk.clear();
  for (int per : kWalkColumns) {
    // finer levels repeat the programs in more groups: one level for the
    // largest models, and none finer than the first that splits nothing
    if (!M->walk.empty() && ((int64_t)P.xunits.size() > 100000 || F <= per)) continue;
    std::vector<ColumnGroup> groups;
    for (int c0 = 0; c0 < F; c0 += per) {
      ColumnGroup g{c0, std::min(per, F - c0), {}};
      for (int c = c0; c < c0 + g.cols; ++c)
        if (!cols[(size_t)c].empty()) g.lists.push_back({c - c0, &cols[(size_t)c]});
      groups.push_back(std::move(g));
    }
    M->walk.emplace_back(new WalkLevel());
    rc = build_level(M, units, groups, wide, 4, *M->walk.back());
    if (rc) return rc;
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
  const int rc = build_level(M, units, groups, false, 2, *L);
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
  for (int64_t g = 0; g < G;) {
    const int64_t bin0 = M->groups[(size_t)g].hist_off;
    list.clear();
    int64_t end = bin0;
    for (; g < G && end - bin0 + ((int64_t)1 << M->groups[(size_t)g].depth) <= kHistWalkBins; ++g) {
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
  hipStream_t s = M->ctx->stream;
  int rc;
  if ((rc = upload(W.ops, prog.ops, s)) || (rc = upload(W.segs, prog.segs, s)) || (rc = upload(W.chunks, chunks, s)) ||
      (rc = upload(W.roots, roots, s)))
    return rc;
  return WDF_OK;
}

int walk_build_explain(wdf_model *M) {
  return guarded([&] { return build_explain(M); });
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
    const HistWalkArgs a{B, ldb, m, hist, W.ops.as<WalkOp>(), W.segs.as<int2>(), W.chunks.as<WalkHistChunk>() + c0,
                         W.roots.as<int64_t>(), std::min(most, W.n_chunks - c0), c0 ? 0 : W.n_roots, M->n_features,
                         M->ctx->n_cu};
    HIP_TRY(launch_hist_walk(a, s));
  }
  return WDF_OK;
}

// level L's columns for n rows: the fewest rows per block that stay within two
// blocks per CU, else 64
static int walk_launch(const wdf_model *M, const WalkLevel &L, const float *tab, const float *X, int64_t n, int64_t ldx,
                       float *out, int64_t ldo, hipStream_t s) {
  const int64_t blocks = 2 * (int64_t)M->ctx->n_cu;
  int rows = 1;
  while (rows < 64 && (n + rows - 1) / rows * L.n_groups > blocks) rows *= 4;
  const WalkArgs a{X, ldx, n, out, ldo, tab, L.ops.as<WalkOp>(), L.segs.as<int2>(), L.groups.as<WalkGroup>(),
                   L.chunks.as<WalkChunk>(), L.runs.as<WalkRun>(), L.entries.as<WalkEntry>(), M->n_features, 0};
  HIP_TRY(launch_walk(a, L.n_groups, L.max_slots, L.wide, L.entry_shift, rows, s));
  return WDF_OK;
}

int walk_explain(const wdf_bg *bg, const float *X, int64_t n, int64_t ldx, float *phi, int64_t ldphi, hipStream_t s) {
  const wdf_model *M = bg->model;
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
