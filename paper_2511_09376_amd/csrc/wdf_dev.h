// Device-side layouts shared by the host code and the static kernels.
#pragma once
#include <stdint.h>

namespace wdf {

// One inner node on a group's path.
struct PathNode {
  float thr;        // x < thr goes left
  int32_t feat;     // split feature
  uint8_t dl;       // NaN goes left when nonzero
  uint8_t dir;      // 0: the group's path continues to the left child, 1: right
  uint8_t merge;    // index of the node's feature among the path's distinct features
  uint8_t first;    // 1 when this is the first node of the path carrying the feature
};

// A group: two sibling leaves (pair) or one leaf whose sibling is an inner node
// (single).  A pair's pattern is the left leaf's; the right leaf's is p ^ 1.
struct Group {
  int32_t tree;
  int32_t depth;      // inner nodes on the path, 0..8
  int32_t dprime;     // distinct features on the path
  int32_t path_off;   // first PathNode of the path
  int64_t hist_off;   // 2^depth histogram bins
  int64_t tab_off;    // depth * 2^depth table entries, position-major
  int32_t col_l;      // contraction column of the left (or single) leaf in its class
  int32_t col_r;      // column of the right leaf, -1 for a single
  float w_l, w_r;     // leaf values (w_r = 0 for a single)
};

// A unit of the explain tables: a group's table, or a "quad": the two pair
// groups below the children of one node, merged into one table indexed by
// (path prefix, split at the node, split at its left child, split at its right
// child) with d + 1 values per entry (d = the pairs' depth).  Explain tables
// are indexed by raw splits (bit 1: the row went left), not by whether the row
// follows the path; `mask` holds the path's right turns, so the pattern of a
// raw index r is r ^ mask.  Layout: E = 2^(depth + quad) entries of nv values,
// stored as ceil(nv / 4) float4 planes [plane][slot], value v in component
// v % 4 of plane v / 4 (unused components 0), so that one 16-byte LDS read
// returns four values of an entry; entry I sits at slot
// I ^ (I >> fold_a) ^ (I >> fold_b) of each plane (a bijection), the shifts
// chosen per unit so that the entries rows are likely to read together fall
// in different groups of LDS banks.
struct XUnit {
  int64_t dst;     // offset in the explain tables (floats, multiple of 4)
  int32_t depth;   // depth of the group(s)
  int32_t quad;    // 1 for a quad
  uint32_t mask;   // right turns: all d positions of a group, the d - 2 prefix positions of a quad
  int32_t nv;      // values per entry: depth + quad
  int32_t fold_a;  // entry I sits at slot I ^ (I >> fold_a) ^ (I >> fold_b) of each plane (0: no term)
  int32_t fold_b;
};

// slot of entry I in a plane of an explain-table unit
constexpr int xunit_slot(const XUnit &u, int I) {
  return I ^ (u.fold_a ? I >> u.fold_a : 0) ^ (u.fold_b ? I >> u.fold_b : 0);
}

// floats of a unit in the explain tables
inline int64_t xunit_floats(const XUnit &u) {
  return 4 * (int64_t)((u.nv + 3) / 4) * ((int64_t)1 << (u.depth + u.quad));
}

// A unit of the specialised interaction tables: one group and one feature i
// at its first path position, with the pair tables of i and each other first
// position (its partners, in path order).  The tables are indexed by the raw
// splits r of the group's path (bit 1: the row went left; the pattern is
// r ^ mask) and stored as planes [plane][slot][width]: 4-wide planes for
// partners 0..3, 4..7 (a last group of three partners takes a 4-wide plane
// with one zero), then one 2- or 1-wide plane for a remaining two or one, so
// that a unit of five partners costs one 16-byte and one 4-byte read.  Entry r
// sits at slot r ^ (r >> 3) ^ (r >> 6) of every plane (a bijection on d bits),
// which spreads entries sharing their low three bits (one group of LDS banks
// for 16-byte rows) over all groups.
struct IvUnit {
  int64_t src;     // the group's pair tables (interaction-table offset)
  int64_t dst;     // offset in the interleaved tables (floats, multiple of 4)
  int32_t depth;   // path positions of the group
  int32_t cnt;     // partners, 1..7
  int32_t q[7];    // pair index of (i, partner s) among the group's position pairs
  int32_t group;   // the group
  uint32_t mask;   // right turns of the group's path, root first (MSB)
};

// 4-wide planes of a unit with cnt partners, and the width of its narrow plane (0, 1 or 2)
constexpr int ivunit_quads(int cnt) { return cnt / 4 + (cnt % 4 == 3 ? 1 : 0); }
constexpr int ivunit_tail(int cnt) { return cnt % 4 == 3 ? 0 : cnt % 4; }
// slot of raw index r in every plane
constexpr uint32_t ivunit_slot(uint32_t r) { return r ^ (r >> 3) ^ (r >> 6); }

// floats of a unit in the interleaved interaction tables (a multiple of 4)
constexpr int64_t ivunit_floats(const IvUnit &u) {
  return (((int64_t)(4 * ivunit_quads(u.cnt) + ivunit_tail(u.cnt)) << u.depth) + 3) & ~(int64_t)3;
}

// The data-driven kernels (k_walk, k_hist_walk) run walk programs: one op per
// tested node of a tree, depth first, on a wave of 64 rows (one per lane).  A
// lane keeps the raw splits of its current path in one register P (root in
// the top bit, bit 1: the row went left); an op drops the levels the walk went
// back up, shifts its split in and, at the last node of a unit, hands out the
// unit's index I = P as slot I ^ (I >> fold_a) ^ (I >> fold_b) ^ mask.
struct WalkOp {
  int32_t feat;
  uint32_t key;   // walk_key(threshold) - bias: the row goes left iff walk_key(x) - bias < key (unsigned)
  uint32_t ctl;   // bits 0-3 levels to drop, bit 4 bias (1: a NaN goes right), bit 5 emit, 8-12 fold_a, 16-20 fold_b (31: no term)
  uint32_t out;   // bits 0-19 where the slot goes (a pattern row of the chunk, or its first bin), 20-31 mask
};
constexpr uint32_t kWalkBias = 1u << 4, kWalkEmit = 1u << 5;
// levels dropped by a segment's first op: all that P may hold (a path, a quad's
// two splits and the padding of a segment), so that segments may run on one
// after another
constexpr int kWalkDropAll = 15;

// Totally ordered image of a float: x < y iff walk_key(x) < walk_key(y), both
// zeros alike, every NaN 0 (below all numbers; a bias of 1 wraps it above them).
constexpr uint32_t walk_key_bits(uint32_t b) {
  return (b & 0x7fffffffu) > 0x7f800000u ? 0u : b == 0x80000000u ? 0x80000000u : (b >> 31) ? ~b : b | 0x80000000u;
}

// One group of output columns: the column range and its chunks of units.
struct WalkGroup {
  int64_t col0;
  int32_t chunk0, chunk1;
};
// Units whose patterns a block holds in LDS together: the tree segments that
// compute them (op ranges) and the column runs that read them.
struct WalkChunk {
  int32_t seg0, seg1, run0, run1;
};
// Zeros for columns [zero0, col), then the sum of entries [e0, e1) for column
// col (none when empty); columns are relative to the group's.
struct WalkRun {
  int32_t zero0, col, e0, e1;
};
// One table value: pattern row slot4 >> 2 of the chunk, tables at float
// 4 tab16 + (slot4 & 3).
struct WalkEntry {
  uint32_t slot4, tab16;
};
// A chunk of the data-driven histogram: groups whose bins fit the LDS.
struct WalkHistChunk {
  int64_t bin0;
  int32_t bins, seg0, seg1, pad;
};

}  // namespace wdf
