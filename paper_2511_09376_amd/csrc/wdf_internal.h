// Internal declarations shared by the host code and the static kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "wdf_dev.h"

namespace wdf {

// The data-driven histogram: hist += counts of the rows of B, chunk by chunk
// of groups; root_bins: the one bin of every tree that is a single leaf.
struct HistWalkArgs {
  const float *X;
  int64_t ldx, m;
  uint32_t *hist;
  const WalkOp *ops;
  const int2 *segs;
  const WalkHistChunk *chunks;
  const int64_t *root_bins;
  int n_chunks, n_root_bins, F, n_cu;
};
constexpr int kWalkXFeatures = 160;  // row keys staged in LDS up to this many features (64 rows: 40 KB)
// LDS of the data-driven histogram: a chunk's bins and 64 rows' keys, so that
// two blocks fit a CU: 12288 bins up to 128 features, fewer up to 160 (refresh of
// 500 uneven trees of 150 features, 100k rows: 7.65 ms with 12288 bins and the
// one block per CU that fits then, 5.22 with 10880; of 128 features 4.31)
constexpr int hist_walk_key_bytes(int F) { return F <= kWalkXFeatures ? F * 64 * 4 : 0; }
constexpr int hist_walk_bins(int F) {
  const int fit = (80 * 1024 - hist_walk_key_bytes(F)) / 4;
  return fit < 12288 ? fit : 12288;
}
constexpr bool hist_walk_two_blocks_fit() {
  for (int F = 1; F <= kWalkXFeatures + 1; ++F)
    if (2 * (hist_walk_bins(F) * 4 + hist_walk_key_bytes(F)) > 160 * 1024) return false;
  return true;
}
static_assert(hist_walk_two_blocks_fit(), "launch_hist_walk plans two blocks per CU");
hipError_t launch_hist_walk(const HistWalkArgs &a, hipStream_t s);
// The data-driven gather: column c of out (out[c * ldo + row]) is the sum of
// its table entries.
struct WalkArgs {
  const float *X;
  int64_t ldx, n;
  float *out;
  int64_t ldo;
  const float *tab;
  const WalkOp *ops;
  const int2 *segs;
  const WalkGroup *groups;
  const WalkChunk *chunks;
  const WalkRun *runs;
  const WalkEntry *entries;
  int F, x_off;  // x_off: byte offset of the row keys in LDS (-1: keys read from X)
};
// wide: pattern rows of 16-bit slots (else 8-bit); entry_shift: log2 of the
// bytes between consecutive slots of a table plane; rows per block: 1, 4, 16,
// 64 or 512
// LDS sizes of the data-driven kernels on the current device (once per context)
hipError_t walk_init();
hipError_t launch_walk(WalkArgs a, int n_groups, int max_slots, bool wide, int entry_shift, int rows, hipStream_t s);
hipError_t launch_patterns(const Group *groups, const PathNode *path, int64_t n_groups, const float *X,
                           int64_t n, int64_t ldx, uint32_t *out, hipStream_t s);
hipError_t launch_columns(const Group *groups, const PathNode *path, int64_t n_groups, const uint32_t *hist,
                          const double *freq, const double *freq_r, double scale, const int64_t *class_off, double *H,
                          hipStream_t s);
// The FP64 products of up to kGemmMaxClasses distinct-feature classes in one
// launch: class i owns waves [c[i].wave0, c[i].wave0 + its 32x32 blocks).
// K is a power of two; for K >= 16, M and H rows must be 16-byte aligned.
constexpr int kGemmMaxClasses = 8;
struct GemmClass {
  const double *M;  // R x K, row-major
  const double *H;  // ncols x K
  double *S;        // ncols x R
  int R, K, ncols, wave0;
};
struct GemmBatch {
  GemmClass c[kGemmMaxClasses];
  int n;
};
// 32x32 output blocks (waves) of one class
inline int gemm_waves(int R, int ncols) { return ((R + 31) / 32) * ((ncols + 31) / 32); }
hipError_t launch_gemm_f64(const GemmBatch &batch, int waves, hipStream_t s);
// The base value: hist, or freq and freq_r (path-dependent).
struct BaseArgs {
  const Group *groups;
  int64_t n_groups;
  const uint32_t *hist;
  const double *freq, *freq_r;
  double scale;
  double *out;
};
hipError_t launch_base(const BaseArgs &b, hipStream_t s);
// gather tables (tab null: none), explain tables and the base value; unit_g0: first group of every unit
hipError_t launch_tables(const XUnit *units, const int64_t *unit_g0, int64_t n_units, const Group *groups,
                         const PathNode *path, const int64_t *s_class_off, const double *S, float *tab, float *xtab,
                         const BaseArgs &base, hipStream_t s);
hipError_t launch_pd_freq(const Group *groups, int64_t n_groups, const double *ratio, const double *ratio_r,
                          double *freq, double *freq_r, hipStream_t s);
// (also clears hist[0, hist_size))
hipError_t launch_quantize(const float *X, int64_t n, int64_t ldx, int F, const float *thr_pad, const int2 *meta,
                           int wide, int words, uint32_t *codes, int64_t ldc, uint32_t *hist, int64_t hist_size,
                           hipStream_t s);
hipError_t launch_expand_iv(const Group *groups, const PathNode *path, int64_t n_groups, const int64_t *iv_off,
                            const int64_t *s_class_off, const double *S, float *tab, hipStream_t s);
hipError_t launch_ivtab(const IvUnit *units, int64_t n_units, const float *tab, float *t2, hipStream_t s);
// patterns of every group into pat (n_groups * n bytes), then the interaction kernel
hipError_t launch_explain_iv(const Group *groups, const PathNode *path, int64_t n_groups, const int32_t *item_off,
                             const int2 *items, const float *tab, const float *X, int64_t n, int64_t ldx, uint8_t *pat,
                             float *out, int64_t ldo, int F, hipStream_t s);
hipError_t launch_fill_u32(uint32_t *p, int64_t n, uint32_t v, hipStream_t s);
// device address, on the current device, of the library's scratch array
// (WDF_NOALLOC_SCRATCH_BYTES bytes) used by the entry points that allocate nothing
hipError_t scratch_address(void **out);

}  // namespace wdf
