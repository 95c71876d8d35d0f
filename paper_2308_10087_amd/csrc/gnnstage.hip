// C-ABI entry points of the stage library: descriptor validation, workspace layout, host
// planning at create time, and the per-chunk launch sequences (Algorithm 1's inner loops and
// the matching backward pass).  All device work is issued on the caller's stream.
#include <stdio.h>
#include "guard.h"
#include <memory>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <string>
#include <utility>
#include <vector>

#include "../../include/gnnstage.h"
#include "common.h"
#include "plan.h"

namespace {

// Row splits of a weight-gradient product (fp32 partial outputs, added in a fixed order).  512 = two workgroups per CU in
// one round: measured on the 2.45 M x 128 x 128 products of the 8-layer configuration, 256 / 384 / 512 / 640 / 768 /
// 1024 splits take 3.08 / 2.62 / 2.56 / 3.24 / 3.01 / 2.91 ms per step.
constexpr int kMaxSplits = 512;
constexpr size_t kAlign = 256;
// Rows of a GraphSage layer whose two products follow each other (the first one's rows are fp32 and are read by the second).
constexpr int64_t kSelfRows = 65536;
// Short rows of a launch, per column, from which they go four to a wave.  With fewer the rows' waves are in flight at one time, and
// four rows one after the other only make the launch's one chain longer.  A row to a wave / four, a pass of two layers in us:
// width 64 4 k rows 80 / 81, 8 k 92 / 91, 12 k 98 / 93; width 128 4 k 90 / 92, 8 k 97 / 98, 12 k 105 / 101; width 256 6 k 113 / 118,
// 12 k 128 / 130, 24 k 173 / 164.  Chunk calls of 75 rows of width 256: 2,160 / 2,613 us for 40 of them.
constexpr int64_t kShortRowsPerColumn = 64;

std::string g_create_error;

// Measurement and test switches.  Defaults are the product path.  The environment is read ONCE per
// gnnstage_workspace_size / gnnstage_create call (both must see the same values) and the result is kept in
// the handle; nothing on the launch path looks at the environment.
//   GNNSTAGE_SPLIT_EDGES (>= 64)      fixed length of the pieces long rows are cut into
//   GNNSTAGE_XCD_CLASSES (1..32)      source-id classes (1 = off)
//   GNNSTAGE_CLASS_MIN_ROW            rows from this length on are cut by class
//   GNNSTAGE_DENSE=0                  no dense blocks
//   GNNSTAGE_DENSE_MIN_NNZ            entries a 128 x 64 block needs to be multiplied as a dense block
//   GNNSTAGE_DENSE_MIN_SHARE          share of all entries that must fall into such blocks
//   GNNSTAGE_DENSE_MIN_ENTRIES        dense entries per chunk below which the plan stays off
//   GNNSTAGE_ORDER=aggregate|transform  one layer order for every GCN layer
//   GNNSTAGE_SPMM_VALU                vector-ALU aggregation for bf16 rows too
//   GNNSTAGE_SPMM_UNROLL (2, 4, 8)    gather slots per wave of the matrix-core aggregation
//   GNNSTAGE_GEMM_WS_MIN_ROWS         rows from which the weight-stationary product is used
//   GNNSTAGE_GEMM_WIDE_MIN_ROWS       rows from which a weight-gradient product of up to 256 x 256 outputs is one workgroup per split
//   GNNSTAGE_WGRAD_DEFER=0            weight gradients per chunk instead of one product per layer at the end of the pass
//   GNNSTAGE_HOT_CLASSES (0 = off, 2..32: on whatever the table size)   classes of the hottest sources
//   GNNSTAGE_HOT_ROWS                 sources per such class
//   GNNSTAGE_HOT_MIN_ROW              rows from this length on are cut by hotness class
//   GNNSTAGE_SHORT_ROW (0 = off, up to 16)   whole rows of at most this many entries are served four to a wave, however few of them
//   GNNSTAGE_LAUNCH_BLOCKS            workgroups that one aggregation launch over several chunks may have
//   GNNSTAGE_PARTIAL_ROOM             bytes for partial rows, and as many for dense tiles, beyond those of the largest chunk
struct Tuning {
  int split_edges = 0;          // 0: from the launch size
  int xcd_classes = 0;          // 0: from the size of the gathered table
  int class_min_row = 128;      // measured: shorter rows than this cost more in partial sums than their locality gains
  bool dense = true;
  int dense_min_nnz = 0;        // 0: the defaults below
  double dense_min_share = 0.2;
  double dense_min_entries = 2e6;
  int order = 0;                // 0 auto, 1 aggregate first, 2 transform first
  bool spmm_valu = false;
  int spmm_unroll = 2;          // two slots leave room for eight waves per SIMD, which measured best on every workload
  int gemm_ws_min_rows = 65536;
  int gemm_wide_min_rows = 65536;  // weight-gradient products from this many rows on read each operand once (one workgroup per split)
  bool wgrad_defer = true;
  int hot_classes = -1;         // -1: 16 for gathered tables beyond 256 MB, none below
  int hot_rows = 0;             // 0: as many rows as fit an XCD's 4 MB L2
  int hot_min_row = 2048;       // measured on the 10 M vertex graph: 512 -> 142.8, 1024 -> 140.6, 2048 -> 140.4 ms per step (off: 143.2)
  // whole rows of at most this many entries are served four to a wave (0: none; -1: see Shape::short_row)
  int short_row = -1;
  int64_t launch_blocks = kMostBlocks;
  int64_t partial_room = -1;    // -1: see make_layout
};

Tuning read_tuning() {
  Tuning t;
  const char *e;
  if ((e = getenv("GNNSTAGE_SPLIT_EDGES")) && atoi(e) >= 64) t.split_edges = atoi(e);
  if ((e = getenv("GNNSTAGE_XCD_CLASSES")) && atoi(e) >= 1 && atoi(e) <= kMaxClasses) t.xcd_classes = atoi(e);
  if ((e = getenv("GNNSTAGE_CLASS_MIN_ROW")) && atoi(e) >= 1) t.class_min_row = atoi(e);
  if ((e = getenv("GNNSTAGE_DENSE")) && atoi(e) == 0) t.dense = false;
  if ((e = getenv("GNNSTAGE_DENSE_MIN_NNZ")) && atoi(e) >= 1) t.dense_min_nnz = atoi(e);
  if ((e = getenv("GNNSTAGE_DENSE_MIN_SHARE"))) t.dense_min_share = atof(e);
  if ((e = getenv("GNNSTAGE_DENSE_MIN_ENTRIES"))) t.dense_min_entries = atof(e);
  if ((e = getenv("GNNSTAGE_ORDER"))) t.order = !strcmp(e, "aggregate") ? 1 : !strcmp(e, "transform") ? 2 : 0;
  if (getenv("GNNSTAGE_SPMM_VALU")) t.spmm_valu = true;
  if ((e = getenv("GNNSTAGE_SPMM_UNROLL"))) t.spmm_unroll = atoi(e);
  if ((e = getenv("GNNSTAGE_GEMM_WS_MIN_ROWS"))) t.gemm_ws_min_rows = atoi(e);
  if ((e = getenv("GNNSTAGE_GEMM_WIDE_MIN_ROWS"))) t.gemm_wide_min_rows = atoi(e);
  if ((e = getenv("GNNSTAGE_WGRAD_DEFER")) && atoi(e) == 0) t.wgrad_defer = false;
  if ((e = getenv("GNNSTAGE_HOT_CLASSES")) && atoi(e) >= 0 && atoi(e) <= kMaxClasses) t.hot_classes = atoi(e);
  if ((e = getenv("GNNSTAGE_HOT_ROWS")) && atoi(e) >= 1) t.hot_rows = atoi(e);
  if ((e = getenv("GNNSTAGE_HOT_MIN_ROW")) && atoi(e) >= 1) t.hot_min_row = atoi(e);
  if ((e = getenv("GNNSTAGE_SHORT_ROW")) && atoi(e) >= 0) t.short_row = std::min(atoi(e), kShortRowMost);
  if ((e = getenv("GNNSTAGE_LAUNCH_BLOCKS")) && atoll(e) >= 1) t.launch_blocks = std::min<int64_t>(atoll(e), kMostBlocks);
  if ((e = getenv("GNNSTAGE_PARTIAL_ROOM")) && atoll(e) >= 0) t.partial_room = atoll(e);
  return t;
}

// Forward aggregations of fp32 stages.  What ReLU passes hangs on the last bit of a pre-activation: a stage of 5 k vertices
// of width 1000 has one or two of 20 M elements so close to zero that another order of the same sum decides otherwise, and one
// such element moves a weight gradient by 2e-3.  So these pieces don't get shorter with the launch: 256 entries at least, as in
// large launches (4.2 M entries and more: longer, see below).  The order of a row's sum follows from the plan of its chunk and the
// row width alone: the pieces (rows of class_min_row entries and more are cut at source-class bounds too, which depend on the
// chunk's entries), the lane groups of the kernel, the phases of the reduce.  (Pieces of 32 here: 6.7 against 7.1 ms per step
// of that stage.)
constexpr int kLeastPieceF32Fwd = 256;

// Longest piece of a row that one wavefront handles in an aggregation over `entries` entries.  A wave
// streams roughly 16 entries per microsecond, so the longest task bounds the tail of the launch: pieces
// shrink with the launch (about 16k pieces' worth of work per launch), within [least, 4096].
int split_edges_for(const Tuning &t, int64_t entries, int least) {
  if (t.split_edges >= 64) return t.split_edges;
  const int64_t step = least == kLeastPieceF32Fwd ? 64 : least;
  int64_t s = (entries / 16384 + step - 1) / step * step;
  if (s < least) s = least;
  if (s > 4096) s = 4096;
  return (int)s;
}

// Source-id classes (one per XCD) pay when one class's slice of the gathered table has a chance to
// live in an XCD's L2 and the memory-side cache; for tables far beyond that they only add partial sums.
int xcd_classes_setting(const Tuning &t, int64_t table_bytes) {
  if (t.xcd_classes >= 1) return t.xcd_classes;
  return table_bytes <= (int64_t)256 << 20 ? 8 : 1;
}

// Hotness classes, for tables that fit no cache.  On a power-law graph a small set of sources takes a large share
// of all gathers (10 M vertices, 21 entries per row: the 130 k most frequent sources are 45 % of the entries), but
// between two uses of such a row an XCD streams far more than its 4 MB L2 holds.  So the hottest sources are cut
// into classes of as many rows as fit one L2, long rows get their entries ordered by hotness and are cut at the
// class bounds, and the pieces of a class run together on one XCD (the class machinery above): a hot row is
// fetched once per launch and XCD instead of once per use.  The rest of every row, and all short rows, gather
// as before.  Off when id-range classes are forced (GNNSTAGE_XCD_CLASSES).
int hot_classes_setting(const Tuning &t, int64_t table_bytes) {
  if (t.xcd_classes >= 1) return 0;
  if (t.hot_classes >= 0) return t.hot_classes >= 2 ? t.hot_classes : 0;
  return table_bytes > (int64_t)256 << 20 ? 16 : 0;
}
int64_t hot_rows_setting(const Tuning &t, int64_t row_bytes) {
  if (t.hot_rows >= 1) return t.hot_rows;
  return std::max<int64_t>(64, ((int64_t)4 << 20) / std::max<int64_t>(row_bytes, 1));
}

// Lower bounds of the source-id classes: equal id ranges, except that a bound moves onto a chunk boundary
// that lies within a quarter of a class width of it.  Chunks that line up with classes (equal chunks, a
// multiple of the class count) then never straddle two classes, and a backward launch touches exactly the
// classes of its processed chunks.
std::vector<int64_t> class_bounds(int64_t n, int classes, const std::vector<int64_t> &chunk_ptr) {
  std::vector<int64_t> lo((size_t)classes + 1);
  for (int q = 0; q <= classes; ++q) lo[(size_t)q] = ((int64_t)q * n + classes - 1) / classes;
  const int64_t tol = n / (4 * (int64_t)classes);
  for (int q = 1; q < classes; ++q) {
    int64_t best = -1;
    for (const int64_t cb : chunk_ptr)
      if (std::llabs(cb - lo[(size_t)q]) <= tol && (best < 0 || std::llabs(cb - lo[(size_t)q]) < std::llabs(best - lo[(size_t)q])))
        best = cb;
    if (best > 0 && best < n) lo[(size_t)q] = best;
  }
  return lo;
}

// Class bounds for the rows [r0, r1) of an index (one chunk's launch): equal shares of those rows' ENTRIES rather than
// of the id range, so that a chunk whose neighbours cluster in a few id ranges (chunks from a locality-aware
// partitioner: about half of a chunk's neighbours are its own vertices) still spreads over all classes, its heavy
// range cut into slices that fit an L2.  A bound moves to a chunk boundary that lies within a quarter of a class share
// (in entries): classes made of whole chunks are skipped as a whole by launches that drop those chunks.  On a
// uniformly numbered graph this gives the equal, chunk-aligned id ranges of class_bounds.
std::vector<int64_t> class_bounds_by_entries(const int64_t *ptr, const int32_t *idx, int64_t n, int64_t r0, int64_t r1, int classes,
                                             const std::vector<int64_t> &chunk_ptr) {
  if (classes <= 1 || idx == nullptr || ptr[r1] == ptr[r0]) return class_bounds(n, classes, chunk_ptr);
  std::vector<int64_t> mass((size_t)n + 1, 0);  // mass[u + 1] = entries of these rows whose source is u, then prefix sums
  for (int64_t e = ptr[r0]; e < ptr[r1]; ++e) mass[(size_t)idx[e] + 1] += 1;
  for (int64_t u = 0; u < n; ++u) mass[(size_t)u + 1] += mass[(size_t)u];
  const int64_t total = mass[(size_t)n];
  const int64_t tol = total / (4 * (int64_t)classes);
  std::vector<int64_t> lo((size_t)classes + 1, 0);
  lo[(size_t)classes] = n;
  for (int q = 1; q < classes; ++q) {
    const int64_t target = total / classes * q + total % classes * q / classes;
    int64_t b = std::lower_bound(mass.begin(), mass.end(), target) - mass.begin();
    int64_t best = -1;
    for (const int64_t cb : chunk_ptr) {
      const int64_t dist = std::llabs(mass[(size_t)cb] - target);
      if (cb > 0 && cb < n && dist <= tol && (best < 0 || dist < std::llabs(mass[(size_t)best] - target))) best = cb;
    }
    if (best >= 0) b = best;
    lo[(size_t)q] = std::min<int64_t>(std::max<int64_t>(b, lo[(size_t)q - 1]), n);
  }
  return lo;
}

// Dense blocks: switched on for bf16 stages whose aggregations all gather rows of width 128 or 256.
// Threshold: entries a 128 x 64 block needs; default: from 3.4 % of its cells upwards, as low as the chunk's launch
// still fits one round of workgroups, 5 % for a chunk that needs several (see dense_max_items); the same for blocks
// kept as weight tiles, whose curve is flat from 278 to 500: 18.7 - 18.9 ms per c1 step with the caller's weights.
int dense_min_nnz(const Tuning &t) { return t.dense_min_nnz >= 1 ? t.dense_min_nnz : kDenseRB * kDenseCB * 34 / 1000; }
// for a chunk whose launch needs several rounds of workgroups: every block costs time there
int dense_min_nnz_many(const Tuning &t) { return t.dense_min_nnz >= 1 ? t.dense_min_nnz : kDenseRB * kDenseCB / 20; }
// Items (runs of at most 32 blocks of one row block) of a launch that fits one round of workgroups: one workgroup
// per item and 128-column half, two workgroups per CU, 256 CUs; a tenth more is harmless because short items end
// early.  Such a launch takes as long as its longest item, so blocks down to the low threshold are free; beyond it
// the extra workgroups wait for a second round.
int64_t dense_max_items(int widest) { return (int64_t)(2 * 256 * 11 / 10) / std::max(1, widest / 128); }
// A dense launch has a fixed cost (its longest item runs 32 blocks one after the other, some tens of
// microseconds); it only pays when it takes a lot of entries off the sparse kernel: at least
// Tuning::dense_min_entries per chunk on average (the sparse kernel gathers about 40 entries per nanosecond).
constexpr int kDenseItemBlocks = kDenseMaxItemBlocks;

// Launch schedule of one direction.  The task arrays are made of sections, each chunk after chunk: the pieces of source class 0,
// 1, ..., then pieces without a class and whole rows, then short rows.  So a launch over any run of chunks finds each section's
// tasks in one stretch.
struct DirTasks {
  int K = 0;
  int n_classes = 0;               // 0: no class sections
  std::vector<int64_t> sec;        // [section][K + 1]: first task of every chunk
  std::vector<int64_t> slot_off, lr_off, item_off;  // K + 1: partial rows, cut rows, dense items of the chunks
  // entries of every chunk's class pieces by the chunk of the gathered vertex ([chunk][class][source chunk]): what a launch
  // that drops unselected entries really gathers from each class
  std::vector<int64_t> cls_entries, cls_total;  // cls_total: of all source chunks, [chunk][class]
  int64_t first(int section, int c) const { return sec[(size_t)section * (K + 1) + c]; }
  int64_t count(int section, int c0, int c1) const { return first(section, c1) - first(section, c0); }
  int64_t total(int c, int q) const { return cls_total[(size_t)c * n_classes + q]; }
  int64_t selected(int c, int q, const int64_t *sel) const {  // of the source chunks whose word is ~0 (the others' are 0)
    const int64_t *e = &cls_entries[((size_t)c * n_classes + q) * K];
    int64_t sum = 0;
    for (int i = 0; i < K; ++i) sum += e[i] & sel[i];
    return sum;
  }
};

// Sizes that depend only on row lengths: number of tasks / long rows / slots of every chunk.
struct PlanCounts {
  std::vector<int64_t> tasks, longs, slots;
  std::vector<int> split;
  int64_t total_slots = 0;
  int64_t total_tasks = 0, total_longs = 0, max_slots = 0;
};

// Upper bounds (from row lengths alone) on tasks / cut rows / slots of every chunk: a row cut by
// source class adds at most one extra piece per class.
PlanCounts count_plan(const Tuning &tune, const int64_t *ptr, const std::vector<int64_t> &chunk_ptr, int classes, int min_row,
                      int least_piece, const uint8_t *force = nullptr) {
  PlanCounts pc;
  const int K = (int)chunk_ptr.size() - 1;
  pc.tasks.assign(K, 0);
  pc.longs.assign(K, 0);
  pc.slots.assign(K, 0);
  pc.split.assign(K, 0);
  for (int c = 0; c < K; ++c) {
    const int split = split_edges_for(tune, ptr[chunk_ptr[c + 1]] - ptr[chunk_ptr[c]], least_piece);
    pc.split[c] = split;
    for (int64_t r = chunk_ptr[c]; r < chunk_ptr[c + 1]; ++r) {
      const int64_t len = ptr[r + 1] - ptr[r];
      const bool by_src = classes > 1 && len >= min_row;
      if (by_src || len > split || (force && force[r])) {
        const int64_t pieces = (len + split - 1) / split + (by_src ? classes + 1 : 0);  // + 1: the run beyond the classes
        pc.tasks[c] += pieces;
        pc.slots[c] += pieces;
        pc.longs[c] += 1;
      } else {
        pc.tasks[c] += 1;
      }
    }
    pc.total_tasks += pc.tasks[c];
    pc.total_longs += pc.longs[c];
    pc.total_slots += pc.slots[c];
    if (pc.slots[c] > pc.max_slots) pc.max_slots = pc.slots[c];
  }
  return pc;
}

// Everything the host plans for one aggregation direction before anything is uploaded.
struct HostDir {
  DensePlan dp;
  const int64_t *ptr = nullptr;   // the index the sparse kernels see: the original one, or the dense plan's remainder
  const int32_t *idx = nullptr;
  int64_t nnz = 0;
  std::vector<uint8_t> force;     // rows with dense parts (they always write partial sums)
  HotOrder hot;                   // active: idx is hot.idx (long rows ordered by hotness), hot.rank the ranks in that order
  int min_row = 128;              // rows from this length on are cut by class
  PlanCounts pc;
  std::vector<int32_t> item_rb, item_nb;
  std::vector<int64_t> item_b0;
  std::vector<ChunkMask> item_chunks;
  std::vector<int64_t> chunk_item_off;  // K + 1
  std::vector<int64_t> rowscale_off;    // K + 1: chunk k owns 128 scale slots per row block
  int64_t max_items = 0;
  bool dense() const { return dp.active; }
  int64_t padded_entries() const {  // entry lists padded to multiples of eight (16-byte loads)
    int64_t t = 0;
    for (int64_t b = 0; b < dp.n_blocks(); ++b) t += (dp.blk_e0[(size_t)b + 1] - dp.blk_e0[(size_t)b] + 7) / 8 * 8;
    return t;
  }
  const uint8_t *force_ptr() const { return dp.active ? force.data() : nullptr; }
};

void host_mask_set(ChunkMask &m, int c) { m.w[c >> 6] |= 1ull << (c & 63); }

bool make_host_dir(const Tuning &tune, const int64_t *ptr, const int32_t *idx, int64_t n, const std::vector<int64_t> &chunk_ptr,
                   int classes, bool hot, bool want_orig, bool try_dense, int dense_width, int least_piece, HostDir &h) {
  const int K = (int)chunk_ptr.size() - 1;
  h.ptr = ptr;
  h.idx = idx;
  h.nnz = ptr[n];
  h.chunk_item_off.assign((size_t)K + 1, 0);
  h.rowscale_off.assign((size_t)K + 1, 0);
  for (int k = 0; k < K; ++k)
    h.rowscale_off[(size_t)k + 1] = h.rowscale_off[(size_t)k] + (chunk_ptr[(size_t)k + 1] - chunk_ptr[(size_t)k] + kDenseRB - 1) / kDenseRB * kDenseRB;
  if (try_dense) {
    // share of all entries that must be dense: the relative threshold, or the absolute one if that asks for more
    const double nnz = (double)ptr[n];
    const double share = std::max(tune.dense_min_share, nnz > 0 ? tune.dense_min_entries * K / nnz : 0.0);
    if (!build_dense_plan(ptr, idx, n, K, chunk_ptr.data(), dense_min_nnz(tune), share, h.dp, kDenseItemBlocks, dense_max_items(dense_width),
                          dense_min_nnz_many(tune)))
      return false;
  }
  if (h.dp.active) {
    const DensePlan &dp = h.dp;
    h.ptr = dp.rem_ptr.data();
    h.idx = dp.rem_idx.data();
    h.nnz = (int64_t)dp.rem_idx.size();
    h.force.assign((size_t)n, 0);
    std::vector<int> chunk_of_cb((size_t)dp.cb_off[(size_t)K]);
    for (int c = 0; c < K; ++c)
      for (int64_t b = dp.cb_off[(size_t)c]; b < dp.cb_off[(size_t)c + 1]; ++b) chunk_of_cb[(size_t)b] = c;
    for (int k = 0; k < K; ++k) {
      int64_t b = dp.chunk_blk_off[(size_t)k];
      const int64_t b_end = dp.chunk_blk_off[(size_t)k + 1];
      while (b < b_end) {  // runs of blocks of one row block, at most kDenseItemBlocks each
        int64_t e = b;
        ChunkMask m{};
        while (e < b_end && dp.blk_rb[(size_t)e] == dp.blk_rb[(size_t)b] && e - b < kDenseItemBlocks) {
          host_mask_set(m, chunk_of_cb[(size_t)dp.blk_cb[(size_t)e]]);
          ++e;
        }
        h.item_rb.push_back(dp.blk_rb[(size_t)b]);
        h.item_b0.push_back(b);
        h.item_nb.push_back((int32_t)(e - b));
        h.item_chunks.push_back(m);
        const int64_t r0 = chunk_ptr[(size_t)k] + (int64_t)dp.blk_rb[(size_t)b] * kDenseRB;
        for (int64_t r = r0; r < std::min<int64_t>(r0 + kDenseRB, chunk_ptr[(size_t)k + 1]); ++r)
          h.force[(size_t)dp.row_perm[(size_t)r]] = 1;
        b = e;
      }
      h.chunk_item_off[(size_t)k + 1] = (int64_t)h.item_rb.size();
      h.max_items = std::max(h.max_items, h.chunk_item_off[(size_t)k + 1] - h.chunk_item_off[(size_t)k]);
    }
  }
  h.min_row = hot ? tune.hot_min_row : tune.class_min_row;
  if (hot && classes > 1) {  // on the index the sparse kernels see (the dense plan's remainder, if there is one)
    if (!build_hot_order(h.ptr, h.idx, n, h.min_row, want_orig, h.hot)) return false;
    h.idx = h.hot.idx.data();
  }
  h.pc = count_plan(tune, h.ptr, chunk_ptr, classes, h.min_row, least_piece, h.force_ptr());
  return true;
}

struct Bump {
  size_t off = 0;
  size_t take(size_t bytes) {
    const size_t at = off;
    off += (bytes + kAlign - 1) / kAlign * kAlign;
    return at;
  }
};

struct Layout {
  size_t row_ptr, pcol, val, t_ptr, prow, tval;
  size_t f_task_row, f_task_e0, f_task_ne, f_task_slot, f_lr_row, f_lr_slot0, f_lr_n;
  size_t b_task_row, b_task_e0, b_task_ne, b_task_slot, b_lr_row, b_lr_slot0, b_lr_n;
  size_t f_slot_class, b_slot_class;
  size_t pass_tables;  // three tables of K entries (PassTableArgs)
  size_t rem_ptr[2];  // row pointers of the remainder index per direction (dense plan active), else unused
  // dense plan per direction (0 forward, 1 transposed)
  size_t d_blk_cb[2], d_blk_e0[2], d_ent_pos[2], d_ent_w[2], d_colslot[2], d_tiles[2];
  size_t d_bits[2], d_colscale[2], d_rowscale[2];  // weights of the form s(row) * s(column): patterns and scales
  size_t d_item_rs[2], d_item_chunk[2], d_item_b0[2], d_item_nb[2], d_item_chunks[2];
  size_t d_lr_dense0[2], d_lr_ndense[2], d_lr_item0[2];
  size_t dense_partial, zero_row;
  size_t partial;
  int64_t item_cap, slot_cap;  // dense items and partial rows that one launch may use
  int64_t self_rows;           // GraphSage: rows of self_fwd
  size_t row_stride;           // elements of a chunk's rows
  size_t ln_stride;            // of the parameter sums of one layer
  int ln_layers;               // layers whose parameter sums wait to be added up at a time
  std::vector<size_t> Z, dZ, Wt, Wn, Tc, Th;
  std::vector<size_t> dY;  // deferred weight gradients: dL/d(pre-activation) of every aggregate-first layer, all n rows
  std::vector<size_t> Wt_self, Wn_self;  // GraphSage: staged copies of W_self (Wt / Wn then hold W_neigh)
  size_t self_fwd = 0, self_bwd = 0;      // GraphSage: h_v W_self (fp32), dY W_self^T where it can't wait in the output rows
  size_t ln_partial = 0;                  // ResGCN+: parameter-gradient scratch
  size_t G[2];
  size_t gemm_partial, bias_partial, gemm_partial_floats, bias_partial_floats;
  size_t total;
};

struct Shape {
  int64_t n = 0, nnz = 0;
  int K = 0, L = 0;
  std::vector<int64_t> chunk_ptr;
  std::vector<int> dims, ld;
  std::vector<char> tf;  // per layer: 1 = transform first (gather rows of width d_{j+1}), 0 = aggregate first
  int dtype = 0, level0_f32 = 0, variant = 0, need_input_grad = 0;
  Tuning tune;
  bool has_bias() const { return variant != GNNSTAGE_GCNII; }
  // One weight-gradient product per layer over all rows at the end of the backward pass instead of one per chunk
  // (the rows of dL/d(pre-activation) are kept for the whole pass): a per-chunk product of a few ten thousand rows
  // runs at its launch and latency floor.
  bool defer_wgrad() const { return tune.wgrad_defer; }
  bool sage() const { return variant == GNNSTAGE_SAGE; }
  bool res() const { return variant == GNNSTAGE_RESGCN; }
  // dY W_self^T of layer j waits in the rows that the layer's transposed aggregation writes and adds it to: those are of the
  // gradient rows' type, and no column of them belongs to two lanes
  bool self_in_place(int j) const { return dims[j] % 8 == 0 && level_elt(j) == elt(); }
  // elements of one weight matrix: GraphSage stacks [W_self ; W_neigh]
  size_t w_half(int j) const { return (size_t)dims[j] * dims[j + 1]; }
  int elt() const { return dtype == GNNSTAGE_BF16 ? 2 : 4; }
  int level_elt(int j) const { return (j == 0 && level0_f32) ? 4 : elt(); }
  // source classes for the aggregation schedule, decided by the widest bf16/fp32 table that is gathered
  int64_t widest_row_bytes() const {  // of the widest row any aggregation of the stage gathers
    int64_t widest = 0;
    for (int j = 0; j < L; ++j)
      widest = std::max<int64_t>(widest, tf[j] ? (int64_t)dims[j + 1] * elt()
                                               : std::max<int64_t>((int64_t)dims[j] * level_elt(j), (int64_t)dims[j] * elt()));
    return widest;
  }
  // classes of the hottest sources instead of id-range classes (tables that fit no cache)
  bool hot() const { return hot_classes_setting(tune, n * widest_row_bytes()) >= 2; }
  int64_t hot_rows() const { return hot_rows_setting(tune, widest_row_bytes()); }
  // Short rows.  Tables that fit no cache: up to 4 entries, summed on the vector ALU with fp32 weights (10 M vertices 141.2 against
  // 143.2 ms per step; up to 8 / 16: 143.2 / 148.0, the launch is bound by the gathers).  Others: up to 16, on the matrix cores.
  bool short_valu() const { return n * widest_row_bytes() > ((int64_t)256 << 20); }
  // (None where every aggregation runs on the vector ALU, a row to a wave: 89 k fp32 vertices of width 100 1.99 ms per pass in row
  // order, 2.08 with the short rows apart.)
  int short_row() const { return tune.short_row >= 0 ? tune.short_row : valu_layers() == L ? 0 : short_valu() ? 4 : kShortRowMost; }
  int classes() const {
    if (hot()) return hot_classes_setting(tune, n * widest_row_bytes());
    return xcd_classes_setting(tune, n * widest_row_bytes());
  }
  // Shortest piece that long rows of small launches are cut into (backward, and bf16 stages).  The vector-ALU kernel has 8 row pieces of a task in
  // flight, the matrix-core kernel turns 128 entries at a time into gathers.  Measured with pieces of 32 / 64 / 128
  // entries on the vector-ALU kernel: 5 k vertices of width 1000, 32 chunks 23.1 / 23.5 / 24.6 ms per step; 89 k vertices of
  // width 100 16.1 / 16.6 / 18.1 ms.  64 / 128 / 256 on the matrix-core kernel: 9.45 / 9.61 / 9.59 ms (300 k vertices of
  // width 128), 13.9 / 13.3 / 13.6 ms (169 k vertices of width 256).
  int least_piece(bool transposed) const {
    if (dtype == GNNSTAGE_F32 && !transposed) return kLeastPieceF32Fwd;
    const int valu = valu_layers();
    return valu == L ? 32 : valu > 0 ? 64 : 128;
  }
  int valu_layers() const {  // whose aggregations run on the vector ALU
    int valu = 0;
    for (int j = 0; j < L; ++j) {
      const bool f32_rows = dtype == GNNSTAGE_F32 || (j == 0 && level0_f32 && !tf[j]);
      valu += f32_rows || (tf[j] ? dims[j + 1] : dims[j]) % 8 != 0 || tune.spmm_valu;
    }
    return valu;
  }
  // dense blocks serve the matrix-core aggregation only: every aggregation of the stage must gather bf16 rows
  // of width 128 or 256
  int dense_width() const {  // the widest rows the dense kernel gathers (one workgroup per 128 columns)
    int wdt = 128;
    for (int j = 0; j < L; ++j) wdt = std::max(wdt, tf[j] ? dims[j + 1] : dims[j]);
    return wdt;
  }
  bool dense_ok() const {
    if (dtype != GNNSTAGE_BF16 || !tune.dense) return false;
    for (int j = 0; j < L; ++j) {
      const int wdt = tf[j] ? dims[j + 1] : dims[j];
      if (wdt != 128 && wdt != 256) return false;
      if (!tf[j] && j == 0 && level0_f32) return false;
    }
    return true;
  }
  // tasks, and what fills every chunk's short rows up to a multiple of four
  int64_t task_capacity(int64_t tasks) const { return tasks + 3 * (int64_t)K; }
  int64_t max_rows() const {
    int64_t m = 0;
    for (int c = 0; c < K; ++c) m = std::max<int64_t>(m, chunk_ptr[c + 1] - chunk_ptr[c]);
    return m;
  }
};

bool read_shape(const gnnstage_desc *d, Shape &s, std::string &err) {
  if (!d) { err = "descriptor is NULL"; return false; }
  if (d->n_vertices <= 0 || d->nnz < 0) { err = "n_vertices must be positive and nnz non-negative"; return false; }
  if (!d->row_ptr || !d->chunk_ptr || !d->dims) { err = "row_ptr, chunk_ptr and dims must not be NULL"; return false; }
  if (d->n_chunks <= 0 || d->n_chunks > kMaxChunks) { err = "n_chunks must be in [1, 256]"; return false; }
  if (d->n_layers <= 0 || d->n_layers > 1024) { err = "n_layers must be in [1, 1024]"; return false; }
  if (d->dtype != GNNSTAGE_F32 && d->dtype != GNNSTAGE_BF16) { err = "unknown dtype"; return false; }
  if (d->variant != GNNSTAGE_GCN && d->variant != GNNSTAGE_GCNII && d->variant != GNNSTAGE_SAGE &&
      d->variant != GNNSTAGE_RESGCN) {
    err = "unknown variant";
    return false;
  }
  s.n = d->n_vertices;
  s.nnz = d->nnz;
  s.K = d->n_chunks;
  s.L = d->n_layers;
  s.dtype = d->dtype;
  s.level0_f32 = (d->dtype == GNNSTAGE_BF16 && d->level0_f32) ? 1 : 0;
  s.variant = d->variant;
  s.need_input_grad = d->need_input_grad ? 1 : 0;
  s.chunk_ptr.assign(d->chunk_ptr, d->chunk_ptr + s.K + 1);
  if (s.chunk_ptr[0] != 0 || s.chunk_ptr[s.K] != s.n) { err = "chunk_ptr must start at 0 and end at n_vertices"; return false; }
  for (int c = 0; c < s.K; ++c)
    if (s.chunk_ptr[c] > s.chunk_ptr[c + 1]) { err = "chunk_ptr must be non-decreasing"; return false; }
  s.dims.assign(d->dims, d->dims + s.L + 1);
  s.ld.resize(s.L + 1);
  for (int j = 0; j <= s.L; ++j) {
    if (s.dims[j] <= 0 || s.dims[j] > (1 << 20)) { err = "every level width must be in [1, 2^20]"; return false; }
    if (s.dtype == GNNSTAGE_BF16 && (s.dims[j] & 1) && !(j == 0 && s.level0_f32)) {
      err = "bf16 levels need an even width";
      return false;
    }
    s.ld[j] = round_up(s.dims[j], 8);
  }
  if (s.variant == GNNSTAGE_GCNII || s.res()) {
    for (int j = 1; j <= s.L; ++j)
      if (s.dims[j] != s.dims[0]) { err = "GCNII and ResGCN+ need equal widths at every level"; return false; }
    if (s.level0_f32) { err = "GCNII and ResGCN+ do not take an fp32 level 0"; return false; }
    if (s.res() && s.dims[0] > kLnMaxWidth) { err = "ResGCN+ rows are limited to 1024 columns"; return false; }
  }
  // Layer order.  (A_hat H) W == A_hat (H W) and the select is per edge, so a GCN layer may apply W
  // before the aggregation; that pays when it narrows the rows the gather has to move.
  s.tune = read_tuning();
  s.tf.assign(s.L, 0);
  for (int j = 0; j < s.L; ++j) {
    if (s.variant != GNNSTAGE_GCN) continue;
    const bool narrower = (size_t)s.dims[j + 1] * s.elt() < (size_t)s.dims[j] * s.level_elt(j);
    s.tf[j] = narrower ? 1 : 0;
    if (s.tune.order == 1) s.tf[j] = 0;
    if (s.tune.order == 2) s.tf[j] = 1;
  }
  if (d->row_ptr[0] != 0 || d->row_ptr[s.n] != s.nnz) { err = "row_ptr must start at 0 and end at nnz"; return false; }
  for (int64_t v = 0; v < s.n; ++v)
    if (d->row_ptr[v] > d->row_ptr[v + 1]) { err = "row_ptr must be non-decreasing"; return false; }
  return true;
}

Layout layout_for(const Shape &s, const HostDir &hf, const HostDir &hb, bool rank1, int64_t item_cap, int64_t slot_cap) {
  const PlanCounts &f = hf.pc, &b = hb.pc;
  Layout l;
  Bump w;
  l.row_ptr = w.take(sizeof(int64_t) * (s.n + 1));
  l.pcol = w.take(sizeof(uint32_t) * hf.nnz);
  l.val = w.take(sizeof(float) * hf.nnz);
  l.t_ptr = w.take(sizeof(int64_t) * (s.n + 1));
  l.prow = w.take(sizeof(uint32_t) * hb.nnz);
  l.tval = w.take(sizeof(float) * hb.nnz);
  for (int dir = 0; dir < 2; ++dir) {
    const HostDir &h = dir ? hb : hf;
    const bool on = h.dense();
    const size_t nb = on ? (size_t)h.dp.n_blocks() : 0, ne = on ? (size_t)h.padded_entries() : 0;
    const size_t ni = h.item_rb.size(), nl = on ? (size_t)h.pc.total_longs : 0;
    l.rem_ptr[dir] = w.take(on ? sizeof(int64_t) * (s.n + 1) : 0);
    l.d_blk_cb[dir] = w.take(sizeof(int32_t) * nb);
    l.d_blk_e0[dir] = w.take(on ? sizeof(int64_t) * (nb + 1) : 0);
    l.d_ent_pos[dir] = w.take(rank1 ? 0 : sizeof(uint16_t) * ne);
    l.d_ent_w[dir] = w.take(rank1 ? 0 : sizeof(uint32_t) * ne);
    l.d_colslot[dir] = w.take(on ? sizeof(uint32_t) * h.dp.colslot_vertex.size() : 0);
    l.d_tiles[dir] = w.take(rank1 ? 0 : sizeof(uint16_t) * nb * 2 * kDenseRB * kDenseCB);
    l.d_bits[dir] = w.take(rank1 ? sizeof(uint32_t) * nb * 256 : 0);
    l.d_colscale[dir] = w.take(on && rank1 ? sizeof(float) * h.dp.colslot_vertex.size() : 0);
    l.d_rowscale[dir] = w.take(on && rank1 ? sizeof(float) * (size_t)h.rowscale_off.back() : 0);
    l.d_item_rs[dir] = w.take(sizeof(int32_t) * ni);
    l.d_item_chunk[dir] = w.take(sizeof(int32_t) * ni);
    l.d_item_b0[dir] = w.take(sizeof(int64_t) * ni);
    l.d_item_nb[dir] = w.take(sizeof(int32_t) * ni);
    l.d_item_chunks[dir] = w.take(sizeof(ChunkMask) * ni);
    l.d_lr_dense0[dir] = w.take(sizeof(int32_t) * nl);
    l.d_lr_ndense[dir] = w.take(sizeof(int32_t) * nl);
    l.d_lr_item0[dir] = w.take(sizeof(int32_t) * nl);
  }
  l.item_cap = item_cap;
  l.slot_cap = slot_cap;
  l.dense_partial = w.take(sizeof(float) * (size_t)item_cap * kDenseRB * s.dense_width());
  l.zero_row = w.take(item_cap > 0 ? 512 : 0);
  const int64_t f_tasks = s.task_capacity(f.total_tasks), b_tasks = s.task_capacity(b.total_tasks);
  l.f_task_row = w.take(sizeof(int32_t) * f_tasks);
  l.f_task_e0 = w.take(sizeof(int64_t) * f_tasks);
  l.f_task_ne = w.take(sizeof(int32_t) * f_tasks);
  l.f_task_slot = w.take(sizeof(int32_t) * f_tasks);
  l.f_lr_row = w.take(sizeof(int32_t) * f.total_longs);
  l.f_lr_slot0 = w.take(sizeof(int32_t) * f.total_longs);
  l.f_lr_n = w.take(sizeof(int32_t) * f.total_longs);
  l.b_task_row = w.take(sizeof(int32_t) * b_tasks);
  l.b_task_e0 = w.take(sizeof(int64_t) * b_tasks);
  l.b_task_ne = w.take(sizeof(int32_t) * b_tasks);
  l.b_task_slot = w.take(sizeof(int32_t) * b_tasks);
  l.b_lr_row = w.take(sizeof(int32_t) * b.total_longs);
  l.b_lr_slot0 = w.take(sizeof(int32_t) * b.total_longs);
  l.b_lr_n = w.take(sizeof(int32_t) * b.total_longs);
  l.f_slot_class = w.take((size_t)f.total_slots);
  l.b_slot_class = w.take((size_t)b.total_slots);
  l.pass_tables = w.take(sizeof(PassChunk) * 3 * (size_t)s.K);
  int max_d = 0, max_ld = 0;
  size_t max_io = 0;
  for (int j = 0; j <= s.L; ++j) {
    max_d = std::max(max_d, s.dims[j]);
    max_ld = std::max(max_ld, s.ld[j]);
  }
  for (int j = 0; j < s.L; ++j) max_io = std::max(max_io, (size_t)s.dims[j] * s.dims[j + 1]);
  l.partial = w.take(sizeof(float) * (size_t)slot_cap * max_d);
  l.row_stride = (size_t)round_up((int)std::min<int64_t>(s.max_rows(), 0x7ffffff0), 8) * max_ld;  // rows of a chunk
  l.ln_stride = (size_t)(kLnMaxWaves / 4) * 2 * max_d;
  l.ln_layers = std::min(s.L, kBatch);
  const size_t elt = s.elt();
  l.Z.resize(s.L);
  l.dZ.resize(s.L);
  l.Wt.resize(s.L);
  l.Wn.resize(s.L);
  l.Tc.assign(s.L, 0);
  l.Th.assign(s.L, 0);
  l.dY.assign(s.L, 0);
  for (int j = 0; j < s.L && s.res(); ++j) {
    // ResGCN+: ReLU(LayerNorm(.)) of the current and of the historical rows, the saved aggregation, and the
    // gradient of the aggregation for ALL rows (the parameter gradient through historical rows needs it)
    l.Tc[j] = w.take((size_t)s.n * s.ld[j] * elt);
    l.Th[j] = w.take((size_t)s.n * s.ld[j] * elt);
    l.Z[j] = w.take((size_t)s.n * s.ld[j] * elt);
    l.dZ[j] = w.take((size_t)s.n * s.ld[j] * elt);
    // deferred weight gradients keep dY of all rows in the table of activated current rows (of the same width): a chunk's rows
    // of that table are written before they are read in a forward pass, and no backward pass reads them.  The gradient of the
    // activated rows of a backward pass waits in the table of historical ones for the same reason.
    l.dY[j] = l.Tc[j];
  }
  if (s.res()) l.ln_partial = w.take(sizeof(float) * l.ln_stride * l.ln_layers);
  for (int j = 0; j < s.L && !s.res(); ++j) {
    if (s.tf[j]) {
      // transform-first layer: transformed current / historical rows, and the masked upstream gradient
      l.Z[j] = 0;
      l.Tc[j] = w.take((size_t)s.n * s.ld[j + 1] * elt);
      l.Th[j] = w.take((size_t)s.n * s.ld[j + 1] * elt);
      l.dZ[j] = w.take((size_t)s.n * s.ld[j + 1] * elt);
    } else {
      l.Z[j] = w.take((size_t)s.n * s.ld[j] * elt);
      l.dZ[j] = (j == 0 && !s.need_input_grad) ? 0 : w.take((size_t)s.n * s.ld[j] * elt);
      if (s.defer_wgrad()) l.dY[j] = w.take((size_t)s.n * s.ld[j + 1] * elt);
    }
  }
  for (int j = 0; j < s.L; ++j) {
    l.Wt[j] = w.take((size_t)s.dims[j + 1] * s.ld[j] * elt);
    l.Wn[j] = w.take((size_t)s.dims[j] * s.ld[j + 1] * elt);
  }
  if (s.sage()) {
    l.Wt_self.resize(s.L);
    l.Wn_self.resize(s.L);
    for (int j = 0; j < s.L; ++j) {
      l.Wt_self[j] = w.take((size_t)s.dims[j + 1] * s.ld[j] * elt);
      l.Wn_self[j] = w.take((size_t)s.dims[j] * s.ld[j + 1] * elt);
    }
    // the rows of a chunk, or a block of 64 k of a whole pass: its fp32 rows are read back from a cache
    l.self_rows = std::max<int64_t>(s.max_rows(), std::min<int64_t>(s.n, kSelfRows));
    l.self_fwd = w.take(sizeof(float) * (size_t)l.self_rows * max_ld);
    int wait_ld = 0;
    for (int j = s.need_input_grad ? 0 : 1; j < s.L; ++j)
      if (!s.self_in_place(j)) wait_ld = std::max(wait_ld, s.ld[j]);
    l.self_bwd = w.take((size_t)s.n * wait_ld * elt);
  }
  l.G[0] = w.take(l.row_stride * elt);
  l.G[1] = w.take(s.defer_wgrad() ? 0 : l.row_stride * elt);
  l.gemm_partial_floats = (size_t)kMaxSplits * max_io;
  l.bias_partial_floats = (size_t)kMaxSplits * max_d;
  l.gemm_partial = w.take(sizeof(float) * l.gemm_partial_floats);
  l.bias_partial = w.take(sizeof(float) * l.bias_partial_floats);
  l.total = w.off;
  return l;
}

// One launch over a whole layer needs room for the partial sums of every chunk: at most 1 GiB beyond that of the largest chunk,
// or a sixteenth of the workspace where that is more; a layer whose sums need more is served in several launches.
Layout make_layout(const Shape &s, const HostDir &hf, const HostDir &hb, bool rank1) {
  const int64_t one_items = std::max(hf.max_items, hb.max_items), one_slots = std::max(hf.pc.max_slots, hb.pc.max_slots);
  const Layout one = layout_for(s, hf, hb, rank1, one_items, one_slots);
  const int64_t all_items = (int64_t)std::max(hf.item_rb.size(), hb.item_rb.size()), all_slots = std::max(hf.pc.total_slots, hb.pc.total_slots);
  const size_t half = s.tune.partial_room >= 0 ? (size_t)s.tune.partial_room : std::max<size_t>((size_t)1 << 30, one.total / 16) / 2;
  int widest = 1;
  for (const int d : s.dims) widest = std::max(widest, d);
  const int64_t item_room = (int64_t)(half / (sizeof(float) * kDenseRB * (size_t)s.dense_width())), slot_room = (int64_t)(half / (sizeof(float) * (size_t)widest));
  return layout_for(s, hf, hb, rank1, std::min(all_items, one_items + item_room), std::min(all_slots, one_slots + slot_room));
}

struct Profiler {
  uint32_t kinds = 0;  // bit k set: launches of kind k are timed
  int n_layers = 0;  // slot n_layers collects launches that belong to no layer
  struct Rec { int kind, layer; hipEvent_t a, b; };
  std::vector<Rec> recs;
  std::vector<hipEvent_t> free_events;
  std::vector<double> ms;          // [kind][layer]
  std::vector<int64_t> launches;   // [kind][layer]
  void init(int L) {
    n_layers = L;
    ms.assign((size_t)GNNSTAGE_NKINDS * (L + 1), 0.0);
    launches.assign((size_t)GNNSTAGE_NKINDS * (L + 1), 0);
  }
  hipEvent_t get() {
    if (!free_events.empty()) {
      hipEvent_t e = free_events.back();
      free_events.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    // timing only: no system-scope fence when the event completes (the default event makes every write of the
    // stream visible to the host, which costs a launch of a few microseconds about as much as the launch itself)
    (void)hipEventCreateWithFlags(&e, hipEventDisableSystemFence);
    return e;
  }
  void collect() {
    for (auto &r : recs) {
      float t = 0.f;
      if (hipEventElapsedTime(&t, r.a, r.b) == hipSuccess) {
        ms[(size_t)r.kind * (n_layers + 1) + r.layer] += t;
        launches[(size_t)r.kind * (n_layers + 1) + r.layer] += 1;
      }
      free_events.push_back(r.a);
      free_events.push_back(r.b);
    }
    recs.clear();
  }
  void destroy() {
    collect();
    for (auto e : free_events) (void)hipEventDestroy(e);
    free_events.clear();
  }
};

}  // namespace

struct gnnstage {
  Shape s;
  Layout lay;
  int vbits = 0;
  float alpha = 0.f;
  std::vector<float> beta;
  // caller-owned device buffers
  std::vector<void *> W, bias, cur, hist;
  std::vector<float *> dW, dbias;
  const void *h0 = nullptr;
  std::vector<const float *> ln_g, ln_b;  // ResGCN+: LayerNorm parameters and their gradients
  std::vector<float *> d_ln_g, d_ln_b;
  float ln_eps = 1e-5f;
  float dropout_p = 0.f;      // ResGCN+: between ReLU and the convolution; GCN, GraphSage: on every layer's output
  uint64_t dropout_seed = 0;  // of the current pass
  // What the setters wrote.  A pass latches both at its first forward call and keeps them until its last backward
  // call, so that the backward pass redraws exactly the decisions of its forward pass whatever the caller sets
  // in between.
  float next_dropout_p = 0.f;
  uint64_t next_dropout_seed = 0;
  // GCN, GraphSage: the stored output of a layer is the value after dropout; a positive one passed ReLU and dropout,
  // so every ReLU mask of the backward pass also scales by 1 / (1 - rate)
  bool output_dropout() const { return dropout_p > 0.f && (s.variant == GNNSTAGE_GCN || s.variant == GNNSTAGE_SAGE); }
  float mask_scale() const { return output_dropout() ? (float)(1.0 / (1.0 - (double)dropout_p)) : 1.f; }
  // the dropout of layer j for a launch whose first row is vertex u0
  LnDropout dropout(int j, int64_t u0) const {
    LnDropout dp{};
    if (dropout_p > 0.f) {
      uint64_t z = dropout_seed + (uint64_t)(j + 1) * 0x9E3779B97F4A7C15ull;  // SplitMix64 output for that state
      z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
      z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
      dp.key = z ^ (z >> 31);
      dp.threshold = (uint32_t)std::ceil((double)dropout_p * 16777216.0);
      dp.scale = (float)(1.0 / (1.0 - (double)dropout_p));
      dp.u0 = u0;
    }
    return dp;
  }
  void *grad_in = nullptr;
  float *grad_h0 = nullptr;
  char *ws = nullptr;
  // host copies for the diagnostics
  std::vector<int64_t> h_row_ptr;
  std::vector<uint32_t> h_pcol;
  // schedules
  DirTasks tasks[2];  // 0 forward, 1 transposed
  // of a pass whose chunks run side by side: entries that backward launches gather from every class ([chunk][class]), of the
  // chunks from the row's own on (0) and of those in front of it (1)
  std::vector<int64_t> kept[2];
  bool tables_written = false;  // the tables in the workspace are those of the present order
  bool dense_on[2] = {false, false};  // dense blocks per direction (0 forward, 1 transposed)
  int64_t dense_entries[2] = {0, 0};  // entries that live in dense blocks
  bool dense_rank1 = false;           // their weights are kept as pattern bits and row / column scales
  int n_classes = 1;
  // pass state (Section 3.3: V_processed, and its backward twin)
  std::vector<int32_t> order;
  ChunkMask fmask{}, bmask{};
  int n_bwd = 0;
  bool cur_stale = false;  // the levels traded places and no complete pass has rewritten the current ones yet
  int gi = 0;              // without deferred weight gradients: which of the two scratch matrices holds dY
  std::vector<char> wgrad_pending;  // per chunk: its backward call ran, its rows' weight-gradient products are still owed
  std::string err;
  Profiler prof;

  template <typename T>
  T *at(size_t off) const { return reinterpret_cast<T *>(ws + off); }
  int level_dtype(int j) const { return (j == 0 && s.level0_f32) ? DT_F32 : (s.dtype == GNNSTAGE_BF16 ? DT_BF16 : DT_F32); }
  int cdtype() const { return s.dtype == GNNSTAGE_BF16 ? DT_BF16 : DT_F32; }
  size_t level_elt(int j) const { return level_dtype(j) == DT_BF16 ? 2 : 4; }
};

namespace {

int fail(gnnstage *st, int code, const std::string &msg) {
  if (st) st->err = msg; else g_create_error = msg;
  return code;
}

struct Timed {
  gnnstage *st;
  hipStream_t s;
  int kind, layer;
  hipEvent_t a = nullptr, b = nullptr;
  Timed(gnnstage *st_, hipStream_t s_, int kind_, int layer_ = -1)
      : st(st_), s(s_), kind(kind_), layer(layer_ < 0 ? st_->prof.n_layers : layer_) {
    if ((st->prof.kinds >> kind) & 1u) {
      a = st->prof.get();
      b = st->prof.get();
      (void)hipEventRecord(a, s);
    }
  }
  ~Timed() {
    if (a != nullptr) {
      (void)hipEventRecord(b, s);
      st->prof.recs.push_back({kind, layer, a, b});
    }
  }
};

#define HIP_TRY(st, expr)                                                                            \
  do {                                                                                               \
    const int e_ = (int)(expr);                                                                      \
    if (e_ != 0)                                                                                     \
      return fail(st, GNNSTAGE_EHIP, std::string(#expr) + ": " + hipGetErrorString((hipError_t)e_)); \
  } while (0)

void mask_set(ChunkMask &m, int c) { m.w[c >> 6] |= 1ull << (c & 63); }

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// What a launch selects: a mask by value (of the chunk that it serves, or one for all rows), or a table of a whole pass.
enum Select { SEL_MASK, SEL_FORWARD, SEL_BACKWARD, SEL_EARLIER };

// A run of chunks that a layer's launches serve: one chunk, which sees mask, or all of a pass, whose rows see the masks of
// the pass tables.
struct Span {
  int c0, c1;
  bool whole;
  ChunkMask mask;
};
int64_t span_row0(const gnnstage *st, const Span &sp) { return st->s.chunk_ptr[(size_t)sp.c0]; }
int64_t span_rows(const gnnstage *st, const Span &sp) { return st->s.chunk_ptr[(size_t)sp.c1] - st->s.chunk_ptr[(size_t)sp.c0]; }
Span chunk_span(int k, const ChunkMask &mask) { return Span{k, k + 1, false, mask}; }
// A single chunk needs no table: its rows select it (forward and on the way back), or nothing (earlier).
bool by_table(const gnnstage *st) { return st->s.K > 1; }
Span whole_span(const gnnstage *st) {
  Span sp{0, st->s.K, true, ChunkMask{}};
  if (!by_table(st)) sp.mask.w[0] = 1;
  return sp;
}
Select span_select(const gnnstage *st, const Span &sp, Select table) { return sp.whole && by_table(st) ? table : SEL_MASK; }

// XCD assignment of the class sections for one launch over chunks [c0, c1).  `drop` = the launch skips unselected entries:
// a class with no entry from a selected chunk has no work and is not served at all.  Every class gets
// a cost (a fixed part per task, one unit per gathered entry, a small part per entry that is read and
// dropped), and the groups of the active classes are dealt to the 8 XCDs like water into buckets of equal
// cost, a class being split between neighbouring XCDs where a bucket boundary falls inside it.
// Every launch comes through here: only one that drops by a mask adds up over source chunks (chunk calls of 250 chunks spent
// 2.6 us per launch on such sums whatever the launch).
void assign_xcds(const gnnstage *st, const DirTasks &t, int c0, int c1, Select sel, const ChunkMask &mask, bool drop, SpmmArgs &a) {
  const int C = t.n_classes, K = st->s.K;
  int64_t chosen[kMaxChunks];
  bool all_chosen = true;
  if (drop && sel == SEL_MASK)
    for (int c = 0; c < K; ++c) {
      chosen[c] = mask_test(mask, (uint32_t)c) ? -1 : 0;
      all_chosen = all_chosen && chosen[c] != 0;
    }
  const bool keeps_all = !drop || (sel == SEL_MASK && all_chosen);
  a.active_classes = 0;
  a.all_classes_active = 1;
  a.n_class_blocks = 0;
  int groups[kMaxClasses];
  double unit[kMaxClasses];  // cost of one group of four tasks
  double total = 0;
  for (XcdRun &x : a.xcd) x = XcdRun{};
  for (int q = 0; q < kMaxClasses; ++q) a.cls_begin[q] = a.cls_end[q] = 0;
  for (int q = 0; q < C; ++q) {
    a.cls_begin[q] = (int32_t)t.first(q, c0);
    a.cls_end[q] = (int32_t)t.first(q, c1);
    const int64_t ntasks = t.count(q, c0, c1);
    groups[q] = 0;
    unit[q] = 0;
    int64_t kept = 0, all = 0;
    for (int r = c0; r < c1; ++r) {
      all += t.total(r, q);
      kept += keeps_all ? t.total(r, q) : sel == SEL_MASK ? t.selected(r, q, chosen) : st->kept[sel == SEL_EARLIER ? 1 : 0][(size_t)r * C + q];
    }
    const bool on = ntasks > 0 && kept > 0;
    if (!on) a.all_classes_active = 0;
    if (!on) continue;
    a.active_classes |= 1u << q;
    groups[q] = (int)((ntasks + 3) / 4);
    const double cost = 32.0 * (double)ntasks + (double)kept + 0.125 * (double)(all - kept);
    unit[q] = cost / groups[q];
    total += cost;
  }
  if (total == 0) return;
  const double quota = total / 8;
  int x = 0, most = 0;
  double used = 0;
  for (int q = 0; q < C; ++q) {
    int g = 0;
    while (g < groups[q]) {
      if (x < 7 && used >= quota - 0.5 * unit[q]) {
        ++x;
        used = 0;
      }
      int take = groups[q] - g;
      if (x < 7) {
        const int room = (int)((quota - used) / unit[q] + 0.5);
        take = std::min(take, std::max(room, 1));
      }
      if (a.xcd[x].groups == 0) {
        a.xcd[x].cls = q;
        a.xcd[x].group0 = g;
      }
      a.xcd[x].groups += take;
      g += take;
      used += take * unit[q];
      most = std::max(most, a.xcd[x].groups);
    }
  }
  a.n_class_blocks = 8 * most;
}

// What launch_stage_weights needs for the tables of a pass over all chunks in this order.
void plan_pass_tables(gnnstage *st, const std::vector<int32_t> &order, PassTableArgs &a) {
  const Shape &s = st->s;
  const DirTasks &t = st->tasks[1];
  a = PassTableArgs{};
  a.K = s.K;
  PassChunk *p = st->at<PassChunk>(st->lay.pass_tables);
  a.forward = p;
  a.backward = p + s.K;
  a.earlier = p + 2 * s.K;
  for (int i = 0; i < s.K; ++i) a.pos[order[(size_t)i]] = (uint8_t)i;
  for (auto &k : st->kept) k.assign((size_t)s.K * t.n_classes, 0);
  for (int r = 0; r < s.K; ++r) {
    a.classes_backward[r] = a.classes_earlier[r] = 0;
    int64_t ahead[kMaxChunks];
    for (int c = 0; c < s.K; ++c) ahead[c] = a.pos[c] < a.pos[r] ? -1 : 0;
    for (int q = 0; q < t.n_classes; ++q) {
      const int64_t earlier = t.selected(r, q, ahead), sum[2] = {t.total(r, q) - earlier, earlier};
      for (int i = 0; i < 2; ++i) st->kept[i][(size_t)r * t.n_classes + q] = sum[i];
      if (sum[0] > 0) a.classes_backward[r] |= 1u << q;
      if (sum[1] > 0) a.classes_earlier[r] |= 1u << q;
    }
  }
}
// The tables of the present pass, where they have not been written with its weights.
int write_pass_tables(gnnstage *st, const std::vector<int32_t> &order, hipStream_t stream) {
  if (st->tables_written || !by_table(st)) return GNNSTAGE_OK;
  PassTableArgs a;
  plan_pass_tables(st, order, a);
  HIP_TRY(st, launch_stage_weights(nullptr, 0, st->cdtype(), &a, stream));
  st->tables_written = true;
  return GNNSTAGE_OK;
}

// The schedule of chunks [c0, c1) of a launch whose operands are in place.
void set_schedule(const gnnstage *st, int dir, int c0, int c1, Select sel, const ChunkMask &mask, SpmmArgs &a) {
  const Layout &lay = st->lay;
  const DirTasks &t = st->tasks[dir];
  a.pidx = st->at<uint32_t>(dir ? lay.prow : lay.pcol);
  a.val = st->at<float>(dir ? lay.tval : lay.val);
  a.task_row = st->at<int32_t>(dir ? lay.b_task_row : lay.f_task_row);
  a.task_e0 = st->at<int64_t>(dir ? lay.b_task_e0 : lay.f_task_e0);
  a.task_ne = st->at<uint32_t>(dir ? lay.b_task_ne : lay.f_task_ne);
  a.task_slot = st->at<int32_t>(dir ? lay.b_task_slot : lay.f_task_slot);
  a.tail0 = t.first(t.n_classes, c0);
  a.n_tail = t.count(t.n_classes, c0, c1);
  a.short0 = t.first(t.n_classes + 1, c0);
  a.n_short = t.count(t.n_classes + 1, c0, c1);
  a.short_rows = st->s.short_valu() ? SHORT_ROWS_VALU : st->s.tune.short_row >= 0 || a.n_short >= kShortRowsPerColumn * a.d ? SHORT_ROWS_MFMA : SHORT_ROWS_SINGLE;
  a.slot_class = st->at<uint8_t>(dir ? lay.b_slot_class : lay.f_slot_class);
  const int64_t l0 = t.lr_off[(size_t)c0];
  a.lr_row = st->at<int32_t>(dir ? lay.b_lr_row : lay.f_lr_row) + l0;
  a.lr_slot0 = st->at<int32_t>(dir ? lay.b_lr_slot0 : lay.f_lr_slot0) + l0;
  a.lr_nslots = st->at<uint32_t>(dir ? lay.b_lr_n : lay.f_lr_n) + l0;
  a.n_long = t.lr_off[(size_t)c1] - l0;
  a.partial = st->at<float>(lay.partial);
  a.slot0 = t.slot_off[(size_t)c0];
  a.vbits = st->vbits;
  a.many_chunks = st->s.K > 64 ? 1 : 0;
  a.force_valu = st->s.tune.spmm_valu ? 1 : 0;
  a.unroll = st->s.tune.spmm_unroll;
  a.long_pieces = st->s.least_piece(dir == 1) == kLeastPieceF32Fwd ? 1 : 0;
  a.mask = mask;
  a.pass = sel == SEL_MASK ? nullptr : st->at<PassChunk>(lay.pass_tables) + (size_t)(sel == SEL_FORWARD ? 0 : sel == SEL_BACKWARD ? 1 : 2) * st->s.K;
  a.drop_unselected = a.src_unsel == nullptr ? 1 : 0;
  if (st->dense_on[dir]) {
    a.lr_dense0 = st->at<int32_t>(lay.d_lr_dense0[dir]) + l0;
    a.lr_ndense = st->at<int32_t>(lay.d_lr_ndense[dir]) + l0;
    a.lr_item0 = st->at<int32_t>(lay.d_lr_item0[dir]) + l0;
    a.item_chunks = st->at<ChunkMask>(lay.d_item_chunks[dir]);
    a.dense_partial = st->at<float>(lay.dense_partial);
    a.item0 = t.item_off[(size_t)c0];
  }
  assign_xcds(st, t, c0, c1, sel, mask, dir == 1, a);  // every transposed launch drops unselected entries
}

// One aggregation over the rows of a span: dense blocks first, then the sparse kernels, then (where chunks have long rows)
// the reduce of their pieces, timed apart; as many chunks at a time as have room for their partial sums and fit a launch.
int run_spmm(gnnstage *st, SpmmArgs a, int src_dtype, int out_dtype, bool transposed, const Span &sp, Select sel, hipStream_t stream, int kind, int layer) {
  const Layout &lay = st->lay;
  const int dir = transposed ? 1 : 0;
  const DirTasks &t = st->tasks[dir];
  for (int c0 = sp.c0, c1; c0 < sp.c1; c0 = c1) {
    for (c1 = c0 + 1; c1 < sp.c1; ++c1)
      if (t.slot_off[(size_t)c1 + 1] - t.slot_off[(size_t)c0] > lay.slot_cap || t.item_off[(size_t)c1 + 1] - t.item_off[(size_t)c0] > lay.item_cap) break;
    set_schedule(st, dir, c0, c1, sel, sp.mask, a);
    while (c1 - c0 > 1 && spmm_blocks(a) > st->s.tune.launch_blocks) {
      c1 = c0 + (c1 - c0) / 2;
      set_schedule(st, dir, c0, c1, sel, sp.mask, a);
    }
    {
      Timed tm(st, stream, kind, layer);
      const int64_t i0 = t.item_off[(size_t)c0], n_items = t.item_off[(size_t)c1] - i0;
      if (st->dense_on[dir] && n_items > 0) {
        if (src_dtype != DT_BF16 || (a.d != 128 && a.d != 256) || a.src_ld != a.d) return hipErrorInvalidValue;
        DenseArgs da{};
        da.item_rs = st->at<int32_t>(lay.d_item_rs[dir]) + i0;
        da.item_chunk = st->at<int32_t>(lay.d_item_chunk[dir]) + i0;
        da.item_b0 = st->at<int64_t>(lay.d_item_b0[dir]) + i0;
        da.item_nb = st->at<int32_t>(lay.d_item_nb[dir]) + i0;
        da.item_chunks = st->at<ChunkMask>(lay.d_item_chunks[dir]) + i0;
        da.n_items = (int32_t)n_items;
        da.blk_cb = st->at<int32_t>(lay.d_blk_cb[dir]);
        if (st->dense_rank1) {
          da.bits = st->at<uint32_t>(lay.d_bits[dir]);
          da.colscale = st->at<float>(lay.d_colscale[dir]);
          da.rowscale = st->at<float>(lay.d_rowscale[dir]);
        } else {
          da.tiles = st->at<bf16_t>(lay.d_tiles[dir]);
        }
        da.zero_row = st->at<char>(lay.zero_row);
        da.colslot = st->at<uint32_t>(lay.d_colslot[dir]);
        da.src_sel = a.src_sel;
        da.src_unsel = a.src_unsel;
        da.d = a.d;
        da.src_ld = a.src_ld;
        da.vbits = a.vbits;
        da.pass = a.pass;
        da.mask = a.mask;
        da.partial = st->at<float>(lay.dense_partial);
        const int e = launch_spmm_dense(da, stream);
        if (e != 0) return e;
      }
      const int e = launch_spmm(a, src_dtype, out_dtype, stream);
      if (e != 0) return e;
    }
    if (a.n_long > 0) {
      Timed tm(st, stream, 7, layer);
      const int e = launch_spmm_reduce(a, src_dtype, out_dtype, stream);
      if (e != 0) return e;
    }
  }
  return 0;
}

// C[M x N] = A . Bt^T for a chunk's rows of a level or of an internal matrix
GemmNtArgs nt_args(const gnnstage *st, const void *A, int a_dtype, int lda, size_t Bt, int ldb, int64_t M, int N, int K) {
  GemmNtArgs g{};
  g.ws_min_rows = st->s.tune.gemm_ws_min_rows;
  g.A = A;
  g.a_dtype = a_dtype;
  g.lda = lda;
  g.Bt = st->at<char>(Bt);
  g.ldb = ldb;
  g.M = (int)M;
  g.N = N;
  g.K = K;
  g.Kp = ldb;
  g.epilogue = EPI_PLAIN;
  return g;
}
void nt_out(GemmNtArgs &g, void *out, int dtype, int ld) {
  g.out = out;
  g.out_dtype = dtype;
  g.out_ld = ld;
}
GemmTnArgs tn_args(const gnnstage *st, const void *A, int a_dtype, int lda, const void *B, int ldb, int64_t M, int I, int O, float scale, float *dW) {
  GemmTnArgs w{};
  w.wide_min_rows = st->s.tune.gemm_wide_min_rows;
  w.A = A;
  w.a_dtype = a_dtype;
  w.lda = lda;
  w.B = B;
  w.ldb = ldb;
  w.M = (int)M;
  w.I = I;
  w.O = O;
  w.scale = scale;
  w.dW = dW;
  w.partial = st->at<float>(st->lay.gemm_partial);
  w.max_splits = kMaxSplits;
  return w;
}
const char *level_rows(const gnnstage *st, const std::vector<void *> &level, int j, int64_t row0) {
  return static_cast<const char *>(level[(size_t)j]) + (size_t)row0 * st->s.dims[(size_t)j] * st->level_elt(j);
}

// ResGCN+: LayerNorm, ReLU, dropout of rows [row0, row0 + M) of a level, and the way back (dr: gradient of the activated rows,
// res: rows [M x ld_{j+1}] of the residual branch or NULL)
LnArgs ln_args(const gnnstage *st, const std::vector<void *> &level, int j, int64_t row0, int64_t M, void *out, int out_dtype, int out_ld) {
  return LnArgs{level_rows(st, level, j, row0), st->level_dtype(j), st->s.dims[j], st->ln_g[j], st->ln_b[j], st->ln_eps, M, st->s.dims[j], out, out_dtype, out_ld,
                st->dropout(j, row0)};
}

// LayerNorm parameter sums of whole passes, which wait in scratch until all layers' (or as many as there is scratch for) are
// added up: a sum over few rows is a launch of its own for each layer otherwise.  The rows of a layer are summed in groups
// of chunks, a group's sums of all layers in one launch.
struct LnSums {
  int n_groups = 0, n_layers = 0;
  LnReduceArgs red[kBatch][kBatch];  // [layer][group]
  int add_up(gnnstage *st, hipStream_t stream) {
    LnReduceArgs list[kBatch * kBatch];
    int n = 0;
    for (int g = 0; g < n_groups; ++g)
      for (int i = 0; i < n_layers; ++i)
        if (red[i][g].n_parts > 0) list[n++] = red[i][g];
    n_layers = 0;
    HIP_TRY(st, launch_ln_param_reduce(list, n, stream));
    return GNNSTAGE_OK;
  }
};
// Backward of layer j's LayerNorm over the rows of a span but those of chunk `without` (-1, or a chunk outside of the span: all): x = level rows, dr (n rows of ld_j)
// the gradient of the activated rows, out (leading dimension out_ld, indexed by absolute row, or NULL) the gradient of x, res (n rows of ld_{j+1} or NULL)
// the residual branch.
int ln_backward(gnnstage *st, LnSums &sums, const std::vector<void *> &level, int j, const Span &sp, int without, const char *dr, char *out, int out_dtype, int out_ld,
                const char *res, hipStream_t stream) {
  const Shape &s = st->s;
  const size_t celt = s.elt();
  LnBackArgs l[kBatch];
  if (without < sp.c0 || without >= sp.c1) without = -1;
  // As many groups as chunks up to eight, of equal numbers of rows: a launch takes as long as its largest group.  The rows of `without`
  // are a gap in them.  (Groups of whole chunks in front of the gap and behind it were up to a quarter larger than others: LayerNorm
  // backward of four layers of 89 k fp32 rows of width 100, 31 of 32 chunks, 342 instead of 325 us.)
  const int n_groups = std::min(sp.c1 - sp.c0, kBatch);
  const int64_t gap0 = without < 0 ? s.n : s.chunk_ptr[(size_t)without], gap1 = without < 0 ? s.n : s.chunk_ptr[(size_t)without + 1];
  const int64_t first = span_row0(st, sp), rows = span_rows(st, sp);
  const int max_waves = kLnMaxWaves / n_groups / 4 * 4;
  float *scratch = st->at<float>(st->lay.ln_partial) + (size_t)sums.n_layers * st->lay.ln_stride;
  for (int g = 0; g < n_groups; ++g) {
    int64_t row0 = first + rows * g / n_groups, end = first + rows * (g + 1) / n_groups;
    if (row0 >= gap0 && row0 < gap1) row0 = std::min(gap1, end);  // a gap at either end is cut off
    if (end > gap0 && end <= gap1) end = std::max(gap0, row0);
    const int64_t M = end - row0;
    LnBackArgs &x = l[g];
    x = LnBackArgs{};
    x.gap_row = std::min(std::max<int64_t>(gap0 - row0, 0), M);
    x.gap_end = std::min(std::max<int64_t>(gap1 - row0, 0), M);
    x.f = ln_args(st, level, j, row0, M, out ? out + (size_t)row0 * out_ld * (out_dtype == DT_BF16 ? 2 : 4) : nullptr, out_dtype, out_ld);
    x.dr = dr + (size_t)row0 * s.ld[j] * celt;
    x.dr_dtype = st->cdtype();
    x.dr_ld = s.ld[j];
    x.res = res ? res + (size_t)row0 * s.ld[j + 1] * celt : nullptr;
    x.res_dtype = st->cdtype();
    x.res_ld = s.ld[j + 1];
    x.partial = scratch + (size_t)g * (max_waves / 4) * 2 * s.dims[j];
    x.dgamma = st->d_ln_g[j];
    x.dbeta = st->d_ln_b[j];
  }
  HIP_TRY(st, launch_ln_relu_backward(l, n_groups, max_waves, sums.red[sums.n_layers], stream));
  sums.n_groups = n_groups;
  sums.n_layers += 1;
  return !sp.whole || sums.n_layers == st->lay.ln_layers ? sums.add_up(st, stream) : (int)GNNSTAGE_OK;
}

// What a pass needs before its first chunk: staged weights; ResGCN+: Rh = f(hist[j]), the activated historical rows; the
// transformed historical rows of transform-first layers (constants of the pass).
int begin_forward(gnnstage *st, const std::vector<int32_t> *order, hipStream_t stream) {
  const Shape &s = st->s;
  const int cd = st->cdtype();
  st->order.clear();
  st->tables_written = false;
  st->fmask = ChunkMask{};
  st->bmask = ChunkMask{};
  st->n_bwd = 0;
  st->wgrad_pending.assign((size_t)s.K, 0);  // what an abandoned backward pass still owed is dropped with it
  st->dropout_p = st->next_dropout_p;
  st->dropout_seed = st->next_dropout_seed;
  {
    Timed t(st, stream, 6);
    std::vector<StageWeightsArgs> w;
    for (int j = 0; j < s.L; ++j) {
      // GraphSage: W[j] = [W_self ; W_neigh]; Wt / Wn take the half that multiplies the aggregation
      const char *Wagg = static_cast<const char *>(st->W[j]) + (s.sage() ? s.w_half(j) * s.elt() : 0);
      w.push_back(StageWeightsArgs{Wagg, s.dims[j], s.dims[j + 1], st->at<char>(st->lay.Wt[j]), s.ld[j], st->at<char>(st->lay.Wn[j]), s.ld[j + 1]});
      if (s.sage())
        w.push_back(StageWeightsArgs{st->W[j], s.dims[j], s.dims[j + 1], st->at<char>(st->lay.Wt_self[j]), s.ld[j], st->at<char>(st->lay.Wn_self[j]), s.ld[j + 1]});
    }
    PassTableArgs tables;
    const bool with_tables = order != nullptr && by_table(st);
    if (with_tables) plan_pass_tables(st, *order, tables);
    HIP_TRY(st, launch_stage_weights(w.data(), (int)w.size(), cd, with_tables ? &tables : nullptr, stream));
    st->tables_written = with_tables;
  }
  for (int j = 0; j < s.L; ++j) {
    if (s.res()) {
      Timed t(st, stream, 1, j);
      const LnArgs a = ln_args(st, st->hist, j, 0, s.n, st->at<char>(st->lay.Th[j]), cd, s.ld[j]);
      HIP_TRY(st, launch_ln_relu(a, stream));
    } else if (s.tf[j]) {
      Timed t(st, stream, 1, j);
      GemmNtArgs g = nt_args(st, st->hist[j], st->level_dtype(j), s.dims[j], st->lay.Wt[j], s.ld[j], s.n, s.dims[j + 1], s.dims[j]);
      nt_out(g, st->at<char>(st->lay.Th[j]), cd, s.ld[j + 1]);
      HIP_TRY(st, launch_gemm_nt(g, cd, stream));
    }
  }
  return GNNSTAGE_OK;
}

// Whether level j never changes: a first stage's input that is its own history.  One table of its rows then serves as current and as
// historical ones.  (A level that is its own history and is computed - above 0, or level 0 of a stage that hands a gradient
// down - holds rows of this pass and of the last one: what is made of the historical rows when the pass begins, and of a
// chunk's current rows with the chunk, are two tables.  A whole pass finds all rows of its level 0 there when it begins: one table.)
bool constant_level(const gnnstage *st, int j) { return j == 0 && !st->s.need_input_grad && st->hist[0] == st->cur[0]; }

// Layer j of a span's chunks (which have rows).  The chunks of a whole pass go side by side: layer j of a chunk reads rows of
// level j alone, of the chunks processed up to its own the current ones and of the others the historical ones, whatever has been computed of
// the levels above; so a pass is one round of launches per layer, not per chunk and layer, and a launch's rows gather from the
// tables of one layer.
//   aggregate first:  Z = A_hat (cur | hist); cur[j + 1] = epilogue(Z W)             GraphSage: + h_v W_self
//   transform first:  Tc = cur W; cur[j + 1] = ReLU(A_hat (Tc | Th) + b)
//   ResGCN+:          r_u = ReLU(LayerNorm_j(h_u)) on whichever row of u is read, z_v = sum_u A_vu r_u,
//                     h'_v = h_v + z_v W_j + b_j; Rc[C_k] = f(cur[j][C_k]) is computed with the chunk
int forward_layer(gnnstage *st, int j, const Span &sp, hipStream_t stream) {
  const Shape &s = st->s;
  const int cd = st->cdtype();
  const size_t celt = s.elt();
  const int64_t row0 = span_row0(st, sp), M = span_rows(st, sp);
  const bool shared = constant_level(st, j) || (sp.whole && st->hist[j] == st->cur[j]);
  if (!shared && s.res()) {
    Timed t(st, stream, 1, j);
    HIP_TRY(st, launch_ln_relu(ln_args(st, st->cur, j, row0, M, st->at<char>(st->lay.Tc[j]) + (size_t)row0 * s.ld[j] * celt, cd, s.ld[j]), stream));
  } else if (!shared && s.tf[j]) {  // the span's current rows
    Timed t(st, stream, 1, j);
    GemmNtArgs g = nt_args(st, level_rows(st, st->cur, j, row0), st->level_dtype(j), s.dims[j], st->lay.Wt[j], s.ld[j], M, s.dims[j + 1], s.dims[j]);
    nt_out(g, st->at<char>(st->lay.Tc[j]) + (size_t)row0 * s.ld[j + 1] * celt, cd, s.ld[j + 1]);
    HIP_TRY(st, launch_gemm_nt(g, cd, stream));
  }
  SpmmArgs a{};
  int src_dtype = cd;
  a.epilogue = SPMM_PLAIN;
  if (s.tf[j] || s.res()) {
    a.src_unsel = st->at<char>(st->lay.Th[j]);
    a.src_sel = shared ? a.src_unsel : st->at<char>(st->lay.Tc[j]);
    a.d = s.tf[j] ? s.dims[j + 1] : s.dims[j];
    a.src_ld = s.tf[j] ? s.ld[j + 1] : s.ld[j];
  } else {
    a.src_sel = st->cur[j];
    a.src_unsel = st->hist[j];
    a.d = s.dims[j];
    a.src_ld = s.dims[j];
    src_dtype = st->level_dtype(j);
  }
  if (s.tf[j]) {
    a.out = st->cur[j + 1];
    a.out_ld = s.dims[j + 1];
    a.epilogue = SPMM_BIAS_RELU;
    a.bias = static_cast<const float *>(st->bias[j]);
  } else {
    a.out = st->at<char>(st->lay.Z[j]);
    a.out_ld = s.ld[j];
  }
  if (s.variant == GNNSTAGE_GCNII) {
    a.epilogue = SPMM_MIX;
    a.aux = st->h0;
    a.aux_ld = s.dims[j];
    a.s_acc = 1.f - st->alpha;
    a.s_aux = st->alpha;
  }
  HIP_TRY(st, run_spmm(st, a, src_dtype, cd, false, sp, span_select(st, sp, SEL_FORWARD), stream, 0, j));
  char *const level = static_cast<char *>(st->cur[j + 1]);
  if (s.tf[j]) {
    if (st->output_dropout())  // on the rows just written, in place
      HIP_TRY(st, launch_dropout_rows(level + (size_t)row0 * s.dims[j + 1] * celt, cd, M, s.dims[j + 1], s.dims[j + 1], st->dropout(j, row0), stream));
    return GNNSTAGE_OK;
  }
  Timed t(st, stream, 1, j);
  // GraphSage: blocks of rows, the vertex's own row through W_self kept in fp32 until the layer's epilogue adds it
  const int64_t step = s.sage() ? st->lay.self_rows : M;
  for (int64_t r = row0; r < row0 + M; r += step) {
    const int64_t m = std::min(step, row0 + M - r);
    if (s.sage()) {
      GemmNtArgs g = nt_args(st, level_rows(st, st->cur, j, r), st->level_dtype(j), s.dims[j], st->lay.Wt_self[j], s.ld[j], m, s.dims[j + 1], s.dims[j]);
      nt_out(g, st->at<float>(st->lay.self_fwd), DT_F32, s.ld[j + 1]);
      HIP_TRY(st, launch_gemm_nt(g, cd, stream));
    }
    GemmNtArgs g = nt_args(st, st->at<char>(st->lay.Z[j]) + (size_t)r * s.ld[j] * celt, cd, s.ld[j], st->lay.Wt[j], s.ld[j], m, s.dims[j + 1], s.dims[j]);
    if (s.variant == GNNSTAGE_GCNII) {
      g.epilogue = EPI_FWD_GCNII;
      g.aux = g.A;
      g.aux_dtype = cd;
      g.aux_ld = s.ld[j];
      g.beta = st->beta[j];
    } else {
      g.epilogue = EPI_FWD_GCN;
      g.bias = static_cast<const float *>(st->bias[j]);
      if (s.sage()) {
        g.epilogue = EPI_FWD_ADD;
        g.aux = st->at<float>(st->lay.self_fwd);
        g.aux_dtype = DT_F32;
        g.aux_ld = s.ld[j + 1];
      } else if (s.res()) {
        g.epilogue = EPI_RES;
        g.aux = level_rows(st, st->cur, j, r);
        g.aux_dtype = st->level_dtype(j);
        g.aux_ld = s.dims[j];
      }
    }
    nt_out(g, level + (size_t)r * s.dims[j + 1] * celt, cd, s.dims[j + 1]);
    if (st->output_dropout()) g.drop = st->dropout(j, r);
    HIP_TRY(st, launch_gemm_nt(g, cd, stream));
  }
  return GNNSTAGE_OK;
}

// dW_j += scale * Z_j^T dY (and the bias gradient) over rows [r0, r0 + M) of an aggregate-first layer: the products of it
void wgrad_products(gnnstage *st, int j, int64_t r0, int64_t M, const char *dY, std::vector<GemmTnArgs> &out) {
  const Shape &s = st->s;
  const int cd = st->cdtype();
  GemmTnArgs w = tn_args(st, st->at<char>(st->lay.Z[j]) + (size_t)r0 * s.ld[j] * s.elt(), cd, s.ld[j], dY, s.ld[j + 1], M, s.dims[j], s.dims[j + 1],
                         s.variant == GNNSTAGE_GCNII ? st->beta[j] : 1.f,
                         st->dW[j] + (s.sage() ? s.w_half(j) : 0));  // GraphSage: W_neigh is the lower half
  if (s.has_bias()) {
    w.dbias = st->dbias[j];
    w.bias_partial = st->at<float>(st->lay.bias_partial);
  }
  out.push_back(w);
  if (s.sage())  // dW_self += h_v^T dY over the rows' own (current) level-j values
    out.push_back(tn_args(st, level_rows(st, st->cur, j, r0), st->level_dtype(j), s.dims[j], dY, s.ld[j + 1], M, s.dims[j], s.dims[j + 1], 1.f, st->dW[j]));
}
int run_products(gnnstage *st, const std::vector<GemmTnArgs> &w, int layer, hipStream_t stream) {
  Timed t(st, stream, 4, layer);
  HIP_TRY(st, launch_gemm_tn_list(w.data(), (int)w.size(), st->lay.gemm_partial_floats, st->lay.bias_partial_floats, st->cdtype(), stream));
  return GNNSTAGE_OK;
}
int wgrad_rows(gnnstage *st, int j, int64_t r0, int64_t M, const char *dY, hipStream_t stream) {
  std::vector<GemmTnArgs> w;
  wgrad_products(st, j, r0, M, dY, w);
  return run_products(st, w, j, stream);
}

// Weight (and bias) gradients of the aggregate-first layers that the backward calls made so far still owe:
// dW_j += scale * Z_j^T dY_j over the rows of every maximal run of chunks whose backward call has run.  A complete
// pass is one run, i.e. one product per layer over all n rows.
int flush_deferred_wgrad(gnnstage *st, hipStream_t stream) {
  const Shape &s = st->s;
  if (!s.defer_wgrad() || st->wgrad_pending.empty()) return GNNSTAGE_OK;
  const size_t celt = s.elt();
  int c = 0;
  while (c < s.K) {
    if (!st->wgrad_pending[(size_t)c]) {
      ++c;
      continue;
    }
    int c1 = c;
    while (c1 < s.K && st->wgrad_pending[(size_t)c1]) st->wgrad_pending[(size_t)c1++] = 0;
    const int64_t r0 = s.chunk_ptr[c], M = s.chunk_ptr[c1] - r0;
    c = c1;
    if (M <= 0) continue;
    if (M > 0x7fffffff) return fail(st, GNNSTAGE_ENOTSUP, "more than 2^31 - 1 rows in one weight-gradient product");
    std::vector<GemmTnArgs> w;
    for (int j = s.L - 1; j >= 0; --j) {
      if (s.tf[j]) continue;  // transform-first layers: finish_transform_first
      wgrad_products(st, j, r0, M, st->at<char>(st->lay.dY[j]) + (size_t)r0 * s.ld[j + 1] * celt, w);
      if (st->prof.kinds == 0) continue;  // (a timed launch belongs to one layer)
      const int rc = run_products(st, w, j, stream);
      if (rc != GNNSTAGE_OK) return rc;
      w.clear();
    }
    const int rc = w.empty() ? (int)GNNSTAGE_OK : run_products(st, w, -1, stream);
    if (rc != GNNSTAGE_OK) return rc;
  }
  return GNNSTAGE_OK;
}

// Whether a product over all rows can count them (and its tiles' rows beyond them) in 32 bits.
bool rows_in_one_product(const gnnstage *st) { return st->s.n <= 0x7fff0000; }

// The spans of the work behind a pass's last backward call: all chunks side by side, one by one while launches are timed (a
// timed launch belongs to one chunk's share).  earlier: with the masks of the chunks in front of each in the forward order.
int finish_spans(gnnstage *st, bool earlier, std::vector<Span> &spans, hipStream_t stream) {
  spans.clear();
  ChunkMask m{};
  if (st->prof.kinds == 0 && rows_in_one_product(st)) {
    spans.push_back(whole_span(st));
    spans[0].mask = ChunkMask{};
    for (int c = 0; c < st->s.K && !earlier; ++c) mask_set(spans[0].mask, (uint32_t)c);
    return earlier ? write_pass_tables(st, st->order, stream) : (int)GNNSTAGE_OK;
  }
  for (int c = 0; c < st->s.K && !earlier; ++c) mask_set(m, c);
  for (size_t i = 0; i < st->order.size(); ++i) {
    const int c = st->order[i];
    if (st->s.chunk_ptr[(size_t)c + 1] > st->s.chunk_ptr[(size_t)c]) spans.push_back(chunk_span(c, m));
    if (earlier) mask_set(m, c);
  }
  return GNNSTAGE_OK;
}

// After the last backward call of a pass: the history-side weight gradient of every transform-first layer, dW += hist^T dT.
// dT sums over the readers that saw the historical row; over all readers where the current side has not been taken (a level
// that serves as both and has no gradient of its own, see backward_layer).
int finish_transform_first(gnnstage *st, hipStream_t stream) {
  const Shape &s = st->s;
  const int cd = st->cdtype();
  std::vector<Span> spans;
  for (int j = 0; j < s.L; ++j) {
    if (!s.tf[j]) continue;
    const bool all = constant_level(st, j);
    const int rc = finish_spans(st, !all, spans, stream);
    if (rc != GNNSTAGE_OK) return rc;
    for (const Span &sp : spans) {
      SpmmArgs a{};
      a.src_sel = st->at<char>(st->lay.dZ[j]);
      a.src_unsel = nullptr;
      a.d = s.dims[j + 1];
      a.src_ld = s.ld[j + 1];
      a.out = st->at<char>(st->lay.Th[j]);  // the transformed historical rows have been read for the last time
      a.out_ld = s.ld[j + 1];
      a.epilogue = SPMM_PLAIN;
      HIP_TRY(st, run_spmm(st, a, cd, cd, true, sp, all ? SEL_MASK : span_select(st, sp, SEL_EARLIER), stream, 2, j));
      Timed t(st, stream, 4, j);
      const int64_t row0 = span_row0(st, sp);
      HIP_TRY(st, launch_gemm_tn(tn_args(st, level_rows(st, st->hist, j, row0), st->level_dtype(j), s.dims[j],
                                         st->at<char>(st->lay.Th[j]) + (size_t)row0 * s.ld[j + 1] * s.elt(), s.ld[j + 1], span_rows(st, sp), s.dims[j], s.dims[j + 1],
                                         1.f, st->dW[j]), cd, stream));
    }
  }
  return GNNSTAGE_OK;
}

// ResGCN+, after the last backward chunk: the LayerNorm of layer j was also applied to the historical rows, so its
// parameters receive gradient through every edge whose reader saw the historical row of u: the readers whose
// chunk came before u's chunk in the forward order.
int res_backward_finish(gnnstage *st, hipStream_t stream) {
  const Shape &s = st->s;
  const int cd = st->cdtype();
  if (s.K == 1) return GNNSTAGE_OK;  // no row was read as a historical one
  std::vector<Span> spans;
  const int rc = finish_spans(st, true, spans, stream);
  if (rc != GNNSTAGE_OK) return rc;
  LnSums sums;
  for (int j = 0; j < s.L; ++j)
    for (const Span &sp : spans) {
      if (!sp.whole && sp.c0 == st->order[0]) continue;  // nothing of it was read as historical rows
      SpmmArgs a{};
      a.src_sel = st->at<char>(st->lay.dZ[j]);
      a.src_unsel = nullptr;
      a.d = s.dims[j];
      a.src_ld = s.ld[j];
      a.out = st->at<char>(st->lay.Th[j]);
      a.out_ld = s.ld[j];
      a.epilogue = SPMM_PLAIN;
      HIP_TRY(st, run_spmm(st, a, cd, cd, true, sp, span_select(st, sp, SEL_EARLIER), stream, 2, j));
      Timed t(st, stream, 4, j);
      // no row of the chunk that came first was read as a historical one: it may hold anything, also what times zero is no number
      const int e = ln_backward(st, sums, st->hist, j, sp, st->order[0], st->at<char>(st->lay.Th[j]), nullptr, cd, 0, nullptr, stream);
      if (e != GNNSTAGE_OK) return e;
    }
  return sums.add_up(st, stream);
}

// Where dY_j = dL/d(pre-activation of layer j) of a chunk's rows lives, [M x ld_{j+1}], zero in the padding
// columns.  With deferred weight gradients: the chunk's rows of a matrix over all n rows (transform-first layers
// keep that matrix anyway, it is what later chunks' transposed aggregations gather); otherwise one of two
// chunk-sized scratch matrices, used alternately.
char *full_dY(const gnnstage *st, int j) { return st->at<char>(st->s.tf[j] ? st->lay.dZ[j] : st->lay.dY[j]); }
char *dY_rows(const gnnstage *st, int64_t row0, int j) {
  if (!st->s.defer_wgrad()) return st->at<char>(st->lay.G[st->gi]);
  return full_dY(st, j) + (size_t)row0 * st->s.ld[(size_t)j + 1] * st->s.elt();
}

// dY of the top layer for rows [row0, row0 + M): the upstream gradient behind the activation's derivative (ResGCN+: no
// activation after the convolution)
int top_dY(gnnstage *st, const void *grad_rows, int64_t row0, int64_t M, char *out, hipStream_t stream) {
  const Shape &s = st->s;
  Timed t(st, stream, 6);
  if (s.res())
    HIP_TRY(st, launch_copy_rows(grad_rows, s.dims[s.L], out, s.ld[s.L], M, s.dims[s.L], st->cdtype(), stream));
  else
    HIP_TRY(st, launch_relu_mask(grad_rows, static_cast<const char *>(st->cur[s.L]) + (size_t)row0 * s.dims[s.L] * s.elt(), st->cdtype(), M, s.dims[s.L],
                                 out, s.ld[s.L], st->mask_scale(), stream));
  return GNNSTAGE_OK;
}

// Layer j of a span's chunks on the way back; layers from the top.  Layer j of a chunk gathers gradient rows of layer j alone, of the chunks
// whose turn has come, so the chunks of a whole pass go side by side here too.
int backward_layer(gnnstage *st, LnSums &sums, int j, const Span &sp, hipStream_t stream) {
  const Shape &s = st->s;
  const int cd = st->cdtype();
  const size_t celt = s.elt();
  const int64_t row0 = span_row0(st, sp), M = span_rows(st, sp);
  const bool defer = s.defer_wgrad(), need_prev = j > 0 || s.need_input_grad;
  char *const dY = dY_rows(st, row0, j);
  // where the gradient of level j goes: leading dimension, type, first row (of all rows, or of the span's alone)
  const int prev_ld = j > 0 ? s.ld[j] : s.dims[0], prev_dtype = st->level_dtype(j);
  const bool prev_all = j == 0 || defer;
  char *const prev = j == 0 ? static_cast<char *>(st->grad_in) : defer ? full_dY(st, j - 1) : st->at<char>(st->lay.G[st->gi ^ 1]);
  char *const prev_rows = prev == nullptr ? nullptr : prev + (prev_all ? (size_t)row0 * prev_ld * (prev_dtype == DT_BF16 ? 2 : 4) : 0);
  // ---- bias gradients of transform-first layers, weight gradients that are not deferred; input-gradient products
  SpmmArgs a{};
  if (s.tf[j]) {
    // bias gradient = column sums of dY: fused into the weight-gradient product where that product reads dY
    // (aggregate-first layers), a kernel of its own for transform-first layers
    if (s.has_bias()) {
      Timed t(st, stream, 4, j);
      HIP_TRY(st, launch_colsum_add(dY, cd, s.ld[j + 1], (int)M, s.dims[j + 1], st->at<float>(st->lay.bias_partial), kMaxSplits, st->dbias[j], stream));
    }
    if (!defer) {
      Timed t(st, stream, 6);
      HIP_TRY(st, launch_copy(dY, full_dY(st, j) + (size_t)row0 * s.ld[j + 1] * celt, (size_t)M * s.ld[j + 1] * celt, stream));
    }
  } else {
    if (!defer) {
      const int rc = wgrad_rows(st, j, row0, M, dY, stream);
      if (rc != GNNSTAGE_OK) return rc;
    }
    if (s.res() || need_prev) {
      Timed t(st, stream, 3, j);
      GemmNtArgs g = nt_args(st, dY, cd, s.ld[j + 1], st->lay.Wn[j], s.ld[j + 1], M, s.dims[j], s.dims[j + 1]);
      nt_out(g, st->at<char>(st->lay.dZ[j]) + (size_t)row0 * s.ld[j] * celt, cd, s.ld[j]);
      if (s.variant == GNNSTAGE_GCNII) {
        g.epilogue = EPI_DGRAD_GCNII;
        g.aux = dY;
        g.aux_dtype = cd;
        g.aux_ld = s.ld[j + 1];
        g.alpha = st->alpha;
        g.beta = st->beta[j];
        g.h0grad = st->grad_h0 ? st->grad_h0 + (size_t)row0 * s.dims[j] : nullptr;
        g.h0_ld = s.dims[j];
      }
      HIP_TRY(st, launch_gemm_nt(g, cd, stream));
      if (s.sage()) {  // the gradient that reaches the chunk's own rows directly: dY W_self^T
        g.Bt = st->at<char>(st->lay.Wn_self[j]);
        const bool in_place = s.self_in_place(j);
        char *const at = in_place ? prev_rows : st->at<char>(st->lay.self_bwd) + (size_t)row0 * s.ld[j] * celt;
        nt_out(g, at, cd, in_place ? prev_ld : s.ld[j]);
        a.add = at;
        a.add_ld = g.out_ld;
        a.add_row0 = row0;
        HIP_TRY(st, launch_gemm_nt(g, cd, stream));
      }
    }
  }
  // ---- transposed aggregation; Section 3.4: nothing flows back from unprocessed vertices
  // transform first: see below; nothing else depends on dT_cur of a level that never changes.
  if (s.tf[j] ? constant_level(st, j) : !s.res() && !need_prev) {
    if (!defer && !s.tf[j]) st->gi ^= 1;
    return GNNSTAGE_OK;
  }
  int out_dtype = cd;
  a.src_sel = s.tf[j] ? full_dY(st, j) : st->at<char>(st->lay.dZ[j]);
  a.src_unsel = nullptr;
  a.d = s.tf[j] ? s.dims[j + 1] : s.dims[j];
  a.src_ld = s.tf[j] ? s.ld[j + 1] : s.ld[j];
  a.epilogue = SPMM_PLAIN;
  a.out_ld = a.src_ld;
  if (s.tf[j] && defer) {
    a.out = st->at<char>(st->lay.Tc[j]);  // the transformed current rows have been read for the last time
  } else if (s.tf[j]) {
    a.out = st->at<char>(st->lay.G[st->gi ^ 1]);
    a.out_row0 = row0;
  } else if (s.res()) {
    a.out = st->at<char>(st->lay.Th[j]);  // and the activated historical ones
  } else {
    a.out = prev;
    a.out_row0 = prev_all ? 0 : row0;
    a.out_ld = prev_ld;
    out_dtype = prev_dtype;
    if (j > 0) {
      a.epilogue = s.sage() ? SPMM_ADD_MASK : SPMM_MASK;
      a.mask_scale = st->mask_scale();
      a.aux = st->cur[j];
      a.aux_ld = s.dims[j];
    } else {
      a.epilogue = s.sage() ? SPMM_ADD : SPMM_PLAIN;
    }
  }
  HIP_TRY(st, run_spmm(st, a, cd, out_dtype, true, sp, span_select(st, sp, SEL_BACKWARD), stream, 2, j));
  // ---- behind it
  if (s.res()) {  // back through ReLU and LayerNorm of the span's own (current) rows, plus the residual branch
    Timed t(st, stream, 4, j);
    char *const all = !need_prev ? nullptr : prev_all ? prev : prev - (size_t)row0 * prev_ld * celt;
    const int rc = ln_backward(st, sums, st->cur, j, sp, -1, st->at<char>(st->lay.Th[j]), all, prev_dtype, prev_ld, dY - (size_t)row0 * s.ld[j + 1] * celt, stream);
    if (rc != GNNSTAGE_OK) return rc;
  } else if (s.tf[j]) {
    // Layer computed as A_hat (H W).  With T = H W:  dL/dW = cur^T dT_cur + hist^T dT_hist, where
    // dT_cur[u] sums A_vu dY[v] over the readers v that saw u's CURRENT row (exactly the vertices
    // already processed in this backward pass) and dT_hist over the readers that saw its history.  The first is taken here, the
    // second, which is known only when every chunk's dY is, after the last chunk (finish_transform_first).
    const char *dT = static_cast<const char *>(a.out) + (defer ? (size_t)row0 * s.ld[j + 1] * celt : 0);
    {
      Timed t(st, stream, 4, j);
      HIP_TRY(st, launch_gemm_tn(tn_args(st, level_rows(st, st->cur, j, row0), st->level_dtype(j), s.dims[j], dT, s.ld[j + 1], M, s.dims[j], s.dims[j + 1], 1.f, st->dW[j]),
                                 cd, stream));
    }
    if (need_prev) {
      Timed t(st, stream, 3, j);
      GemmNtArgs g = nt_args(st, dT, cd, s.ld[j + 1], st->lay.Wn[j], s.ld[j + 1], M, s.dims[j], s.dims[j + 1]);
      nt_out(g, j > 0 && !defer ? st->at<char>(st->lay.G[st->gi]) : prev_rows, prev_dtype, prev_ld);  // without deferral dY_j is dead by now and its scratch is reused
      if (j > 0) {
        g.epilogue = EPI_MASK;
        g.mask_scale = st->mask_scale();
        g.aux = level_rows(st, st->cur, j, row0);
        g.aux_dtype = cd;
        g.aux_ld = s.dims[j];
        g.out_pad = s.ld[j];
      }
      HIP_TRY(st, launch_gemm_nt(g, cd, stream));
    }
  }
  if (!defer && !s.tf[j]) st->gi ^= 1;
  return GNNSTAGE_OK;
}

// what the last call of a pass owes beyond its own rows: the deferred weight-gradient products, then the
// history-side gradients
int end_backward(gnnstage *st, hipStream_t stream) {
  if (st->n_bwd != st->s.K) return GNNSTAGE_OK;
  const int rc = flush_deferred_wgrad(st, stream);
  if (rc != GNNSTAGE_OK) return rc;
  return st->s.res() ? res_backward_finish(st, stream) : finish_transform_first(st, stream);
}

// Whether a pass may run layer by layer over all of its chunks.
bool whole_pass_ok(const gnnstage *st, const int32_t *order, int n) {
  if (n != st->s.K || !st->s.defer_wgrad() || st->prof.kinds != 0) return false;  // (timed launches belong to one chunk each)
  if (!rows_in_one_product(st)) return false;
  // a level above 0 that is its own history: what a chunk does not select are the rows of the last pass, which the level below
  // would have overwritten
  for (int j = 1; j < st->s.L; ++j)
    if (st->hist[j] == st->cur[j]) return false;
  std::vector<char> seen((size_t)n, 0);
  for (int i = 0; i < n; ++i) {
    if (order[i] < 0 || order[i] >= n || seen[(size_t)order[i]]) return false;
    seen[(size_t)order[i]] = 1;
  }
  return true;
}

}  // namespace

extern "C" int gnnstage_version(void) { return 100; }

extern "C" int64_t gnnstage_dense_entries(const gnnstage_t *st, int32_t transposed) {
  if (!st) return GNNSTAGE_EINVAL;
  return st->dense_entries[transposed ? 1 : 0];
}

extern "C" const char *gnnstage_last_error(const gnnstage_t *st) { return st ? st->err.c_str() : g_create_error.c_str(); }

namespace {
// transposed index and the per-direction plans: what both the size query and create need
struct HostPlan {
  std::vector<int64_t> t_ptr, t_edge;
  std::vector<int32_t> t_row;
  HostDir f, b;
};

int make_host_plan(const gnnstage_desc *d, const Shape &s, bool want_edge, HostPlan &hp, std::string &err) {
  if (s.nnz > 0 && !d->col_idx) {
    err = "col_idx is NULL";
    return GNNSTAGE_EINVAL;
  }
  hp.t_ptr.assign((size_t)s.n + 1, 0);
  hp.t_row.resize((size_t)s.nnz);
  if (want_edge) hp.t_edge.resize((size_t)s.nnz);
  if (gnnstage_plan_transpose(s.n, d->row_ptr, d->col_idx, hp.t_ptr.data(), hp.t_row.data(),
                              want_edge ? hp.t_edge.data() : nullptr) != GNNSTAGE_OK) {
    err = "col_idx is NULL or has an entry outside [0, n_vertices)";
    return GNNSTAGE_EINVAL;
  }
  const bool dense = s.dense_ok();
  if (!make_host_dir(s.tune, d->row_ptr, d->col_idx, s.n, s.chunk_ptr, s.classes(), s.hot(), want_edge, dense, s.dense_width(), s.least_piece(false), hp.f) ||
      !make_host_dir(s.tune, hp.t_ptr.data(), hp.t_row.data(), s.n, s.chunk_ptr, s.classes(), s.hot(), want_edge, dense, s.dense_width(), s.least_piece(true), hp.b)) {
    err = "cannot plan the aggregation";
    return GNNSTAGE_EINVAL;
  }
  return GNNSTAGE_OK;
}

uint16_t bf16_bits_rne(float f) {  // finite inputs: round to nearest even, as the device conversion does
  uint32_t u;
  memcpy(&u, &f, 4);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
float bf16_bits_to_f32(uint16_t h) {
  const uint32_t u = (uint32_t)h << 16;
  float f;
  memcpy(&f, &u, 4);
  return f;
}
}  // namespace

extern "C" size_t gnnstage_workspace_size(const gnnstage_desc *desc) try {
  Shape s;
  std::string err;
  if (!read_shape(desc, s, err)) {
    g_create_error = err;
    return 0;
  }
  HostPlan hp;
  if (make_host_plan(desc, s, false, hp, err) != GNNSTAGE_OK) {
    g_create_error = err;
    return 0;
  }
  return make_layout(s, hp.f, hp.b, desc->edge_val == nullptr).total;
}
GNNSTAGE_GUARD_SIZE

extern "C" int gnnstage_create(const gnnstage_desc *d, gnnstage_t **out) try {
  if (!out) return fail(nullptr, GNNSTAGE_EINVAL, "out is NULL");
  *out = nullptr;
  Shape s;
  std::string err;
  if (!read_shape(d, s, err)) return fail(nullptr, GNNSTAGE_EINVAL, err);
  // The library computes the weights itself: w(v, u) = s_row(v) s_col(u), which the dense blocks keep as patterns.
  const bool rank1 = d->edge_val == nullptr;
  // GraphSage without weights: the mean aggregator, 1 / |N(v)| on every entry of row v; the sparse kernels take
  // it from here on like weights the caller gave
  std::vector<float> mean_val;
  gnnstage_desc with_mean;
  if (s.sage() && !d->edge_val && d->row_ptr) {
    mean_val.resize((size_t)s.nnz);
    for (int64_t v = 0; v < s.n; ++v) {
      const int64_t e0 = d->row_ptr[v], e1 = d->row_ptr[v + 1];
      if (e0 < 0 || e1 < e0 || e1 > s.nnz) return fail(nullptr, GNNSTAGE_EINVAL, "row_ptr is not a valid CSR pointer array");
      for (int64_t e = e0; e < e1; ++e) mean_val[(size_t)e] = 1.f / (float)(e1 - e0);
    }
    with_mean = *d;
    with_mean.edge_val = mean_val.data();
    d = &with_mean;
  }
  if (!d->W || !d->cur || !d->hist) return fail(nullptr, GNNSTAGE_EINVAL, "W, cur and hist must not be NULL");
  if (!d->dW) return fail(nullptr, GNNSTAGE_EINVAL, "dW must not be NULL");
  if (s.has_bias() && (!d->bias || !d->dbias)) return fail(nullptr, GNNSTAGE_EINVAL, "GCN and GraphSage need bias and dbias");
  if (s.variant == GNNSTAGE_GCNII && (!d->beta || !d->h0)) return fail(nullptr, GNNSTAGE_EINVAL, "GCNII needs beta and h0");
  if (s.res()) {
    if (!d->ln_gamma || !d->ln_beta || !d->d_ln_gamma || !d->d_ln_beta)
      return fail(nullptr, GNNSTAGE_EINVAL, "ResGCN+ needs ln_gamma, ln_beta and their gradient arrays");
    for (int j = 0; j < s.L; ++j)
      if (!d->ln_gamma[j] || !d->ln_beta[j] || !d->d_ln_gamma[j] || !d->d_ln_beta[j])
        return fail(nullptr, GNNSTAGE_EINVAL, "a LayerNorm parameter pointer is NULL");
    if (!(d->ln_eps > 0.f)) return fail(nullptr, GNNSTAGE_EINVAL, "ln_eps must be positive");
  }
  if (!(d->dropout_p >= 0.f && d->dropout_p < 1.f)) return fail(nullptr, GNNSTAGE_EINVAL, "dropout_p must be in [0, 1)");
  if (d->dropout_p > 0.f && s.variant == GNNSTAGE_GCNII) return fail(nullptr, GNNSTAGE_EINVAL, "no dropout in GCNII layers");
  if (s.need_input_grad && !d->grad_in) return fail(nullptr, GNNSTAGE_EINVAL, "need_input_grad set but grad_in is NULL");
  if (!d->workspace || (reinterpret_cast<uintptr_t>(d->workspace) & (kAlign - 1)))
    return fail(nullptr, GNNSTAGE_EINVAL, "workspace must be a 256-byte aligned device pointer");
  for (int j = 0; j <= s.L; ++j) {
    if (!d->cur[j] || !aligned16(d->cur[j])) return fail(nullptr, GNNSTAGE_EINVAL, "cur[j] NULL or not 16-byte aligned");
    if (j < s.L) {
      if (!d->hist[j] || !aligned16(d->hist[j])) return fail(nullptr, GNNSTAGE_EINVAL, "hist[j] NULL or not 16-byte aligned");
      if (!d->W[j] || !d->dW[j]) return fail(nullptr, GNNSTAGE_EINVAL, "W[j] / dW[j] NULL");
      if (s.has_bias() && (!d->bias[j] || !d->dbias[j])) return fail(nullptr, GNNSTAGE_EINVAL, "bias[j] / dbias[j] NULL");
    }
  }
  if ((d->h0 && !aligned16(d->h0)) || (d->grad_in && !aligned16(d->grad_in)))
    return fail(nullptr, GNNSTAGE_EINVAL, "h0 / grad_in not 16-byte aligned");

  // ---- host planning -------------------------------------------------------------------
  HostPlan hp;
  int rc = make_host_plan(d, s, d->edge_val != nullptr, hp, err);
  if (rc != GNNSTAGE_OK) return fail(nullptr, rc, err);
  const std::vector<int64_t> &t_ptr = hp.t_ptr, &t_edge = hp.t_edge;
  int vbits = 0;
  std::vector<uint32_t> pcol((size_t)hp.f.nnz), prow((size_t)hp.b.nnz);
  rc = gnnstage_plan_pack(s.n, hp.f.nnz, hp.f.idx, s.K, s.chunk_ptr.data(), pcol.data(), &vbits);
  if (rc == GNNSTAGE_ENOTSUP)
    return fail(nullptr, rc, "vertex-id bits + chunk-id bits exceed the 32-bit packed index word");
  if (rc != GNNSTAGE_OK) return fail(nullptr, rc, "cannot pack column indices");
  rc = gnnstage_plan_pack(s.n, hp.b.nnz, hp.b.idx, s.K, s.chunk_ptr.data(), prow.data(), &vbits);
  if (rc != GNNSTAGE_OK) return fail(nullptr, rc, "cannot pack row indices");

  Layout lay = make_layout(s, hp.f, hp.b, rank1);
  if (d->workspace_bytes < lay.total) {
    char buf[160];
    snprintf(buf, sizeof buf, "workspace too small: %zu bytes given, %zu needed", d->workspace_bytes, lay.total);
    return fail(nullptr, GNNSTAGE_ENOMEM, buf);
  }

  std::unique_ptr<gnnstage> holder(new gnnstage());  // freed on every early return, and when something below throws
  gnnstage *st = holder.get();
  st->s = s;
  st->lay = lay;
  st->vbits = vbits;
  st->alpha = d->alpha;
  if (s.res()) {
    for (int j = 0; j < s.L; ++j) {
      st->ln_g.push_back(static_cast<const float *>(d->ln_gamma[j]));
      st->ln_b.push_back(static_cast<const float *>(d->ln_beta[j]));
      st->d_ln_g.push_back(d->d_ln_gamma[j]);
      st->d_ln_b.push_back(d->d_ln_beta[j]);
    }
    st->ln_eps = d->ln_eps;
  }
  st->dropout_p = st->next_dropout_p = d->dropout_p;
  if (d->beta) st->beta.assign(d->beta, d->beta + s.L); else st->beta.assign(s.L, 0.f);
  st->W.assign(d->W, d->W + s.L);
  st->cur.assign(d->cur, d->cur + s.L + 1);
  st->hist.assign(d->hist, d->hist + s.L);
  st->dW.assign(d->dW, d->dW + s.L);
  if (d->bias) st->bias.assign(d->bias, d->bias + s.L); else st->bias.assign(s.L, nullptr);
  if (d->dbias) st->dbias.assign(d->dbias, d->dbias + s.L); else st->dbias.assign(s.L, nullptr);
  st->h0 = d->h0;
  st->grad_in = d->grad_in;
  st->grad_h0 = d->grad_h0;
  st->ws = static_cast<char *>(d->workspace);
  st->prof.init(s.L);
  st->n_classes = s.classes();
  st->h_row_ptr.assign(d->row_ptr, d->row_ptr + s.n + 1);
  if (hp.f.dense()) {  // the diagnostics walk the whole index, not the remainder
    st->h_pcol.resize((size_t)s.nnz);
    if (gnnstage_plan_pack(s.n, s.nnz, d->col_idx, s.K, s.chunk_ptr.data(), st->h_pcol.data(), &vbits) != GNNSTAGE_OK)
      return fail(nullptr, GNNSTAGE_EINVAL, "cannot pack column indices");
  } else {
    st->h_pcol = pcol;
  }

  // schedules: built on the host chunk by chunk, put into sections (DirTasks), uploaded into the preallocated arrays
  const int classes = s.classes();
  auto build = [&](const HostDir &h, const uint32_t *packed, int dir) -> int {
    const int64_t *ptr = h.ptr;
    const int32_t *idx = h.idx;
    const PlanCounts &pc = h.pc;
    DirTasks &t = st->tasks[dir];
    t.K = s.K;
    t.n_classes = classes > 1 ? classes : 0;
    const int n_sec = t.n_classes + 2;
    struct Section {  // room for the most it can hold, of which only what is written takes memory
      std::unique_ptr<int32_t[]> row, slot;
      std::unique_ptr<int64_t[]> e0;
      std::unique_ptr<uint32_t[]> ne;
      int64_t size = 0;
      explicit Section(int64_t most)
          : row(new int32_t[(size_t)most]), slot(new int32_t[(size_t)most]), e0(new int64_t[(size_t)most]), ne(new uint32_t[(size_t)most]) {}
      void add(int32_t r, int64_t e, uint32_t n, int32_t sl) {
        row[(size_t)size] = r;
        e0[(size_t)size] = e;
        ne[(size_t)size] = n;
        slot[(size_t)size++] = sl;
      }
    };
    std::vector<Section> sec;
    for (int q = 0; q < n_sec; ++q) sec.emplace_back(q < t.n_classes ? pc.total_slots : s.task_capacity(pc.total_tasks));  // class pieces have slots
    std::vector<std::vector<int64_t>> upto((size_t)n_sec, std::vector<int64_t>(1, 0));  // tasks of a section up to every chunk's end
    t.slot_off.assign(1, 0);
    t.lr_off.assign(1, 0);
    t.item_off.assign(h.chunk_item_off.begin(), h.chunk_item_off.end());
    t.cls_entries.assign((size_t)s.K * t.n_classes * s.K, 0);
    t.cls_total.assign((size_t)s.K * t.n_classes, 0);
    std::vector<uint8_t> slot_class;
    std::vector<int32_t> lrow, lslot0, ldense0, lndense, litem0;
    std::vector<uint32_t> ln;
    const int short_row = s.short_row() > 0 ? s.short_row() : -1;  // -1: no row is
    std::vector<int32_t> row, ne, slot;
    std::vector<int64_t> e0;
    for (int c = 0; c < s.K; ++c) {
      const int64_t cap = std::max<int64_t>(pc.tasks[c], 1);
      row.resize((size_t)cap);
      ne.resize((size_t)cap);
      slot.resize((size_t)cap);
      e0.resize((size_t)cap);
      int64_t ns = 0;
      std::vector<int64_t> coff(classes + 1, 0);
      std::vector<uint8_t> sclass((size_t)std::max<int64_t>(pc.slots[c], 1), 255);
      // class bounds: equal shares of the chunk's entries over the id range, or (hotness classes) slices of
      // hot_rows ranks each, the ranks beyond the last slice belonging to no class
      std::vector<int64_t> cls_lo;
      if (h.hot.active) {
        cls_lo.resize((size_t)classes + 1);
        for (int q = 0; q <= classes; ++q) cls_lo[(size_t)q] = std::min<int64_t>((int64_t)q * s.hot_rows(), s.n);
      } else {
        cls_lo = class_bounds_by_entries(ptr, idx, s.n, s.chunk_ptr[c], s.chunk_ptr[c + 1], classes, s.chunk_ptr);
      }
      const int64_t got = pc.tasks[c] == 0 ? 0 : gnnstage_plan_tasks(ptr, h.hot.active ? h.hot.rank.data() : idx, s.n, s.chunk_ptr[c], s.chunk_ptr[c + 1],
                                              pc.split[c], classes, cls_lo.data(), h.min_row, h.force_ptr(), cap, row.data(),
                                              e0.data(), ne.data(), slot.data(), &ns, coff.data(), sclass.data());
      if (got < 0 || got > pc.tasks[c] || ns > pc.slots[c]) return GNNSTAGE_EINVAL;
      const int64_t slot0 = t.slot_off.back(), l0 = t.lr_off.back();
      const uint32_t chunk_bits = (uint32_t)c << kTaskChunkShift;
      Section &tail = sec[(size_t)t.n_classes], &shorts = sec[(size_t)n_sec - 1];
      int64_t i = 0;
      for (int q = 0; q < t.n_classes; ++q) {
        Section &x = sec[(size_t)q];
        int64_t *entries = &t.cls_entries[((size_t)c * t.n_classes + q) * s.K];
        for (; i < coff[(size_t)q + 1]; ++i) {
          x.add(row[(size_t)i], e0[(size_t)i], (uint32_t)ne[(size_t)i] | chunk_bits, (int32_t)(slot0 + slot[(size_t)i]));
          for (int64_t e = e0[(size_t)i]; e < e0[(size_t)i] + ne[(size_t)i]; ++e) entries[packed[e] >> vbits] += 1;
          t.cls_total[(size_t)c * t.n_classes + q] += ne[(size_t)i];
        }
      }
      for (; i < got; ++i) {
        if ((uint32_t)ne[(size_t)i] > kTaskCountMask) return GNNSTAGE_ENOTSUP;
        const bool piece = slot[(size_t)i] >= 0;
        Section &x = !piece && ne[(size_t)i] <= short_row ? shorts : tail;
        x.add(row[(size_t)i], e0[(size_t)i], (uint32_t)ne[(size_t)i] | chunk_bits, piece ? (int32_t)(slot0 + slot[(size_t)i]) : -1);
      }
      while (shorts.size % 4 != 0) shorts.add(-1, 0, chunk_bits, -1);
      for (int q = 0; q < n_sec; ++q) upto[(size_t)q].push_back(sec[(size_t)q].size);
      slot_class.insert(slot_class.end(), sclass.begin(), sclass.begin() + ns);
      t.slot_off.push_back(slot0 + ns);
      // cut rows: their slots are consecutive, so sorting the pieces by slot groups them by row
      std::vector<std::pair<int32_t, int32_t>> sr;
      for (int64_t i = 0; i < got; ++i)
        if (slot[(size_t)i] >= 0) sr.emplace_back(slot[(size_t)i], row[(size_t)i]);
      std::sort(sr.begin(), sr.end());
      auto add_long = [&](int32_t r, int32_t first_slot) {
        lrow.push_back(r);
        lslot0.push_back(first_slot);
        ln.push_back(chunk_bits);
        ldense0.push_back(0);
        lndense.push_back(0);
        litem0.push_back(0);
      };
      for (const auto &p : sr) {
        if ((int64_t)lrow.size() == l0 || lrow.back() != p.second) add_long(p.second, (int32_t)(slot0 + p.first));
        ln.back() += 1;
      }
      // rows of dense row blocks: their dense partial rows join the pieces (a row without any piece is added)
      const int64_t it_end = t.item_off[(size_t)c + 1];
      if (it_end > t.item_off[(size_t)c]) {
        std::vector<int64_t> where((size_t)(s.chunk_ptr[c + 1] - s.chunk_ptr[c]), -1);
        for (size_t i = (size_t)l0; i < lrow.size(); ++i) where[(size_t)(lrow[i] - s.chunk_ptr[c])] = (int64_t)i;
        int64_t it = t.item_off[(size_t)c];
        while (it < it_end) {
          int64_t it2 = it;
          while (it2 < it_end && h.item_rb[(size_t)it2] == h.item_rb[(size_t)it]) ++it2;
          const int64_t p0 = (int64_t)h.item_rb[(size_t)it] * kDenseRB;
          const int64_t p1 = std::min<int64_t>(p0 + kDenseRB, s.chunk_ptr[c + 1] - s.chunk_ptr[c]);
          if ((it + 1) * kDenseRB > 0x7fffffff) return GNNSTAGE_ENOTSUP;
          for (int64_t pp = p0; pp < p1; ++pp) {
            const int32_t r = h.dp.row_perm[(size_t)(s.chunk_ptr[c] + pp)];
            int64_t at = where[(size_t)(r - s.chunk_ptr[c])];
            if (at < 0) {
              at = (int64_t)lrow.size();
              add_long(r, (int32_t)slot0);
            }
            ldense0[(size_t)at] = (int32_t)(it * kDenseRB + (pp - p0));
            lndense[(size_t)at] = (int32_t)(it2 - it);
            litem0[(size_t)at] = (int32_t)it;
          }
          it = it2;
        }
      }
      t.lr_off.push_back((int64_t)lrow.size());
      if (t.lr_off.back() - l0 > pc.longs[c] || t.slot_off.back() > 0x7fffffff) return GNNSTAGE_ENOTSUP;
    }
    int64_t at = 0;
    auto up = [&](size_t off, const void *src, size_t elt, size_t count, int64_t first) {
      return count == 0 || hipMemcpy(st->at<char>(off) + (size_t)first * elt, src, count * elt, hipMemcpyHostToDevice) == hipSuccess;
    };
    for (int q = 0; q < n_sec; ++q) {
      const Section &x = sec[(size_t)q];
      for (const int64_t u : upto[(size_t)q]) t.sec.push_back(at + u);
      const size_t n = (size_t)x.size;
      if (at + x.size > s.task_capacity(pc.total_tasks)) return GNNSTAGE_ENOTSUP;
      if (!up(dir ? lay.b_task_row : lay.f_task_row, x.row.get(), 4, n, at) || !up(dir ? lay.b_task_e0 : lay.f_task_e0, x.e0.get(), 8, n, at) ||
          !up(dir ? lay.b_task_ne : lay.f_task_ne, x.ne.get(), 4, n, at) || !up(dir ? lay.b_task_slot : lay.f_task_slot, x.slot.get(), 4, n, at))
        return GNNSTAGE_EHIP;
      at += x.size;
    }
    if (at > 0x7fffffff) return GNNSTAGE_ENOTSUP;  // sections are indexed in 32 bits
    if (!up(dir ? lay.b_slot_class : lay.f_slot_class, slot_class.data(), 1, slot_class.size(), 0) || !up(dir ? lay.b_lr_row : lay.f_lr_row, lrow.data(), 4, lrow.size(), 0) ||
        !up(dir ? lay.b_lr_slot0 : lay.f_lr_slot0, lslot0.data(), 4, lslot0.size(), 0) || !up(dir ? lay.b_lr_n : lay.f_lr_n, ln.data(), 4, ln.size(), 0))
      return GNNSTAGE_EHIP;
    if (h.dense() && (!up(lay.d_lr_dense0[dir], ldense0.data(), 4, ldense0.size(), 0) || !up(lay.d_lr_ndense[dir], lndense.data(), 4, lndense.size(), 0) ||
                      !up(lay.d_lr_item0[dir], litem0.data(), 4, litem0.size(), 0)))
      return GNNSTAGE_EHIP;
    return GNNSTAGE_OK;
  };

  auto bail = [&](int code, const std::string &msg) { return fail(nullptr, code, msg); };
  if (hipMemcpy(st->at<int64_t>(lay.row_ptr), d->row_ptr, sizeof(int64_t) * (s.n + 1), hipMemcpyHostToDevice) != hipSuccess ||
      hipMemcpy(st->at<int64_t>(lay.t_ptr), t_ptr.data(), sizeof(int64_t) * (s.n + 1), hipMemcpyHostToDevice) != hipSuccess ||
      (hp.f.nnz > 0 && hipMemcpy(st->at<uint32_t>(lay.pcol), pcol.data(), sizeof(uint32_t) * hp.f.nnz, hipMemcpyHostToDevice) != hipSuccess) ||
      (hp.b.nnz > 0 && hipMemcpy(st->at<uint32_t>(lay.prow), prow.data(), sizeof(uint32_t) * hp.b.nnz, hipMemcpyHostToDevice) != hipSuccess))
    return bail(GNNSTAGE_EHIP, std::string("uploading the graph failed: ") + hipGetErrorString(hipGetLastError()));
  for (int dir = 0; dir < 2; ++dir) {  // dense plans
    const HostDir &h = dir ? hp.b : hp.f;
    if (!h.dense()) continue;
    const DensePlan &dp = h.dp;
    const size_t nb = (size_t)dp.n_blocks(), ne = dp.ent_pos.size(), ni = h.item_rb.size();  // ne: real entries, without padding
    std::vector<int32_t> item_rs(ni), item_chunk(ni);
    for (int c = 0; c < s.K; ++c)
      for (int64_t i = h.chunk_item_off[(size_t)c]; i < h.chunk_item_off[(size_t)c + 1]; ++i) {
        item_chunk[(size_t)i] = c;
        item_rs[(size_t)i] = (int32_t)(h.rowscale_off[(size_t)c] + (int64_t)h.item_rb[(size_t)i] * kDenseRB);
      }
    std::vector<uint32_t> colslot(dp.colslot_vertex.size());
    std::vector<int32_t> chunk_of((size_t)s.n);
    for (int c = 0; c < s.K; ++c)
      for (int64_t v = s.chunk_ptr[c]; v < s.chunk_ptr[c + 1]; ++v) chunk_of[(size_t)v] = c;
    for (size_t i = 0; i < colslot.size(); ++i) {
      const int32_t v = dp.colslot_vertex[i];
      colslot[i] = v < 0 ? 0xffffffffu : ((uint32_t)v | ((uint32_t)chunk_of[(size_t)v] << vbits));
    }
    if (hipMemcpy(st->at<int64_t>(lay.rem_ptr[dir]), dp.rem_ptr.data(), sizeof(int64_t) * (s.n + 1), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(st->at<int32_t>(lay.d_blk_cb[dir]), dp.blk_cb.data(), sizeof(int32_t) * nb, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(st->at<uint32_t>(lay.d_colslot[dir]), colslot.data(), sizeof(uint32_t) * colslot.size(), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(st->at<int32_t>(lay.d_item_rs[dir]), item_rs.data(), sizeof(int32_t) * ni, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(st->at<int32_t>(lay.d_item_chunk[dir]), item_chunk.data(), sizeof(int32_t) * ni, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(st->at<int64_t>(lay.d_item_b0[dir]), h.item_b0.data(), sizeof(int64_t) * ni, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(st->at<int32_t>(lay.d_item_nb[dir]), h.item_nb.data(), sizeof(int32_t) * ni, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(st->at<ChunkMask>(lay.d_item_chunks[dir]), h.item_chunks.data(), sizeof(ChunkMask) * ni, hipMemcpyHostToDevice) != hipSuccess)
      return bail(GNNSTAGE_EHIP, std::string("uploading the dense blocks failed: ") + hipGetErrorString(hipGetLastError()));
    if (rank1) {
      // patterns and the two scale vectors.  GCN normalisation: s_row = s_col = 1 / sqrt(row length in A + I).
      // Mean aggregator: 1 / |N(v)| belongs to the destination v, which is the row of a forward block and the
      // column of a block of the transposed index.
      auto row_len = [&](int64_t v) { return d->row_ptr[v + 1] - d->row_ptr[v]; };
      auto inv_sqrt = [&](int64_t v) { return (float)(1.0 / sqrt((double)row_len(v))); };
      auto inv_len = [&](int64_t v) { return row_len(v) > 0 ? 1.f / (float)row_len(v) : 0.f; };
      auto row_scale = [&](int64_t v) { return !s.sage() ? inv_sqrt(v) : dir == 0 ? inv_len(v) : 1.f; };
      auto col_scale = [&](int64_t v) { return !s.sage() ? inv_sqrt(v) : dir == 0 ? 1.f : inv_len(v); };
      std::vector<uint32_t> bits(nb * 256, 0u);
      for (size_t b = 0; b < nb; ++b)
        for (int64_t e = dp.blk_e0[b]; e < dp.blk_e0[b + 1]; ++e) {
          const uint32_t pos = dp.ent_pos[(size_t)e], r = pos >> 8, c = pos & 255u;
          bits[b * 256 + r * 2 + (c >> 5)] |= 1u << (c & 31u);
        }
      std::vector<float> colscale(colslot.size(), 0.f), rowscale((size_t)h.rowscale_off.back(), 0.f);
      for (size_t i = 0; i < colslot.size(); ++i)
        if (dp.colslot_vertex[i] >= 0) colscale[i] = col_scale(dp.colslot_vertex[i]);
      for (int k = 0; k < s.K; ++k)
        for (int64_t pp = 0; pp < s.chunk_ptr[k + 1] - s.chunk_ptr[k]; ++pp)
          rowscale[(size_t)(h.rowscale_off[(size_t)k] + pp)] = row_scale(dp.row_perm[(size_t)(s.chunk_ptr[k] + pp)]);
      if (hipMemcpy(st->at<uint32_t>(lay.d_bits[dir]), bits.data(), sizeof(uint32_t) * bits.size(), hipMemcpyHostToDevice) != hipSuccess ||
          hipMemcpy(st->at<float>(lay.d_colscale[dir]), colscale.data(), sizeof(float) * colscale.size(), hipMemcpyHostToDevice) != hipSuccess ||
          hipMemcpy(st->at<float>(lay.d_rowscale[dir]), rowscale.data(), sizeof(float) * rowscale.size(), hipMemcpyHostToDevice) != hipSuccess)
        return bail(GNNSTAGE_EHIP, "uploading the dense patterns failed");
    } else {
      const size_t ne_pad = (size_t)h.padded_entries();
      std::vector<uint32_t> ent_w(ne_pad, 0u);
      std::vector<uint16_t> ent_pos(ne_pad, (uint16_t)0xffff);
      std::vector<int64_t> blk_e0(nb + 1, 0);
      for (int k = 0; k < s.K; ++k)
        for (int64_t b = dp.chunk_blk_off[(size_t)k]; b < dp.chunk_blk_off[(size_t)k + 1]; ++b) {
          int64_t at = blk_e0[(size_t)b];
          for (int64_t e = dp.blk_e0[(size_t)b]; e < dp.blk_e0[(size_t)b + 1]; ++e, ++at) {
            const uint32_t pos = dp.ent_pos[(size_t)e];
            const int64_t e_csr = dir ? t_edge[(size_t)dp.ent_orig[(size_t)e]] : dp.ent_orig[(size_t)e];
            const float wgt = d->edge_val[e_csr];
            const uint16_t hi = bf16_bits_rne(wgt), lo = bf16_bits_rne(wgt - bf16_bits_to_f32(hi));
            ent_w[(size_t)at] = (uint32_t)hi | ((uint32_t)lo << 16);
            ent_pos[(size_t)at] = (uint16_t)pos;
          }
          blk_e0[(size_t)b + 1] = (at + 7) / 8 * 8;
        }
      if (hipMemcpy(st->at<int64_t>(lay.d_blk_e0[dir]), blk_e0.data(), sizeof(int64_t) * (nb + 1), hipMemcpyHostToDevice) != hipSuccess ||
          hipMemcpy(st->at<uint16_t>(lay.d_ent_pos[dir]), ent_pos.data(), sizeof(uint16_t) * ne_pad, hipMemcpyHostToDevice) != hipSuccess ||
          hipMemcpy(st->at<uint32_t>(lay.d_ent_w[dir]), ent_w.data(), sizeof(uint32_t) * ne_pad, hipMemcpyHostToDevice) != hipSuccess)
        return bail(GNNSTAGE_EHIP, "uploading the dense entries failed");
      if (launch_fill_zero(st->at<char>(lay.d_tiles[dir]), sizeof(uint16_t) * nb * 2 * kDenseRB * kDenseCB, nullptr) != 0 ||
          launch_dense_expand(st->at<int64_t>(lay.d_blk_e0[dir]), st->at<uint16_t>(lay.d_ent_pos[dir]),
                              st->at<uint32_t>(lay.d_ent_w[dir]), st->at<char>(lay.d_tiles[dir]), (int64_t)nb, nullptr) != 0)
        return bail(GNNSTAGE_EHIP, "expanding the dense blocks failed");
    }
    st->dense_rank1 = rank1;
    if (launch_fill_zero(st->at<char>(lay.zero_row), 512, nullptr) != 0) return bail(GNNSTAGE_EHIP, "clearing the zero row failed");
    st->dense_on[dir] = true;
    st->dense_entries[dir] = (int64_t)ne;
  }
  if (d->edge_val) {
    std::vector<float> fval, tval((size_t)hp.b.nnz);
    const float *fv = d->edge_val;
    // entry i of the index a direction's sparse kernels see -> its position in that direction's full index:
    // through the hotness order (if any), then through the dense plan's remainder (if any)
    auto full_pos = [](const HostDir &h, int64_t i) {
      if (h.hot.active) i = h.hot.orig[(size_t)i];
      return h.dense() ? h.dp.rem_orig[(size_t)i] : i;
    };
    if (hp.f.dense() || hp.f.hot.active) {
      fval.resize((size_t)hp.f.nnz);
      for (int64_t i = 0; i < hp.f.nnz; ++i) fval[(size_t)i] = d->edge_val[full_pos(hp.f, i)];
      fv = fval.data();
    }
    for (int64_t i = 0; i < hp.b.nnz; ++i) tval[(size_t)i] = d->edge_val[t_edge[(size_t)full_pos(hp.b, i)]];
    if ((hp.f.nnz > 0 && hipMemcpy(st->at<float>(lay.val), fv, sizeof(float) * hp.f.nnz, hipMemcpyHostToDevice) != hipSuccess) ||
        (hp.b.nnz > 0 && hipMemcpy(st->at<float>(lay.tval), tval.data(), sizeof(float) * hp.b.nnz, hipMemcpyHostToDevice) != hipSuccess))
      return bail(GNNSTAGE_EHIP, "uploading edge values failed");
  } else {
    // Section 2.1 weights from the row lengths of A + I, for the (remaining) CSR entries and for their transposed copies
    const int64_t *rp = st->at<int64_t>(lay.row_ptr);
    const int64_t *fp = hp.f.dense() ? st->at<int64_t>(lay.rem_ptr[0]) : rp;
    const int64_t *bp = hp.b.dense() ? st->at<int64_t>(lay.rem_ptr[1]) : st->at<int64_t>(lay.t_ptr);
    if (launch_gcn_norm(fp, st->at<uint32_t>(lay.pcol), vbits, rp, s.n, st->at<float>(lay.val), nullptr) != 0 ||
        launch_gcn_norm(bp, st->at<uint32_t>(lay.prow), vbits, rp, s.n, st->at<float>(lay.tval), nullptr) != 0)
      return bail(GNNSTAGE_EHIP, "normalisation kernel launch failed");
  }
  rc = build(hp.f, pcol.data(), 0);
  if (rc == GNNSTAGE_OK) rc = build(hp.b, prow.data(), 1);
  if (rc != GNNSTAGE_OK) return bail(rc, "building the launch schedule failed");
  if (hipDeviceSynchronize() != hipSuccess) return bail(GNNSTAGE_EHIP, "device synchronisation failed after create");
  *out = holder.release();
  return GNNSTAGE_OK;
}
GNNSTAGE_GUARD_INT

extern "C" int gnnstage_destroy(gnnstage_t *st) try {
  if (!st) return GNNSTAGE_EINVAL;
  const hipError_t e = hipDeviceSynchronize();
  st->prof.destroy();
  delete st;
  return e == hipSuccess ? GNNSTAGE_OK : GNNSTAGE_EHIP;
}
GNNSTAGE_GUARD_INT

extern "C" int stage_forward_chunk(gnnstage_t *st, int32_t k, int32_t pos, void *hip_stream) try {
  if (!st) return GNNSTAGE_EINVAL;
  const Shape &s = st->s;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (k < 0 || k >= s.K) return fail(st, GNNSTAGE_ERANGE, "chunk id out of range");
  if (pos == 0) {  // a new pass: V_processed <- empty
    const int rc = begin_forward(st, nullptr, stream);
    if (rc != GNNSTAGE_OK) return rc;
  }
  if (pos != (int32_t)st->order.size()) return fail(st, GNNSTAGE_EORDER, "pos_in_pass does not continue the current pass");
  if (mask_test(st->fmask, (uint32_t)k)) return fail(st, GNNSTAGE_EORDER, "chunk already processed in this pass");
  st->order.push_back(k);
  mask_set(st->fmask, k);  // C_k joins V_processed before its layers run
  if ((int)st->order.size() == s.K) st->cur_stale = false;  // after this call every current row is of this pass
  const Span sp = chunk_span(k, st->fmask);
  for (int j = 0; j < s.L && span_rows(st, sp) > 0; ++j) {
    const int rc = forward_layer(st, j, sp, stream);
    if (rc != GNNSTAGE_OK) return rc;
  }
  return GNNSTAGE_OK;
}
GNNSTAGE_GUARD_INT

extern "C" int gnnstage_forward_pass(gnnstage_t *st, const int32_t *order, int32_t n_order, void *hip_stream) try {
  if (!st || (n_order > 0 && !order)) return GNNSTAGE_EINVAL;
  if (!whole_pass_ok(st, order, n_order)) {
    for (int32_t p = 0; p < n_order; ++p) {
      const int rc = stage_forward_chunk(st, order[p], p, hip_stream);
      if (rc != GNNSTAGE_OK) return rc;
    }
    return GNNSTAGE_OK;
  }
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  std::vector<int32_t> ks(order, order + n_order);
  int rc = begin_forward(st, &ks, stream);
  if (rc != GNNSTAGE_OK) return rc;
  for (int j = 0; j < st->s.L && rc == GNNSTAGE_OK; ++j) rc = forward_layer(st, j, whole_span(st), stream);
  if (rc != GNNSTAGE_OK) return rc;
  // only now: a pass that failed half-way is none to run backward or to refresh the history from
  st->order.swap(ks);
  for (int32_t k : st->order) mask_set(st->fmask, k);
  st->cur_stale = false;
  return GNNSTAGE_OK;
}
GNNSTAGE_GUARD_INT

extern "C" int gnnstage_flush_weight_gradients(gnnstage_t *st, void *hip_stream) try {
  if (!st) return GNNSTAGE_EINVAL;
  return flush_deferred_wgrad(st, static_cast<hipStream_t>(hip_stream));
}
GNNSTAGE_GUARD_INT

extern "C" int stage_backward_chunk(gnnstage_t *st, int32_t k, const void *grad_out_rows, void *hip_stream) try {
  if (!st) return GNNSTAGE_EINVAL;
  const Shape &s = st->s;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (k < 0 || k >= s.K) return fail(st, GNNSTAGE_ERANGE, "chunk id out of range");
  if ((int)st->order.size() != s.K) return fail(st, GNNSTAGE_EORDER, "backward before the forward pass covered every chunk");
  if (st->n_bwd >= s.K) return fail(st, GNNSTAGE_EORDER, "backward pass already complete");
  if (st->order[s.K - 1 - st->n_bwd] != k) return fail(st, GNNSTAGE_EORDER, "backward must walk the chunks in reverse forward order");
  const int64_t row0 = s.chunk_ptr[(size_t)k], M = s.chunk_ptr[(size_t)k + 1] - row0;
  if (M > 0 && !grad_out_rows) return fail(st, GNNSTAGE_EINVAL, "grad_out_rows is NULL");
  st->n_bwd += 1;
  mask_set(st->bmask, k);
  // an empty chunk has no rows of its own, but the end-of-pass work still runs when it is the last call of the pass
  if (M > 0) {
    if (s.defer_wgrad()) st->wgrad_pending[(size_t)k] = 1;
    st->gi = 0;
    int rc = top_dY(st, grad_out_rows, row0, M, dY_rows(st, row0, s.L - 1), stream);
    LnSums sums;
    for (int j = s.L - 1; j >= 0 && rc == GNNSTAGE_OK; --j) rc = backward_layer(st, sums, j, chunk_span(k, st->bmask), stream);
    if (rc != GNNSTAGE_OK) return rc;
  }
  return end_backward(st, stream);
}
GNNSTAGE_GUARD_INT

extern "C" int gnnstage_backward_pass(gnnstage_t *st, const int32_t *order, int32_t n_order, const void *grad_out, void *hip_stream) try {
  if (!st || (n_order > 0 && !order)) return GNNSTAGE_EINVAL;
  const Shape &s = st->s;
  if (!grad_out || !whole_pass_ok(st, order, n_order) || st->n_bwd != 0 || (int)st->order.size() != s.K ||
      !std::equal(st->order.begin(), st->order.end(), order)) {
    for (int32_t p = n_order - 1; p >= 0; --p) {
      const int32_t k = order[p];
      if (k < 0 || k >= s.K) return fail(st, GNNSTAGE_ERANGE, "chunk id out of range");
      const char *rows = static_cast<const char *>(grad_out);
      const int rc = stage_backward_chunk(st, k, rows ? rows + (size_t)s.chunk_ptr[(size_t)k] * s.dims[s.L] * s.elt() : nullptr, hip_stream);
      if (rc != GNNSTAGE_OK) return rc;
    }
    return GNNSTAGE_OK;
  }
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  int rc = write_pass_tables(st, st->order, stream);
  if (rc != GNNSTAGE_OK) return rc;
  st->n_bwd = s.K;  // there is no second try, whatever fails below: part of the sums may be added by then
  for (int32_t k = 0; k < s.K; ++k) mask_set(st->bmask, k);
  LnSums sums;
  rc = top_dY(st, grad_out, 0, s.n, full_dY(st, s.L - 1), stream);
  for (int j = s.L - 1; j >= 0 && rc == GNNSTAGE_OK; --j) rc = backward_layer(st, sums, j, whole_span(st), stream);
  if (rc == GNNSTAGE_OK) rc = sums.add_up(st, stream);
  if (rc != GNNSTAGE_OK) return rc;
  for (int32_t k = 0; k < s.K; ++k) st->wgrad_pending[(size_t)k] = s.chunk_ptr[(size_t)k + 1] > s.chunk_ptr[(size_t)k] ? 1 : 0;
  return end_backward(st, stream);
}
GNNSTAGE_GUARD_INT

extern "C" int update_history(gnnstage_t *st, void *hip_stream) try {
  if (!st) return GNNSTAGE_EINVAL;
  const Shape &s = st->s;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  if (st->cur_stale)
    return fail(st, GNNSTAGE_EORDER, "the current levels hold stale rows until a complete pass follows gnnstage_update_history_swap");
  Timed t(st, stream, 5);
  std::vector<CopyArgs> c;
  for (int j = 0; j < s.L; ++j)
    if (st->hist[j] != st->cur[j]) c.push_back(CopyArgs{st->cur[j], st->hist[j], (size_t)s.n * s.dims[j] * st->level_elt(j)});
  // in one launch, unless a level's buffer is part of another's
  bool apart = true;
  for (size_t i = 0; i < c.size(); ++i)
    for (size_t k = 0; k < c.size(); ++k) {
      const char *dst = static_cast<const char *>(c[i].dst), *src = static_cast<const char *>(c[k].src), *other = static_cast<const char *>(c[k].dst);
      if (dst < src + c[k].bytes && src < dst + c[i].bytes) apart = false;
      if (i != k && dst < other + c[k].bytes && other < dst + c[i].bytes) apart = false;
    }
  if (apart) {
    HIP_TRY(st, launch_copies(c.data(), (int)c.size(), stream));
  } else {
    for (const CopyArgs &x : c) HIP_TRY(st, launch_copies(&x, 1, stream));
  }
  return GNNSTAGE_OK;
}
GNNSTAGE_GUARD_INT

extern "C" int gnnstage_update_history_swap(gnnstage_t *st, void *hip_stream) try {
  if (!st) return GNNSTAGE_EINVAL;
  const Shape &s = st->s;
  if ((int)st->order.size() != s.K || (st->n_bwd > 0 && st->n_bwd < s.K) || st->cur_stale)
    return fail(st, GNNSTAGE_EORDER, "the levels trade places only behind a complete pass");
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  Timed t(st, stream, 5);
  if (st->hist[0] != st->cur[0])  // level 0 is written by the caller: it keeps its buffers
    HIP_TRY(st, launch_copy(st->cur[0], st->hist[0], (size_t)s.n * s.dims[0] * st->level_elt(0), stream));
  for (int j = 1; j < s.L; ++j)
    if (st->hist[j] != st->cur[j]) {
      std::swap(st->hist[j], st->cur[j]);
      st->cur_stale = true;
    }
  return GNNSTAGE_OK;
}
GNNSTAGE_GUARD_INT

extern "C" int gnnstage_level_buffers(const gnnstage_t *st, int32_t level, void **cur, void **hist) {
  if (!st || level < 0 || level > st->s.L) return GNNSTAGE_EINVAL;
  if (cur) *cur = st->cur[(size_t)level];
  if (hist) *hist = level < st->s.L ? st->hist[(size_t)level] : nullptr;
  return GNNSTAGE_OK;
}

extern "C" int gnnstage_debug_select_counts(gnnstage_t *st, int32_t k, int32_t *out) try {
  if (!st || !out) return GNNSTAGE_EINVAL;
  const Shape &s = st->s;
  if (k < 0 || k >= s.K) return fail(st, GNNSTAGE_ERANGE, "chunk id out of range");
  ChunkMask m = st->fmask;
  mask_set(m, k);
  const uint32_t vb = (uint32_t)st->vbits;
  for (int64_t v = s.chunk_ptr[k]; v < s.chunk_ptr[k + 1]; ++v) {
    int32_t c = 0;
    for (int64_t e = st->h_row_ptr[v]; e < st->h_row_ptr[v + 1]; ++e) c += mask_test(m, st->h_pcol[(size_t)e] >> vb) ? 1 : 0;
    out[v - s.chunk_ptr[k]] = c;
  }
  return GNNSTAGE_OK;
}
GNNSTAGE_GUARD_INT

extern "C" int gnnstage_layer_order(const gnnstage_t *st, int32_t layer) {
  if (!st || layer < 0 || layer >= st->s.L) return GNNSTAGE_EINVAL;
  return st->s.tf[layer] ? 1 : 0;
}

extern "C" int gnnstage_set_dropout_rate(gnnstage_t *st, float dropout_p) {
  if (!st) return GNNSTAGE_EINVAL;
  if ((!st->order.empty() && (int)st->order.size() < st->s.K) || (st->n_bwd > 0 && st->n_bwd < st->s.K))
    return fail(st, GNNSTAGE_EORDER, "the dropout rate cannot change inside a forward or a backward pass");
  if (!(dropout_p >= 0.f && dropout_p < 1.f)) return fail(st, GNNSTAGE_EINVAL, "dropout_p must be in [0, 1)");
  if (dropout_p > 0.f && st->s.variant == GNNSTAGE_GCNII) return fail(st, GNNSTAGE_EINVAL, "no dropout in GCNII layers");
  st->next_dropout_p = dropout_p;  // latched by the next pass's first forward call
  return GNNSTAGE_OK;
}

extern "C" int gnnstage_set_dropout_seed(gnnstage_t *st, uint64_t seed) {
  if (!st) return GNNSTAGE_EINVAL;
  if ((!st->order.empty() && (int)st->order.size() < st->s.K) || (st->n_bwd > 0 && st->n_bwd < st->s.K))
    return fail(st, GNNSTAGE_EORDER, "the dropout seed cannot change inside a forward or a backward pass");
  st->next_dropout_seed = seed;  // latched by the next pass's first forward call
  return GNNSTAGE_OK;
}

extern "C" int64_t gnnstage_query(const gnnstage_t *st, int32_t what, int32_t index) {
  if (!st) return GNNSTAGE_EINVAL;
  const Shape &s = st->s;
  switch (what) {
    case GNNSTAGE_Q_VERTICES: return s.n;
    case GNNSTAGE_Q_CHUNKS: return s.K;
    case GNNSTAGE_Q_LAYERS: return s.L;
    case GNNSTAGE_Q_DTYPE: return s.dtype;
    case GNNSTAGE_Q_LEVEL0_F32: return s.level0_f32;
    case GNNSTAGE_Q_VARIANT: return s.variant;
    case GNNSTAGE_Q_NEED_INPUT_GRAD: return s.need_input_grad;
    case GNNSTAGE_Q_WIDTH: return (index >= 0 && index <= s.L) ? s.dims[(size_t)index] : GNNSTAGE_EINVAL;
    case GNNSTAGE_Q_CHUNK_PTR: return (index >= 0 && index <= s.K) ? s.chunk_ptr[(size_t)index] : GNNSTAGE_EINVAL;
    default: return GNNSTAGE_EINVAL;
  }
}

extern "C" void *gnnstage_buffer(const gnnstage_t *st, int32_t which, int32_t index) {
  if (!st) return nullptr;
  switch (which) {
    case GNNSTAGE_B_CUR: return (index >= 0 && index <= st->s.L) ? st->cur[(size_t)index] : nullptr;
    case GNNSTAGE_B_HIST: return (index >= 0 && index < st->s.L) ? st->hist[(size_t)index] : nullptr;
    case GNNSTAGE_B_GRAD_IN: return st->s.need_input_grad ? st->grad_in : nullptr;
    default: return nullptr;
  }
}

extern "C" int gnnstage_profile_enable(gnnstage_t *st, int32_t on) {
  if (!st) return GNNSTAGE_EINVAL;
  st->prof.kinds = on != 0 ? (1u << GNNSTAGE_NKINDS) - 1u : 0u;
  return GNNSTAGE_OK;
}

extern "C" int gnnstage_profile_select(gnnstage_t *st, uint32_t kind_mask) {
  if (!st || (kind_mask >> GNNSTAGE_NKINDS) != 0) return GNNSTAGE_EINVAL;
  st->prof.kinds = kind_mask;
  return GNNSTAGE_OK;
}

extern "C" int gnnstage_profile_read(gnnstage_t *st, int32_t kind, int32_t layer, double *ms, int64_t *launches) try {
  if (!st || kind < 0 || kind >= GNNSTAGE_NKINDS || layer >= st->s.L) return GNNSTAGE_EINVAL;
  if (hipDeviceSynchronize() != hipSuccess) return fail(st, GNNSTAGE_EHIP, "device synchronisation failed");
  st->prof.collect();
  double t = 0;
  int64_t n = 0;
  const int L1 = st->s.L + 1;
  for (int j = 0; j < L1; ++j) {
    if (layer >= 0 && j != layer) continue;
    t += st->prof.ms[(size_t)kind * L1 + j];
    n += st->prof.launches[(size_t)kind * L1 + j];
  }
  if (ms) *ms = t;
  if (launches) *launches = n;
  return GNNSTAGE_OK;
}
GNNSTAGE_GUARD_INT

extern "C" int gnnstage_profile_reset(gnnstage_t *st) try {
  if (!st) return GNNSTAGE_EINVAL;
  if (hipDeviceSynchronize() != hipSuccess) return fail(st, GNNSTAGE_EHIP, "device synchronisation failed");
  st->prof.collect();
  st->prof.init(st->s.L);
  return GNNSTAGE_OK;
}
GNNSTAGE_GUARD_INT
