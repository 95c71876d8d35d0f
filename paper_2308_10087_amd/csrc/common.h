// Shared declarations of the gnnstage HIP library (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

typedef __bf16 bf16_t;

// Which chunks count as processed (Section 3.3, V_processed), one bit per chunk id.
// Passed by value as a kernel argument; supports up to 256 chunks.
struct ChunkMask {
  uint64_t w[4];
};
constexpr int kMaxChunks = 256;
constexpr int kMaxClasses = 32;  // source-id classes of the aggregation schedule (a 32-bit activity mask)

// Workgroups of 256 along an axis of a grid: the runtime takes fewer than 2^32 work-items there.
constexpr int64_t kMostBlocks = ((int64_t)1 << 24) - 1;
// Kernels with a thread per element (or vector of elements) of a matrix: launch(first row, rows, workgroups) for as many rows at a time as a
// grid has threads.
template <typename F>
static inline int for_row_slabs(int64_t M, int64_t threads_per_row, F launch) {
  const int64_t most = kMostBlocks * 256 / threads_per_row;
  for (int64_t r = 0; r < M; r += most) {
    const int64_t m = M - r < most ? M - r : most;
    launch(r, m, (unsigned)((m * threads_per_row + 255) / 256));
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  return hipSuccess;
}

// The word is picked with selects, not with an indexed access: a kernel that holds the mask as an argument
// would otherwise fetch the word from memory and wait for it (and for every other load in flight).
__host__ __device__ inline bool mask_test(const ChunkMask &m, uint32_t c) {
  const uint64_t lo = (c & 64u) ? m.w[1] : m.w[0], hi = (c & 64u) ? m.w[3] : m.w[2];
  return (((c & 128u) ? hi : lo) >> (c & 63u)) & 1ull;
}

// ---- aggregation (SpMM with current/history select) ---------------------------------
// The same for a mask that a whole wave holds, all of whose lanes ask at once.  Up to 64 chunks (many false, uniform) it is one
// shift of the first word; above that lane i holds the mask's 32-bit word i and answers for it.  Selects among four words
// instead cost an aggregation kernel eight registers, which it does not have to spare (62 against 54).
struct WaveMask {
  uint64_t first;
  uint32_t word;
};
__device__ inline WaveMask wave_mask(const ChunkMask &m, bool many) {
  WaveMask w{m.w[0], 0u};
  if (many) {
#pragma unroll
    for (int i = 0; i < 8; ++i) w.word = (threadIdx.x & 63) == i ? (uint32_t)(m.w[i >> 1] >> (32 * (i & 1))) : w.word;
  }
  return w;
}
__device__ inline bool mask_test(const WaveMask &m, uint32_t c, bool many) {
  if (many) return (((uint32_t)__builtin_amdgcn_ds_bpermute((int)(c >> 5) << 2, (int)m.word) >> (c & 31u)) & 1u) != 0;
  return ((m.first >> (c & 63u)) & 1ull) != 0;
}

enum SpmmEpilogue : int {
  SPMM_PLAIN = 0,     // out = acc
  SPMM_MIX = 1,       // out = s_acc * acc + s_aux * aux[row]      (GCNII initial residual)
  SPMM_MASK = 2,      // out = aux[row] > 0 ? acc : 0              (ReLU derivative on the way back)
  SPMM_BIAS_RELU = 3, // out = max(acc + bias[c], 0)               (transform-first layers)
  SPMM_ADD = 4,       // out = acc + add[row - add_row0]           (GraphSage: the gradient through W_self joins)
  SPMM_ADD_MASK = 5   // out = aux[row] > 0 ? acc + add[row - add_row0] : 0
};
__host__ __device__ inline bool spmm_reads_aux(int e) { return e == SPMM_MIX || e == SPMM_MASK || e == SPMM_ADD_MASK; }
__host__ __device__ inline bool spmm_reads_add(int e) { return e == SPMM_ADD || e == SPMM_ADD_MASK; }

// Dropout behind an activation: threshold = ceil(rate * 2^24) (0: none), scale = 1 / (1 - rate), key = the
// layer's key of this pass, u0 = vertex id of the launch's first row.  Feature c of vertex u (rows of d features)
// survives when the top 24 bits of SplitMix64(key + (u * d + c + 1) * golden) reach the threshold.
struct LnDropout {
  uint32_t threshold;
  float scale;
  uint64_t key;
  int64_t u0;
};
__host__ __device__ inline uint64_t splitmix64_dev(uint64_t z) {
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}
__host__ __device__ inline bool dropout_keep(const LnDropout &dp, int64_t u, int d, int c) {
  const uint64_t r = splitmix64_dev(dp.key + (uint64_t)(u * d + c + 1) * 0x9E3779B97F4A7C15ull);
  return (uint32_t)(r >> 40) >= dp.threshold;
}

// What a row chunk selects in a launch over many chunks: the source chunks it reads as processed, and the source classes
// from which it gathers anything (launches that drop unselected entries).  One entry per row chunk, written by
// launch_stage_weights; 64 bytes, read through the scalar cache.
struct PassChunk {
  ChunkMask mask;
  uint32_t classes;
  uint32_t pad[7];
};
static_assert(sizeof(PassChunk) == 64, "one scalar load of sixteen words");

// One scalar load.  (Three arrays indexed by the XCD, one of them of bytes, are not: the compiler takes the index of one as
// the base of the next, and the scalar unit drops the low bits of such an address.)
struct alignas(16) XcdRun {
  int32_t cls, group0, groups, unused;
};

enum ShortRows : int32_t { SHORT_ROWS_MFMA, SHORT_ROWS_VALU, SHORT_ROWS_SINGLE };  // VALU: fp32 weights on the vector ALU

struct SpmmArgs {
  // sparse structure: packed index words (vertex | chunk << vbits) and weights
  const uint32_t *pidx;
  const float *val;
  // launch schedule
  const int32_t *task_row;   // -1: a filler behind a chunk's short rows
  const int64_t *task_e0;
  const uint32_t *task_ne;   // entries | row chunk << kTaskChunkShift
  const int32_t *task_slot;  // partial row, counted over all chunks; -1: the task finishes its row
  // XCD-aware serving order.  Class c's pieces are tasks [cls_begin[c], cls_end[c]).  Workgroups are dealt round-robin to the
  // 8 XCDs; the groups of four tasks of the active classes, one class after the other, are cut into eight runs, and XCD x
  // (workgroups with index % 8 == x) serves xcd[x].groups of them from group xcd[x].group0 of class xcd[x].cls on.
  // Workgroups from n_class_blocks on serve the tail, tasks [tail0, tail0 + n_tail), and the short rows.
  int32_t cls_begin[kMaxClasses], cls_end[kMaxClasses];
  XcdRun xcd[8];
  int32_t n_class_blocks;
  int64_t tail0, n_tail;
  // Whole rows of at most a few entries (no partial slot), every chunk's filled up to a multiple of four.  Where there are many of
  // them the matrix-core kernel gives them to extra workgroups of the same launch whose waves serve four rows each: a wave per
  // row would spend its life waiting for three dependent round trips to move a kilobyte or two.  Few of them (SHORT_ROWS_SINGLE), the
  // vector-ALU kernel and rows wider than 256 columns: a row to a wave like any other task.
  int64_t short0, n_short;
  // The two lists' workgroups are dealt out evenly, so that the launch goes through both in about the order of their rows:
  // workgroup p behind the class pieces serves short rows if p mix crosses a whole number of 2^32 (set by the launcher).
  // First all of the one and then of the other is slower where the gathers bound the launch: 3.6 M entries of 512-byte rows
  // 192 against 177 us.
  uint64_t mix;
  int32_t short_rows;     // ShortRows
  const uint8_t *slot_class;  // class of every partial slot (255: none); pieces of inactive classes are not run
  uint32_t active_classes;
  int32_t all_classes_active;
  // long rows: pieces summed by the reduce kernel
  const int32_t *lr_row;
  const int32_t *lr_slot0;
  const uint32_t *lr_nslots;  // pieces | row chunk << kTaskChunkShift
  int64_t n_long;
  float *partial;   // [n_slots][d] fp32, first row: slot slot0
  int64_t slot0;
  // dense-block partial sums of a cut row: rows lr_dense0[i] + 128 * g (g < lr_ndense[i]), counted over all chunks, of
  // dense_partial, one per item of the row's row block; lr_item0[i] is the first of those items (for the activity test)
  const int32_t *lr_dense0;
  const int32_t *lr_ndense;
  const int32_t *lr_item0;
  const ChunkMask *item_chunks;
  const float *dense_partial;  // first row: item item0
  int64_t item0;
  int32_t drop_unselected;  // the launch skips unselected entries: items without a chunk in the mask were not run
  // gathered operand: rows of width d, leading dimension src_ld
  const void *src_sel;    // read when the neighbour's chunk is in the mask
  const void *src_unsel;  // read otherwise; nullptr => the entry contributes zero
  int32_t d;
  int32_t src_ld;
  int32_t vbits;
  int32_t many_chunks;    // more than 64
  const PassChunk *pass;  // masks by row chunk; nullptr: mask for all rows
  ChunkMask mask;
  // output rows: out[(row - out_row0) * out_ld + c], c < d; columns [d, out_ld) get zeros
  void *out;
  int32_t out_ld;
  int64_t out_row0;
  // epilogue
  int32_t epilogue;
  const void *aux;  // indexed by absolute row, leading dimension aux_ld, same dtype as src
  int32_t aux_ld;
  float s_acc, s_aux;
  const float *bias;  // SPMM_BIAS_RELU
  const void *add;    // SPMM_ADD / SPMM_ADD_MASK: rows indexed by row - add_row0, same dtype as src; may be the output rows
  int32_t add_ld;     // themselves where d is a multiple of 8 (no column then belongs to two lanes)
  int64_t add_row0;
  float mask_scale = 1.f;  // SPMM_MASK / SPMM_ADD_MASK: what passes the mask is scaled (1 / (1 - rate) of that dropout)
  // kernel choice (measurement and test switches, set by the stage from what it read at create)
  int32_t force_valu = 0;  // vector-ALU aggregation for bf16 rows too
  int32_t long_pieces = 0; // rows are cut into pieces of 256 entries or more (forward aggregations of fp32 stages)
  int32_t unroll = 2;      // gather slots per wave of the matrix-core aggregation: 2, 4 or 8
};
constexpr int kShortRowMost = 16;    // entries of a short row: one per lane of its group
constexpr int kTaskChunkShift = 24;  // a piece or an uncut row has fewer than 2^24 entries
constexpr uint32_t kTaskCountMask = (1u << kTaskChunkShift) - 1u;
static_assert(kMaxChunks <= 256, "the chunk shares a word with a count");
static_assert(sizeof(SpmmArgs) <= 4096, "kernel arguments");
// The most workgroups that a launch of these operands, or of the reduce behind it, has along an axis: what a launch over several
// chunks must keep to kMostBlocks (67 M whole rows, or 16.7 M cut ones).
static inline int64_t spmm_blocks(const SpmmArgs &a) {
  const int64_t main = a.n_class_blocks + (a.n_tail + 3) / 4 + a.n_short / 4 + 7;  // + 7: rounded up to eight for wide rows
  return main > a.n_long ? main : a.n_long;
}

// What every wave needs of the operands to find its task and its mask, in one round trip: the compiler moves each of these loads behind
// the branch that needs it, five round trips in a row in front of the task's (a launch over 1,078 fp32 rows of width 100 7.2 us, 6.7 so;
// over 19 bf16 rows of width 256 5.5 and 5.2).
struct SpmmHead {
  uint64_t mix;
  int64_t tail0, n_tail, short0, n_short;
  uint64_t mask0;
  const PassChunk *pass;
  int32_t n_class_blocks, short_rows;
};
__device__ inline SpmmHead spmm_head(const SpmmArgs &a) {
  SpmmHead h{a.mix, a.tail0, a.n_tail, a.short0, a.n_short, a.mask.w[0], a.pass, a.n_class_blocks, a.short_rows};
  asm volatile("" : "+s"(h.mix), "+s"(h.tail0), "+s"(h.n_tail), "+s"(h.short0), "+s"(h.n_short), "+s"(h.mask0), "+s"(h.pass), "+s"(h.n_class_blocks), "+s"(h.short_rows));
  return h;
}
// workgroup b behind the class pieces: whether it serves short rows, and how many of its kind come before it
struct SpmmTurn {
  bool is_short;
  uint32_t index;
};
__device__ inline SpmmTurn spmm_turn(const SpmmHead &h, unsigned b) {
  const uint64_t p = b - (unsigned)h.n_class_blocks;
  const uint32_t before = (uint32_t)(p * h.mix >> 32), upto = (uint32_t)((p + 1) * h.mix >> 32);
  return SpmmTurn{upto > before, upto > before ? before : (uint32_t)p - before};
}
// which task the wave `wave` of workgroup `b` runs (-1: none); cls: its class (-1: none)
__device__ inline int64_t spmm_task_index(const SpmmArgs &a, const SpmmHead &h, unsigned b, int wave, int &cls) {
  cls = -1;
  if (b < (unsigned)h.n_class_blocks) {
    const XcdRun run = a.xcd[b & 7];
    int g = (int)(b >> 3);
    if (g >= run.groups) return -1;
    g += run.group0;
    for (int q = run.cls; q < kMaxClasses; ++q) {  // the runs cover exactly the active classes' groups
      const int t0 = a.cls_begin[q], nt = a.cls_end[q] - t0, ng = ((a.active_classes >> q) & 1u) ? (nt + 3) >> 2 : 0;
      if (g < ng) {
        const int t = g * 4 + wave;
        cls = q;
        return t < nt ? t0 + t : -1;
      }
      g -= ng;
    }
    return -1;
  }
  const SpmmTurn w = spmm_turn(h, b);
  const int64_t t = (int64_t)w.index * 4 + wave;
  return w.is_short ? (t < h.n_short ? h.short0 + t : -1) : t < h.n_tail ? h.tail0 + t : -1;
}
// The mask of a row chunk; chunk is the same for the whole wave.  The table is read through the scalar cache: by the time
// a wave has its index words it has its mask.
__device__ inline ChunkMask spmm_row_mask(const PassChunk *pass, const ChunkMask &mask, uint32_t chunk, uint32_t &classes) {
  classes = 0xffffffffu;
  if (pass == nullptr) return mask;
  typedef __attribute__((address_space(4))) const PassChunk const_chunk;
  const const_chunk *p = (const const_chunk *)(uintptr_t)(pass + chunk);
  ChunkMask m;
#pragma unroll
  for (int i = 0; i < 4; ++i) m.w[i] = p->mask.w[i];
  classes = p->classes;
  return m;
}
__device__ inline ChunkMask spmm_row_mask(const SpmmArgs &a, const SpmmHead &h, uint32_t chunk, uint32_t &classes) {
  ChunkMask m = a.mask;
  m.w[0] = h.mask0;
  return spmm_row_mask(h.pass, m, chunk, classes);
}

// ---- several launches in one -------------------------------------------------------------------
// Launches of one kernel that do not depend on each other run as one, operand sets side by side: sub-launch z is the grid's
// plane z, so that a workgroup's operands are one load away.  Planes are as wide as the widest sub-launch; workgroups past the
// end of theirs return.
constexpr int kBatch = 8;  // the kernel arguments stay below 4 KB
template <typename A>
struct Batch {
  A sub[kBatch];
};

// ---- dense blocks of an aggregation (bf16 rows of width 128 or 256) ---------------------------
// After ordering rows and columns by degree, the blocks that hold many entries are multiplied as dense
// 128 x 64 tiles on the matrix cores; the sparse kernels above only see the remaining entries.  An item
// is a run of blocks of one row block; it leaves a 128 x d fp32 tile of partial sums that the reduce
// kernel adds to the rows' sparse pieces.
constexpr int kDenseRB = 128, kDenseCB = 64;
constexpr int kDenseMaxItemBlocks = 32;  // blocks one workgroup multiplies before it writes its partial tile
struct DenseArgs {
  const int32_t *item_rs;         // first row-scale slot of every item of this launch
  const int32_t *item_chunk;      // its row chunk
  const int64_t *item_b0;         // its first block
  const int32_t *item_nb;         // and how many
  const ChunkMask *item_chunks;   // chunks its blocks' columns come from
  int32_t n_items;
  const int32_t *blk_cb;          // column block of every block: column slots 64 * cb ...
  const bf16_t *tiles;            // per block two 128 x 64 weight tiles (nearest bf16, then the remainder's bf16) as
                                  // launch_dense_expand writes them: [32-row group][16-column step][lane][8 values]
  // weights of the form s(row) * s(column) instead (bits != nullptr): per block 256 words of pattern bits
  // (word t: row t / 2, columns 32 * (t % 2) ..), s per column slot (0 = padding) and per row position of the chunk
  const uint32_t *bits;
  const float *colscale;
  const float *rowscale;          // 128 slots per row block, zero past a chunk's last row
  const void *zero_row;           // at least 512 bytes of zeros, 16-byte aligned
  const uint32_t *colslot;        // vertex | chunk << vbits of every column slot, 0xffffffff = padding
  const void *src_sel;            // rows of vertices whose chunk is in the mask
  const void *src_unsel;          // rows of the others; nullptr => they contribute zero
  int32_t d, src_ld, vbits;
  const PassChunk *pass;          // as in SpmmArgs
  ChunkMask mask;
  float *partial;                 // [n_items][128][d]
};
int launch_spmm_dense(const DenseArgs &a, hipStream_t s);
// Writes the weight tiles of n_blocks blocks (cleared by the caller) from their entry lists: entries
// [blk_e0[b], blk_e0[b + 1]) of block b, position = row << 8 | column (0xffff = padding), weight as two bf16
// halves (nearest bf16 in the low half of the word, the remainder's bf16 in the high half).
int launch_dense_expand(const int64_t *blk_e0, const uint16_t *ent_pos, const uint32_t *ent_w, void *tiles, int64_t n_blocks,
                        hipStream_t s);

enum DType : int { DT_F32 = 0, DT_BF16 = 1 };

// src dtype -> out dtype; returns hipError_t as int.  launch_spmm runs the per-task kernel,
// launch_spmm_reduce adds the pieces of long rows (needed whenever a.n_long > 0).
int launch_spmm(const SpmmArgs &a, int src_dtype, int out_dtype, hipStream_t s);
int launch_spmm_reduce(const SpmmArgs &a, int src_dtype, int out_dtype, hipStream_t s);

// The tables of a pass whose chunks run side by side, from the chunks' places in the forward order (pos[chunk]).  Row chunk c
// selects: forward, the chunks up to its own; backward, those from its own on (their backward work comes first); earlier,
// those in front of it (the readers that saw the historical rows of c).  classes_*: see PassChunk, for the last two.
struct PassTableArgs {
  PassChunk *forward, *backward, *earlier;  // [K] each
  int32_t K;
  uint8_t pos[kMaxChunks];
  uint32_t classes_backward[kMaxChunks], classes_earlier[kMaxChunks];
};
static_assert(sizeof(PassTableArgs) <= 3072, "kernel arguments");

// ---- dense transforms -------------------------------------------------------------------
enum GemmEpilogue : int {
  EPI_FWD_GCN = 0,     // out = ReLU(acc + bias[n])
  EPI_FWD_GCNII = 1,   // out = ReLU((1-beta) aux[m][n] + beta acc)
  EPI_PLAIN = 2,       // out = acc
  EPI_DGRAD_GCNII = 3, // dp = (1-beta) aux[m][n] + beta acc; out = (1-alpha) dp; h0grad[m][n] += alpha dp
  EPI_MASK = 4,        // out = aux[m][n] > 0 ? acc : 0
  EPI_FWD_ADD = 5,     // out = ReLU(acc + bias[n] + aux[m][n])   (GraphSage: aux = h_v W_self)
  EPI_RES = 6          // out = acc + bias[n] + aux[m][n]         (ResGCN+: aux = h_v, no activation)
};

// C[M x N] = A[M x K] . Bt[N x Kp]^T.  Bt is an internal buffer: K-contiguous rows, zero padded to Kp,
// Kp % 8 == 0, compute dtype.  A is either such a padded buffer too, or any row-major matrix of fp32 or
// bf16 elements with K valid columns (read with bounds checks).
struct GemmNtArgs {
  const void *A;
  int32_t a_dtype;
  int32_t lda;
  const void *Bt;
  int32_t ldb;
  int32_t M, N, K, Kp;
  int32_t epilogue;
  const float *bias;
  const void *aux;
  int32_t aux_dtype;
  int32_t aux_ld;
  float alpha, beta;
  float *h0grad;  // fp32, pre-offset to the first row
  int32_t h0_ld;
  void *out;
  int32_t out_dtype;
  int32_t out_ld;
  int32_t out_pad;  // columns [N, out_pad) of every output row are written as zeros (0: none)
  int32_t vec_epi;  // set by the launcher: the epilogue may use 16-byte accesses
  float mask_scale = 1.f;  // EPI_MASK: what passes the mask is scaled (1 / (1 - rate) of that dropout)
  LnDropout drop{};        // EPI_FWD_GCN / EPI_FWD_ADD: dropout of the layer's output (threshold 0: none)
  int32_t ws_min_rows = 65536;  // rows from which the weight-stationary kernel is used (tests force it on small inputs)
};
int launch_gemm_nt(const GemmNtArgs &a, int compute_dtype, hipStream_t s);

// dW[I x O] += scale * A[M x I]^T . B[M x O]   (reduction over the M rows of the chunk).
// B is an internal padded buffer in the compute dtype; A as for the NT product.
struct GemmTnArgs {
  const void *A;
  int32_t a_dtype;
  int32_t lda;
  const void *B;
  int32_t ldb;
  int32_t M, I, O;
  float scale;
  float *dW;       // fp32 [I][O]
  float *partial;  // fp32 scratch [splits][I][O]
  int32_t max_splits;
  float *dbias;         // optional: dbias[o] += column sums of B, fused into the product
  float *bias_partial;  // fp32 scratch [splits][O]
  int32_t wide_min_rows = 65536;  // bf16 operands from this many rows on, with more than one 128 x 128 output tile: one
                                  // workgroup per row split computes the whole output (tests force it on small inputs)
};
int launch_gemm_tn(const GemmTnArgs &a, int compute_dtype, hipStream_t s);
// n of them that have the same scratch (partial: partial_floats, bias_partial: bias_floats), as many at a time as it holds and
// as add to different buffers
int launch_gemm_tn_list(const GemmTnArgs *a, int n, size_t partial_floats, size_t bias_floats, int compute_dtype, hipStream_t s);
// dst[o] += sum over the M rows of B[.][o]; partial: fp32 scratch [max_splits][O]
int launch_colsum_add(const void *B, int dtype, int ldb, int M, int O, float *partial, int max_splits, float *dst,
                      hipStream_t s);

// ---- LayerNorm + ReLU in front of the aggregation (ResGCN+ variant) -------------------------------
constexpr int kLnMaxWidth = 1024;  // a row lives in the registers of one wavefront
constexpr int kLnMaxWaves = 8192;  // wavefronts of one backward launch; the parameter-gradient scratch holds one
                                   // 2 x d block of sums per workgroup of four
// out[r][c] = Dropout(ReLU(gamma[c] * (x[r][c] - mean_r) / sqrt(var_r + eps) + beta[c])), c < d; zeros up to out_ld
struct LnArgs {
  const void *x;
  int32_t x_dtype, x_ld;
  const float *gamma, *beta;
  float eps;
  int64_t M;
  int32_t d;
  void *out;
  int32_t out_dtype, out_ld;
  LnDropout drop;
};
// Backward of the same for M rows (the fields above: out, which may be NULL, receives the gradient of x): dr is the gradient of
// the activated rows, res (or NULL) rows that are added to out (the residual branch); dgamma / dbeta get "+=" of the column
// sums in a fixed order (partial: fp32 scratch, kLnMaxWaves / 4 * 2 * d).  Rows [gap_row, gap_end) take no part and are not read;
// the first row does.
struct LnBackArgs {
  LnArgs f;
  const void *dr;
  int32_t dr_dtype, dr_ld;
  const void *res;
  int32_t res_dtype, res_ld;
  float *partial;
  float *dgamma, *dbeta;
  int64_t gap_row, gap_end;
  int32_t blocks;  // set by the launcher
};
static_assert(sizeof(Batch<LnBackArgs>) <= 4096, "kernel arguments");
// What a backward launch leaves to add up: n_parts blocks of [gamma sums | beta sums] that go to dgamma and dbeta.
struct LnReduceArgs {
  const float *partial;
  int32_t n_parts, d;
  float *dgamma, *dbeta;
};
int launch_ln_relu(const LnArgs &a, hipStream_t s);
// n <= kBatch of them, with scratch of their own, of at most max_waves wavefronts each; red[i]: what is left to add up
int launch_ln_relu_backward(const LnBackArgs *a, int n, int max_waves, LnReduceArgs *red, hipStream_t s);
int launch_ln_param_reduce(const LnReduceArgs *red, int n, hipStream_t s);
// dst[r][c] = src[r][c] for c < d, zero for d <= c < dst_ld
int launch_copy_rows(const void *src, int src_ld, void *dst, int dst_ld, int64_t M, int d, int dtype, hipStream_t s);

// ---- small kernels ------------------------------------------------------------------------
// Wt[N][Kp] (transposed) and Wn[K][Np] (plain) zero-padded copies of W[K][N] in the compute dtype
struct StageWeightsArgs {
  const void *W;
  int32_t K, N;
  void *Wt;
  int32_t Kp;
  void *Wn;
  int32_t Np;
};
// n weights in launches of up to kBatch; tables (or NULL): written by a workgroup of the first one
int launch_stage_weights(const StageWeightsArgs *w, int n, int dtype, const PassTableArgs *tables, hipStream_t s);
// x[r][c] <- survives ? x[r][c] * scale : 0 in place, r < M, c < d (rows of leading dimension ld; dp.u0 = vertex of row 0)
int launch_dropout_rows(void *x, int dtype, int64_t M, int d, int ld, const LnDropout &dp, hipStream_t s);
// out[m][c] = level[m][c] > 0 ? g[m][c] * scale : 0 for c < d, zeros up to out_ld (the ReLU derivative on the way back; scale = 1 / (1 - rate) of a dropout behind it)
int launch_relu_mask(const void *g, const void *level, int dtype, int64_t M, int d, void *out, int out_ld, float scale,
                     hipStream_t s);
int launch_copy(const void *src, void *dst, size_t bytes, hipStream_t s);
struct CopyArgs {
  const void *src;
  void *dst;
  size_t bytes;
};
int launch_copies(const CopyArgs *c, int n, hipStream_t s);  // that do not overlap, in launches of up to kBatch
int launch_fill_zero(void *dst, size_t bytes, hipStream_t s);
struct FillArgs {
  void *dst;
  size_t bytes;
};
int launch_fills_zero(const FillArgs *f, int n, hipStream_t s);  // planes of launches of up to kFills
constexpr int kFills = 32;
// symmetric normalisation weights from row lengths: val[e] = 1/sqrt(len(row) * len(other))
int launch_gcn_norm(const int64_t *ptr, const uint32_t *pidx, int vbits, const int64_t *len_ptr, int64_t n,
                    float *val, hipStream_t s);

static inline int round_up(int x, int m) { return (x + m - 1) / m * m; }
