// Neighbour aggregation with the current-vs-history select fused into the gather
// (Algorithm 1, the AGGREGATE line; Section 3.3), and its transposed twin for the
// backward pass where unselected entries contribute zero (Section 3.4, technique 3).
//
// One wavefront per task.  A task is a whole sparse row, or a piece of a long row (power-law
// hubs are cut so that no wave owns more than a fixed number of entries; the pieces write
// fp32 partial sums that a second small kernel adds in a fixed order, so results do not
// depend on scheduling).  Two kernels share that schedule:
//  * spmm_kernel, the vector-ALU form for fp32 rows and odd widths: the 64 lanes form G = 64/LPR
//    groups of LPR lanes, each group gathers one neighbour row per step with 16/8/4-byte loads;
//    entry metadata (packed index, weight) is loaded 64 entries at a time, one per lane, and
//    broadcast through lane permutes; dropped entries are first compacted inside the wave.
//  * spmm_ring_kernel, for bf16 rows whose width is a multiple of 8: entries become address
//    records in a wave-private LDS ring and the weighted sum runs on the matrix cores.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace {

// V consecutive elements of a row.  Rows are only known to be 4-byte aligned (a width of 100 bf16 columns, say); a global
// access of 4, 8 or 16 bytes needs no more than that.  (bf16 columns from an odd one on are not even that: store_cols.)
template <typename T, int V>
struct alignas(sizeof(T) * V < 4 ? sizeof(T) * V : 4) Pack {
  T v[V];
};

__device__ inline float to_f32(float x) { return x; }
__device__ inline float to_f32(bf16_t x) { return (float)x; }
template <typename T>
__device__ inline T from_f32(float x);
template <>
__device__ inline float from_f32<float>(float x) { return x; }
template <>
__device__ inline bf16_t from_f32<bf16_t>(float x) { return (bf16_t)x; }

// The row of the auxiliary matrix that the mixing and masking epilogues read (zeros for the others).
template <typename Tin, int VEC>
__device__ inline Pack<Tin, VEC> load_aux(const SpmmArgs &a, int64_t row, int c) {
  if (spmm_reads_aux(a.epilogue))
    return *reinterpret_cast<const Pack<Tin, VEC> *>(static_cast<const Tin *>(a.aux) + (size_t)row * a.aux_ld + c);
  Pack<Tin, VEC> z;
#pragma unroll
  for (int t = 0; t < VEC; ++t) z.v[t] = from_f32<Tin>(0.f);
  return z;
}

// Stores columns c .. c + VEC - 1 of an output row.  fp32 rows of odd width that are aggregated into bf16 rows (raw features)
// end in a vector that starts at an odd column, two bytes off the 4-byte grid: that one goes element by element.  Rows of
// bf16 sources have even widths and even first columns throughout.
template <typename Tin, typename Tout, int VEC>
__device__ inline void store_cols(Tout *p, int c, const float (&r)[VEC]) {
  if constexpr (sizeof(Tout) < sizeof(Tin)) {
    if (c & 1) {
#pragma unroll
      for (int t = 0; t < VEC; ++t) p[c + t] = from_f32<Tout>(r[t]);
      return;
    }
  }
  Pack<Tout, VEC> o;
#pragma unroll
  for (int t = 0; t < VEC; ++t) o.v[t] = from_f32<Tout>(r[t]);
  *reinterpret_cast<Pack<Tout, VEC> *>(p + c) = o;
}

// Applies the epilogue to VEC consecutive columns of one output row and stores them; x is load_aux of the
// same columns (a caller with other loads in flight asks for it early).
template <typename Tin, typename Tout, int VEC>
__device__ inline void finish_cols(const SpmmArgs &a, int64_t row, int c, const float (&acc)[VEC], const Pack<Tin, VEC> &x) {
  float r[VEC];
  if (a.epilogue == SPMM_PLAIN) {
#pragma unroll
    for (int t = 0; t < VEC; ++t) r[t] = acc[t];
  } else if (a.epilogue == SPMM_BIAS_RELU) {
#pragma unroll
    for (int t = 0; t < VEC; ++t) {
      const float y = acc[t] + a.bias[c + t];
      r[t] = y > 0.f ? y : 0.f;
    }
  } else if (spmm_reads_add(a.epilogue)) {
    const Pack<Tin, VEC> y = *reinterpret_cast<const Pack<Tin, VEC> *>(
        static_cast<const Tin *>(a.add) + (size_t)(row - a.add_row0) * a.add_ld + c);
#pragma unroll
    for (int t = 0; t < VEC; ++t) {
      const float sum = acc[t] + to_f32(y.v[t]);
      r[t] = a.epilogue == SPMM_ADD ? sum : to_f32(x.v[t]) > 0.f ? sum * a.mask_scale : 0.f;
    }
  } else if (a.epilogue == SPMM_MIX) {
#pragma unroll
    // one rounding for the dominant (1 - alpha) term: with rows on the bf16 grid the exact mix often sits
    // exactly half-way between two bf16 values, and rounding the large product separately would push all
    // of those ties the same way
    for (int t = 0; t < VEC; ++t) r[t] = __builtin_fmaf(a.s_acc, acc[t], a.s_aux * to_f32(x.v[t]));
  } else {
#pragma unroll
    for (int t = 0; t < VEC; ++t) r[t] = to_f32(x.v[t]) > 0.f ? acc[t] * a.mask_scale : 0.f;
  }
  store_cols<Tin, Tout, VEC>(static_cast<Tout *>(a.out) + (size_t)(row - a.out_row0) * a.out_ld, c, r);
}

template <typename Tin, typename Tout, int VEC>
__device__ inline void finish_cols(const SpmmArgs &a, int64_t row, int c, const float (&acc)[VEC]) {
  finish_cols<Tin, Tout, VEC>(a, row, c, acc, load_aux<Tin, VEC>(a, row, c));
}

template <typename Tout>
__device__ inline void zero_pad_cols(const SpmmArgs &a, int64_t row, int lane) {
  const int c = a.d + lane;
  if (c < a.out_ld) static_cast<Tout *>(a.out)[(size_t)(row - a.out_row0) * a.out_ld + c] = from_f32<Tout>(0.f);
}

// The vector-ALU aggregation (fp32 rows; bf16 rows whose width is no multiple of 8).  A wave runs one task over one tile
// of LPR * VEC columns; G = 64 / LPR groups of lanes each own every G-th entry, U entries of a group are in flight.
// What bounds it is how many row pieces are outstanding: of a wave (a loop that gathers one step, adds it and goes on
// waits for memory once per step; a wave that works out every entry's address by itself spends 25 instructions on it) and
// of the launch (column tiles of wide rows run as waves of their own, and long rows are cut into short pieces where the
// launch is small and the sums are not the ones that decide which elements pass ReLU).  Measured, one launch before and after: 12 k entries of
// 4,000-byte rows 117 -> 7.9 us, 17 k entries of 400-byte rows 20 -> 6.0 us, 111 k entries of 200-byte bf16 rows
// 72 -> 8.1 us (2.7 TB/s gathered), 312 k entries of 512-byte fp32 rows 60 -> 24 us (6.7 TB/s).
// A row's last vector moves back so that it ends with the row: it repeats columns of its neighbour lane, which both
// lanes sum and store alike, and every width is read in 16-byte accesses.
template <typename Tin, typename Tout, int VEC, int LPR, int U>
__global__ __launch_bounds__(256) void spmm_kernel(const SpmmArgs a) {
  typedef Tin vec_t __attribute__((ext_vector_type(VEC), aligned(4)));
  constexpr int G = 64 / LPR;
  constexpr int TILE_W = LPR * VEC;
  const int lane = threadIdx.x & 63;
  int cls;
  const SpmmHead head = spmm_head(a);
  const int64_t task = spmm_task_index(a, head, blockIdx.x, threadIdx.x >> 6, cls);
  if (task < 0) return;  // whole wave leaves together
  const int grp = lane / LPR, lig = lane % LPR;
  const int d = a.d;
  const int col = blockIdx.y * TILE_W + lig * VEC;
  const bool on = col < d;
  const int c = col + VEC <= d ? col : d - VEC;
  // task fields are the same for the whole wave: keep them in scalar registers, so that every loop
  // bound below is provably wave-uniform (the lane permutes need all lanes in step)
  const int32_t row_raw = a.task_row[task], slot_raw = a.task_slot[task];
  const int64_t e0_raw = a.task_e0[task];
  const uint32_t ne_raw = a.task_ne[task];
  __builtin_amdgcn_sched_barrier(0);  // one round trip, also for the wave whose task turns out to be a filler
  const int64_t row = __builtin_amdgcn_readfirstlane(row_raw);
  if (row < 0) return;  // filler
  const int64_t e0 = ((int64_t)__builtin_amdgcn_readfirstlane((int)(e0_raw >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)(e0_raw & 0xffffffff));
  const uint32_t ne_chunk = (uint32_t)__builtin_amdgcn_readfirstlane((int)ne_raw);
  const int ne = (int)(ne_chunk & kTaskCountMask);
  const int slot = __builtin_amdgcn_readfirstlane(slot_raw);
  uint32_t chunk_classes;
  const bool many = a.many_chunks != 0;
  const WaveMask mask = wave_mask(spmm_row_mask(a, head, ne_chunk >> kTaskChunkShift, chunk_classes), many);
  if (cls >= 0 && !((chunk_classes >> cls) & 1u)) return;  // nothing of this class is gathered for the row's chunk
  const uint32_t vmask = (1u << a.vbits) - 1u;
  const bool drop_unsel = a.src_unsel == nullptr;
  const char *base_sel = static_cast<const char *>(a.src_sel);
  const char *base_unsel = drop_unsel ? base_sel : static_cast<const char *>(a.src_unsel);
  const uint32_t row_bytes = (uint32_t)a.src_ld * (uint32_t)sizeof(Tin), col_bytes = (uint32_t)c * (uint32_t)sizeof(Tin);

  float acc[VEC];
#pragma unroll
  for (int t = 0; t < VEC; ++t) acc[t] = 0.f;

  // the index words and weights of the next 64 entries are in flight while the current ones are gathered
  uint32_t pc_next = 0;
  float w_next = 0.f;
  auto load_meta = [&](int base) {
    if (base + lane < ne) {
      pc_next = a.pidx[e0 + base + lane];
      w_next = a.val[e0 + base + lane];
    }
  };
  load_meta(0);
  for (int base = 0; base < ne; base += 64) {
    int n = ne - base < 64 ? ne - base : 64;
    // one lane works out the row address of one entry; the lanes that gather it only add their column
    const bool sel = mask_test(mask, pc_next >> a.vbits, many);
    const uint64_t at = reinterpret_cast<uint64_t>(sel ? base_sel : base_unsel) + (uint64_t)(pc_next & vmask) * row_bytes;
    int at_lo = (int)(uint32_t)at, at_hi = (int)(at >> 32), w = __float_as_int(w_next);
    const bool keep = lane < n && (sel || !drop_unsel);
    load_meta(base + 64);
    if (drop_unsel) {  // wave-uniform: compact the kept entries to the low lanes
      const uint64_t bal = __ballot(keep);
      const int nk = __popcll(bal);
      const int rk = __popcll(bal & ((1ull << lane) - 1ull));
      const int dest = keep ? rk : nk + (lane - rk);
      at_lo = __builtin_amdgcn_ds_permute(dest << 2, at_lo);
      at_hi = __builtin_amdgcn_ds_permute(dest << 2, at_hi);
      w = __builtin_amdgcn_ds_permute(dest << 2, w);
      n = __builtin_amdgcn_readfirstlane(nk);
    }
    // entries i, i + G, ... of every group: N of them in flight; CHECK: some may lie past the end
    auto gather = [&](auto count, auto check, int i) {
      constexpr int N = decltype(count)::value;
      constexpr bool CHECK = decltype(check)::value;
      Pack<Tin, VEC> x[N];
      float ww[N];
#pragma unroll
      for (int u = 0; u < N; ++u) {
        const int idx = i + u * G + grp;
        uint64_t rp;
        if constexpr (G == 1) {  // the entry is the same for the whole wave
          rp = (uint32_t)__builtin_amdgcn_readlane(at_lo, idx & 63) | (uint64_t)(uint32_t)__builtin_amdgcn_readlane(at_hi, idx & 63) << 32;
          ww[u] = __int_as_float(__builtin_amdgcn_readlane(w, idx & 63));
        } else {
          rp = (uint32_t)__shfl(at_lo, idx & 63) | (uint64_t)(uint32_t)__shfl(at_hi, idx & 63) << 32;
          ww[u] = __int_as_float(__shfl(w, idx & 63));
        }
        if (!CHECK || idx < n) {
          const vec_t v = *(const __attribute__((address_space(1))) vec_t *)(rp + col_bytes);
#pragma unroll
          for (int t = 0; t < VEC; ++t) x[u].v[t] = v[t];
        } else {
          ww[u] = 0.f;
#pragma unroll
          for (int t = 0; t < VEC; ++t) x[u].v[t] = from_f32<Tin>(0.f);
        }
      }
      __builtin_amdgcn_sched_barrier(0);  // every load is issued before the first is waited for
#pragma unroll
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int t = 0; t < VEC; ++t) acc[t] = __builtin_fmaf(ww[u], to_f32(x[u].v[t]), acc[t]);
    };
    int i = 0;
    for (; i + G * U <= n; i += G * U) gather(std::integral_constant<int, U>{}, std::false_type{}, i);
    constexpr int TU = U < 8 ? U : 8;
    for (; i < n; i += G * TU) gather(std::integral_constant<int, TU>{}, std::true_type{}, i);
  }
  // add the G groups' partial rows (same columns live LPR lanes apart)
#pragma unroll
  for (int off = LPR; off < 64; off <<= 1)
#pragma unroll
    for (int t = 0; t < VEC; ++t) acc[t] += __shfl_xor(acc[t], off);

  if (grp == 0) {
    if (on) {
      if (slot >= 0) {
        Pack<float, VEC> o;
#pragma unroll
        for (int t = 0; t < VEC; ++t) o.v[t] = acc[t];
        *reinterpret_cast<Pack<float, VEC> *>(a.partial + (size_t)(slot - a.slot0) * d + c) = o;
      } else {
        finish_cols<Tin, Tout, VEC>(a, row, c, acc);
      }
    }
    if (slot < 0 && blockIdx.y == 0) zero_pad_cols<Tout>(a, row, lig);
  }
}

// Sums the pieces of every cut row, then applies the epilogue.  One workgroup per row: 8 phases x 32
// column vectors; phase p adds the slots p, p+8, p+16, ... (hub rows have hundreds of pieces), then the 8
// phase sums are added in order.  The order is fixed, so results are reproducible.
// A workgroup moves a few KB, so what it costs is its chain of dependent memory round trips.  There are
// two: the row's header words, then everything else at once.  Pieces that may not count (a class or an item
// that did not run in this launch holds stale sums) are loaded anyway, together with the word that says so,
// and left out by a select; the epilogue's auxiliary row is asked for before the sums.
template <typename Tin, typename Tout, int VEC>
__global__ __launch_bounds__(256) void spmm_reduce_kernel(const SpmmArgs a) {
  __shared__ float red[8][32][VEC];
  const int64_t i = blockIdx.x;
  const int ph = threadIdx.x >> 5, cv = threadIdx.x & 31;
  const bool dense = a.lr_ndense != nullptr;
  const int64_t row = a.lr_row[i];
  const int slot0 = a.lr_slot0[i];
  const uint32_t ns_chunk = a.lr_nslots[i], chunk = ns_chunk >> kTaskChunkShift;
  const int ns = (int)(ns_chunk & kTaskCountMask);
  const int nd = dense ? a.lr_ndense[i] : 0;
  const int dense0 = dense ? a.lr_dense0[i] : 0, item0 = dense ? a.lr_item0[i] : 0;
  // pieces of classes that were not run in this launch (all their entries unselected) hold stale data
  const bool check = a.slot_class != nullptr && (a.all_classes_active == 0 || a.pass != nullptr) && a.drop_unselected;
  ChunkMask mask = a.mask;
  uint32_t classes = a.active_classes;
  if (a.pass != nullptr && a.drop_unselected) {
    mask = a.pass[chunk].mask;
    classes &= a.pass[chunk].classes;
  }
  {
    const int col = (int)blockIdx.y * 32 * VEC + cv * VEC;
    const bool on = col < a.d;
    const int c = col + VEC <= a.d ? col : a.d - VEC;  // the row's last vector ends with the row
    float acc[VEC];
#pragma unroll
    for (int t = 0; t < VEC; ++t) acc[t] = 0.f;
    Pack<Tin, VEC> xa;
    if (on) {
      if (ph == 0) xa = load_aux<Tin, VEC>(a, row, c);
      for (int s = ph; s < ns; s += 8) {
        const uint32_t sc = check ? a.slot_class[slot0 + s] : 32u;
        const Pack<float, VEC> x = *reinterpret_cast<const Pack<float, VEC> *>(a.partial + (size_t)(slot0 + s - a.slot0) * a.d + c);
        __builtin_amdgcn_sched_barrier(0);
        const bool use = sc >= 32u || ((classes >> sc) & 1u);
#pragma unroll
        for (int t = 0; t < VEC; ++t) acc[t] += use ? x.v[t] : 0.f;
      }
      // the row's parts from dense blocks: one partial row per item of its row block
      for (int g = ph; g < nd; g += 8) {
        bool use = true;
        if (a.drop_unselected) {  // an item without a selected chunk was not run
          const ChunkMask m = a.item_chunks[item0 + g];
          use = ((m.w[0] & mask.w[0]) | (m.w[1] & mask.w[1]) | (m.w[2] & mask.w[2]) | (m.w[3] & mask.w[3])) != 0;
        }
        const Pack<float, VEC> x =
            *reinterpret_cast<const Pack<float, VEC> *>(a.dense_partial + ((size_t)dense0 + (size_t)(g - a.item0) * kDenseRB) * a.d + c);
#pragma unroll
        for (int t = 0; t < VEC; ++t) acc[t] += use ? x.v[t] : 0.f;
      }
    }
#pragma unroll
    for (int t = 0; t < VEC; ++t) red[ph][cv][t] = acc[t];
    __syncthreads();
    if (ph == 0 && on) {
#pragma unroll
      for (int p = 1; p < 8; ++p)
#pragma unroll
        for (int t = 0; t < VEC; ++t) acc[t] += red[p][cv][t];
      finish_cols<Tin, Tout, VEC>(a, row, c, acc, xa);
    }
  }
  if (threadIdx.x < 64 && blockIdx.y == 0) zero_pad_cols<Tout>(a, row, threadIdx.x);
}

// ---- bf16 sources: the weighted row sum on the matrix cores ---------------------------------
// A gathered 16-byte piece (8 consecutive bf16 columns of one neighbour row) is exactly one lane's
// A-operand fragment of v_mfma_f32_16x16x32_bf16: lane l supplies A[m = l%16][k = 8*(l/16) .. +8].
// Reading m as "8-column block" and k as (neighbour slot g = l/16, column t inside the block), the
// B operand  B[8g + t][n] = w_g * [t == n % 8]  turns the instruction into
//     D[m][n] += sum_g w_g * X[u_g][8m + n % 8]
// i.e. four neighbours (one per 16-lane group) times a 128-column tile are scaled by their edge
// weights and accumulated in fp32 with no bf16->fp32 conversion and no vector FMA.  Columns n < 8 of B
// carry the upper bf16 half of the fp32 weight, columns n >= 8 the remainder, and the two halves of D
// are added at the end, so the weight keeps 16 mantissa bits.  (A non-finite input value also poisons
// the other 7 columns of its 8-column block, since 0 * inf = nan inside the dot product.)
typedef bf16_t bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) bf16x8_t global_bf16x8_t;  // a load through it is a global load

// A record of the gather loops: row address and the weight as two bf16.
__device__ inline uint32_t pack_weight(float w) {
  const bf16_t hi = (bf16_t)w;
  const bf16_t lo = (bf16_t)(w - (float)hi);
  return (uint32_t)__builtin_bit_cast(uint16_t, hi) | ((uint32_t)__builtin_bit_cast(uint16_t, lo) << 16);
}
// What a lane contributes to the B operand: selw moves its half of the packed weight (columns 0 .. 7 the upper, 8 .. 15 the lower)
// into bf16 element pos & 1 of a word and zeroes the other, wword says which of the four words that is.
struct WeightLane {
  uint32_t selw;
  int wword;
};
__device__ inline WeightLane weight_lane(int lig) {
  const int pos = lig & 7;
  const uint32_t b0 = lig >= 8 ? 2u : 0u;
  return WeightLane{(pos & 1) ? (((b0 + 1u) << 24) | (b0 << 16) | 0x0c0cu) : (0x0c0c0000u | ((b0 + 1u) << 8) | b0), pos >> 1};
}
__device__ inline bf16x8_t weight_operand(const WeightLane &l, uint32_t packed) {
  const uint32_t wbits = __builtin_amdgcn_perm(0u, packed, l.selw);
  u32x4_t bw;
  bw[0] = l.wword == 0 ? wbits : 0u;
  bw[1] = l.wword == 1 ? wbits : 0u;
  bw[2] = l.wword == 2 ? wbits : 0u;
  bw[3] = l.wword == 3 ? wbits : 0u;
  return __builtin_bit_cast(bf16x8_t, bw);
}
// Accumulators of one row -> its columns in LDS.  Element i of lane l is D[m = 4*(l/16) + i][n = l%16]; column = 8m + n%8, the
// halves n < 8 and n >= 8 are the two parts of the weight.
template <int NT>
__device__ inline void row_to_lds(const f32x4_t (&acc)[NT], float *rowbuf, int lane) {
#pragma unroll
  for (int h = 0; h < NT; ++h)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float v = acc[h][i] + __shfl_xor(acc[h][i], 8);
      if (!(lane & 8)) rowbuf[h * 128 + (4 * (lane >> 4) + i) * 8 + (lane & 7)] = v;
    }
}
__device__ inline void lds_written() {  // the wave's own LDS writes have landed
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Short rows (at most kShortRowMost entries: the bulk of a power-law graph's rows).  A wave per row spends its life in a chain
// of memory round trips (task, index words, gathers, the epilogue's row) to move a kilobyte or two, and what a launch of many
// short rows takes is rounds of such chains: a backward launch, which gathers half of the entries, took nine tenths of a forward
// one.  Here a wave serves four rows in one chain: a 16-lane group reads the index words of one, one per lane; the kept
// entries of the four rows become one run of records, each row's filled up to a multiple of four with zero weights, so that
// the gather loop sees steps of four records as in spmm_ring_kernel and a row's sum has the same bits as there; at a row's last
// step its accumulators go to LDS (behind the records, the last row's in their place); the epilogue's rows are asked for with the
// index words.  `first` = index of the first row of this wave among the launch's short rows.  The four rows are of one chunk
// (fillers see to it).
template <typename Tout, int NT, bool FULL>
__device__ __forceinline__ void spmm_short_rows(const SpmmArgs &a, int64_t first, u32x4_t *ring) {
  constexpr int U = 2;           // steps in flight
  constexpr int LR = NT * 16;    // lanes that hold a row's columns behind the sums
  constexpr int NR = 64 / LR;    // rows stored at a time
  constexpr int NP = 4 / NR;
  static_assert(NT == 1 || NT == 2, "the sums of three rows of 256 columns fit behind the records");
  if (first >= a.n_short) return;  // whole waves: n_short is a multiple of four
  const int lane = threadIdx.x & 63, lig = lane & 15, g = lane >> 4;
  auto rowbuf = [&](int r) { return reinterpret_cast<float *>(ring + (r < 3 ? 4 * kShortRowMost + r * (NT * 32) : 0)); };  // NT * 128 floats
  const int64_t task = a.short0 + first + g;
  const uint32_t ne_chunk = a.task_ne[task];
  const int64_t e0 = a.task_e0[task];
  const bool drop_unsel = a.src_unsel == nullptr, many = a.many_chunks != 0;
  const int ne = (int)(ne_chunk & kTaskCountMask);  // 0 of a filler
  const int d = a.d, c_out = (lane % LR) * 8;
  int32_t row_out[NP];  // rows that this lane stores columns c_out .. of
  Pack<bf16_t, 8> xa[NP];
#pragma unroll
  for (int p = 0; p < NP; ++p) row_out[p] = a.task_row[a.short0 + first + p * NR + lane / LR];
  uint32_t pc = 0;
  float w_own = 0.f;
  if (lig < ne) {
    pc = a.pidx[e0 + lig];
    w_own = a.val[e0 + lig];
  }
#pragma unroll
  for (int p = 0; p < NP; ++p)
    if (NT == 1 && row_out[p] >= 0 && c_out < d) xa[p] = load_aux<bf16_t, 8>(a, row_out[p], c_out);
  uint32_t classes;
  const WaveMask mask = wave_mask(spmm_row_mask(a.pass, a.mask, (uint32_t)__builtin_amdgcn_readfirstlane((int)ne_chunk) >> kTaskChunkShift, classes), many);
  const bool sel = mask_test(mask, pc >> a.vbits, many);
  const bool keep = lig < ne && (sel || !drop_unsel);
  const uint64_t bal = __ballot(keep);
  int end[4];  // steps up to every row's last
  int steps = 0, my0 = 0;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    if (r == g) my0 = steps;
    steps += (__popc((uint32_t)(bal >> (16 * r)) & 0xffffu) + 3) >> 2;
    end[r] = steps;
  }
  const uint32_t bits = (uint32_t)(bal >> (16 * g)) & 0xffffu;
  const int nk = __popc(bits);
  const uint64_t at = reinterpret_cast<uint64_t>(sel ? a.src_sel : a.src_unsel) + (uint64_t)(pc & ((1u << a.vbits) - 1u)) * ((uint32_t)a.src_ld * 2u);
  // fillers of the last step: a kept row of the same sum, weight zero
  const int pad_from = (g * 16 + (bits ? __ffs(bits) - 1 : 0)) << 2;
  const uint32_t pad_lo = (uint32_t)__builtin_amdgcn_ds_bpermute(pad_from, (int)(uint32_t)at);
  const uint32_t pad_hi = (uint32_t)__builtin_amdgcn_ds_bpermute(pad_from, (int)(uint32_t)(at >> 32));
  if (keep) ring[my0 * 4 + __popc(bits & ((1u << lig) - 1u))] = u32x4_t{(uint32_t)at, (uint32_t)(at >> 32), pack_weight(w_own), 0u};
  if (lig >= nk && lig < ((nk + 3) & ~3)) ring[my0 * 4 + lig] = u32x4_t{pad_lo, pad_hi, 0u, 0u};
  lds_written();
  const WeightLane wl = weight_lane(lig);
  const bf16x8_t zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  f32x4_t acc[NT];
#pragma unroll
  for (int h = 0; h < NT; ++h) acc[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  bf16x8_t x[U][NT];
  uint32_t wk[U];
  auto issue = [&](int step, int u) {
    const u32x4_t rec = ring[step * 4 + g];
    const global_bf16x8_t *p = reinterpret_cast<const global_bf16x8_t *>(((uint64_t)rec[1] << 32 | rec[0]) + (uint32_t)lig * 16u);
    wk[u] = rec[2];
#pragma unroll
    for (int h = 0; h < NT; ++h) x[u][h] = (FULL || h * 128 + lig * 8 < d) ? p[h * 16] : zero8;
    __builtin_amdgcn_sched_barrier(0);
  };
  int r = 0;  // rows finished
  auto finish_rows = [&](int done) {  // those whose last step is among the first `done`
    while (r < 4 && (r == 0 ? end[0] : r == 1 ? end[1] : r == 2 ? end[2] : end[3]) <= done) {
      row_to_lds<NT>(acc, rowbuf(r), lane);
#pragma unroll
      for (int h = 0; h < NT; ++h) acc[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      ++r;
    }
  };
  finish_rows(0);
#pragma unroll
  for (int u = 0; u < U; ++u)
    if (u < steps) issue(u, u);
  for (int k = 0; k < steps; k += U) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k + u < steps) {  // uniform, like all control flow around the matrix instruction
        const bf16x8_t bfrag = weight_operand(wl, wk[u]);
#pragma unroll
        for (int h = 0; h < NT; ++h) acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[u][h], bfrag, acc[h], 0, 0, 0);
        if (k + u + U < steps) issue(k + u + U, u);
        finish_rows(k + u + 1);
      }
    }
  }
#pragma unroll
  for (int p = 0; p < NP; ++p)  // (registers for both rows of a lane are free only now)
    if (NT == 2 && row_out[p] >= 0 && c_out < d) xa[p] = load_aux<bf16_t, 8>(a, row_out[p], c_out);
  lds_written();
#pragma unroll 1
  for (int p = 0; p < NP; ++p) {
    const float *sums = rowbuf(p * NR + lane / LR) + c_out;
    const int32_t row = p == 0 ? row_out[0] : row_out[NP - 1];
    if (row < 0) continue;
    if (c_out < d) {
      float v[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = sums[t];
      finish_cols<bf16_t, Tout, 8>(a, row, c_out, v, p == 0 ? xa[0] : xa[NP - 1]);
    }
    zero_pad_cols<Tout>(a, row, lane % LR);
  }
}

// Short rows of tables that fit no cache (at most four entries, weights in fp32): every 16-lane group owns one row: a lane keeps
// 8 columns of each 128-column tile in fp32 registers and the sum runs on the vector ALU; two to four of the row's entries are in
// flight per lane.  Entries that a backward launch drops are not loaded at all.
template <typename Tout, int NT, bool FULL, bool MANY>
__device__ __forceinline__ void spmm_short_rows_valu(const SpmmArgs &a, int64_t first) {
  if (first >= a.n_short) return;  // whole waves: n_short is a multiple of four
  const int lane = threadIdx.x & 63, lig = lane & 15;
  const int64_t task = a.short0 + first + (lane >> 4);
  const uint32_t ne_chunk = a.task_ne[task];
  const int64_t row = a.task_row[task], e0 = a.task_e0[task];
  uint32_t classes;
  const ChunkMask mask = spmm_row_mask(a.pass, a.mask, (uint32_t)__builtin_amdgcn_readfirstlane((int)ne_chunk) >> kTaskChunkShift, classes);
  const uint32_t vmask = (1u << a.vbits) - 1u;
  const bool drop_unsel = a.src_unsel == nullptr;
  const char *base_sel = static_cast<const char *>(a.src_sel);
  const char *base_unsel = drop_unsel ? base_sel : static_cast<const char *>(a.src_unsel);
  const size_t row_bytes = (size_t)a.src_ld * 2u;
  const int d = a.d;
  if (row < 0) return;
  const int ne = (int)(ne_chunk & kTaskCountMask);
  float acc[NT][8];
#pragma unroll
  for (int h = 0; h < NT; ++h)
#pragma unroll
    for (int c = 0; c < 8; ++c) acc[h][c] = 0.f;
  constexpr int SU = MANY ? 1 : NT == 1 ? 4 : 2;  // entries in flight per lane (16 bytes x NT each); MANY: more than 64 chunks
  for (int i = 0; i < ne; i += SU) {
    bf16x8_t x[SU][NT];
    float w[SU];
#pragma unroll
    for (int u = 0; u < SU; ++u) {
      w[u] = 0.f;
#pragma unroll
      for (int h = 0; h < NT; ++h) x[u][h] = bf16x8_t{0, 0, 0, 0, 0, 0, 0, 0};
      if (i + u < ne) {
        const uint32_t pc = a.pidx[e0 + i + u];
        const bool sel = MANY ? mask_test(mask, pc >> a.vbits) : ((mask.w[0] >> (pc >> a.vbits)) & 1ull) != 0;
        if (sel || !drop_unsel) {
          w[u] = a.val[e0 + i + u];
          const char *p = (sel ? base_sel : base_unsel) + (size_t)(pc & vmask) * row_bytes + (size_t)lig * 16u;
#pragma unroll
          for (int h = 0; h < NT; ++h)
            if (FULL || h * 128 + lig * 8 < d) x[u][h] = *reinterpret_cast<const bf16x8_t *>(p + h * 256);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < SU; ++u)
#pragma unroll
      for (int h = 0; h < NT; ++h)
#pragma unroll
        for (int c = 0; c < 8; ++c) acc[h][c] = __builtin_fmaf(w[u], (float)x[u][h][c], acc[h][c]);
  }
#pragma unroll
  for (int h = 0; h < NT; ++h) {
    const int c = h * 128 + lig * 8;
    if (FULL || c < d) finish_cols<bf16_t, Tout, 8>(a, row, c, acc[h]);
  }
  zero_pad_cols<Tout>(a, row, lig);
}

// Entry metadata is turned, once per entry, into a 16-byte record {row address, packed weight halves}
// and appended to a wave-private ring in LDS; unselected entries of a backward launch are simply not
// appended, so the gather loop sees one dense stream of kept entries across the 64-entry metadata
// batches.  A wave alternates between two phases.  Phase A turns KB batches of metadata (loaded during
// the previous phase B) into records.  Phase B gathers: it works in steps of four records (one per
// 16-lane group) and owns U register slots; slot u holds the pieces of step s with s % U == u.  In the
// steady loop every slot is multiplied into the accumulators and immediately refilled with the loads of
// step s + U, unconditionally, so the number of younger loads at every wait is a compile-time constant
// and U - 1 steps of gathers stay in flight while one is consumed.  Per step the vector ALU only adds
// the lane offset to the record's address and expands the weight (one byte permute, four selects).
// Waves per SIMD: seven where their registers hold the loop.  Four column blocks need 86; held to 72 they went through scratch
// memory inside the loop: two forward aggregations of 250 k rows of width 512 took 890 us and take 597 us with five waves
// (width 384 1,090 -> 584; six waves still spill: 742, 753).
template <typename Tout, int NT, int U, bool FULL>
__global__ __launch_bounds__(256, NT * U > 8 ? 1 : NT == 4 ? 5 : 7) void spmm_ring_kernel(const SpmmArgs a) {
  constexpr int TILE_W = NT * 128;
  constexpr int KB = 2;    // metadata batches per phase
  constexpr int R = 256;   // ring capacity in records: a phase appends at most 64 * KB, fewer than 8 * U are left over
  static_assert(TILE_W * sizeof(float) <= R * sizeof(u32x4_t), "the output row reuses the ring's memory");
  static_assert(NT > 2 || 4 * kShortRowMost * sizeof(u32x4_t) + 3 * TILE_W * sizeof(float) <= R * sizeof(u32x4_t), "and so do those of short rows");
  static_assert((U & (U - 1)) == 0 && U <= 8, "slot count");
  __shared__ u32x4_t ring_all[4][R];
  const SpmmHead head = spmm_head(a);
  if constexpr (NT <= 2) {
    const SpmmTurn turn = spmm_turn(head, blockIdx.x);
    if ((int)blockIdx.x >= head.n_class_blocks && turn.is_short && head.short_rows != SHORT_ROWS_SINGLE) {  // 16 short rows
      const int64_t first = (int64_t)turn.index * 16 + (threadIdx.x >> 6) * 4;
      if (head.short_rows == SHORT_ROWS_MFMA)
        spmm_short_rows<Tout, NT, FULL>(a, first, ring_all[threadIdx.x >> 6]);
      else if (a.many_chunks != 0)
        spmm_short_rows_valu<Tout, NT, FULL, true>(a, first);
      else
        spmm_short_rows_valu<Tout, NT, FULL, false>(a, first);
      return;
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int cls;
  const int64_t task = spmm_task_index(a, head, blockIdx.x, wave, cls);
  if (task < 0) return;  // whole wave leaves together (no block-wide barrier below)
  u32x4_t *ring = ring_all[wave];
  const int g = lane >> 4, lig = lane & 15;
  const int tile0 = blockIdx.y * TILE_W;
  // Task fields are the same for the whole wave: keep them in scalar registers.  The matrix instruction
  // ignores the execution mask, so all control flow around it must be provably wave-uniform.
  const int32_t row_raw = a.task_row[task], slot_raw = a.task_slot[task];
  const int64_t e0_raw = a.task_e0[task];
  const uint32_t ne_raw = a.task_ne[task];
  __builtin_amdgcn_sched_barrier(0);  // one round trip, also for the wave whose task turns out to be a filler
  const int64_t row = __builtin_amdgcn_readfirstlane(row_raw);
  if (row < 0) return;  // filler
  const int64_t e0 = ((int64_t)__builtin_amdgcn_readfirstlane((int)(e0_raw >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)(e0_raw & 0xffffffff));
  const uint32_t ne_chunk = (uint32_t)__builtin_amdgcn_readfirstlane((int)ne_raw);
  const int ne = (int)(ne_chunk & kTaskCountMask);
  const int slot = __builtin_amdgcn_readfirstlane(slot_raw);
  uint32_t chunk_classes;
  const bool many = a.many_chunks != 0;
  const WaveMask mask = wave_mask(spmm_row_mask(a, head, ne_chunk >> kTaskChunkShift, chunk_classes), many);
  if (cls >= 0 && !((chunk_classes >> cls) & 1u)) return;  // nothing of this class is gathered for the row's chunk
  const uint32_t vmask = (1u << a.vbits) - 1u;
  const bool drop_unsel = a.src_unsel == nullptr;
  const char *base_sel = static_cast<const char *>(a.src_sel) + (size_t)tile0 * 2;
  const char *base_unsel = drop_unsel ? base_sel : static_cast<const char *>(a.src_unsel) + (size_t)tile0 * 2;
  const int d = a.d;
  const uint32_t row_bytes = (uint32_t)a.src_ld * 2u;
  const uint32_t lane_off = (uint32_t)lig * 16u;
  const WeightLane wl = weight_lane(lig);

  f32x4_t acc[NT];
#pragma unroll
  for (int h = 0; h < NT; ++h) acc[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  const bf16x8_t zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  bf16x8_t x[U][NT];
  uint32_t wk[U];
  uint64_t rec_addr = 0;  // record of the next step to issue, read one step ahead
  uint32_t rec_w = 0;

  auto read_record = [&](int step) {
    const uint32_t *rec = reinterpret_cast<const uint32_t *>(&ring[((step << 2) + g) & (R - 1)]);
    rec_addr = *reinterpret_cast<const uint64_t *>(rec);
    rec_w = rec[2];
  };
  // gathers of step `step` into slot u; the record was read before, the following one is requested now
  // (past the last appended record this reads stale ring memory that nobody uses)
  auto issue = [&](int step, int u) {
    const global_bf16x8_t *p = reinterpret_cast<const global_bf16x8_t *>(rec_addr + lane_off);
    wk[u] = rec_w;
#pragma unroll
    for (int h = 0; h < NT; ++h) x[u][h] = (FULL || tile0 + h * 128 + lig * 8 < d) ? p[h * 16] : zero8;
    read_record(step + 1);
    // keep the slots in program order: the wait in front of a slot's product then only covers that slot's
    // own loads and leaves the younger gathers in flight
    __builtin_amdgcn_sched_barrier(0);
  };
  auto consume = [&](int u) {
    const bf16x8_t bfrag = weight_operand(wl, wk[u]);
#pragma unroll
    for (int h = 0; h < NT; ++h) acc[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[u][h], bfrag, acc[h], 0, 0, 0);
    __builtin_amdgcn_sched_barrier(0);
  };

  const int nb = (ne + 63) >> 6;  // metadata batches
  int bprod = 0;                  // batches turned into records so far
  int produced = 0;               // records appended so far
  int issued = 0;                 // steps whose gathers have been issued (and, between phases, multiplied)
  uint32_t pad_lo = 0, pad_hi = 0;  // address of some kept row, for the zero-weight records that fill the last step

  uint32_t pcs[KB];
  float ws[KB];
  auto prefetch = [&](int b0) {  // clamped index: lanes past the end re-read the last entry and are not kept
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      int i = ((b0 + k) << 6) + lane;
      i = i < ne ? i : ne - 1;
      pcs[k] = a.pidx[e0 + i];
      ws[k] = a.val[e0 + i];
    }
  };
  if (ne > 0) prefetch(0);
  while (bprod < nb) {
    // ---- phase A: KB batches of metadata become records
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const int nraw = ne - ((bprod + k) << 6);  // entries left from this batch on (may be <= 0)
      const uint32_t pc = pcs[k];
      const float w = ws[k];
      const bool sel = mask_test(mask, pc >> a.vbits, many);
      const bool keep = lane < nraw && (sel || !drop_unsel);
      const uint64_t addr = reinterpret_cast<uint64_t>(sel ? base_sel : base_unsel) + (uint64_t)(pc & vmask) * row_bytes;
      const uint32_t wpk = pack_weight(w);
      const uint64_t bal = __ballot(keep);
      const int nk = __builtin_amdgcn_readfirstlane(__popcll(bal));
      const int rk = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
      if (keep) ring[(produced + rk) & (R - 1)] = u32x4_t{(uint32_t)addr, (uint32_t)(addr >> 32), wpk, 0u};
      if (nk > 0) {
        const int first = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)bal) - 1);
        pad_lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)addr, first);
        pad_hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(addr >> 32), first);
      }
      produced += nk;
    }
    bprod += KB;
    const bool final = bprod >= nb;
    if (!final) prefetch(bprod);  // lands while this phase's gathers run
    if (final) {  // complete the last step with zero-weight records that point at a row of the sum
      const int padn = (-produced) & 3;
      if (lane < padn) ring[(produced + lane) & (R - 1)] = u32x4_t{pad_lo, pad_hi, 0u, 0u};
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    const int avail = final ? (produced + 3) >> 2 : produced >> 2;  // steps that may be issued
    const int count = avail - issued;
    if (!final && count < 2 * U) continue;  // too few kept entries for a steady loop: collect more first
    // ---- phase B: steps issued .. avail - 1
    read_record(issued);
    int k = 0;
    if (count >= 2 * U) {
#pragma unroll
      for (int u = 0; u < U; ++u) issue(issued + u, u);
      for (; k + 2 * U <= count; k += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
          consume(u);
          issue(issued + k + U + u, u);
        }
      }
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (u < count) issue(issued + u, u);
    }
    // steps k .. k + U - 1 (those below count) are in their slots; fewer than U further steps remain
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k + u < count) consume(u);
      if (k + U + u < count) issue(issued + k + U + u, u);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + U + u < count) consume(u);
    issued = avail;
  }
  float *rowbuf = reinterpret_cast<float *>(ring);  // every record has been read: the ring's memory is free
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  row_to_lds<NT>(acc, rowbuf, lane);
  lds_written();
  // natural layout again: lane q owns 8 consecutive columns
#pragma unroll
  for (int r = 0; r < (NT * 16 + 63) / 64; ++r) {
    const int q = lane + 64 * r;
    const int c = tile0 + q * 8;
    if (q < NT * 16 && c < d) {
      float v[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) v[t] = rowbuf[q * 8 + t];
      if (slot >= 0) {
        Pack<float, 8> o;
#pragma unroll
        for (int t = 0; t < 8; ++t) o.v[t] = v[t];
        *reinterpret_cast<Pack<float, 8> *>(a.partial + (size_t)(slot - a.slot0) * d + c) = o;
      } else {
        finish_cols<bf16_t, Tout, 8>(a, row, c, v);
      }
    }
  }
  if (slot < 0 && blockIdx.y == 0) zero_pad_cols<Tout>(a, row, lane);
}

typedef void (*spmm_fn)(const SpmmArgs);
struct Shape {
  int vec, lpr;
  spmm_fn main, reduce;
};

template <typename Tin, typename Tout, int VEC, int LPR, int U>
constexpr Shape shape_of() {
  return Shape{VEC, LPR, spmm_kernel<Tin, Tout, VEC, LPR, U>, spmm_reduce_kernel<Tin, Tout, VEC>};
}

// 16 bytes per lane wherever the row has that many, as few lanes per row as cover it (more rows in flight per wave), rows
// wider than 64 lanes cut into tiles; 4 bytes per lane for the narrowest rows.
// deep: 16 entries of a group in flight instead of 4 or 8, for launches of few waves with long pieces, where a wave has
// only its own loads to hide latency behind.  fp32 stages, 32 chunks, deep / not: 34 k vertices of width 100 5.07 / 5.51 ms per
// step, 89 k 11.2 / 11.8, 5 k of width 1000 7.13 / 7.34.  Short pieces lose the registers for nothing: 47 k vertices of
// width 100 in bf16 (pieces of 32) 4.01 / 3.74 ms.
template <typename Tin, typename Tout>
const Shape *pick_for(int d, bool deep) {
  constexpr int V = 16 / sizeof(Tin), V1 = 4 / sizeof(Tin);
  static const Shape tab[] = {shape_of<Tin, Tout, V1, 16, 4>(), shape_of<Tin, Tout, V, 16, 4>(), shape_of<Tin, Tout, V, 32, 4>(),
                              shape_of<Tin, Tout, V, 64, 8>()};
  if constexpr (std::is_same_v<Tin, float> && std::is_same_v<Tout, float>) {
    static const Shape deep_tab[] = {shape_of<Tin, Tout, V1, 16, 16>(), shape_of<Tin, Tout, V, 16, 16>(), shape_of<Tin, Tout, V, 32, 16>(),
                                     shape_of<Tin, Tout, V, 64, 16>()};
    if (deep) return &deep_tab[d < V ? 0 : d <= 16 * V ? 1 : d <= 32 * V ? 2 : 3];
  }
  return &tab[d < V ? 0 : d <= 16 * V ? 1 : d <= 32 * V ? 2 : 3];
}
constexpr int64_t kDeepWaves = 8192;  // two rounds of the four waves per SIMD that the deep instances' registers leave

}  // namespace

static const Shape *pick_shape(const SpmmArgs &a, int src_dtype, int out_dtype) {
  const bool deep = a.long_pieces && (a.n_class_blocks * (int64_t)4 + a.n_tail + a.n_short) * ((a.d + 255) / 256) <= kDeepWaves;
  if (src_dtype == DT_BF16) {
    if (a.d % 2 != 0) return nullptr;  // rejected at create time
    return out_dtype == DT_BF16 ? pick_for<bf16_t, bf16_t>(a.d, deep) : pick_for<bf16_t, float>(a.d, deep);
  }
  return out_dtype == DT_BF16 ? pick_for<float, bf16_t>(a.d, deep) : pick_for<float, float>(a.d, deep);
}

static bool mfma_path(const SpmmArgs &a, int src_dtype) {
  const bool off = a.force_valu != 0;  // measurement switch
  const bool has_aux = spmm_reads_aux(a.epilogue);
  return !off && src_dtype == DT_BF16 && a.d % 8 == 0 && a.src_ld % 8 == 0 && a.out_ld % 8 == 0 &&
         (!has_aux || a.aux_ld % 8 == 0) && (!spmm_reads_add(a.epilogue) || a.add_ld % 8 == 0);
}

template <typename Tout, int NT>
static spmm_fn ring_fn(const SpmmArgs &a, int unroll) {
  const bool full = a.d == NT * 128;
  if (unroll >= 8) return full ? spmm_ring_kernel<Tout, NT, 8, true> : spmm_ring_kernel<Tout, NT, 8, false>;
  if (unroll >= 4) return full ? spmm_ring_kernel<Tout, NT, 4, true> : spmm_ring_kernel<Tout, NT, 4, false>;
  return full ? spmm_ring_kernel<Tout, NT, 2, true> : spmm_ring_kernel<Tout, NT, 2, false>;
}
template <typename Tout>
static spmm_fn ring_for(const SpmmArgs &a) {
  const int unroll = a.unroll;  // 4 or 8 trade waves per SIMD for deeper per-wave queues (tests run all three)
  return a.d <= 128 ? ring_fn<Tout, 1>(a, unroll) : a.d <= 256 ? ring_fn<Tout, 2>(a, unroll) : ring_fn<Tout, 4>(a, unroll >= 8 ? 4 : 2);
}

static int launch_checked(spmm_fn fn, dim3 grid, const SpmmArgs &a, hipStream_t s) {
  hipLaunchKernelGGL(fn, grid, dim3(256), 0, s, a);
  return (int)hipGetLastError();
}

int launch_spmm(const SpmmArgs &a_in, int src_dtype, int out_dtype, hipStream_t s) {
  SpmmArgs a = a_in;
  const bool mfma = mfma_path(a, src_dtype);
  // short rows: 16 to a workgroup where four rows of them fit a wave's registers, else one to a wave like the others
  const int64_t tail_blocks = (a.n_tail + 3) / 4, short_blocks = mfma && a.d <= 256 && a.short_rows != SHORT_ROWS_SINGLE ? (a.n_short + 15) / 16 : a.n_short / 4;
  int64_t gx = a.n_class_blocks + tail_blocks + short_blocks;
  if (gx <= 0) return hipSuccess;
  if (gx + 7 > kMostBlocks) return hipErrorInvalidValue;
  // rounded up: the count of short workgroups comes out exactly (below 2^32 workgroups), and none behind the last one
  a.mix = short_blocks > 0 ? (((uint64_t)short_blocks << 32) + (uint64_t)(tail_blocks + short_blocks) - 1) / (uint64_t)(tail_blocks + short_blocks) : 0;
  if (mfma)
    return launch_checked(out_dtype == DT_BF16 ? ring_for<bf16_t>(a) : ring_for<float>(a), dim3((unsigned)gx, a.d <= 256 ? 1u : (unsigned)((a.d + 511) / 512)), a, s);
  const Shape *best = pick_shape(a, src_dtype, out_dtype);
  if (!best) return hipErrorInvalidValue;
  const int tile_w = best->lpr * best->vec;
  const unsigned gy = (unsigned)((a.d + tile_w - 1) / tile_w);
  if (gy > 1) gx = (gx + 7) / 8 * 8;  // every column tile starts on the same XCD (tasks past the end do nothing)
  return launch_checked(best->main, dim3((unsigned)gx, gy), a, s);
}

int launch_spmm_reduce(const SpmmArgs &a, int src_dtype, int out_dtype, hipStream_t s) {
  if (a.n_long <= 0) return hipSuccess;
  if (a.n_long > kMostBlocks) return hipErrorInvalidValue;
  const Shape *best = pick_shape(a, src_dtype, out_dtype);
  if (!best) return hipErrorInvalidValue;
  return launch_checked(best->reduce, dim3((unsigned)a.n_long, (unsigned)((a.d + 32 * best->vec - 1) / (32 * best->vec))), a, s);
}
