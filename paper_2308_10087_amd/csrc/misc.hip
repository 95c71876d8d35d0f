// Small kernels around the two hot operations: weight staging, the ReLU-derivative mask on
// the upstream gradient, the history copy (Section 3.4, second technique), zero fill, and the
// symmetric normalisation weights of Section 2.1.
#include <algorithm>

#include "common.h"

namespace {

__device__ inline float to_f32(float x) { return x; }
__device__ inline float to_f32(bf16_t x) { return (float)x; }
template <typename T>
__device__ inline T from_f32(float x);
template <>
__device__ inline float from_f32<float>(float x) { return x; }
template <>
__device__ inline bf16_t from_f32<bf16_t>(float x) { return (bf16_t)x; }

// Row chunk c's entries of a pass's tables; pos: places of the chunks in the forward order, in LDS.
__device__ inline void write_pass_chunk(const PassTableArgs &a, const int *pos, int c) {
  PassChunk f{}, b{}, e{};
  const int p = pos[c];
  for (int k = 0; k < a.K; ++k) {
    const uint64_t bit = 1ull << (k & 63);
    const int pk = pos[k];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (k >> 6 != i) continue;
      f.mask.w[i] |= pk <= p ? bit : 0;
      b.mask.w[i] |= pk >= p ? bit : 0;
      e.mask.w[i] |= pk < p ? bit : 0;
    }
  }
  f.classes = 0xffffffffu;
  b.classes = a.classes_backward[c];
  e.classes = a.classes_earlier[c];
  a.forward[c] = f;
  a.backward[c] = b;
  a.earlier[c] = e;
}

// Wt[n][k] = W[k][n] (k < K, else 0; row stride Kp) and Wn[k][n] = W[k][n] (n < N, else 0; row stride Np), a 32 x 32 tile of one
// weight (plane of the grid) per workgroup, turned in LDS; the plane behind the weights writes a pass's tables.  What a pass
// needs before its first layer is one launch: 5 launches of 2.3 - 2.9 us for four 64 x 64 weights and the tables, 4 of 10 us for
// 1000 x 1000 (strided reads).
struct StageArgs {
  StageWeightsArgs w[kBatch];
  int32_t n;
  PassTableArgs tables;
};
static_assert(sizeof(StageArgs) <= 4096 && kMaxChunks == 256, "kernel arguments; a thread per chunk");
template <typename T>
__global__ __launch_bounds__(256) void stage_weights_kernel(const StageArgs a) {
  __shared__ T tile[32][33];
  __shared__ int pos[kMaxChunks];
  if ((int)blockIdx.y >= a.n) {
    if (blockIdx.x > 0) return;
    const int c = threadIdx.x;
    pos[c] = c < a.tables.K ? a.tables.pos[c] : 0;
    __syncthreads();
    if (c < a.tables.K) write_pass_chunk(a.tables, pos, c);
    return;
  }
  const StageWeightsArgs w = a.w[blockIdx.y];
  const int tk = (max(w.K, w.Kp) + 31) / 32, tn = (max(w.N, w.Np) + 31) / 32;
  if ((int)blockIdx.x >= tk * tn) return;
  const int k0 = (int)blockIdx.x / tn * 32, n0 = (int)blockIdx.x % tn * 32;
  const int x = threadIdx.x & 31, y = threadIdx.x >> 5;
  const T *W = static_cast<const T *>(w.W);
  T *Wt = static_cast<T *>(w.Wt), *Wn = static_cast<T *>(w.Wn);
#pragma unroll
  for (int i = 0; i < 32; i += 8) {
    const int k = k0 + y + i, n = n0 + x;
    const T v = k < w.K && n < w.N ? W[(size_t)k * w.N + n] : from_f32<T>(0.f);
    if (k < w.K && n < w.Np) Wn[(size_t)k * w.Np + n] = v;
    tile[y + i][x] = v;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 32; i += 8) {
    const int n = n0 + y + i, k = k0 + x;
    if (n < w.N && k < w.Kp) Wt[(size_t)n * w.Kp + k] = tile[x][y + i];
  }
}

// 8 elements per thread with 16-byte accesses (d and out_ld multiples of 8, aligned pointers)
template <typename T>
__global__ __launch_bounds__(256) void relu_mask_vec_kernel(const T *g, const T *level, int64_t M, int d, T *out, float scale) {
  typedef T vec_t __attribute__((ext_vector_type(8)));
  const int64_t idx = ((int64_t)blockIdx.x * 256 + threadIdx.x) * 8;
  if (idx >= M * d) return;
  const T *gp = g + idx, *lp = level + idx;
  T *op = out + idx;
  if constexpr (sizeof(T) == 2) {
    const vec_t x = *reinterpret_cast<const vec_t *>(gp), l = *reinterpret_cast<const vec_t *>(lp);
    vec_t r;
#pragma unroll
    for (int t = 0; t < 8; ++t) r[t] = to_f32(l[t]) > 0.f ? from_f32<T>(to_f32(x[t]) * scale) : from_f32<T>(0.f);
    *reinterpret_cast<vec_t *>(op) = r;
  } else {
    typedef T half_t __attribute__((ext_vector_type(4)));
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const half_t x = *reinterpret_cast<const half_t *>(gp + 4 * h), l = *reinterpret_cast<const half_t *>(lp + 4 * h);
      half_t r;
#pragma unroll
      for (int t = 0; t < 4; ++t) r[t] = to_f32(l[t]) > 0.f ? from_f32<T>(to_f32(x[t]) * scale) : from_f32<T>(0.f);
      *reinterpret_cast<half_t *>(op + 4 * h) = r;
    }
  }
}

// Dropout on rows that a layer has just written: 8 consecutive columns per thread when the row allows it.
template <typename T, int VEC>
__global__ __launch_bounds__(256) void dropout_rows_kernel(T *x, int64_t M, int d, int ld, LnDropout dp) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int per_row = d / VEC;
  if (idx >= M * per_row) return;
  const int64_t r = idx / per_row;
  const int c = (int)(idx % per_row) * VEC;
  typedef T vec_t __attribute__((ext_vector_type(VEC)));
  vec_t *p = reinterpret_cast<vec_t *>(x + r * ld + c);
  vec_t v = *p;
#pragma unroll
  for (int t = 0; t < VEC; ++t) v[t] = dropout_keep(dp, dp.u0 + r, d, c + t) ? from_f32<T>(to_f32(v[t]) * dp.scale) : from_f32<T>(0.f);
  *p = v;
}

template <typename T>
__global__ __launch_bounds__(256) void relu_mask_kernel(const T *g, const T *level, int64_t M, int d, T *out, int out_ld, float scale) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= M * out_ld) return;
  const int64_t m = idx / out_ld;
  const int c = (int)(idx % out_ld);
  float r = 0.f;
  if (c < d && to_f32(level[m * d + c]) > 0.f) r = to_f32(g[m * d + c]) * scale;
  out[idx] = from_f32<T>(r);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// 16-byte copy with a byte tail.  A workgroup walks contiguous segments (256 KB for large buffers, down to 16 KB for
// small ones so that enough workgroups take part; 2,048 workgroups take the segments round-robin), four 16-byte
// words per thread in flight, loads and stores non-temporal: the bytes are not read
// again soon and need not displace anything in the caches.  Measured against other forms on a 5 GB buffer (read +
// written per second): grid-stride over 4,096 workgroups 4.6 - 4.8 TB/s, over 65,536 workgroups 5.3 TB/s, this form
// 5.4 TB/s, a device-to-device hipMemcpyAsync 4.3 TB/s, a read-only pass 5.3 - 5.7 TB/s, a write-only pass 5.1 TB/s.
// Several copies that do not overlap are planes of one launch.
struct CopyPlane {
  const u32x4 *src;
  u32x4 *dst;
  size_t n16, seg;
  int32_t tail;
};
__global__ __launch_bounds__(256) void copy_kernel(const Batch<CopyPlane> ba) {
  const CopyPlane a = ba.sub[blockIdx.y];
  const u32x4 *src = a.src;
  u32x4 *dst = a.dst;
  const size_t n16 = a.n16, seg = a.seg;
  const size_t nseg = (n16 + seg - 1) / seg;
  for (size_t sg = blockIdx.x; sg < nseg; sg += gridDim.x) {
    const size_t b = sg * seg, e = b + seg < n16 ? b + seg : n16;
    size_t i = b + threadIdx.x;
    for (; i + 3 * 256 < e; i += 4 * 256) {
      u32x4 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = __builtin_nontemporal_load(src + i + u * 256);
#pragma unroll
      for (int u = 0; u < 4; ++u) __builtin_nontemporal_store(v[u], dst + i + u * 256);
    }
    for (; i < e; i += 256) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
  }
  if (blockIdx.x == 0 && (int)threadIdx.x < a.tail)
    reinterpret_cast<uint8_t *>(dst + n16)[threadIdx.x] = reinterpret_cast<const uint8_t *>(src + n16)[threadIdx.x];
}

struct FillPlanes {
  struct {
    u32x4 *dst;
    size_t n16;
    int32_t tail;
  } p[kFills];
};
__global__ __launch_bounds__(256) void fill_zero_kernel(const FillPlanes a) {
  u32x4 *dst = a.p[blockIdx.y].dst;
  const size_t n16 = a.p[blockIdx.y].n16;
  const size_t stride = (size_t)gridDim.x * 256;
  const u32x4 z = {0u, 0u, 0u, 0u};
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n16; i += stride) dst[i] = z;
  if (blockIdx.x == 0 && (int)threadIdx.x < a.p[blockIdx.y].tail) reinterpret_cast<uint8_t *>(dst + n16)[threadIdx.x] = 0;
}

// One wave per sparse row: val[e] = 1 / sqrt(len(row) * len(other endpoint)), lengths taken from
// len_ptr (the CSR row pointer of A + I), computed in fp64 and rounded once to fp32.
__global__ __launch_bounds__(256) void gcn_norm_kernel(const int64_t *ptr, const uint32_t *pidx, int vbits,
                                                       const int64_t *len_ptr, int64_t n, float *val) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= n) return;
  const int lane = threadIdx.x & 63;
  const uint32_t vmask = (1u << vbits) - 1u;
  const double dv = (double)(len_ptr[row + 1] - len_ptr[row]);
  for (int64_t e = ptr[row] + lane; e < ptr[row + 1]; e += 64) {
    const int64_t u = pidx[e] & vmask;
    const double du = (double)(len_ptr[u + 1] - len_ptr[u]);
    val[e] = (float)(1.0 / sqrt(dv * du));
  }
}

}  // namespace

int launch_stage_weights(const StageWeightsArgs *w, int n, int dtype, const PassTableArgs *tables, hipStream_t s) {
  for (int i0 = 0; i0 < n || tables != nullptr; i0 += kBatch) {
    StageArgs a{};
    a.n = std::max(0, std::min(kBatch, n - i0));
    unsigned gx = 1;
    for (int i = 0; i < a.n; ++i) {
      a.w[i] = w[i0 + i];
      gx = std::max(gx, (unsigned)((std::max(a.w[i].K, a.w[i].Kp) + 31) / 32 * ((std::max(a.w[i].N, a.w[i].Np) + 31) / 32)));
    }
    const unsigned gy = (unsigned)a.n + (tables != nullptr ? 1u : 0u);
    if (tables != nullptr) a.tables = *tables;
    tables = nullptr;
    hipLaunchKernelGGL(dtype == DT_BF16 ? stage_weights_kernel<bf16_t> : stage_weights_kernel<float>, dim3(gx, gy), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  return hipSuccess;
}

template <typename T, int VEC>
static int dropout_rows(T *x, int64_t M, int d, int ld, const LnDropout &dp, hipStream_t s) {
  return for_row_slabs(M, d / VEC, [&](int64_t r, int64_t m, unsigned gx) {
    LnDropout at = dp;
    at.u0 += r;
    hipLaunchKernelGGL((dropout_rows_kernel<T, VEC>), dim3(gx), dim3(256), 0, s, x + (size_t)r * ld, m, d, ld, at);
  });
}
int launch_dropout_rows(void *x, int dtype, int64_t M, int d, int ld, const LnDropout &dp, hipStream_t s) {
  if (M <= 0 || d <= 0 || dp.threshold == 0) return hipSuccess;
  if (dtype != DT_BF16) return dropout_rows<float, 1>(static_cast<float *>(x), M, d, ld, dp, s);
  const bool vec = d % 8 == 0 && ld % 8 == 0 && (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
  return vec ? dropout_rows<bf16_t, 8>(static_cast<bf16_t *>(x), M, d, ld, dp, s) : dropout_rows<bf16_t, 1>(static_cast<bf16_t *>(x), M, d, ld, dp, s);
}

template <typename T>
static int relu_mask(const T *g, const T *level, int64_t M, int d, T *out, int out_ld, float scale, hipStream_t s) {
  const auto al = [](const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  const bool vec = d % 8 == 0 && out_ld == d && al(g) && al(level) && al(out);
  return for_row_slabs(M, vec ? d / 8 : out_ld, [&](int64_t r, int64_t m, unsigned gx) {
    const T *gr = g + (size_t)r * d, *lr = level + (size_t)r * d;
    T *o = out + (size_t)r * out_ld;
    if (vec)
      hipLaunchKernelGGL(relu_mask_vec_kernel<T>, dim3(gx), dim3(256), 0, s, gr, lr, m, d, o, scale);
    else
      hipLaunchKernelGGL(relu_mask_kernel<T>, dim3(gx), dim3(256), 0, s, gr, lr, m, d, o, out_ld, scale);
  });
}
int launch_relu_mask(const void *g, const void *level, int dtype, int64_t M, int d, void *out, int out_ld, float scale,
                     hipStream_t s) {
  if (dtype == DT_BF16)
    return relu_mask(static_cast<const bf16_t *>(g), static_cast<const bf16_t *>(level), M, d, static_cast<bf16_t *>(out), out_ld, scale, s);
  return relu_mask(static_cast<const float *>(g), static_cast<const float *>(level), M, d, static_cast<float *>(out), out_ld, scale, s);
}

static unsigned stream_grid(size_t n16) {
  size_t blocks = (n16 + 255) / 256;
  if (blocks > 256 * 16) blocks = 256 * 16;  // 16 blocks per CU, grid-stride beyond that
  if (blocks == 0) blocks = 1;
  return (unsigned)blocks;
}

// ---- what the memory system gives a row gather (diagnostic) --------------------------------------------
// Every 16-lane group reads whole rows of row_bytes (16 bytes per lane and step) at pseudo-random row numbers,
// eight rows in flight per group, and folds what it read into one word so that no load can be dropped.  A share
// of the draws goes to the first hot_rows rows (a power-law graph's hubs); the others are uniform over the table.
namespace {
__device__ inline uint32_t mix32(uint32_t x) {
  x ^= x >> 16;
  x *= 0x7feb352du;
  x ^= x >> 15;
  x *= 0x846ca68bu;
  return x ^ (x >> 16);
}

template <int MODE>  // 0: plain loads, 1: non-temporal loads, 2: plain loads, hot rows scattered, 3: non-temporal loads for the cold draws only
__global__ __launch_bounds__(256) void gather_probe_kernel(const u32x4 *table, uint32_t n_rows, int row_vecs, int rows_per_group,
                                                           uint32_t hot_rows, uint32_t hot_threshold, uint32_t seed, uint32_t *sink) {
  const uint32_t group = (blockIdx.x * 256u + threadIdx.x) >> 4;
  const int lig = threadIdx.x & 15;
  u32x4 acc = {0u, 0u, 0u, 0u};
  for (int i = 0; i < rows_per_group; i += 8) {
    u32x4 x[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const uint32_t h = mix32(seed + group * 0x9e3779b9u + (uint32_t)(i + u));
      const uint32_t pick = mix32(h ^ 0x85ebca6bu);
      uint32_t row = (pick < hot_threshold) ? h % hot_rows : h % n_rows;
      if (MODE == 2 && pick < hot_threshold) row *= n_rows / hot_rows;  // the hot rows spread evenly over the table
      const u32x4 *p = table + (size_t)row * row_vecs + lig;
      const bool nt = MODE == 1 || (MODE == 3 && pick >= hot_threshold);
      x[u] = nt ? __builtin_nontemporal_load(p) : p[0];
      for (int v = 16; v < row_vecs; v += 16) {
        const u32x4 y = nt ? __builtin_nontemporal_load(p + v) : p[v];
        x[u] ^= y;
      }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) acc ^= x[u];
  }
  if ((acc[0] ^ acc[1] ^ acc[2] ^ acc[3]) == 0x12345677u) sink[0] = group;  // practically never true; keeps the loads alive
}

}  // namespace

// Times n_launches launches of the probe on `stream` with HIP events and reports bytes gathered per second.
// table: DEVICE, n_rows rows of row_bytes (a multiple of 256, at most 4096); sink: DEVICE, 4 bytes.
extern "C" int gnnstage_debug_gather_rate(const void *table, int64_t n_rows, int32_t row_bytes, int64_t gathers_per_launch,
                                          int32_t n_launches, int64_t hot_rows, double hot_share, int32_t mode, uint32_t seed,
                                          void *sink, void *hip_stream, double *bytes_per_second) {
  if (!table || !sink || !bytes_per_second || n_rows < 1 || n_rows > 0xffffffffll || row_bytes < 256 || row_bytes > 4096 ||
      row_bytes % 256 != 0 || gathers_per_launch < 1 || n_launches < 1 || hot_rows < 0 || hot_rows > n_rows ||
      !(hot_share >= 0.0 && hot_share <= 1.0) || (hot_share > 0.0 && hot_rows < 1) || mode < 0 || mode > 3)
    return -1;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const int blocks = 256 * 8;  // eight workgroups of four waves per compute unit: full occupancy
  const int64_t groups = (int64_t)blocks * 16;
  int64_t per_group = (gathers_per_launch + groups - 1) / groups;
  per_group = (per_group + 7) / 8 * 8;
  if (per_group > (1 << 24)) return -1;
  const uint32_t thr = hot_share >= 1.0 ? 0xffffffffu : (uint32_t)(hot_share * 4294967296.0);
  hipEvent_t a = nullptr, b = nullptr;
  if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) return -5;
  auto launch = [&](uint32_t sd) {
    const u32x4 *t = static_cast<const u32x4 *>(table);
    const uint32_t hr = (uint32_t)std::max<int64_t>(hot_rows, 1);
    uint32_t *sk = static_cast<uint32_t *>(sink);
    if (mode == 3)
      hipLaunchKernelGGL(gather_probe_kernel<3>, dim3(blocks), dim3(256), 0, s, t, (uint32_t)n_rows, row_bytes / 16, (int)per_group, hr, thr, sd, sk);
    else if (mode == 2)
      hipLaunchKernelGGL(gather_probe_kernel<2>, dim3(blocks), dim3(256), 0, s, t, (uint32_t)n_rows, row_bytes / 16, (int)per_group, hr, thr, sd, sk);
    else if (mode == 1)
      hipLaunchKernelGGL(gather_probe_kernel<1>, dim3(blocks), dim3(256), 0, s, t, (uint32_t)n_rows, row_bytes / 16, (int)per_group, hr, thr, sd, sk);
    else
      hipLaunchKernelGGL(gather_probe_kernel<0>, dim3(blocks), dim3(256), 0, s, t, (uint32_t)n_rows, row_bytes / 16, (int)per_group, hr, thr, sd, sk);
  };
  launch(seed);  // warm-up
  (void)hipEventRecord(a, s);
  for (int i = 0; i < n_launches; ++i) launch(seed + 1u + (uint32_t)i);
  (void)hipEventRecord(b, s);
  float ms = 0.f;
  const bool ok = hipEventSynchronize(b) == hipSuccess && hipEventElapsedTime(&ms, a, b) == hipSuccess && hipGetLastError() == hipSuccess;
  (void)hipEventDestroy(a);
  (void)hipEventDestroy(b);
  if (!ok || !(ms > 0.f)) return -5;
  *bytes_per_second = (double)per_group * (double)groups * (double)row_bytes * n_launches / ((double)ms * 1e-3);
  return 0;
}

int launch_copies(const CopyArgs *c, int n, hipStream_t s) {
  for (int i0 = 0; i0 < n; i0 += kBatch) {
    Batch<CopyPlane> b{};
    unsigned grid = 0, m = 0;
    for (int i = i0; i < std::min(n, i0 + kBatch); ++i) {
      if (c[i].bytes == 0) continue;
      const size_t n16 = c[i].bytes / 16;
      // segment length in 16-byte words: a 2,048th of the buffer, in steps of 16 KB, between 16 KB and 256 KB
      size_t seg = ((n16 / 2048 + 1023) / 1024) * 1024;
      seg = seg < 1024 ? 1024 : seg > 16384 ? 16384 : seg;
      const size_t nseg = (n16 + seg - 1) / seg;
      b.sub[m++] = CopyPlane{static_cast<const u32x4 *>(c[i].src), static_cast<u32x4 *>(c[i].dst), n16, seg, (int32_t)(c[i].bytes % 16)};
      grid = std::max(grid, (unsigned)(nseg < 1 ? 1 : nseg > 2048 ? 2048 : nseg));
    }
    if (m == 0) continue;
    hipLaunchKernelGGL(copy_kernel, dim3(grid, m), dim3(256), 0, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  return hipSuccess;
}
int launch_copy(const void *src, void *dst, size_t bytes, hipStream_t s) {
  const CopyArgs c{src, dst, bytes};
  return launch_copies(&c, 1, s);
}

int launch_fills_zero(const FillArgs *f, int n, hipStream_t s) {
  for (int i = 0; i < n;) {
    FillPlanes a{};
    unsigned m = 0, grid = 1;
    for (; i < n && m < (unsigned)kFills; ++i) {
      if (f[i].bytes == 0) continue;
      const size_t n16 = f[i].bytes / 16;
      a.p[m].dst = static_cast<u32x4 *>(f[i].dst);
      a.p[m].n16 = n16;
      a.p[m++].tail = (int32_t)(f[i].bytes % 16);
      grid = std::max(grid, stream_grid(n16));
    }
    if (m == 0) continue;
    hipLaunchKernelGGL(fill_zero_kernel, dim3(grid, m), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  return hipSuccess;
}
int launch_fill_zero(void *dst, size_t bytes, hipStream_t s) {
  const FillArgs f{dst, bytes};
  return launch_fills_zero(&f, 1, s);
}

int launch_gcn_norm(const int64_t *ptr, const uint32_t *pidx, int vbits, const int64_t *len_ptr, int64_t n, float *val,
                    hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(gcn_norm_kernel, dim3((unsigned)((n + 3) / 4)), dim3(256), 0, s, ptr, pidx, vbits, len_ptr, n, val);
  return (int)hipGetLastError();
}
