// Row-wise LayerNorm + ReLU in front of the aggregation (ResGCN+ variant), its backward, and a row copy
// with padding.  One wavefront per vertex row; rows are strided over the launched wavefronts.
//
// LayerNorm over the d features of one vertex: y = gamma * (x - mean) / sqrt(var + eps) + beta with the
// biased variance; the layer's input to the aggregation is r = ReLU(y).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <functional>

#include "common.h"

namespace {

__device__ inline float ld_elt(const void *p, int dtype, size_t i) {
  return dtype == DT_BF16 ? (float)static_cast<const bf16_t *>(p)[i] : static_cast<const float *>(p)[i];
}
__device__ inline void st_elt(void *p, int dtype, size_t i, float v) {
  if (dtype == DT_BF16)
    static_cast<bf16_t *>(p)[i] = (bf16_t)v;
  else
    static_cast<float *>(p)[i] = v;
}

__device__ inline float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// NI = columns per lane (lane, lane + 64, ...): the row lives in registers between the passes
template <int NI>
__global__ __launch_bounds__(256) void ln_relu_kernel(const LnArgs a) {
  const unsigned block = blockIdx.x, blocks = gridDim.x;
  const void *x = a.x;
  void *out = a.out;
  const float *gamma = a.gamma, *beta = a.beta;
  const float eps = a.eps;
  const int64_t M = a.M;
  const int x_dtype = a.x_dtype, x_ld = a.x_ld, d = a.d, out_dtype = a.out_dtype, out_ld = a.out_ld;
  const LnDropout dp = a.drop;
  const int lane = threadIdx.x & 63;
  const int64_t w0 = (int64_t)block * 4 + (threadIdx.x >> 6), nw = (int64_t)blocks * 4;
  for (int64_t r = w0; r < M; r += nw) {
    float v[NI];
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      v[i] = c < d ? ld_elt(x, x_dtype, (size_t)r * x_ld + c) : 0.f;
      sum += v[i];
    }
    const float mean = wave_sum(sum) / (float)d;
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      const float t = c < d ? v[i] - mean : 0.f;
      sq += t * t;
    }
    const float rstd = 1.f / sqrtf(wave_sum(sq) / (float)d + eps);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < out_ld) {
        float y = 0.f;
        if (c < d) {
          y = gamma[c] * ((v[i] - mean) * rstd) + beta[c];
          y = y > 0.f ? y : 0.f;
          if (dp.threshold > 0) y = dropout_keep(dp, dp.u0 + r, d, c) ? y * dp.scale : 0.f;
        }
        st_elt(out, out_dtype, (size_t)r * out_ld + c, y);
      }
    }
  }
}

// dr -> dx (+ res) for the rows of the launch; the column sums of the parameter gradients are added over the
// four wavefronts of a workgroup in LDS and go to partial[workgroup][0][c] (gamma) and partial[workgroup][1][c]
// (beta); ln_param_reduce_kernel adds those in a fixed order.
// LONG: a wavefront adds kLnChain rows in one chain and then to its sums in LDS: over all rows of a layer a wavefront has hundreds (8 M
// rows in 32 chunks: 977), whose one chain was off 64 bits by 5.2e-7 of the root of the sum of squares; in chains of 32 it is 1.8e-7.
// Fewer rows: an instance without that, which a launch over a chunk of some ten thousand rows would pay 0.3 - 0.4 us for.
constexpr int kLnChain = 32;
template <typename T, int NI, bool LONG>
__global__ __launch_bounds__(256) void ln_relu_backward_kernel(const Batch<LnBackArgs> ba) {
  const LnBackArgs b = ba.sub[blockIdx.z];
  const LnArgs &a = b.f;
  const unsigned block = blockIdx.x, blocks = b.blocks;
  if (block >= blocks) return;
  const T *x = static_cast<const T *>(a.x), *dr = static_cast<const T *>(b.dr), *res = static_cast<const T *>(b.res);
  T *out = static_cast<T *>(a.out);
  const float *gamma = a.gamma, *beta = a.beta;
  float *partial = b.partial;
  const float eps = a.eps;
  const int64_t M = a.M;
  const int x_ld = a.x_ld, d = a.d, out_ld = a.out_ld, dr_ld = b.dr_ld, res_ld = b.res_ld;
  const LnDropout dp = a.drop;
  __shared__ float red[4][2][NI * 64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int64_t w0 = (int64_t)block * 4 + (threadIdx.x >> 6), nw = (int64_t)blocks * 4;
  float dg[NI], db[NI], gam[NI], bet[NI];
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    const int c = lane + 64 * i;
    dg[i] = db[i] = 0.f;
    gam[i] = c < d ? gamma[c] : 0.f;
    bet[i] = c < d ? beta[c] : 0.f;
  }
  const int64_t gap_row = b.gap_row, gap_end = b.gap_end;
  int chain = 0;
  bool waiting = false;  // earlier chains' sums wait in LDS
  for (int64_t r = w0; r < M; r += nw) {
    if (r >= gap_row && r < gap_end) continue;
    if (LONG && chain == kLnChain) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        float *g = &red[wave][0][lane + 64 * i], *b = &red[wave][1][lane + 64 * i];
        *g = waiting ? *g + dg[i] : dg[i];
        *b = waiting ? *b + db[i] : db[i];
        dg[i] = db[i] = 0.f;
      }
      waiting = true;
      chain = 0;
    }
    ++chain;
    float xh[NI], dxh[NI];
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      xh[i] = c < d ? (float)x[(size_t)r * x_ld + c] : 0.f;
      sum += xh[i];
    }
    const float mean = wave_sum(sum) / (float)d;
    float sq = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      xh[i] = c < d ? xh[i] - mean : 0.f;
      sq += xh[i] * xh[i];
    }
    const float rstd = 1.f / sqrtf(wave_sum(sq) / (float)d + eps);
    float m1 = 0.f, m2 = 0.f;
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      xh[i] *= rstd;
      float dn = 0.f;
      if (c < d) {
        const float y = gam[i] * xh[i] + bet[i];
        dn = y > 0.f ? (float)dr[(size_t)r * dr_ld + c] : 0.f;  // ReLU derivative, strict
        if (dp.threshold > 0) dn = dropout_keep(dp, dp.u0 + r, d, c) ? dn * dp.scale : 0.f;
      }
      dg[i] += dn * xh[i];
      db[i] += dn;
      dxh[i] = dn * gam[i];
      m1 += dxh[i];
      m2 += dxh[i] * xh[i];
    }
    m1 = wave_sum(m1) / (float)d;
    m2 = wave_sum(m2) / (float)d;
    if (out != nullptr) {
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        const int c = lane + 64 * i;
        if (c < out_ld) {
          float v = 0.f;
          if (c < d) {
            v = rstd * (dxh[i] - m1 - xh[i] * m2);
            if (res != nullptr) v += (float)res[(size_t)r * res_ld + c];
          }
          out[(size_t)r * out_ld + c] = (T)v;
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    float *g = &red[wave][0][lane + 64 * i], *b = &red[wave][1][lane + 64 * i];
    if (LONG && waiting) {
      dg[i] += *g;
      db[i] += *b;
    }
    if (wave > 0) {
      *g = dg[i];
      *b = db[i];
    }
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int c = lane + 64 * i;
      if (c < d) {
        partial[((size_t)block * 2 + 0) * d + c] = ((dg[i] + red[1][0][c]) + red[2][0][c]) + red[3][0][c];
        partial[((size_t)block * 2 + 1) * d + c] = ((db[i] + red[1][1][c]) + red[2][1][c]) + red[3][1][c];
      }
    }
  }
}

// ---- bf16 rows whose width is 8 x a power of two: LPR lanes per row, 16 bytes per lane, 64 / LPR rows per
// wavefront at a time (the same arithmetic as above, with the loads and stores vectorised)
typedef bf16_t bf16x8_ln __attribute__((ext_vector_type(8)));

template <int LPR>
__device__ inline float group_sum(float v) {
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

template <int LPR>
__global__ __launch_bounds__(256) void ln_relu_vec_kernel(const LnArgs a) {
  const unsigned block = blockIdx.x, blocks = gridDim.x;
  const bf16_t *x = static_cast<const bf16_t *>(a.x);
  bf16_t *out = static_cast<bf16_t *>(a.out);
  const float *gamma = a.gamma, *beta = a.beta;
  const float eps = a.eps;
  const int64_t M = a.M;
  const int x_ld = a.x_ld, out_ld = a.out_ld;
  const LnDropout dp = a.drop;
  constexpr int RPW = 64 / LPR, d = LPR * 8;
  const int lane = threadIdx.x & 63, sub = lane % LPR, rw = lane / LPR;
  const int64_t w0 = (int64_t)block * 4 + (threadIdx.x >> 6), nw = (int64_t)blocks * 4;
  float gam[8], bet[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    gam[t] = gamma[sub * 8 + t];
    bet[t] = beta[sub * 8 + t];
  }
  for (int64_t r0 = w0 * RPW; r0 < M; r0 += nw * RPW) {
    const int64_t r = r0 + rw;
    const bool on = r < M;
    const int64_t rr = on ? r : M - 1;  // lanes past the end repeat the last row and do not store
    const bf16x8_ln xv = *reinterpret_cast<const bf16x8_ln *>(x + (size_t)rr * x_ld + sub * 8);
    float v[8], sum = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      v[t] = (float)xv[t];
      sum += v[t];
    }
    const float mean = group_sum<LPR>(sum) / (float)d;
    float sq = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) sq += (v[t] - mean) * (v[t] - mean);
    const float rstd = 1.f / sqrtf(group_sum<LPR>(sq) / (float)d + eps);
    bf16x8_ln o;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      float y = gam[t] * ((v[t] - mean) * rstd) + bet[t];
      y = y > 0.f ? y : 0.f;
      if (dp.threshold > 0) y = dropout_keep(dp, dp.u0 + rr, d, sub * 8 + t) ? y * dp.scale : 0.f;
      o[t] = (bf16_t)y;
    }
    if (on) *reinterpret_cast<bf16x8_ln *>(out + (size_t)r * out_ld + sub * 8) = o;
  }
}

template <int LPR, bool LONG>
__global__ __launch_bounds__(256) void ln_relu_backward_vec_kernel(const Batch<LnBackArgs> ba) {
  const LnBackArgs b = ba.sub[blockIdx.z];
  const LnArgs &a = b.f;
  const unsigned block = blockIdx.x, blocks = b.blocks;
  if (block >= blocks) return;
  const bf16_t *x = static_cast<const bf16_t *>(a.x), *dr = static_cast<const bf16_t *>(b.dr), *res = static_cast<const bf16_t *>(b.res);
  bf16_t *out = static_cast<bf16_t *>(a.out);
  const float *gamma = a.gamma, *beta = a.beta;
  float *partial = b.partial;
  const float eps = a.eps;
  const int64_t M = a.M;
  const int x_ld = a.x_ld, out_ld = a.out_ld, dr_ld = b.dr_ld, res_ld = b.res_ld;
  const LnDropout dp = a.drop;
  constexpr int RPW = 64 / LPR, d = LPR * 8;
  __shared__ float red[4][2][LONG ? RPW : 1][LPR * 8];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, sub = lane % LPR, rw = lane / LPR;
  const int64_t w0 = (int64_t)block * 4 + (threadIdx.x >> 6), nw = (int64_t)blocks * 4;
  float gam[8], bet[8], dg[8], db[8];
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    gam[t] = gamma[sub * 8 + t];
    bet[t] = beta[sub * 8 + t];
    dg[t] = db[t] = 0.f;
  }
  const int64_t gap_row = b.gap_row, gap_end = b.gap_end;
  int chain = 0;
  bool waiting = false;
  for (int64_t r0 = w0 * RPW; r0 < M; r0 += nw * RPW) {
    if (LONG && chain == kLnChain) {
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        float *g = &red[wave][0][rw][sub * 8 + t], *b = &red[wave][1][rw][sub * 8 + t];
        *g = waiting ? *g + dg[t] : dg[t];
        *b = waiting ? *b + db[t] : db[t];
        dg[t] = db[t] = 0.f;
      }
      waiting = true;
      chain = 0;
    }
    ++chain;
    const int64_t r = r0 + rw;
    const bool on = r < M && (r < gap_row || r >= gap_end);
    const int64_t rr = on ? r : 0;
    const bf16x8_ln xv = *reinterpret_cast<const bf16x8_ln *>(x + (size_t)rr * x_ld + sub * 8);
    const bf16x8_ln dv = *reinterpret_cast<const bf16x8_ln *>(dr + (size_t)rr * dr_ld + sub * 8);
    bf16x8_ln rv;
    if (res != nullptr) rv = *reinterpret_cast<const bf16x8_ln *>(res + (size_t)rr * res_ld + sub * 8);
    float xh[8], dxh[8], sum = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      xh[t] = (float)xv[t];
      sum += xh[t];
    }
    const float mean = group_sum<LPR>(sum) / (float)d;
    float sq = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      xh[t] -= mean;
      sq += xh[t] * xh[t];
    }
    const float rstd = 1.f / sqrtf(group_sum<LPR>(sq) / (float)d + eps);
    float m1 = 0.f, m2 = 0.f;
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      xh[t] *= rstd;
      const float y = gam[t] * xh[t] + bet[t];
      float dn = (on && y > 0.f) ? (float)dv[t] : 0.f;  // ReLU derivative, strict; repeated rows add nothing
      if (dp.threshold > 0) dn = dropout_keep(dp, dp.u0 + rr, d, sub * 8 + t) ? dn * dp.scale : 0.f;
      dg[t] += dn * xh[t];
      db[t] += dn;
      dxh[t] = dn * gam[t];
      m1 += dxh[t];
      m2 += dxh[t] * xh[t];
    }
    m1 = group_sum<LPR>(m1) / (float)d;
    m2 = group_sum<LPR>(m2) / (float)d;
    if (out != nullptr && on) {
      bf16x8_ln o;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        float v = rstd * (dxh[t] - m1 - xh[t] * m2);
        if (res != nullptr) v += (float)rv[t];
        o[t] = (bf16_t)v;
      }
      *reinterpret_cast<bf16x8_ln *>(out + (size_t)r * out_ld + sub * 8) = o;
    }
  }
  // column sums: over the row groups of the wavefront (fixed order), then over the four wavefronts in LDS
#pragma unroll
  for (int t = 0; t < 8; ++t) {
    if (LONG && waiting) {
      dg[t] += red[wave][0][rw][sub * 8 + t];
      db[t] += red[wave][1][rw][sub * 8 + t];
    }
#pragma unroll
    for (int o = LPR; o < 64; o <<= 1) {
      dg[t] += __shfl_xor(dg[t], o);
      db[t] += __shfl_xor(db[t], o);
    }
  }
  if (wave > 0 && rw == 0) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      red[wave][0][0][sub * 8 + t] = dg[t];
      red[wave][1][0][sub * 8 + t] = db[t];
    }
  }
  __syncthreads();
  if (wave == 0 && rw == 0) {
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const int c = sub * 8 + t;
      partial[((size_t)block * 2 + 0) * d + c] = ((dg[t] + red[1][0][0][c]) + red[2][0][0][c]) + red[3][0][0][c];
      partial[((size_t)block * 2 + 1) * d + c] = ((db[t] + red[1][1][0][c]) + red[2][1][0][c]) + red[3][1][0][c];
    }
  }
}

// widths served by the vectorised kernels: 64, 128, 256, 512 bf16 columns, 16-byte aligned rows
inline int vec_lanes(int d, int dtype, const void *p, int ld) {
  if (dtype != DT_BF16 || ld % 8 != 0 || (reinterpret_cast<uintptr_t>(p) & 15u)) return 0;
  return (d == 64 || d == 128 || d == 256 || d == 512) ? d / 8 : 0;
}

// One workgroup per 64 entries of the 2 x d sums: 16 wavefronts each add every 16th partial row, then the 16
// slice sums are added in order.  n_parts: the partial rows of a sub-launch are its workgroups in the launch before.
__global__ __launch_bounds__(1024) void ln_param_reduce_kernel(const Batch<LnReduceArgs> ba) {
  const LnReduceArgs &a = ba.sub[blockIdx.z];
  const unsigned block = blockIdx.x;
  const float *partial = a.partial;
  float *dgamma = a.dgamma, *dbeta = a.dbeta;
  const int n_parts = a.n_parts, d = a.d;
  __shared__ float red[16][64];
  const int lane = threadIdx.x & 63, slice = threadIdx.x >> 6;
  const int idx = block * 64 + lane;  // position in [gamma sums | beta sums]
  float s = 0.f;
  if (idx < 2 * d) {
#pragma unroll 8
    for (int w = slice; w < n_parts; w += 16) s += partial[(size_t)w * 2 * d + idx];
  }
  red[slice][lane] = s;
  __syncthreads();
  if (slice == 0 && idx < 2 * d) {
    float t = red[0][lane];
#pragma unroll
    for (int q = 1; q < 16; ++q) t += red[q][lane];
    float *dst = idx < d ? dgamma + idx : dbeta + (idx - d);
    *dst += t;
  }
}

__global__ __launch_bounds__(256) void copy_rows_kernel(const void *src, int src_ld, void *dst, int dst_ld, int64_t M, int d, int dtype) {
  const int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (idx >= M * dst_ld) return;
  const int64_t r = idx / dst_ld;
  const int c = (int)(idx % dst_ld);
  st_elt(dst, dtype, (size_t)idx, c < d ? ld_elt(src, dtype, (size_t)r * src_ld + c) : 0.f);
}

int waves_for(int64_t M, int max_waves) {
  int64_t w = (M + 3) / 4 * 4;  // whole workgroups
  if (w > max_waves) w = max_waves / 4 * 4;
  if (w < 4) w = 4;
  return (int)w;
}

}  // namespace

static void set_blocks(LnBackArgs &a, unsigned g) { a.blocks = (int32_t)g; }
static void set_blocks(LnReduceArgs &, unsigned) {}
// Runs sub-launches [0, n) (kernel fn[i], gx[i] workgroups; 0: nothing to do), those of one kernel together.
template <typename A, typename Fn>
static int launch_merged(const A *const *a, const Fn *fn, const unsigned *gx, int n, unsigned threads, hipStream_t s) {
  bool done[kBatch] = {};
  for (int i = 0; i < n; ++i) {
    if (done[i] || gx[i] == 0) continue;
    Batch<A> b;
    unsigned m = 0, width = 0;
    for (int j = i; j < n; ++j) {
      if (done[j] || gx[j] == 0 || fn[j] != fn[i]) continue;
      done[j] = true;
      b.sub[m] = *a[j];
      set_blocks(b.sub[m++], gx[j]);
      width = std::max(width, gx[j]);
    }
    hipLaunchKernelGGL(fn[i], dim3(width, 1, m), dim3(threads), 0, s, b);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return (int)e;
  }
  return hipSuccess;
}

// whether two parameter reduces have elements of their destinations in common
static bool adds_to_the_same(const LnReduceArgs &a, const LnReduceArgs &b) {
  const float *da[2] = {a.dgamma, a.dbeta}, *db[2] = {b.dgamma, b.dbeta};
  for (const float *x : da)
    for (const float *y : db)
      if (std::less<const float *>()(x, y + b.d) && std::less<const float *>()(y, x + a.d)) return true;
  return false;
}

int launch_ln_relu(const LnArgs &a, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.d > kLnMaxWidth || a.out_ld > kLnMaxWidth) return hipErrorInvalidValue;
  void (*fn)(const LnArgs);
  unsigned gx;
  const int lpr = (a.out_dtype == DT_BF16 && a.out_ld == a.d && vec_lanes(a.d, a.out_dtype, a.out, a.out_ld)) ? vec_lanes(a.d, a.x_dtype, a.x, a.x_ld) : 0;
  if (lpr) {
    const int rpw = 64 / lpr;
    gx = (unsigned)(waves_for((a.M + rpw - 1) / rpw, 16384) / 4);
    fn = lpr == 8 ? ln_relu_vec_kernel<8> : lpr == 16 ? ln_relu_vec_kernel<16> : lpr == 32 ? ln_relu_vec_kernel<32> : ln_relu_vec_kernel<64>;
  } else {
    const int ni = (std::max(a.d, a.out_ld) + 63) / 64;
    gx = (unsigned)(waves_for(a.M, 16384) / 4);
    fn = ni <= 1 ? ln_relu_kernel<1> : ni <= 2 ? ln_relu_kernel<2> : ni <= 4 ? ln_relu_kernel<4> : ni <= 8 ? ln_relu_kernel<8> : ln_relu_kernel<16>;
  }
  hipLaunchKernelGGL(fn, dim3(gx), dim3(256), 0, s, a);
  return (int)hipGetLastError();
}

int launch_ln_relu_backward(const LnBackArgs *l, int n, int max_waves, LnReduceArgs *red, hipStream_t s) {
  if (n > kBatch) return hipErrorInvalidValue;
  typedef void (*fn_t)(const Batch<LnBackArgs>);
  const LnBackArgs *ptr[kBatch];
  fn_t fn[kBatch];
  unsigned gx[kBatch];
  for (int i = 0; i < n; ++i) {
    const LnBackArgs &b = l[i];
    const LnArgs &a = b.f;
    ptr[i] = &b;
    fn[i] = nullptr;
    gx[i] = 0;
    red[i] = LnReduceArgs{};
    if (a.M <= 0) continue;
    if (a.d > kLnMaxWidth || (a.out && a.out_ld > kLnMaxWidth)) return hipErrorInvalidValue;
    int lpr = vec_lanes(a.d, a.x_dtype, a.x, a.x_ld);
    if (lpr && (!vec_lanes(a.d, b.dr_dtype, b.dr, b.dr_ld) || (b.res && !vec_lanes(a.d, b.res_dtype, b.res, b.res_ld)) ||
                (a.out && !vec_lanes(a.d, a.out_dtype, a.out, a.out_ld))))
      lpr = 0;
    if (lpr) {
      const int rpw = 64 / lpr;
      gx[i] = (unsigned)(waves_for((a.M + rpw - 1) / rpw, max_waves) / 4);
      const bool more = a.M > (int64_t)gx[i] * 4 * rpw * kLnChain;
#define LN_VEC(L) (more ? ln_relu_backward_vec_kernel<L, true> : ln_relu_backward_vec_kernel<L, false>)
      fn[i] = lpr == 8 ? LN_VEC(8) : lpr == 16 ? LN_VEC(16) : lpr == 32 ? LN_VEC(32) : LN_VEC(64);
#undef LN_VEC
    } else {
      const int ni = (std::max(a.d, a.out ? a.out_ld : a.d) + 63) / 64;
      gx[i] = (unsigned)(waves_for(a.M, max_waves) / 4);
      const bool more = a.M > (int64_t)gx[i] * 4 * kLnChain;
      if (b.dr_dtype != a.x_dtype || (b.res && b.res_dtype != a.x_dtype) || (a.out && a.out_dtype != a.x_dtype)) return hipErrorInvalidValue;
#define LN_ROW(T, N) (more ? ln_relu_backward_kernel<T, N, true> : ln_relu_backward_kernel<T, N, false>)
#define LN_ROWS(T) (ni <= 1 ? LN_ROW(T, 1) : ni <= 2 ? LN_ROW(T, 2) : ni <= 4 ? LN_ROW(T, 4) : ni <= 8 ? LN_ROW(T, 8) : LN_ROW(T, 16))
      fn[i] = a.x_dtype == DT_BF16 ? LN_ROWS(bf16_t) : LN_ROWS(float);
#undef LN_ROWS
#undef LN_ROW
    }
    red[i] = LnReduceArgs{b.partial, (int32_t)gx[i], a.d, b.dgamma, b.dbeta};
  }
  return launch_merged(ptr, fn, gx, n, 256, s);
}

// The sums are added to the parameter gradients without atomics.  Layers may share those buffers (tied parameters), and the
// groups of a layer's rows do, so a launch takes the sums up to the first that would add to a buffer again; that one starts
// the next launch.
int launch_ln_param_reduce(const LnReduceArgs *red, int n, hipStream_t s) {
  for (int i0 = 0, i1; i0 < n; i0 = i1) {
    const LnReduceArgs *ptr[kBatch];
    void (*fn[kBatch])(const Batch<LnReduceArgs>);
    unsigned gx[kBatch];
    for (i1 = i0; i1 < n && i1 - i0 < kBatch; ++i1) {
      bool again = false;
      for (int i = i0; i < i1; ++i) again = again || adds_to_the_same(red[i], red[i1]);
      if (again) break;
      ptr[i1 - i0] = &red[i1];
      fn[i1 - i0] = ln_param_reduce_kernel;
      gx[i1 - i0] = red[i1].n_parts > 0 ? (unsigned)((2 * red[i1].d + 63) / 64) : 0;
    }
    const int e = launch_merged(ptr, fn, gx, i1 - i0, 1024, s);
    if (e != 0) return e;
  }
  return hipSuccess;
}

int launch_copy_rows(const void *src, int src_ld, void *dst, int dst_ld, int64_t M, int d, int dtype, hipStream_t s) {
  const size_t elt = dtype == DT_BF16 ? 2 : 4;
  return for_row_slabs(M, dst_ld, [&](int64_t r, int64_t m, unsigned gx) {
    hipLaunchKernelGGL(copy_rows_kernel, dim3(gx), dim3(256), 0, s, static_cast<const char *>(src) + (size_t)r * src_ld * elt, src_ld,
                       static_cast<char *>(dst) + (size_t)r * dst_ld * elt, dst_ld, m, d, dtype);
  });
}
