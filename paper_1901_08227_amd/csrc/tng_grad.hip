// Local-gradient kernels of libtng (Algorithm 1: "each server calculates local gradient"), gfx950.
//
// Logistic regression is two matrix-vector products per worker (z = X_B w, g = X_B^T r) with a
// different X_B per worker and a single vector on the other side, so there is no dense
// matrix-matrix contraction to put on the matrix cores: both passes stream the minibatch rows
// with coalesced 16-byte loads and are bound by HBM bandwidth.  Gradients are compared with a
// tolerance, so these kernels use fused multiply-adds explicitly; the Rosenbrock gradient keeps a
// fixed expression tree without them and is reproducible bit for bit.
#include "tng_device.hpp"
#include "tng_kernels.hpp"

#include <mutex>

namespace tng {

namespace {

constexpr int kWavesPerBlock = kBlock / kWave;

// Background: index "uniformly sampled" -- idx = (draw * n_rows) >> 32, draws from stream 1.
__device__ __forceinline__ uint32_t minibatch_row(uint32_t k0, uint32_t k1, uint32_t iter, uint32_t m, uint32_t j,
                                                  uint64_t n_rows) {
  const U32x4 r = philox4x32_10(j >> 2, m, iter, 1u, k0, k1);
  const uint32_t lane = j & 3u;
  const uint32_t x = lane == 0 ? r.x : lane == 1 ? r.y : lane == 2 ? r.z : r.w;
  return (uint32_t)(((uint64_t)x * n_rows) >> 32);
}

__global__ __launch_bounds__(kBlock) void minibatch_indices_kernel(uint32_t k0, uint32_t k1, uint32_t iter,
                                                                   uint32_t batch,
                                                                   const uint64_t* __restrict__ n_rows,
                                                                   uint32_t* __restrict__ idx) {
  const uint32_t m = blockIdx.y;
  const uint32_t j = blockIdx.x * kBlock + threadIdx.x;
  if (j >= batch) return;
  idx[(uint64_t)m * batch + j] = minibatch_row(k0, k1, iter, m, j, n_rows[m]);
}

__device__ __forceinline__ float block_sum(float v, float* red) {
  v = wave_sum(v);
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  if (lane == 0) red[wave] = v;
  __syncthreads();
  float s = red[0];
#pragma unroll
  for (int k = 1; k < kWavesPerBlock; ++k) s += red[k];
  return s;
}

// Maximum of non-negative values over the workgroup (any size up to 1024 threads); valid in thread 0.  red: 16 floats of LDS.
__device__ __forceinline__ float block_max(float v, float* red) {
  v = wave_max_nonneg(v);
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  __syncthreads();  // red may still be read from an earlier call
  if (lane == 0) red[wave] = v;
  __syncthreads();
  const int nw = (blockDim.x + kWave - 1) / kWave;
  float r = red[0];
  for (int k = 1; k < nw; ++k) r = fmaxf(r, red[k]);
  return r;
}

// Largest |normalize(g)| over the four components of a float4 of gradient values (fused scale pass).
__device__ __forceinline__ float absmax4(const ScaleFusion& f, const float4& g, const float4& r1, const float4& r2) {
  return fmaxf(fmaxf(fabsf(normalize_dyn(f.norm, g.x, r1.x, r2.x, f.eps)), fabsf(normalize_dyn(f.norm, g.y, r1.y, r2.y, f.eps))),
               fmaxf(fabsf(normalize_dyn(f.norm, g.z, r1.z, r2.z, f.eps)), fabsf(normalize_dyn(f.norm, g.w, r1.w, r2.w, f.eps))));
}

// References of elements e0 .. e0 + 3 (any 4-byte alignment).
__device__ __forceinline__ void load_refs4(const ScaleFusion& f, uint64_t e0, float4& r1, float4& r2) {
  r1 = make_float4(0.f, 0.f, 0.f, 0.f);
  r2 = make_float4(1.f, 1.f, 1.f, 1.f);
  if (f.norm != kNormNone) r1 = load4_at(f.gref, e0);
  if (f.norm == kNormComb) r2 = load4_at(f.gref2, e0);
}

// A thread owns the four columns 4 q .. 4 q + 3 of a row of d >= 4; the last thread of a row whose length is no
// multiple of 4 takes the last four instead and repeats up to three columns of its neighbour's, with the same
// operations and so the same results.  (The last d mod 4 columns had launches of their own: 14 us for three columns
// at a minibatch of 128, one dependent load per row.)
__device__ __forceinline__ uint64_t first_column(uint64_t q, uint64_t d) { return 4 * q + 4 <= d ? 4 * q : d - 4; }

// The same two helpers with the kind of normalisation known at compile time: no branch around the loads,
// so the compiler can count them (see the pipelined CSR gradient kernel).
template <int NORM>
__device__ __forceinline__ void load_refs4_t(const ScaleFusion& f, uint64_t q, float4& r1, float4& r2) {
  r1 = make_float4(0.f, 0.f, 0.f, 0.f);
  r2 = make_float4(1.f, 1.f, 1.f, 1.f);
  if (NORM != kNormNone) r1 = reinterpret_cast<const float4*>(f.gref)[q];
  if (NORM == kNormComb) r2 = reinterpret_cast<const float4*>(f.gref2)[q];
}

// The same of elements e0 .. e0 + 3 of d; past the end such that a gradient of 0 normalises to 0.
template <int NORM>
__device__ __forceinline__ void load_refs4_end(const ScaleFusion& f, uint64_t e0, uint64_t d, float4& r1, float4& r2) {
  r1 = make_float4(0.f, 0.f, 0.f, 0.f);
  r2 = make_float4(1.f, 1.f, 1.f, 1.f);
  if (NORM != kNormNone) r1 = load4_within(f.gref, e0, d, NORM == kNormQuot ? 1.f : 0.f);
  if (NORM == kNormComb) r2 = load4_within(f.gref2, e0, d, 1.f);
}

template <int NORM>
__device__ __forceinline__ float absmax4_t(const ScaleFusion& f, const float4& g, const float4& r1, const float4& r2) {
  return fmaxf(fmaxf(fabsf(normalize_dyn(NORM, g.x, r1.x, r2.x, f.eps)), fabsf(normalize_dyn(NORM, g.y, r1.y, r2.y, f.eps))),
               fmaxf(fabsf(normalize_dyn(NORM, g.z, r1.z, r2.z, f.eps)), fabsf(normalize_dyn(NORM, g.w, r1.w, r2.w, f.eps))));
}

// sigma(z) - y without cancellation for the labels 0 and 1.
__device__ __forceinline__ float logistic_residual(float z, float y) {
  const float e = expf(-fabsf(z));           // in (0, 1]
  const float small = e / (1.0f + e);          // sigma(-|z|)
  const float big = 1.0f / (1.0f + e);         // sigma(|z|)
  const float sig = z >= 0.f ? big : small;
  if (y == 1.0f) return z >= 0.f ? -small : -big;  // sigma(z) - 1 = -sigma(-z)
  if (y == 0.0f) return sig;
  return sig - y;
}

// z_i = x_i . w and r_i = sigma(z_i) - y_i for ROWS minibatch rows per workgroup (w is fetched once
// for all of them; each row keeps the accumulation order it has with ROWS = 1).
template <bool VEC, int ROWS>
__global__ __launch_bounds__(kBlock) void logreg_dense_resid_kernel(const float* const* __restrict__ Xs,
                                                                    const float* const* __restrict__ ys,
                                                                    const uint64_t* __restrict__ n_rows,
                                                                    uint32_t* __restrict__ idx,
                                                                    const float* __restrict__ w,
                                                                    float* __restrict__ resid, uint64_t d,
                                                                    uint32_t batch, uint32_t k0, uint32_t k1,
                                                                    uint32_t iter) {
  __shared__ float red[kWavesPerBlock];
  const uint32_t m = blockIdx.y, i0 = blockIdx.x * ROWS;
  // the row ids are drawn here (one launch fewer) and left in idx for the accumulation pass
  uint32_t row[ROWS];
  GlobalPtr<float> x[ROWS];
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    row[r] = minibatch_row(k0, k1, iter, m, min(i0 + r, batch - 1), n_rows[m]);  // a short last group repeats its last row
    if (threadIdx.x == 0 && i0 + r < batch) idx[(uint64_t)m * batch + i0 + r] = row[r];
    x[r] = as_global(Xs[m]) + (uint64_t)row[r] * d;
  }
  float acc[ROWS];
  if (VEC) {
    const float4* w4 = reinterpret_cast<const float4*>(w);
    const uint64_t nvec = d / 4;
    float a0[ROWS], a1[ROWS], a2[ROWS], a3[ROWS];
#pragma unroll
    for (int r = 0; r < ROWS; ++r) a0[r] = a1[r] = a2[r] = a3[r] = 0.f;
#pragma unroll 8 / ROWS
    for (uint64_t k = threadIdx.x; k < nvec; k += kBlock) {
      const float4 wv = w4[k];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) {
        const float4 xv = load4_stream_any(x[r], k);
        a0[r] = __builtin_fmaf(xv.x, wv.x, a0[r]);
        a1[r] = __builtin_fmaf(xv.y, wv.y, a1[r]);
        a2[r] = __builtin_fmaf(xv.z, wv.z, a2[r]);
        a3[r] = __builtin_fmaf(xv.w, wv.w, a3[r]);
      }
    }
    if (4 * nvec + threadIdx.x < d) {  // the last d mod 4 columns
      const uint64_t k = 4 * nvec + threadIdx.x;
      const float wk = w[k];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) a0[r] = __builtin_fmaf(x[r][k], wk, a0[r]);
    }
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = (a0[r] + a1[r]) + (a2[r] + a3[r]);
  } else {
#pragma unroll
    for (int r = 0; r < ROWS; ++r) acc[r] = 0.f;
    for (uint64_t k = threadIdx.x; k < d; k += kBlock) {
      const float wk = w[k];
#pragma unroll
      for (int r = 0; r < ROWS; ++r) acc[r] = __builtin_fmaf(x[r][k], wk, acc[r]);
    }
  }
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    if (r > 0) __syncthreads();  // red is reused
    const float z = block_sum(acc[r], red);
    if (threadIdx.x == 0 && i0 + r < batch)
      resid[(uint64_t)m * batch + i0 + r] = logistic_residual(z, as_global(ys[m])[row[r]]);
  }
}

// g_m[k] = (1/B) sum_i r_i X[idx_i][k] + l2 w[k]; a thread owns 4 (VEC) or 1 columns.
template <bool VEC, bool FUSE>
__global__ __launch_bounds__(kBlock) void logreg_dense_grad_kernel(const float* const* __restrict__ Xs,
                                                                   const uint32_t* __restrict__ idx,
                                                                   const float* __restrict__ resid,
                                                                   const float* __restrict__ w,
                                                                   float* __restrict__ g, uint64_t d,
                                                                   uint32_t batch, float inv_b, float l2,
                                                                   ScaleFusion fuse) {
  __shared__ float sR[kBlock];
  __shared__ uint32_t sRow[kBlock];
  __shared__ float red[16];
  const uint32_t m = blockIdx.y;
  const GlobalPtr<float> X = as_global(Xs[m]);
  const uint64_t index = (uint64_t)blockIdx.x * kBlock + threadIdx.x;  // float4 (VEC) or float index
  const bool active = index < (VEC ? (d + 3) / 4 : d);
  const uint64_t col = VEC ? first_column(index, d) : index;
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (uint32_t base = 0; base < batch; base += kBlock) {
    __syncthreads();
    if (base + threadIdx.x < batch) {
      sR[threadIdx.x] = resid[(uint64_t)m * batch + base + threadIdx.x];
      sRow[threadIdx.x] = idx[(uint64_t)m * batch + base + threadIdx.x];
    }
    __syncthreads();
    if (active) {
      const uint32_t cnt = min((uint32_t)kBlock, batch - base);
      if (VEC) {
#pragma unroll 8
        for (uint32_t i = 0; i < cnt; ++i) {
          const float4 xv = load4_stream_any(X + (uint64_t)sRow[i] * d + col, 0);
          const float r = sR[i];
          acc.x = __builtin_fmaf(r, xv.x, acc.x);
          acc.y = __builtin_fmaf(r, xv.y, acc.y);
          acc.z = __builtin_fmaf(r, xv.z, acc.z);
          acc.w = __builtin_fmaf(r, xv.w, acc.w);
        }
      } else {
#pragma unroll 8
        for (uint32_t i = 0; i < cnt; ++i) acc.x = __builtin_fmaf(sR[i], X[(uint64_t)sRow[i] * d + col], acc.x);
      }
    }
  }
  float amax = 0.f;
  if (active) {
    if (VEC) {
      const float4 wv = load4_at(w, col);
      float4 o;
      o.x = __builtin_fmaf(l2, wv.x, acc.x * inv_b);
      o.y = __builtin_fmaf(l2, wv.y, acc.y * inv_b);
      o.z = __builtin_fmaf(l2, wv.z, acc.z * inv_b);
      o.w = __builtin_fmaf(l2, wv.w, acc.w * inv_b);
      store4_any(g + (uint64_t)m * d + col, 0, o);
      if (FUSE) {
        float4 r1, r2;
        load_refs4(fuse, col, r1, r2);
        amax = absmax4(fuse, o, r1, r2);
      }
    } else {
      g[(uint64_t)m * d + col] = __builtin_fmaf(l2, w[col], acc.x * inv_b);
    }
  }
  if (FUSE) {
    amax = block_max(amax, red);
    if (threadIdx.x == 0) fuse.partials[(uint64_t)blockIdx.x * gridDim.y + m] = amax;
  }
}

// The same for problems with few columns: 1024 threads, COLS float4
// columns times RG row groups; the minibatch rows are dealt round-robin to the row groups, which run
// side by side, and their partial sums are added in the fixed order ((p0 + p1) + p2) + ...  Cuts the
// chain of dependent row fetches to 1/RG; narrow column blocks (32 x 32) also spread a tiny problem
// over eight times as many compute units, each of which can only pull so many bytes per microsecond.
constexpr int kSplitThreads = 1024;
template <int COLS, bool FUSE>
__global__ __launch_bounds__(kSplitThreads) void logreg_dense_grad_split_kernel(
    const float* const* __restrict__ Xs, const uint32_t* __restrict__ idx, const float* __restrict__ resid,
    const float* __restrict__ w, float* __restrict__ g, uint64_t d, uint32_t batch, float inv_b, float l2,
    ScaleFusion fuse) {
  constexpr int RG = kSplitThreads / COLS;
  __shared__ float sR[kBlock];
  __shared__ uint32_t sRow[kBlock];
  __shared__ float4 sAcc[RG - 1][COLS];
  __shared__ float red[16];
  const uint32_t m = blockIdx.y;
  const uint32_t tx = threadIdx.x % COLS, rg = threadIdx.x / COLS;
  const GlobalPtr<float> X = as_global(Xs[m]);
  const uint64_t index = (uint64_t)blockIdx.x * COLS + tx;  // float4 index
  const bool active = index < (d + 3) / 4;
  const uint64_t col = first_column(index, d);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (uint32_t base = 0; base < batch; base += kBlock) {
    __syncthreads();
    if (threadIdx.x < (uint32_t)kBlock && base + threadIdx.x < batch) {
      sR[threadIdx.x] = resid[(uint64_t)m * batch + base + threadIdx.x];
      sRow[threadIdx.x] = idx[(uint64_t)m * batch + base + threadIdx.x];
    }
    __syncthreads();
    if (active) {
      const uint32_t cnt = min((uint32_t)kBlock, batch - base);
#pragma unroll 8
      for (uint32_t i = rg; i < cnt; i += RG) {
        const float4 xv = load4_stream_any(X + (uint64_t)sRow[i] * d + col, 0);
        const float r = sR[i];
        acc.x = __builtin_fmaf(r, xv.x, acc.x);
        acc.y = __builtin_fmaf(r, xv.y, acc.y);
        acc.z = __builtin_fmaf(r, xv.z, acc.z);
        acc.w = __builtin_fmaf(r, xv.w, acc.w);
      }
    }
  }
  if (rg > 0) sAcc[rg - 1][tx] = acc;
  __syncthreads();
  float amax = 0.f;
  if (active && rg == 0) {
#pragma unroll
    for (int k = 0; k < RG - 1; ++k) {
      const float4 p = sAcc[k][tx];
      acc.x = acc.x + p.x;
      acc.y = acc.y + p.y;
      acc.z = acc.z + p.z;
      acc.w = acc.w + p.w;
    }
    const float4 wv = load4_at(w, col);
    float4 o;
    o.x = __builtin_fmaf(l2, wv.x, acc.x * inv_b);
    o.y = __builtin_fmaf(l2, wv.y, acc.y * inv_b);
    o.z = __builtin_fmaf(l2, wv.z, acc.z * inv_b);
    o.w = __builtin_fmaf(l2, wv.w, acc.w * inv_b);
    store4_any(g + (uint64_t)m * d + col, 0, o);
    if (FUSE) {
      float4 r1, r2;
      load_refs4(fuse, col, r1, r2);
      amax = absmax4(fuse, o, r1, r2);
    }
  }
  if (FUSE) {
    amax = block_max(amax, red);
    if (threadIdx.x == 0) fuse.partials[(uint64_t)blockIdx.x * gridDim.y + m] = amax;
  }
}

// ------------------------------------------------------------------------------------------
// Dense problems whose gradients fit one workgroup (M * d <= 4096): what bounds an iteration is its launches, about 4.4 us
// of the host each, so there are two.  The first takes the rows once: a thread keeps its float4 column of kSmallRows
// rows in registers between the dot products and the accumulation, and a workgroup leaves the partial gradient of its
// share of a worker's minibatch (parts[m][s][4 ceil(d / 4)], zero past d).  The second, one workgroup, adds those in
// order and (STEP) does all the rest of the iteration: a thread has one float4 of one worker.
// Iterations, three launches against these two: d = 1000, M = 4, B = 64 13.8 -> 12.1 us (5.1 + 6.8: the one workgroup
// reads 128 KiB of partial gradients), B = 512 23.5 -> 17.7; d = 64, M = 1, B = 8 13.2 -> 9.6 (the launches); d = 100, M = 32,
// B = 512 35.6 -> 19.3.  More rows per trip mean fewer partial gradients: 4 rows 12.9, 8 rows 12.1 us at d = 1000.
// ------------------------------------------------------------------------------------------
constexpr int kSmallRows = 8;

// Columns 4 q .. 4 q + 3 of a row of d >= 4, 0 past its end.
__device__ __forceinline__ float4 load4_row_end(GlobalPtr<float> row, uint32_t q, uint32_t d) {
  const uint32_t col = min(4 * q, d - 4), past = 4 * q - col;  // columns of the float4 that lie past the end
  const float4 v = load4_stream_any(row + col, 0);
  return make_float4(past == 0 ? v.x : past == 1 ? v.y : past == 2 ? v.z : v.w,
                     past == 0 ? v.y : past == 1 ? v.z : past == 2 ? v.w : 0.f,
                     past == 0 ? v.z : past == 1 ? v.w : 0.f, past == 0 ? v.w : 0.f);
}

__global__ __launch_bounds__(kBlock) void logreg_dense_small_kernel(const float* const* __restrict__ Xs,
                                                                    const float* const* __restrict__ ys,
                                                                    const uint64_t* __restrict__ n_rows,
                                                                    uint32_t* __restrict__ idx,
                                                                    const float* __restrict__ w,
                                                                    float4* __restrict__ parts, uint32_t d,
                                                                    uint32_t batch, uint32_t k0, uint32_t k1,
                                                                    uint32_t iter) {
  __shared__ float red[2][kSmallRows][kWavesPerBlock];
  const uint32_t m = blockIdx.y, s = blockIdx.x, S = gridDim.x, t = threadIdx.x;
  const uint32_t nvec = (d + 3) / 4;
  const uint32_t q = min(t, nvec - 1);  // idle threads fetch the last column
  const GlobalPtr<float> X = as_global(Xs[m]), y = as_global(ys[m]);
  const uint64_t n = n_rows[m];
  const float4 wv = t < nvec ? load4_row_end(as_global(w), q, d) : make_float4(0.f, 0.f, 0.f, 0.f);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  uint32_t parity = 0;
  for (uint32_t i0 = s; i0 < batch; i0 += S * kSmallRows, parity ^= 1u) {
    // lane r draws row r of the trip; a short last trip fetches its first row in place of those that it lacks
    const uint32_t mine = i0 + (t % kSmallRows) * S;
    const uint32_t drawn = minibatch_row(k0, k1, iter, m, mine < batch ? mine : i0, n);
    if (t < (uint32_t)kSmallRows && mine < batch) idx[(uint64_t)m * batch + mine] = drawn;
    const float label = y[drawn];
    float4 x[kSmallRows];
#pragma unroll
    for (int r = 0; r < kSmallRows; ++r)
      x[r] = load4_row_end(X + (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)drawn, r) * d, q, d);
#pragma unroll
    for (int r = 0; r < kSmallRows; ++r) {
      const float p = __builtin_fmaf(x[r].x, wv.x, x[r].y * wv.y) + __builtin_fmaf(x[r].z, wv.z, x[r].w * wv.w);
      const float z = wave_sum_uniform(t < nvec ? p : 0.f);
      if (t % kWave == 0) red[parity][r][t / kWave] = z;
    }
    __syncthreads();  // (two sets of slots alternate: one barrier per trip is enough)
    // lane r of every wavefront makes the residual of row r
    float z = red[parity][t % kSmallRows][0];
#pragma unroll
    for (int k = 1; k < kWavesPerBlock; ++k) z += red[parity][t % kSmallRows][k];
    const float residual = logistic_residual(z, label);
#pragma unroll
    for (int r = 0; r < kSmallRows; ++r) {
      if (i0 + (uint32_t)r * S >= batch) break;
      const float res = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(residual), r));
      acc.x = __builtin_fmaf(res, x[r].x, acc.x);
      acc.y = __builtin_fmaf(res, x[r].y, acc.y);
      acc.z = __builtin_fmaf(res, x[r].z, acc.z);
      acc.w = __builtin_fmaf(res, x[r].w, acc.w);
    }
  }
  if (t < nvec) parts[((uint64_t)m * S + s) * nvec + t] = acc;
}

typedef uint8_t __attribute__((may_alias)) lds_byte;
typedef uint16_t __attribute__((may_alias)) lds_half;
constexpr uint32_t kSmallThreads = 1024;
template <int NORM, int BITS, bool STEP, bool EIGHTS>
__global__ __launch_bounds__(kSmallThreads) void logreg_dense_small_finish_kernel(
    const float4* __restrict__ parts, uint32_t S, float* w, float* __restrict__ g, uint32_t d, uint32_t M, float inv_b,
    float l2, const float* gref, const float* gref2, float eps, float* __restrict__ scales, uint32_t* __restrict__ codes,
    uint32_t words, uint32_t k0, uint32_t k1, uint32_t iter, float* __restrict__ vbar, float* refout, float inv_m,
    float lr) {
  __shared__ float4 value[STEP ? kSmallThreads : 1];
  __shared__ uint32_t packed[STEP ? kSmallThreads : 1];  // [M][words]
  __shared__ uint32_t top[STEP ? kSmallThreads : 1];     // the workers' scales as bits
  const uint32_t nvec = (d + 3) / 4, t = threadIdx.x;
  const bool active = t < M * nvec;
  const uint32_t m = active ? t / nvec : M - 1, q = active ? t % nvec : nvec - 1;
  if (STEP) packed[t] = top[t] = 0u;
  // The parts are added in order.  Whole eights of them (EIGHTS; most minibatches: 57 to 64, 121 to 128, 185 to 192 and more than 248
  // rows) eight at a time, the iterate and the references asked for behind the last eight; otherwise the first one and then
  // eight at a time and the rest.  (d = 1000, M = 4: 8 parts 12.6 -> 12.2 us per iteration, 32 parts 17.7 -> 17.4; d = 69, M = 5, 32
  // parts 14.5 -> 13.9.  A last batch that repeats its last part instead of being shorter: d = 300, M = 4, 25 parts 11.9 -> 12.6.
  // Sixteen at a time: 32 parts 21.0.  What follows asked for ahead of 32 parts: 4 us more.)
  const float4* part = parts + (uint64_t)m * S * nvec + q;
  float4 acc, wv, r1 = make_float4(0.f, 0.f, 0.f, 0.f), r2 = make_float4(1.f, 1.f, 1.f, 1.f);
  auto add = [&](const float4& v) { acc = make_float4(acc.x + v.x, acc.y + v.y, acc.z + v.z, acc.w + v.w); };
  auto references = [&] {
    if (STEP && (NORM == kNormSub || NORM == kNormComb)) r1 = load4_within(gref, 4 * q, d, 0.f);
    if (STEP && NORM == kNormQuot) r1 = load4_within(gref, 4 * q, d, 1.f);
    if (STEP && NORM == kNormComb) r2 = load4_within(gref2, 4 * q, d, 1.f);
  };
  if (EIGHTS) {
    acc = make_float4(-0.f, -0.f, -0.f, -0.f);  // (-0 + x is x, the sign of a zero included)
    float4 v[8];
    for (uint32_t s = 8; s < S; s += 8, part += 8 * nvec) {
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) v[k] = part[k * nvec];
#pragma unroll
      for (uint32_t k = 0; k < 8; ++k) add(v[k]);
    }
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) v[k] = part[k * nvec];
    wv = load4_within(w, 4 * q, d, 0.f);
    references();
#pragma unroll
    for (uint32_t k = 0; k < 8; ++k) add(v[k]);
  } else {
    acc = parts[(uint64_t)m * S * nvec + q];
#pragma unroll 8
    for (uint32_t s = 1; s < S; ++s) add(parts[((uint64_t)m * S + s) * nvec + q]);
    wv = load4_within(w, 4 * q, d, 0.f);
  }
  const float4 o = make_float4(__builtin_fmaf(l2, wv.x, acc.x * inv_b), __builtin_fmaf(l2, wv.y, acc.y * inv_b),
                               __builtin_fmaf(l2, wv.z, acc.z * inv_b), __builtin_fmaf(l2, wv.w, acc.w * inv_b));
  if (active) store4_within(g + (uint64_t)m * d, 4 * q, d, o);
  if (!STEP) return;

  if (!EIGHTS) references();
  if (NORM == kNormQuot) r1 = make_float4(clamp_ref(r1.x, eps), clamp_ref(r1.y, eps), clamp_ref(r1.z, eps), clamp_ref(r1.w, eps));
  if (NORM == kNormComb) r2 = make_float4(clamp_ref(r2.x, eps), clamp_ref(r2.y, eps), clamp_ref(r2.z, eps), clamp_ref(r2.w, eps));
  const float4 v = make_float4(normalize<NORM>(o.x, r1.x, r2.x), normalize<NORM>(o.y, r1.y, r2.y),
                               normalize<NORM>(o.z, r1.z, r2.z), normalize<NORM>(o.w, r1.w, r2.w));
  // (past the end the gradient is 0 and its references such that it normalises to 0)
  const float amax = active ? fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))) : 0.f;
  __syncthreads();
  const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
  if ((uint32_t)__builtin_amdgcn_readlane((int)m, kWave - 1) == first) {  // one worker's wavefront
    const float wmax = wave_max_nonneg(amax);
    if (t % kWave == 0) atomicMax(&top[first], __float_as_uint(wmax));
  } else {
    atomicMax(&top[m], __float_as_uint(amax));
  }
  __syncthreads();
  const float R = __uint_as_float(top[m]) < 0x1p-126f ? 0.f : __uint_as_float(top[m]);
  if (active && q == 0) scales[m] = R;
  float4 val = make_float4(0.f, 0.f, 0.f, 0.f);
  if (active && R != 0.f) {
    constexpr float LEVELS = (float)((1 << (BITS - 1)) - 1);
    const float inv_r = 1.0f / R, step = R / LEVELS;
    const U32x4 rnd = philox4x32_10(q, m, iter, 0u, k0, k1);
    const uint32_t frag = quantize4_and_values<BITS>(v, inv_r, rnd, R, step, val);
    if (BITS == 2)
      reinterpret_cast<lds_byte*>(packed + m * words)[q] = (uint8_t)frag;
    else
      reinterpret_cast<lds_half*>(packed + m * words)[q] = (uint16_t)frag;
  }
  value[t] = val;
  __syncthreads();
  if (t < M * words) store_word_through(codes + t, packed[t]);
  if (t < nvec) {  // the server: m = 0 here, so q, the references and w are those of the thread's float4
    float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
    for (uint32_t k = 0; k < M; ++k) {
      const float4 p = value[k * nvec + t];
      sum.x = sum.x + p.x;
      sum.y = sum.y + p.y;
      sum.z = sum.z + p.z;
      sum.w = sum.w + p.w;
    }
    const float4 u = make_float4(denormalize<NORM>(sum.x * inv_m, r1.x, r2.x), denormalize<NORM>(sum.y * inv_m, r1.y, r2.y),
                                 denormalize<NORM>(sum.z * inv_m, r1.z, r2.z), denormalize<NORM>(sum.w * inv_m, r1.w, r2.w));
    const float px = lr * u.x, py = lr * u.y, pz = lr * u.z, pw = lr * u.w;
    store4_within(vbar, 4 * t, d, u);
    store4_within(w, 4 * t, d, make_float4(wv.x - px, wv.y - py, wv.z - pz, wv.w - pw));
    if (refout != nullptr) store4_within(refout, 4 * t, d, u);
  }
}

// ------------------------------------------------------------------------------------------
// Dense problems of up to 32 K columns: the rows are read once here too.  A workgroup takes several of its worker's
// minibatch rows at a time, all their loads in flight together, and holds them in registers, NV float4 columns a thread, from
// the dot products to the accumulation into its partial gradient; w and the partial gradient stay in registers as well.
// logreg_dense_mid_parts_kernel adds the S partial gradients of a worker (parts[m][s][ceil(d / 4)] float4).
// Bound by memory where the rows are many (d = 16000, M = 32, B = 512: 1 GiB of rows in an iteration of 174 us, 6.4 TB/s in this
// kernel) and by latency where a workgroup has one trip.  Iterations, the residual and the accumulation pass (rows read
// twice) / this: d = 10007, M = 8, B = 128 26.9 / 20.9 us, M = 32, B = 512 231 / 122; d = 16000, M = 32, B = 512 324 / 174;
// d = 5003, M = 16, B = 512 70.9 / 44.6; d = 2048, M = 32, B = 256 34.1 / 24.1; d = 1000, M = 32, B = 512 42.3 / 26.9; d = 300,
// M = 20, B = 64 16.5 / 14.6.
// Up to 4 float4 columns a thread two workgroups share a compute unit (128 registers), one fetching while the other
// computes; beyond, one with twice the registers and four rows at a time is faster (with the partial gradients added by a
// thread per column still: d = 10007, M = 8, B = 128 24.0, two of three rows each 26.7; d = 16000, M = 16, B = 512 95.8, two of one row
// 106).  Beyond 16 K columns the workgroup has 1024 threads and
// takes one or two rows.  There, and at 16 K, rows went through LDS and registers one at a time, or twice through memory
// where d was no multiple of 4: d = 32768, M = 16, B = 512 223 / 178, d = 32765 355 / 184, d = 20000, M = 16, B = 200 94.8 / 60.2,
// d = 16384, M = 16, B = 512 136 / 98; their partial gradients were a chain of up to 256 loads, d = 32768, M = 1, B = 512 146 / 32.4.
// ------------------------------------------------------------------------------------------
constexpr int kMidThreads = 512, kMidThreadsLong = 1024;
constexpr uint64_t kMidMostColumns = 16 * 1024;  // for kMidThreads: 8 float4 a thread
constexpr int dense_mid_rows(int t, int nv) {    // rows at a time
  return t == kMidThreadsLong ? (nv <= 5 ? 2 : 1) : nv <= 2 ? 8 : 4;
}
constexpr int dense_mid_per_unit(int t, int nv) { return t != kMidThreadsLong && nv <= 4 ? 2 : 1; }  // workgroups per compute unit
inline int dense_mid_threads(uint64_t d) { return d <= 4 * kBlock ? kBlock : d <= kMidMostColumns ? kMidThreads : kMidThreadsLong; }
inline int dense_mid_columns(uint64_t d) {
  const uint64_t t = (uint64_t)dense_mid_threads(d);
  return (int)(((d + 3) / 4 + t - 1) / t);
}
template <int T, int NV>
__global__ __launch_bounds__(T, T / 256 * dense_mid_per_unit(T, NV)) void logreg_dense_mid_kernel(const float* const* __restrict__ Xs,
                                                                const float* const* __restrict__ ys,
                                                                const uint64_t* __restrict__ n_rows,
                                                                uint32_t* __restrict__ idx, const float* __restrict__ w,
                                                                float4* __restrict__ parts, uint32_t d, uint32_t batch,
                                                                uint32_t k0, uint32_t k1, uint32_t iter) {
  constexpr int R = dense_mid_rows(T, NV);
  __shared__ float red[2][R][T / kWave];
  const uint32_t m = blockIdx.y, s = blockIdx.x, S = gridDim.x, t = threadIdx.x;
  const uint32_t nvec = (d + 3) / 4;
  const GlobalPtr<float> X = as_global(Xs[m]), y = as_global(ys[m]);
  const uint64_t n = n_rows[m];
  // All float4 but the last of a thread lie inside the row ((NV - 1) T < ceil(d / 4) <= NV T); the last may repeat columns of its
  // neighbour's, and idle threads fetch the row's last columns.
  const uint32_t q_last = t + (uint32_t)(NV - 1) * T;
  const uint32_t c_first = 4 * t, c_last = (uint32_t)first_column(min(q_last, nvec - 1), d);
  const uint32_t repeated = q_last < nvec ? 4 * q_last - c_last : 4u;  // of its four columns: they count once in the dot product
  auto columns = [&](auto row, int k) { return k < NV - 1 ? row + 4 * k * T + c_first : row + c_last; };
  float4 wv[NV], acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    wv[k] = load4_at(columns(w, k), 0);
    acc[k] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  uint32_t parity = 0;
  for (uint32_t i0 = s; i0 < batch; i0 += S * R, parity ^= 1u) {
    // lane r draws row r of the trip; a short last trip fetches its first row in place of those that it lacks
    const uint32_t mine = i0 + (t % kWave % R) * S;
    const uint32_t drawn = minibatch_row(k0, k1, iter, m, mine < batch ? mine : i0, n);
    if (t < (uint32_t)R && mine < batch) idx[(uint64_t)m * batch + mine] = drawn;
    const float label = y[drawn];
    float4 x[R][NV];
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const GlobalPtr<float> row = X + (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)drawn, r) * d;
#pragma unroll
      for (int k = 0; k < NV; ++k) x[r][k] = load4_stream_any(columns(row, k), 0);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float z0 = 0.f, z1 = 0.f, z2 = 0.f, z3 = 0.f;
#pragma unroll
      for (int k = 0; k < NV - 1; ++k) {
        z0 = __builtin_fmaf(x[r][k].x, wv[k].x, z0);
        z1 = __builtin_fmaf(x[r][k].y, wv[k].y, z1);
        z2 = __builtin_fmaf(x[r][k].z, wv[k].z, z2);
        z3 = __builtin_fmaf(x[r][k].w, wv[k].w, z3);
      }
      const float4 xl = x[r][NV - 1], wl = wv[NV - 1];  // (left out by choice, not by a factor of 0: an infinite x would make it NaN)
      z0 = repeated > 0 ? z0 : __builtin_fmaf(xl.x, wl.x, z0);
      z1 = repeated > 1 ? z1 : __builtin_fmaf(xl.y, wl.y, z1);
      z2 = repeated > 2 ? z2 : __builtin_fmaf(xl.z, wl.z, z2);
      z3 = repeated > 3 ? z3 : __builtin_fmaf(xl.w, wl.w, z3);
      const float z = wave_sum_uniform((z0 + z1) + (z2 + z3));
      if (t % kWave == 0) red[parity][r][t / kWave] = z;
    }
    __syncthreads();  // (two sets of slots alternate: one barrier per trip is enough)
    // lane r of every wavefront makes the residual of row r
    float z = red[parity][t % kWave % R][0];
#pragma unroll
    for (int k = 1; k < T / kWave; ++k) z += red[parity][t % kWave % R][k];
    const float residual = logistic_residual(z, label);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      if (i0 + (uint32_t)r * S >= batch) break;
      const float res = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(residual), r));
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        acc[k].x = __builtin_fmaf(res, x[r][k].x, acc[k].x);
        acc[k].y = __builtin_fmaf(res, x[r][k].y, acc[k].y);
        acc[k].z = __builtin_fmaf(res, x[r][k].z, acc[k].z);
        acc[k].w = __builtin_fmaf(res, x[r][k].w, acc[k].w);
      }
    }
  }
  float4* out = parts + ((uint64_t)m * S + s) * nvec;
#pragma unroll
  for (int k = 0; k < NV; ++k)
    if (k < NV - 1 || q_last < nvec) out[t + (uint32_t)k * T] = acc[k];
}

// g_m = (1/B) (sum over the S partial gradients of worker m) + l2 w.  kMidCols float4 columns a workgroup; the partial gradients
// are dealt to its row groups, whose sums are added in order (a thread per column is a chain of up to 256 loads: d = 2^16, M = 1,
// B = 512 160 us, 58 this way).
constexpr int kMidCols = 32, kMidGroups = kBlock / kMidCols;
template <bool FUSE>
__global__ __launch_bounds__(kBlock) void logreg_dense_mid_parts_kernel(
    const float4* __restrict__ parts, const float* __restrict__ w, float* __restrict__ g, uint64_t d, uint32_t S, float inv_b,
    float l2, ScaleFusion fuse) {
  __shared__ float4 sums[kMidGroups - 1][kMidCols];
  __shared__ float red[16];
  const uint32_t m = blockIdx.y, tx = threadIdx.x % kMidCols, rg = threadIdx.x / kMidCols;
  const uint32_t nvec = (uint32_t)((d + 3) / 4), index = blockIdx.x * kMidCols + tx;
  const bool active = index < nvec;
  const float4* p = parts + (uint64_t)m * S * nvec + min(index, nvec - 1);
  const uint64_t col = first_column(min(index, nvec - 1), d);
  const float4 wv = load4_at(w, col);
  float4 r1 = make_float4(0.f, 0.f, 0.f, 0.f), r2 = r1;
  if (FUSE) load_refs4(fuse, col, r1, r2);
  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 8
  for (uint32_t s = rg; s < S; s += kMidGroups) {
    const float4 v = p[(uint64_t)s * nvec];
    acc.x += v.x;
    acc.y += v.y;
    acc.z += v.z;
    acc.w += v.w;
  }
  if (rg > 0) sums[rg - 1][tx] = acc;
  __syncthreads();
  float amax = 0.f;
  if (active && rg == 0) {
#pragma unroll
    for (int k = 0; k < kMidGroups - 1; ++k) {
      const float4 v = sums[k][tx];
      acc.x += v.x;
      acc.y += v.y;
      acc.z += v.z;
      acc.w += v.w;
    }
    float4 o;
    o.x = __builtin_fmaf(l2, wv.x, acc.x * inv_b);
    o.y = __builtin_fmaf(l2, wv.y, acc.y * inv_b);
    o.z = __builtin_fmaf(l2, wv.z, acc.z * inv_b);
    o.w = __builtin_fmaf(l2, wv.w, acc.w * inv_b);
    store4_any(g + (uint64_t)m * d + col, 0, o);
    if (FUSE) amax = absmax4(fuse, o, r1, r2);
  }
  if (FUSE) {
    amax = block_max(amax, red);
    if (threadIdx.x == 0) fuse.partials[(uint64_t)blockIdx.x * gridDim.y + m] = amax;
  }
}

// The same with a thread per column, for few partial gradients of many columns in whole float4: fewer partial maxima are left
// to the tail (d = 2^16, M = 16, B = 256: 219.5 us in groups of 32 columns, 216.4).
template <bool FUSE>
__global__ __launch_bounds__(kBlock) void logreg_dense_parts_kernel(const float* __restrict__ parts,
                                                                    const float* __restrict__ w, float* __restrict__ g,
                                                                    uint64_t d, uint32_t S, float inv_b, float l2,
                                                                    ScaleFusion fuse) {
  __shared__ float red[16];
  const uint32_t m = blockIdx.y;
  const uint64_t col = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool active = col < d / 4;
  float amax = 0.f;
  if (active) {
    const float4* __restrict__ p = reinterpret_cast<const float4*>(parts + (uint64_t)m * S * d) + col;
    float4 acc = load_stream(p);
    for (uint32_t s = 1; s < S; ++s) {
      const float4 v = load_stream(p + (uint64_t)s * (d / 4));
      acc.x += v.x;
      acc.y += v.y;
      acc.z += v.z;
      acc.w += v.w;
    }
    const float4 wv = reinterpret_cast<const float4*>(w)[col];
    float4 o;
    o.x = __builtin_fmaf(l2, wv.x, acc.x * inv_b);
    o.y = __builtin_fmaf(l2, wv.y, acc.y * inv_b);
    o.z = __builtin_fmaf(l2, wv.z, acc.z * inv_b);
    o.w = __builtin_fmaf(l2, wv.w, acc.w * inv_b);
    reinterpret_cast<float4*>(g + (uint64_t)m * d)[col] = o;
    if (FUSE) {
      float4 r1, r2;
      load_refs4(fuse, 4 * col, r1, r2);
      amax = absmax4(fuse, o, r1, r2);
    }
  }
  if (FUSE) {
    amax = block_max(amax, red);
    if (threadIdx.x == 0) fuse.partials[(uint64_t)blockIdx.x * gridDim.y + m] = amax;
  }
}

// One pass over the minibatch rows of dense problems of 64 K columns: a workgroup takes whole rows, one at a time, and
// KEEPS the row on chip between the two uses it has -- the
// dot product z = x . w, and, once sigma(z) - y is known, the accumulation r x into the workgroup's
// partial gradient -- so that X_B is read from memory once instead of twice (the separate residual and
// accumulation passes each stream it at 6.2 TB/s, which is all the memory system gives; re-reading a
// block right after it was read, out of the 256 MB last-level cache, measured no faster than HBM).
// A row of 256 KiB fits neither store alone: each of the 512 threads (one workgroup per compute
// unit, so 256 registers per thread) parks NL = 16 float4 of the row in LDS (128 KiB per
// workgroup; a thread reads back only what it wrote) and holds the other NR = 16 in registers, next to its
// NV float4 of partial gradient.  The LDS half is loaded from memory straight into LDS, so that the whole
// row is requested at once.
// The workgroups of a worker split its minibatch rows; their partial gradients go to scratch
// parts[m][s][d], and dense_parts_launch has them added.
constexpr int kRowsThreads = 512;
constexpr int kRowsWaves = kRowsThreads / kWave;
// 16 bytes per lane from memory straight into LDS: lane l of the wavefront writes the l-th 16 bytes behind
// dst, which is the same for the whole wavefront; counted by vmcnt like any load.  Non-temporal (policy bit
// 2): the row is read once.  (The builtin exists in the device pass only.)
constexpr int kRowsStagger = 55;  // s_sleep units of 64 clocks: about 1.7 microseconds
typedef __attribute__((address_space(3))) void* LdsPtr;
__device__ __forceinline__ void load16_to_lds(GlobalPtr<v4f_t> src, LdsPtr dst) {
#if defined(__HIP_DEVICE_COMPILE__)
  __builtin_amdgcn_global_load_lds(src, dst, 16, 0, 2);
#endif
}
constexpr int kRowsLds = 16;  // float4 per thread kept in LDS
constexpr uint64_t kRowsColumns = 1 << 16;
__global__ __launch_bounds__(kRowsThreads) void logreg_dense_rows_kernel(const float* const* __restrict__ Xs,
                                                                         const float* const* __restrict__ ys,
                                                                         const uint64_t* __restrict__ n_rows,
                                                                         uint32_t* __restrict__ idx,
                                                                         const float* __restrict__ w,
                                                                         float* __restrict__ parts, uint64_t d,
                                                                         uint32_t batch, uint32_t k0, uint32_t k1,
                                                                         uint32_t iter) {
  constexpr int NV = (int)(kRowsColumns / (4 * kRowsThreads)), NL = kRowsLds, NR = NV - NL;
  constexpr int TR = 4;  // float4 of the LDS half read back at a time when the row is added
  constexpr int TW = 8;  // float4 of w on their way at a time
  static_assert(NL % TR == 0 && NL % TW == 0 && NR % TW == 0, "both halves are worked through in whole batches");
  constexpr int kWaitVmem = 0x0F70;         // s_waitcnt vmcnt(0)
  constexpr int kWaitLds = 0xC07F;          // s_waitcnt lgkmcnt(0)
  extern __shared__ float4 rowl[];  // [NL][kRowsThreads]
  __shared__ float red[2][kRowsWaves];
  const uint32_t m = blockIdx.y, s = blockIdx.x, S = gridDim.x, t = threadIdx.x;
  const uint32_t wave_first = (uint32_t)__builtin_amdgcn_readfirstlane((int)(t / kWave)) * kWave;  // a scalar
  const GlobalPtr<float> X = as_global(Xs[m]);
  const GlobalPtr<float> y = as_global(ys[m]);
  const uint64_t n = n_rows[m];
  const float4* __restrict__ w4 = reinterpret_cast<const float4*>(w);
  // float4 column k of the thread: LDS half first (k < NL), register half after
  // (the thread index goes through an opaque copy per use site: otherwise the compiler computes all NV
  // column addresses of x and of w once, ahead of the row loop, and keeps them in 3 NV registers)
  auto opaque_t = [&]() {
    uint32_t v = t;
    asm volatile("" : "+v"(v));
    return v;
  };
  auto column_of = [&](uint32_t tt, int k) { return tt + (uint32_t)k * kRowsThreads; };
  float4 acc[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) acc[k] = make_float4(0.f, 0.f, 0.f, 0.f);
  // A row is fetched (memory busy, arithmetic idle) and then worked on (the reverse), and workgroups that start
  // together stay in step: every compute unit fetches at once and the memory system idles while all of them
  // compute.  A quarter of the workgroups therefore starts at once and the others 1.7, 3.4 and 5.1 microseconds
  // later (about the length of the arithmetic on a row), so that the fetches of some fall into the arithmetic of
  // the others.  Measured at d = 2^16, M = 16, B = 256: iteration 0.236 -> 0.224 ms, this kernel 200
  // microseconds (with twice the delay 0.230 ms; with eight steps of 0.7 microseconds 204 microseconds).
  for (uint32_t q = (blockIdx.x + blockIdx.y * gridDim.x) % 4u; q > 0; --q) __builtin_amdgcn_s_sleep(kRowsStagger);
  uint32_t parity = 0;
  for (uint32_t i = s; i < batch; i += S, parity ^= 1u) {
    const uint32_t row = minibatch_row(k0, k1, iter, m, i, n);
    if (t == 0) idx[(uint64_t)m * batch + i] = row;
    const GlobalPtr<float> x = X + (uint64_t)row * d;
    // Requests of a row, in the order in which they come back: the first batch of w (out of the caches), the
    // register half, then the LDS half, which goes from memory straight into LDS (16 bytes per lane, lane l of
    // a wavefront to the l-th float4 behind the wavefront's address: each thread's own slot) -- so the whole
    // row, 256 KiB at d = 2^16, is in flight at once and no register carries the LDS half.
    float4 wa[TW];
    {
      const uint32_t tt = opaque_t();
#pragma unroll
      for (int k = 0; k < TW; ++k) wa[k] = w4[column_of(tt, k)];
    }
    float4 xr[NR];
    {
      const uint32_t tt = opaque_t();
#pragma unroll
      for (int k = 0; k < NR; ++k) xr[k] = load4_stream(x, column_of(tt, NL + k));
    }
    {
      const uint32_t tt = opaque_t();
#pragma unroll
      for (int k = 0; k < NL; ++k)
        load16_to_lds(reinterpret_cast<GlobalPtr<v4f_t>>(x) + column_of(tt, k),
                      (LdsPtr)(rowl + k * kRowsThreads + wave_first));
    }
    __builtin_amdgcn_s_waitcnt(kWaitVmem);  // everything requested above has arrived, the LDS half in LDS
    asm volatile("" ::: "memory");
    float z0 = 0.f, z1 = 0.f, z2 = 0.f, z3 = 0.f;
#pragma unroll
    for (int k0b = 0; k0b < NL; k0b += TW) {
      if (k0b > 0) {
        const uint32_t tt = opaque_t();
#pragma unroll
        for (int k = 0; k < TW; ++k) wa[k] = w4[column_of(tt, k0b + k)];
      }
      const uint32_t tt = opaque_t();
#pragma unroll
      for (int k = 0; k < TW; ++k) {
        const float4 xv = rowl[(k0b + k) * kRowsThreads + tt];
        z0 = __builtin_fmaf(xv.x, wa[k].x, z0);
        z1 = __builtin_fmaf(xv.y, wa[k].y, z1);
        z2 = __builtin_fmaf(xv.z, wa[k].z, z2);
        z3 = __builtin_fmaf(xv.w, wa[k].w, z3);
      }
      asm volatile("" ::: "memory");  // keeps the next batch's loads behind this batch's use: registers are the scarce thing here
    }
#pragma unroll
    for (int k0b = 0; k0b < NR; k0b += TW) {
      const uint32_t tt = opaque_t();
#pragma unroll
      for (int k = 0; k < TW; ++k) wa[k] = w4[column_of(tt, NL + k0b + k)];
#pragma unroll
      for (int k = 0; k < TW; ++k) {
        z0 = __builtin_fmaf(xr[k0b + k].x, wa[k].x, z0);
        z1 = __builtin_fmaf(xr[k0b + k].y, wa[k].y, z1);
        z2 = __builtin_fmaf(xr[k0b + k].z, wa[k].z, z2);
        z3 = __builtin_fmaf(xr[k0b + k].w, wa[k].w, z3);
      }
      asm volatile("" ::: "memory");
    }
    // z over the workgroup (two sets of slots alternate, so that one barrier per row is enough)
    const float zw = wave_sum((z0 + z1) + (z2 + z3));
    if (t % kWave == 0) red[parity][t / kWave] = zw;
    __syncthreads();
    float z = red[parity][0];
#pragma unroll
    for (int k = 1; k < kRowsWaves; ++k) z += red[parity][k];
    const float r = logistic_residual(z, y[row]);
#pragma unroll
    for (int k = 0; k < NR; ++k) {
      acc[NL + k].x = __builtin_fmaf(r, xr[k].x, acc[NL + k].x);
      acc[NL + k].y = __builtin_fmaf(r, xr[k].y, acc[NL + k].y);
      acc[NL + k].z = __builtin_fmaf(r, xr[k].z, acc[NL + k].z);
      acc[NL + k].w = __builtin_fmaf(r, xr[k].w, acc[NL + k].w);
    }
#pragma unroll
    for (int k0b = 0; k0b < NL; k0b += TR) {
      const uint32_t tt = opaque_t();
#pragma unroll
      for (int k = k0b; k < k0b + TR; ++k) {
        const float4 xv = rowl[k * kRowsThreads + tt];
        acc[k].x = __builtin_fmaf(r, xv.x, acc[k].x);
        acc[k].y = __builtin_fmaf(r, xv.y, acc[k].y);
        acc[k].z = __builtin_fmaf(r, xv.z, acc[k].z);
        acc[k].w = __builtin_fmaf(r, xv.w, acc[k].w);
      }
      asm volatile("" ::: "memory");
    }
    __builtin_amdgcn_s_waitcnt(kWaitLds);  // this row's LDS reads are done before the next row's loads write there
    asm volatile("" ::: "memory");
  }
  float4* __restrict__ out = reinterpret_cast<float4*>(parts + ((uint64_t)m * S + s) * d);
#pragma unroll
  for (int k = 0; k < NV; ++k) store_stream(out + column_of(t, k), acc[k]);
}

// ------------------------------------------------------------------------------------------
// CSR logistic regression, column-tiled.
//
// Gathering w[col] and scattering into g[col] one stored entry at a time costs a 64-byte memory
// transaction per 4 useful bytes (measured: 9.5 ms + 26 ms per step at d = 2^24, M = 64, B = 512).
// Instead the columns are cut into tiles of 2^kCsrTileShift coordinates and a workgroup owns one
// (worker, tile): the tile of w, then the tile of g, lives in LDS, and every minibatch row
// contributes the contiguous segment of its (ascending) columns that falls into the tile.
//   1. csr_bounds_kernel   one coalesced pass over the minibatch rows' column ids: for every row
//                          and tile, the offset of the first entry at or beyond the tile start;
//   2. csr_z_kernel        per (row, tile) partial dot product sum val * w_tile[col];
//      csr_z_reduce_kernel z_i = sum of the partials over the tiles;
//   3. csr_grad_kernel     r_i = sigma(z_i) - y_i; g_tile[col] += (r_i / B) val in LDS, then the whole
//                          tile is written once (+ l2 w): no zero fill, no global atomics.
// The g tile is accumulated in fp64: on this hardware an fp32 LDS atomic add serialises over the
// lanes (~170 clocks per wavefront instruction) while the fp64 one runs at ~12; as a side effect g
// is the correctly rounded sum almost always, whatever the order of the additions.
// Entries are read twice in segment-sized pieces, g is written once.
// ------------------------------------------------------------------------------------------
constexpr int kCsrThreads = 1024;  // 16 wavefronts
constexpr int kCsrRows = 512;      // minibatch rows staged in LDS per trip
// A lane takes two entries of a row segment at once (16 bytes of pairs), and few lanes share a segment.  What bounds these
// passes, next to the bytes, is how many instructions a wavefront issues per entry: with an entry per lane, 32 lanes to a
// segment and a branch around every load and use, the dot products took 600 vector and 850 scalar instructions per
// wavefront and 512 rows, about two thirds of their time, and the segments' loads by themselves ran 25 to 30 % slower than
// with 16 bytes per lane (1.21 -> 0.92 ms for the segments of 2^14 columns, 64 workers, 512 rows of 16777 pairs).  Iteration
// at d = 2^24, M = 64, B = 512, 0.1 % density 4276 -> 3899 us (dot products 1180 -> 959, gradient 2055 -> 1903); d = 2^16, M = 8 19.1 ->
// 17.8.  What the gradient pass then waited for was its own order, see csr_grad_workers_kernel.
constexpr int kCsrLanes = 8;                  // lanes that share one row segment
constexpr int kCsrUnroll = 4;                 // row segments per lane group and trip
constexpr uint32_t kCsrStep = 2 * kCsrLanes;  // entries that a load of each lane covers
constexpr int kCsrLoads = 2;                  // such loads per segment of a tile (mean segment: 16 entries at 0.1 % density)
constexpr int kCsrWideLoads = 3;              // the same for two tiles
constexpr uint32_t kCsrGroups = kCsrThreads / kCsrLanes;
static_assert(kCsrGroups * kCsrUnroll == kCsrRows && kCsrRows <= kCsrThreads, "one sweep of the lane groups covers one trip");

// The stored entries of one worker's shard, in either of the two layouts the library takes: separate
// column and value arrays, or one array of (column, value) pairs.  With pairs a row segment of a
// tile is one contiguous piece of 8 bytes per entry instead of two pieces of 4: segments are short
// (16 entries per row and tile at 0.1 % density), and what such reads deliver is set by the 128-byte
// memory lines they touch, so one piece of twice the length moves the same entries in about two
// thirds of the line traffic, with half the load instructions.
typedef int v2i_t __attribute__((ext_vector_type(2)));
typedef int v2i_u_t __attribute__((ext_vector_type(2), aligned(4)));
typedef float v2f_u_t __attribute__((ext_vector_type(2), aligned(4)));
typedef int v4i_u_t __attribute__((ext_vector_type(4), aligned(8)));
struct CsrTwo {
  int32_t col[2];
  float val[2];
};
// Which column tile (of n, one per workgroup along x) workgroup bx takes.  Workgroups are handed to the
// eight compute dies in turn (bx mod 8), each die with an L2 of its own: die k gets the k-th eighth of the
// tiles, in order, so that the workgroups running side by side on a die are on ADJACENT tiles and the memory
// lines shared by the end of one tile's row segment and the start of the next tile's are fetched from HBM
// once (a bijection for any n; only the traffic depends on how the hardware really deals workgroups out).
__device__ __forceinline__ uint32_t tile_of_workgroup(uint32_t bx, uint32_t n) {
  constexpr uint32_t kDies = 8;
  if (n % kDies != 0) return bx;  // rows of the grid would start on different dies: keep the plain order
  return (bx % kDies) * (n / kDies) + bx / kDies;
}

template <bool PAIRS>
struct CsrEntries {
  GlobalPtr<int32_t> c;  // column ids, or the pairs viewed as 32-bit words (column at 2 pos, value at 2 pos + 1)
  GlobalPtr<float> v;    // values (unused with pairs)
  __device__ __forceinline__ CsrEntries(const int32_t* cols, const float* vals) : c(as_global(cols)), v(as_global(vals)) {}
  __device__ __forceinline__ int32_t col(int64_t pos) const { return PAIRS ? c[2 * pos] : c[pos]; }
  __device__ __forceinline__ void load(int64_t pos, int32_t& col, float& val) const {
    if (PAIRS) {
      const v2i_t p = reinterpret_cast<GlobalPtr<v2i_t>>(c)[pos];
      col = p.x;
      val = __int_as_float(p.y);
    } else {
      col = c[pos];
      val = v[pos];
    }
  }
  // Entries pos and pos + 1.
  __device__ __forceinline__ CsrTwo load2(int64_t pos) const {
    if (PAIRS) {
      const v4i_u_t p = *reinterpret_cast<GlobalPtr<v4i_u_t>>(c + 2 * pos);
      return CsrTwo{{p.x, p.z}, {__int_as_float(p.y), __int_as_float(p.w)}};
    }
    const v2i_u_t ci = *reinterpret_cast<GlobalPtr<v2i_u_t>>(c + pos);
    const v2f_u_t vi = *reinterpret_cast<GlobalPtr<v2f_u_t>>(v + pos);
    return CsrTwo{{ci.x, ci.y}, {vi.x, vi.y}};
  }
  // The position that load2 reads dummy at (16 valid bytes, 8-byte aligned), for segments without entries; two arrays have
  // no such position: they are read at dummy by load2_any.
  __device__ __forceinline__ int64_t position_of(const void* dummy) const {
    return PAIRS ? ((int64_t)reinterpret_cast<uintptr_t>(dummy) - (int64_t)reinterpret_cast<uintptr_t>((const int32_t*)c)) / 8 : 0;
  }
  __device__ __forceinline__ CsrTwo load2_any(bool any, int64_t pos, const void* dummy) const {
    if (PAIRS) return load2(pos);
    const v2i_u_t ci = *(any ? reinterpret_cast<GlobalPtr<v2i_u_t>>(c + pos) : (GlobalPtr<v2i_u_t>)dummy);
    const v2f_u_t vi = *(any ? reinterpret_cast<GlobalPtr<v2f_u_t>>(v + pos) : (GlobalPtr<v2f_u_t>)dummy);
    return CsrTwo{{ci.x, ci.y}, {vi.x, vi.y}};
  }
};

// rowbase[m][i] = position of minibatch row i in worker m's col / val arrays; bounds[m][t][i]
// (tile-major, so that a workgroup reads the bounds of all its rows contiguously) = offset within
// the row of the first entry whose column is at or beyond the start of tile t; t = 0 .. ntiles.
template <bool PAIRS>
__global__ __launch_bounds__(kBlock) void csr_bounds_kernel(const int64_t* const* __restrict__ rowptrs,
                                                            const int32_t* const* __restrict__ cols,
                                                            const uint32_t* __restrict__ idx,
                                                            int64_t* __restrict__ rowbase,
                                                            uint32_t* __restrict__ bounds, uint32_t batch,
                                                            uint32_t ntiles, uint32_t tile_shift) {
  const uint32_t m = blockIdx.y, i = blockIdx.x;
  const uint32_t row = idx[(uint64_t)m * batch + i];
  const int64_t a = as_global(rowptrs[m])[row];
  const uint32_t nnz = (uint32_t)(as_global(rowptrs[m])[row + 1] - a);
  const CsrEntries<PAIRS> e(cols[m], nullptr);
  if (threadIdx.x == 0) rowbase[(uint64_t)m * batch + i] = a;
  uint32_t* __restrict__ out = bounds + (uint64_t)m * (ntiles + 1) * batch + i;
  // entry k opens every tile after the tile of entry k-1 up to its own tile
  for (uint32_t k = threadIdx.x; k <= nnz; k += kBlock) {
    const uint32_t prev = k == 0 ? 0u : ((uint32_t)e.col(a + k - 1) >> tile_shift) + 1u;
    const uint32_t cur = k == nnz ? ntiles : ((uint32_t)e.col(a + k) >> tile_shift);
    for (uint32_t t = prev; t <= cur; ++t) out[(uint64_t)t * batch] = k;
  }
}

// One-off: the same offsets for every row of every shard, row-major (index[m][row][t]).
template <bool PAIRS>
__global__ __launch_bounds__(kBlock) void csr_tile_index_kernel(const int64_t* const* __restrict__ rowptrs,
                                                                const int32_t* const* __restrict__ cols,
                                                                const uint64_t* __restrict__ n_rows,
                                                                const uint32_t* const* __restrict__ index,
                                                                uint32_t ntiles, uint32_t tile_shift) {
  const uint32_t m = blockIdx.y;
  const uint64_t row = blockIdx.x;
  if (row >= n_rows[m]) return;
  const int64_t a = as_global(rowptrs[m])[row];
  const uint32_t nnz = (uint32_t)(as_global(rowptrs[m])[row + 1] - a);
  const CsrEntries<PAIRS> e(cols[m], nullptr);
  uint32_t* __restrict__ out = const_cast<uint32_t*>(index[m]) + row * (ntiles + 1);
  for (uint32_t k = threadIdx.x; k <= nnz; k += kBlock) {
    const uint32_t prev = k == 0 ? 0u : ((uint32_t)e.col(a + k - 1) >> tile_shift) + 1u;
    const uint32_t cur = k == nnz ? ntiles : ((uint32_t)e.col(a + k) >> tile_shift);
    for (uint32_t t = prev; t <= cur; ++t) out[t] = k;
  }
}

// Checks of caller-supplied CSR shards (tng_validate_csr).  Stage 1: the row pointers of worker m are
// non-negative, non-decreasing, end within the nnz[m] stored entries, and no row holds 2^32 entries or
// more.  Stage 2 (only launched when stage 1 found nothing, so every access below is in range): the
// column ids of every row lie in [0, d) and ascend strictly.  A violation sets a bit of *flag.
__global__ __launch_bounds__(kBlock) void csr_validate_rowptr_kernel(const int64_t* const* __restrict__ rowptrs,
                                                                     const uint64_t* __restrict__ n_rows,
                                                                     const uint64_t* __restrict__ nnz,
                                                                     uint32_t* __restrict__ flag) {
  const uint32_t m = blockIdx.y;
  const uint64_t n = n_rows[m];
  const GlobalPtr<int64_t> rp = as_global(rowptrs[m]);
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  uint32_t bad = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) {
    const int64_t a = rp[i], b = rp[i + 1];
    if (a < 0 || b < a || (uint64_t)b > nnz[m] || (uint64_t)(b - a) >= (1ull << 32)) bad = 1u;
  }
  if (bad != 0) atomicOr(flag, 1u);
}

template <bool PAIRS>
__global__ __launch_bounds__(kBlock) void csr_validate_cols_kernel(const int64_t* const* __restrict__ rowptrs,
                                                                   const int32_t* const* __restrict__ cols,
                                                                   const uint64_t* __restrict__ n_rows, uint64_t d,
                                                                   uint32_t* __restrict__ flag) {
  const uint32_t m = blockIdx.y;
  const uint64_t n = n_rows[m];
  uint32_t bad = 0;
  for (uint64_t row = blockIdx.x; row < n; row += gridDim.x) {
    const int64_t a = as_global(rowptrs[m])[row], b = as_global(rowptrs[m])[row + 1];
    const CsrEntries<PAIRS> e(cols[m], nullptr);
    for (int64_t k = a + threadIdx.x; k < b; k += kBlock) {
      const int32_t cur = e.col(k);
      if (cur < 0 || (uint64_t)cur >= d) bad |= 2u;
      if (k > a && e.col(k - 1) >= cur) bad |= 4u;
    }
  }
  if (bad != 0) atomicOr(flag, bad);
}

// Per iteration, with the index: the index rows of the minibatch are transposed into the tile-major
// bounds array (64 rows x 128 tiles through LDS, both sides coalesced), and rowbase is filled.  The row ids come to LDS
// first, so that all of a thread's 32 loads are in flight at once (iteration at d = 2^24, 64 workers, minibatch 512: 4345
// us with 64 x 64 blocks and a dependent load of the row id before each of 16 loads, 4287 this way).
constexpr int kGatherRows = 64, kGatherTiles = 128;
__global__ __launch_bounds__(kBlock) void csr_gather_bounds_kernel(const int64_t* const* __restrict__ rowptrs,
                                                                   const uint32_t* const* __restrict__ index,
                                                                   const uint32_t* __restrict__ idx,
                                                                   int64_t* __restrict__ rowbase,
                                                                   uint32_t* __restrict__ bounds, uint32_t batch,
                                                                   uint32_t ntiles) {
  constexpr int kLoads = kGatherRows * kGatherTiles / kBlock;
  __shared__ uint32_t row_ids[kGatherRows];
  __shared__ uint32_t tile[kGatherRows][kGatherTiles + 1];
  const uint32_t m = blockIdx.z;
  const uint32_t t0 = blockIdx.x * kGatherTiles, i0 = blockIdx.y * kGatherRows;
  if (threadIdx.x < (uint32_t)kGatherRows) {
    const uint64_t o = (uint64_t)m * batch + min(i0 + threadIdx.x, batch - 1);
    const uint32_t row = idx[o];
    row_ids[threadIdx.x] = row;
    if (blockIdx.x == 0 && i0 + threadIdx.x < batch) rowbase[o] = as_global(rowptrs[m])[row];
  }
  __syncthreads();
  {
    const uint32_t tx = threadIdx.x % kGatherTiles, ty = threadIdx.x / kGatherTiles;
    const GlobalPtr<uint32_t> src = as_global(index[m]) + min(t0 + tx, ntiles);
    uint32_t v[kLoads];
#pragma unroll
    for (int k = 0; k < kLoads; ++k)
      v[k] = src[(uint64_t)row_ids[ty + (uint32_t)k * (kBlock / kGatherTiles)] * (ntiles + 1)];
#pragma unroll
    for (int k = 0; k < kLoads; ++k) tile[ty + (uint32_t)k * (kBlock / kGatherTiles)][tx] = v[k];
  }
  __syncthreads();
  const uint32_t tx = threadIdx.x % kGatherRows, ty = threadIdx.x / kGatherRows;
  if (i0 + tx < batch) {
#pragma unroll 8
    for (uint32_t r = ty; r < (uint32_t)kGatherTiles; r += kBlock / kGatherRows)
      if (t0 + r <= ntiles) bounds[((uint64_t)m * (ntiles + 1) + t0 + r) * batch + i0 + tx] = tile[tx][r];
  }
}

// What the lanes need of one row segment, staged in LDS by a thread per row: an even number of entries from pos on, and the
// factor of the row.  A segment of odd length is taken with the entry before it, which is skipped (it is some other
// segment's: reading one past the end could leave the array); only a segment at the very start of the array has none before it:
// its last entry is taken by itself (kCsrHead).
struct __align__(16) CsrSeg {
  int64_t pos;
  uint32_t n;  // entries, kCsrSkip, kCsrHead
  float r;
};
constexpr uint32_t kCsrSkip = 0x80000000u, kCsrHead = 0x40000000u, kCsrCount = 0x3FFFFFFFu;

template <bool PAIRS>
__device__ __forceinline__ CsrSeg csr_segment(const CsrEntries<PAIRS>& e, int64_t start, uint32_t len, float r, const void* dummy) {
  const bool odd = (len & 1u) != 0, head = odd && start == 0;
  const uint32_t n = odd ? (head ? len - 1 : len + 1) : len;
  CsrSeg s;
  s.pos = n == 0 ? e.position_of(dummy) : odd && !head ? start - 1 : start;
  s.n = n | (head ? kCsrHead : odd ? kCsrSkip : 0u);
  s.r = r;
  return s;
}

// Stages minibatch rows first .. first + kCsrRows - 1 of worker m in tile t (those past the minibatch without entries).
template <bool PAIRS>
__device__ __forceinline__ void csr_stage_segments(const CsrEntries<PAIRS>& e, const int64_t* __restrict__ rowbase,
                                                   const uint32_t* __restrict__ bounds, const float* __restrict__ resid,
                                                   uint32_t m, uint32_t batch, uint32_t ntiles, uint32_t t,
                                                   uint32_t first, CsrSeg* seg) {
  if (threadIdx.x >= (uint32_t)kCsrRows) return;
  const uint32_t j = min(first + threadIdx.x, batch - 1);
  const uint32_t* __restrict__ b = bounds + ((uint64_t)m * (ntiles + 1) + t) * batch + j;
  const uint64_t o = (uint64_t)m * batch + j;
  const uint32_t lo = b[0], hi = b[batch];
  const float r = resid != nullptr ? resid[o] : 0.f;
  seg[threadIdx.x] = csr_segment(e, rowbase[o] + lo, first + threadIdx.x < batch ? hi - lo : 0u, r, rowbase + (uint64_t)m * batch);
}

// The first Q kCsrStep entries of U row segments.
template <int U, int Q>
struct CsrBatch {
  uint32_t n[U];
  float r[U];
  CsrTwo two[U][Q];
};

// All loads are issued before any is used and none sits under a condition (the compiler cannot count such loads and makes
// every later wait a wait for all of them): lanes beyond the end of a segment read its last pair again.
template <bool PAIRS, int U, int Q>
__device__ __forceinline__ void csr_request(const CsrEntries<PAIRS>& e, const CsrSeg* seg, uint32_t gl, const void* dummy,
                                            CsrBatch<U, Q>& b) {
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const CsrSeg s = seg[u];
    b.n[u] = s.n;
    b.r[u] = s.r;
    const uint32_t n = s.n & kCsrCount, last = n != 0 ? n - 2 : 0u;
#pragma unroll
    for (int q = 0; q < Q; ++q) b.two[u][q] = e.load2_any(n != 0, s.pos + min(2 * gl + q * kCsrStep, last), dummy);
  }
}

// A load on a rare path has to end there: one that no lane used would count as under way where the paths join again, and the first
// instruction behind that writes to its registers would wait for every load in flight.
__device__ __forceinline__ void csr_arrived(const CsrTwo& e) { asm volatile("" : : "v"(e.col[0]), "v"(e.val[0]), "v"(e.col[1]), "v"(e.val[1])); }

// use(whether, column, value, u, c) for the lane's entries of the batch and of what is behind it; entries that are not the
// lane's come with whether = false (and anything for column and value).  c = 0 .. 3 says which entries of every 2 kCsrStep these
// are: the first or second of the lane's two, in an even or odd load.  LOADS per segment and trip behind the batch.
template <int LOADS, bool PAIRS, int U, int Q, typename F>
__device__ __forceinline__ void csr_use(const CsrEntries<PAIRS>& e, const CsrSeg* seg, uint32_t gl, const void* dummy,
                                        const CsrBatch<U, Q>& b, const F& use) {
  uint32_t longest = 0, any = 0;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t n = b.n[u] & kCsrCount;
    longest = max(longest, n);
    any |= b.n[u];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
      const bool in = 2 * gl + q * kCsrStep < n;
      const bool skip = q == 0 && gl == 0 && (b.n[u] & kCsrSkip) != 0;
      use(in && !skip, b.two[u][q].col[0], b.two[u][q].val[0], u, 2 * (q & 1));
      use(in, b.two[u][q].col[1], b.two[u][q].val[1], u, 2 * (q & 1) + 1);
    }
  }
  for (uint32_t k = Q * kCsrStep; __builtin_amdgcn_ballot_w64(longest > k) != 0ull; k += LOADS * kCsrStep) {
    CsrTwo two[U][LOADS];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t n = b.n[u] & kCsrCount;
#pragma unroll
      for (int q = 0; q < LOADS; ++q)
        two[u][q] = e.load2_any(n != 0, seg[u].pos + min(2 * gl + k + q * kCsrStep, n != 0 ? n - 2 : 0u), dummy);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int q = 0; q < LOADS; ++q) {
        const bool in = 2 * gl + k + q * kCsrStep < (b.n[u] & kCsrCount);
        use(in, two[u][q].col[0], two[u][q].val[0], u, 2 * ((Q + q) & 1));
        use(in, two[u][q].col[1], two[u][q].val[1], u, 2 * ((Q + q) & 1) + 1);
        csr_arrived(two[u][q]);
      }
    }
  }
  if (__builtin_amdgcn_ballot_w64((any & kCsrHead) != 0) != 0ull) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t at = b.n[u] & kCsrCount;
      if (2 * gl == at % kCsrStep && (b.n[u] & kCsrHead) != 0) {
        int32_t c;
        float v;
        e.load(at, c, v);
        use(at / kCsrStep % 2 == 0, c, v, u, 0);
        use(at / kCsrStep % 2 == 1, c, v, u, 2);
        asm volatile("" : : "v"(c), "v"(v));  // (as csr_arrived)
      }
    }
  }
}

// The dot products of U row segments with the tile of w.  An entry's place in its segment modulo 2 kCsrStep = 32 says which of 32
// running sums it goes to, in order; those are added in pairs 16 places apart, then 8, 4, 2 and 1.  (What matters is that the
// chains are of at most 2^tile_shift / 32 products.  With one sum per lane they were four times as long, and the error of z
// against 64 bits 1.1 times as large at 64 entries per segment, twice at 4096.)  The places 16 apart are in the lane, as are
// those 1 apart; in between, lane pairs exchange halves of what they have until each has one sum left.  A segment with an entry
// skipped in front of it has every place shifted by one, under which the pairs stay what they are.
template <int CTRL>
__device__ __forceinline__ float csr_lane_move(float v) {
  return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), CTRL, 0xF, 0xF, false));
}
// Which of the group's places a lane takes: those of lanes 0 .. 3 as they come and those of lanes 4 .. 7 the other way round, so that
// the mirror image of a lane is the one that is 8 entries apart.
__device__ __forceinline__ uint32_t csr_place(uint32_t gl) { return gl < 4 ? gl : 11 - gl; }
// Lane gl is left with sum gl U / kCsrLanes.
template <int U>
__device__ __forceinline__ float csr_group_sums(const float (&acc)[U][4], uint32_t gl) {
  static_assert(kCsrLanes == 8 && (U == 1 || U == 2 || U == 4), "the exchange below");
  constexpr int kMirror = 0x141, kSwap2 = 0x4E, kSwap1 = 0xB1;  // row_half_mirror, quad_perm [2, 3, 0, 1] and [1, 0, 3, 2]
  if constexpr (U == 1) {
    float t[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      t[c] = acc[0][c] + acc[0][c + 2];
      t[c] += csr_lane_move<kMirror>(t[c]);
      t[c] += csr_lane_move<kSwap2>(t[c]);
      t[c] += csr_lane_move<kSwap1>(t[c]);
    }
    return t[0] + t[1];
  } else {
    const bool b4 = (gl & 4u) != 0, b2 = (gl & 2u) != 0, b1 = (gl & 1u) != 0;
    float r[U / 2][2];
#pragma unroll
    for (int k = 0; k < U / 2; ++k) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        const float lower = acc[k][c] + acc[k][c + 2], upper = acc[k + U / 2][c] + acc[k + U / 2][c + 2];
        r[k][c] = (b4 ? upper : lower) + csr_lane_move<kMirror>(b4 ? lower : upper);
      }
    }
    if constexpr (U == 2) {
      float t = (b2 ? r[0][1] : r[0][0]) + csr_lane_move<kSwap2>(b2 ? r[0][0] : r[0][1]);
      t += csr_lane_move<kSwap1>(t);
      return t + csr_lane_move<kSwap2>(t);
    } else {
      float s[2];
#pragma unroll
      for (int c = 0; c < 2; ++c) s[c] = (b2 ? r[1][c] : r[0][c]) + csr_lane_move<kSwap2>(b2 ? r[0][c] : r[1][c]);
      const float t = (b1 ? s[1] : s[0]) + csr_lane_move<kSwap1>(b1 ? s[0] : s[1]);
      return t + csr_lane_move<kSwap1>(t);
    }
  }
}
template <bool PAIRS, int U, int Q>
__device__ __forceinline__ float csr_dot(const CsrEntries<PAIRS>& e, const CsrSeg* seg, uint32_t gl, const void* dummy,
                                         const CsrBatch<U, Q>& b, const float* wtile, uint64_t c0) {
  float acc[U][4] = {};
  csr_use<U == 1 ? 4 : 2>(e, seg, csr_place(gl), dummy, b, [&](bool in, int32_t c, float v, int u, int a) {
    // (left out by choice, not by a factor of 0: the tile's first column may be infinite)
    const float sum = __builtin_fmaf(v, wtile[in ? (uint32_t)c - (uint32_t)c0 : 0u], acc[u][a]);
    acc[u][a] = in ? sum : acc[u][a];
  });
  return csr_group_sums(acc, gl);
}

template <bool PAIRS>
__global__ __launch_bounds__(kCsrThreads) void csr_z_kernel(const int32_t* const* __restrict__ cols,
                                                            const float* const* __restrict__ vals,
                                                            const int64_t* __restrict__ rowbase,
                                                            const uint32_t* __restrict__ bounds,
                                                            const float* __restrict__ w, float* __restrict__ zparts,
                                                            uint64_t d, uint32_t batch, uint32_t ntiles,
                                                            uint32_t tile_shift) {
  extern __shared__ float wtile[];  // w over the tile's columns
  __shared__ CsrSeg seg[kCsrRows];
  // workers vary fastest across the grid: the workgroups that run side by side share one tile of w
  const uint32_t m = blockIdx.x, t = blockIdx.y;
  const uint32_t T = 1u << tile_shift;
  const uint64_t c0 = (uint64_t)t << tile_shift;
  float* __restrict__ zpart = zparts + ((uint64_t)m * ntiles + t) * batch;
  if (tile_shift == kCsrTileShift && c0 + T <= d && (reinterpret_cast<uintptr_t>(w) & 15u) == 0) {
    // full-size tile: all its loads in flight at once, then the LDS stores
    constexpr int kVec = (1 << kCsrTileShift) / (4 * kCsrThreads);
    const float4* __restrict__ w4 = reinterpret_cast<const float4*>(w + c0);
    float4* tile4 = reinterpret_cast<float4*>(wtile);
    float4 tmp[kVec];
#pragma unroll
    for (int q = 0; q < kVec; ++q) tmp[q] = w4[q * kCsrThreads + threadIdx.x];
#pragma unroll
    for (int q = 0; q < kVec; ++q) tile4[q * kCsrThreads + threadIdx.x] = tmp[q];
  } else {
    for (uint32_t j = threadIdx.x; j < T; j += kCsrThreads) wtile[j] = c0 + j < d ? w[c0 + j] : 0.f;
  }
  const CsrEntries<PAIRS> e(cols[m], vals[m]);
  const uint32_t group = threadIdx.x / kCsrLanes, gl = threadIdx.x % kCsrLanes;
  const void* dummy = rowbase + (uint64_t)m * batch;
  for (uint32_t first = 0; first < batch; first += kCsrRows) {
    __syncthreads();
    csr_stage_segments(e, rowbase, bounds, nullptr, m, batch, ntiles, t, first, seg);
    __syncthreads();
    const uint32_t j0 = group * kCsrUnroll;
    CsrBatch<kCsrUnroll, kCsrLoads> b;
    csr_request(e, seg + j0, csr_place(gl), dummy, b);
    const float sum = csr_dot(e, seg + j0, gl, dummy, b, wtile, c0);
    const uint32_t i = first + j0 + gl / (kCsrLanes / kCsrUnroll);
    if (gl % (kCsrLanes / kCsrUnroll) == 0 && i < batch) zpart[i] = sum;
  }
}

// Workgroup barrier that orders LDS traffic only: global loads and stores still in flight are not
// waited for (__syncthreads would wait until every one of them has come back).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The same pass with two adjacent tiles of w (2^15 columns, 128 KiB) in LDS and kCsrWideLoads loads per
// segment: the row segments are twice as long, so fewer of the 128-byte memory lines they touch are
// partial ones.  (Random contiguous segments deliver 2.2 TB/s of useful bytes at 64 bytes per
// segment and 3.2 TB/s at 128; this pass is bound by exactly that.)  One partial sum per row and pair
// of tiles: zparts[m][pair][i].
//
// A trip is P pieces of U segments per lane group: one segment while up to three such pieces hold a trip's part of the minibatch
// (csr_pieces), so that it does not go through pieces of empty segments (iterations M = 8, d = 2^23, B = 64 252 us with four of them, 199
// with one; M = 3, d = 2^22, B = 200 77.0 / 71.9 with two; with three here and in the gradient pass instead of two of two and four d =
// 2^22, M = 9, B = 257 209 / 200; d = 2^24, M = 8, B = 260 461 / 449; 40 entries a row, d = 2^22, M = 32, B = 260 296 / 280; 400, B = 700
// 488 / 479), else two pieces of two.  All pieces but one are on their way while one is worked on: at d = 2^24, M = 64, B = 512 959 us with
// two halves of which one is asked for ahead of the other's arithmetic, 928 with each asked for behind its own, 923 with four pieces of one
// segment (iterations alike: 3296 / 3295).  Where most segments are empty the pass is bound by its vector instructions, of which four
// pieces have more, and by what a step costs by itself: d = 2^22, M = 64, 40 entries a row 100 us with four pieces and two divisions and
// four loads a step, 92 with a step carried along, 89 so; d = 2^21, M = 32, 20 entries a row 38.1 / 37.1 / 36.3.
// ONE: a workgroup has one step (one worker, one trip) and asks for nothing ahead, which would be two rounds of bounds and one of entries
// that are not there: d = 2^21, M = 4, 200 entries a row, B = 512 12.4 us, of the iteration's 52.5, and 49.6 this way; d = 2^24, M = 3, B =
// 512 294 / 283; d = 2^22, M = 8, 40 entries a row, B = 512 116 / 110.
inline int csr_pieces(uint32_t batch) {  // of the minibatch in as few trips as there have to be, dealt out evenly
  const uint32_t trips = (batch + kCsrRows - 1) / kCsrRows, rows = (batch + trips - 1) / trips;
  return (int)((rows + kCsrGroups - 1) / kCsrGroups);
}
template <bool PAIRS, int P, int U, bool ONE>
__global__ __launch_bounds__(kCsrThreads) void csr_z_wide_kernel(const int32_t* const* __restrict__ cols,
                                                                 const float* const* __restrict__ vals,
                                                                 const int64_t* __restrict__ rowbase,
                                                                 const uint32_t* __restrict__ bounds,
                                                                 const float* __restrict__ w,
                                                                 float* __restrict__ zparts, uint64_t d,
                                                                 uint32_t batch, uint32_t ntiles, uint32_t npairs,
                                                                 uint32_t M, uint32_t workers_per_block) {
  constexpr int kPieceRows = U * (int)kCsrGroups, kRows = P * kPieceRows;
  extern __shared__ float wtile[];  // w over the columns of both tiles
  __shared__ CsrSeg seg[ONE ? 1 : 3][kRows];  // of this step, the next one and the one after it
  const uint32_t pair = tile_of_workgroup(blockIdx.x, npairs);
  const uint32_t t_lo = 2 * pair, t_hi = min(2 * pair + 2, ntiles);
  constexpr uint32_t T = 2u << kCsrTileShift;
  const uint64_t c0 = (uint64_t)t_lo << kCsrTileShift;
  // The tiles of w serve several workers in turn.  A step is one trip of kRows minibatch rows of one worker, taken in
  // pieces: a piece is asked for again, of the next step, as soon as it has been worked on, so that all others are on their way while one
  // is worked on.  The segment bounds are fetched three steps ahead and staged two ahead (every thread fetches, the row
  // index clamped, so that no load sits under a condition); past the last step the segments are empty.
  static_assert(kCsrThreads >= kRows, "one thread per staged row");
  const uint32_t m_first = blockIdx.y * workers_per_block, m_last = min(m_first + workers_per_block, M);
  struct Step {  // (carried along: made from a number it was a division and two loads for each of the four in the loop)
    uint32_t m, first;  // worker, first row; past the last step m_last and above
    CsrEntries<PAIRS> e;
    const int64_t* rowbase;
  };
  auto step_at = [&](uint32_t m, uint32_t first) {
    const uint32_t mc = min(m, m_last - 1);
    return Step{m, first, CsrEntries<PAIRS>(cols[mc], vals[mc]), rowbase + (uint64_t)mc * batch};
  };
  auto behind = [&](const Step& s) { return s.first + kRows < batch ? step_at(s.m, s.first + kRows) : step_at(s.m + 1, 0); };
  struct Bounds {
    uint32_t lo, hi;
    int64_t base;
  };
  auto fetch = [&](const Step& s) {
    const uint32_t j = s.first + min(threadIdx.x, min((uint32_t)kRows, batch - s.first) - 1u);
    const uint32_t* __restrict__ b = bounds + (uint64_t)min(s.m, m_last - 1) * (ntiles + 1) * batch;
    return Bounds{b[(uint64_t)t_lo * batch + j], b[(uint64_t)t_hi * batch + j], s.rowbase[j]};
  };
  // Those of the first three steps are asked for together, ahead of the tiles of w: one after the other behind the tiles, each with its
  // wait, they held up the workgroups of few steps (iterations at d = 2^20, M = 8, B = 512 48.7 -> 48.2 us, B = 1000 64.3 -> 63.4; d = 2^22,
  // M = 8, B = 512 143.8 -> 142.3, with the same order in the gradient pass).
  Step now = step_at(m_first, 0), next = ONE ? now : behind(now), third = ONE ? now : behind(next);
  const Bounds first_bounds = fetch(now), second_bounds = ONE ? first_bounds : fetch(next);
  Bounds fetched = ONE ? first_bounds : fetch(third);
  if (c0 + T <= d && (reinterpret_cast<uintptr_t>(w) & 15u) == 0) {
    constexpr int kVec = (int)(T / (4 * kCsrThreads));  // 8 float4 per thread, four in flight at a time
    const float4* __restrict__ w4 = reinterpret_cast<const float4*>(w + c0);
    float4* tile4 = reinterpret_cast<float4*>(wtile);
#pragma unroll
    for (int q0 = 0; q0 < kVec; q0 += 4) {
      float4 tmp[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) tmp[q] = w4[(q0 + q) * kCsrThreads + threadIdx.x];
#pragma unroll
      for (int q = 0; q < 4; ++q) tile4[(q0 + q) * kCsrThreads + threadIdx.x] = tmp[q];
    }
  } else {
    for (uint32_t j = threadIdx.x; j < T; j += kCsrThreads) wtile[j] = c0 + j < d ? w[c0 + j] : 0.f;
  }
  const uint32_t group = threadIdx.x / kCsrLanes, gl = threadIdx.x % kCsrLanes;
  auto stage = [&](const Step& s, uint32_t buf, const Bounds& f) {
    if (threadIdx.x < (uint32_t)kRows)
      seg[buf][threadIdx.x] = csr_segment(s.e, f.base + f.lo, s.m < m_last && s.first + threadIdx.x < batch ? f.hi - f.lo : 0u, 0.f, s.rowbase);
  };
  typedef CsrBatch<U, kCsrWideLoads> Piece;
  Piece pieces[P];
  auto request = [&](const Step& s, uint32_t buf, int k) {
    csr_request(s.e, seg[buf] + k * kPieceRows + group * U, csr_place(gl), s.rowbase, pieces[k]);
  };
  auto dot = [&](const Step& s, uint32_t buf, int k) {
    const uint32_t j0 = k * kPieceRows + group * U;
    const float sum = csr_dot(s.e, seg[buf] + j0, gl, s.rowbase, pieces[k], wtile, c0);
    const uint32_t i = s.first + j0 + gl / (kCsrLanes / U);
    if (gl % (kCsrLanes / U) == 0 && i < batch) zparts[((uint64_t)s.m * npairs + pair) * batch + i] = sum;
  };
  stage(now, 0, first_bounds);
  if (!ONE) stage(next, 1, second_bounds);
  __syncthreads();
#pragma unroll
  for (int k = 0; k < P; ++k) request(now, 0, k);
  if (ONE) {
#pragma unroll
    for (int k = 0; k < P; ++k) dot(now, 0, k);
    return;
  }
  uint32_t buf = 0;
  while (now.m < m_last) {
    const uint32_t buf1 = buf == 2 ? 0 : buf + 1, buf2 = buf1 == 2 ? 0 : buf1 + 1;
    const Step fourth = behind(third);
#pragma unroll
    for (int k = 0; k < P; ++k) {
      dot(now, buf, k);
      request(next, buf1, k);
      if (k == 0) {
        stage(third, buf2, fetched);
        fetched = fetch(fourth);
      }
    }
    lds_barrier();  // the bounds of the third step are in place
    buf = buf1;
    now = next;
    next = third;
    third = fourth;
  }
}

// r[m][i] = (sigma(z_i) - y_i) / B with z_i = sum over the tiles of the partial dot products
// zpart[m][t][i]: what the gradient pass multiplies every stored entry of row i by.  A workgroup takes
// kReduceRows rows of one worker; four groups of threads add a quarter of the partial sums each (four
// accumulators per thread, fixed order), and the quarters are added in order.
constexpr int kReduceRows = kBlock / 4;
__global__ __launch_bounds__(kBlock) void csr_z_reduce_kernel(const float* __restrict__ zpart,
                                                              const float* const* __restrict__ ys,
                                                              const uint32_t* __restrict__ idx, float* __restrict__ r,
                                                              uint32_t batch, uint32_t ntiles, float inv_b) {
  __shared__ float quarter_sum[3][kReduceRows];
  const uint32_t m = blockIdx.y;
  const uint32_t lane_row = threadIdx.x % kReduceRows, quarter = threadIdx.x / kReduceRows;
  const uint32_t i = min(blockIdx.x * kReduceRows + lane_row, batch - 1);  // clamped: every thread meets the barrier
  const uint32_t per = (ntiles + 3) / 4;
  const uint32_t t_begin = min(quarter * per, ntiles), t_end = min(t_begin + per, ntiles);
  const float* __restrict__ p = zpart + (uint64_t)m * ntiles * batch + i;
  float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
  uint32_t t = t_begin;
  for (; t + 4 <= t_end; t += 4) {
    a0 += p[(uint64_t)t * batch];
    a1 += p[(uint64_t)(t + 1) * batch];
    a2 += p[(uint64_t)(t + 2) * batch];
    a3 += p[(uint64_t)(t + 3) * batch];
  }
  for (; t < t_end; ++t) a0 += p[(uint64_t)t * batch];
  const float part = (a0 + a1) + (a2 + a3);
  if (quarter > 0) quarter_sum[quarter - 1][lane_row] = part;
  __syncthreads();
  if (quarter == 0 && blockIdx.x * kReduceRows + lane_row < batch) {
    const float z = ((part + quarter_sum[0][lane_row]) + quarter_sum[1][lane_row]) + quarter_sum[2][lane_row];
    const uint64_t o = (uint64_t)m * batch + i;
    r[o] = logistic_residual(z, as_global(ys[m])[idx[o]]) * inv_b;
  }
}

// Gradient pass: one workgroup per (worker, tile); every minibatch row adds (r_i / B) val into the
// fp64 tile in LDS, and the finished tile is written once (+ l2 w).  FUSE: the write-out also leaves
// the tile's largest |normalize(g)| for the scale pass (partials[tile][worker]), which then need not
// read g again: +0.35 ms here against a 0.7 ms pass saved at d = 2^24, M = 64.
// Where the time goes at d = 2^24, M = 64, B = 512 (2.47 ms): without the adds 2.32 ms, without the
// write-out of g 1.96 ms -- the rest is reading the entries in 66-byte segments, at the rate such
// segments are delivered at all (see the paired dot-product pass).
// Taken apart the same way, zeroing + write-out alone take 0.85 ms and staging + entry loads alone
// 1.50 ms: per compute unit the phases simply add up.  Variants that measured slower or no faster:
// prefetching the next tile's entries during the write-out (software pipelining over a run of
// tiles); tiles of half the width with two workgroups per compute unit, so that one writes while
// the other reads (2.79 ms: the segments of 33 bytes cost more than the overlap gains); fetching the
// entries of two adjacent tiles at once into registers (one wavefront per row, segment descriptors
// as wavefront-uniform values, no spills) and working through the tiles in two phases with the first
// tile's stores left in flight (2.66 ms: its loads alone 1.26 ms, its write-out alone 1.06 ms, both
// together more than their sum -- the random reads and the streaming writes compete in memory);
// a run of four tiles per workgroup with the next tile's segment bounds prefetched, the tile cleared
// by its own write-out and barriers that wait for LDS traffic only (+0.3 ms).  What the variants that
// keep a workgroup alive across tiles have in common: loads and stores share one in-order counter,
// so the wait for the next tile's entries is also a wait for the previous tile's stores to be
// acknowledged, while a workgroup that ends after its write-out leaves them to drain behind it.
template <bool FUSE, bool PAIRS>
__global__ __launch_bounds__(kCsrThreads) void csr_grad_kernel(const int32_t* const* __restrict__ cols,
                                                               const float* const* __restrict__ vals,
                                                               const int64_t* __restrict__ rowbase,
                                                               const uint32_t* __restrict__ bounds,
                                                               const float* __restrict__ resid,
                                                               const float* __restrict__ w, float* __restrict__ g,
                                                               uint64_t d, uint32_t batch, uint32_t ntiles,
                                                               uint32_t tile_shift, float l2, ScaleFusion fuse) {
  extern __shared__ double gtile[];  // g over the tile's columns, accumulated in fp64
  __shared__ CsrSeg seg[kCsrRows];
  __shared__ float red[kCsrThreads / kWave];
  const uint32_t m = blockIdx.x, t = blockIdx.y;
  const uint32_t T = 1u << tile_shift;
  const uint64_t c0 = (uint64_t)t << tile_shift;
  for (uint32_t j = threadIdx.x; j < T; j += kCsrThreads) gtile[j] = 0.0;
  // fused scale pass: the reference of the thread's columns, fetched first so that nothing waits for it
  constexpr int kPer = (1 << kCsrTileShift) / (4 * kCsrThreads);
  float4 r1[kPer], r2[kPer];
  if (FUSE) {
#pragma unroll
    for (int k = 0; k < kPer; ++k) load_refs4(fuse, c0 + 4 * ((uint32_t)k * kCsrThreads + threadIdx.x), r1[k], r2[k]);
  }
  const CsrEntries<PAIRS> e(cols[m], vals[m]);
  const uint32_t group = threadIdx.x / kCsrLanes, gl = threadIdx.x % kCsrLanes;
  const void* dummy = rowbase + (uint64_t)m * batch;
  for (uint32_t first = 0; first < batch; first += kCsrRows) {
    __syncthreads();
    csr_stage_segments(e, rowbase, bounds, resid, m, batch, ntiles, t, first, seg);
    __syncthreads();
    const uint32_t j0 = group * kCsrUnroll;
    CsrBatch<kCsrUnroll, kCsrLoads> b;
    csr_request(e, seg + j0, gl, dummy, b);
    csr_use<1>(e, seg + j0, gl, dummy, b, [&](bool in, int32_t c, float v, int u, int) {
      if (in) atomicAdd(&gtile[(uint32_t)c - (uint32_t)c0], (double)(b.r[u] * v));
    });
  }
  float* __restrict__ out = g + (uint64_t)m * d;
  if (FUSE) {
    // Fused scale pass (the launcher has checked: full tiles of 2^kCsrTileShift columns, no l2 term,
    // aligned rows).  The reference of the thread's columns is fetched before the barrier, so the wait
    // for it runs while the slower wavefronts finish their adds.
    __syncthreads();
    float4* __restrict__ out4 = reinterpret_cast<float4*>(out + c0);
    float amax = 0.f;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint32_t q = (uint32_t)k * kCsrThreads + threadIdx.x;
      const float4 o = make_float4((float)gtile[4 * q], (float)gtile[4 * q + 1], (float)gtile[4 * q + 2],
                                   (float)gtile[4 * q + 3]);
      store_stream(out4 + q, o);
      amax = fmaxf(amax, absmax4(fuse, o, r1[k], r2[k]));
    }
    amax = wave_max_nonneg(amax);
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = amax;
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
      for (int k = 1; k < kCsrThreads / kWave; ++k) amax = fmaxf(amax, red[k]);
      fuse.partials[(uint64_t)t * gridDim.x + m] = amax;
    }
    return;
  }
  __syncthreads();
  if (c0 + T <= d && T % 4 == 0 && l2 == 0.f && ((reinterpret_cast<uintptr_t>(out) | (d * 4)) & 15u) == 0) {
    float4* __restrict__ out4 = reinterpret_cast<float4*>(out + c0);
    for (uint32_t q = threadIdx.x; q < T / 4; q += kCsrThreads)
      store_stream(out4 + q, make_float4((float)gtile[4 * q], (float)gtile[4 * q + 1], (float)gtile[4 * q + 2],
                                         (float)gtile[4 * q + 3]));
  } else {
    for (uint32_t j = threadIdx.x; j < T; j += kCsrThreads) {
      if (c0 + j < d) out[c0 + j] = l2 != 0.f ? __builtin_fmaf(l2, w[c0 + j], (float)gtile[j]) : (float)gtile[j];
    }
  }
}

// Where the pipelined kernels below keep column c of a tile (2^kCsrTileShift columns, from a multiple of that on): the four
// columns of a thread's float4 as two pairs, the first pairs of all threads in the lower half of the tile, the second in
// the upper, so that the lanes of a wavefront read and clear 16 bytes each next to one another (with the columns in order they
// are 32 bytes apart and meet on half of the banks).
__device__ __forceinline__ uint32_t csr_slot(uint32_t c) {
  constexpr uint32_t T = 1u << kCsrTileShift;
  return ((c >> 1) & (T / 2 - 2)) | (c & 1u) | ((c & 2u) * (T / 4));
}
// Columns 4 q .. 4 q + 3 of the tile, which are cleared.
__device__ __forceinline__ float4 csr_take4(double* gtile, uint32_t q) {
  typedef double v2d_t __attribute__((ext_vector_type(2)));
  v2d_t* lower = reinterpret_cast<v2d_t*>(gtile) + q;
  v2d_t* upper = lower + (1u << kCsrTileShift) / 4;
  const v2d_t a = *lower, b = *upper;
  *lower = *upper = v2d_t{0.0, 0.0};
  return make_float4((float)a.x, (float)a.y, (float)b.x, (float)b.y);
}

// The gradient pass with the fused scale pass for the common case -- full tiles, no l2 term, at most
// kCsrRows minibatch rows, 16-byte aligned rows of g -- as a software pipeline over a run of tiles of one
// worker.  With one 128 KiB workgroup per compute unit nothing else hides a tile's chain of
// dependent memory round trips (segment bounds, then entries, then the write-out), so the workgroup
// overlaps them itself:
//   while tile t's entries are added into the LDS tile, the segment bounds of tile t+1 are on their way;
//   after the barrier that ends the adds, the entries of tile t+1 are requested BEFORE tile t is written
//   out: loads and stores retire through one in-order counter, so the wait for those entries at the
//   top of the next round only has to leave the (younger) stores outstanding, and the write-out, the
//   clearing of the tile and the stores' acknowledgement all run under the entries' latency.
// The barriers order LDS traffic only.  Lanes beyond a segment's length hold its last pair once more, which csr_use tells
// them to leave out.
template <bool PAIRS, int NORM>
__global__ __launch_bounds__(kCsrThreads) void csr_grad_run_kernel(const int32_t* const* __restrict__ cols,
                                                                   const float* const* __restrict__ vals,
                                                                   const int64_t* __restrict__ rowbase,
                                                                   const uint32_t* __restrict__ bounds,
                                                                   const float* __restrict__ resid,
                                                                   float* __restrict__ g, uint64_t d, uint32_t batch,
                                                                   uint32_t ntiles, ScaleFusion fuse) {
  extern __shared__ double gtile[];  // g over the tile's columns, accumulated in fp64
  __shared__ CsrSeg seg[2][kCsrRows];
  // By parity of the round: read behind the next round's first barrier, where wavefronts that are ahead already store their own maxima
  // of that round.
  __shared__ float red[2][kCsrThreads / kWave];
  constexpr uint32_t T = 1u << kCsrTileShift;
  constexpr int kPer = (int)(T / (4 * kCsrThreads));
  const uint32_t m = blockIdx.x;
  // Workgroup r of a worker takes tiles r, r + stride, r + 2 stride, ... (stride = workgroups per worker):
  // the workgroups of one worker that run side by side are then on ADJACENT tiles, and the 128-byte memory
  // lines that hold the end of one tile's row segment and the start of the next tile's are fetched from
  // HBM once and shared in the caches (with consecutive tiles per workgroup they were fetched twice, a
  // round apart: 7.8 GB read per launch instead of 4.6 at d = 2^24, 64 workers).
  const uint32_t stride = gridDim.y;
  const uint32_t t_first = blockIdx.y;
  const uint32_t row = min(threadIdx.x, batch - 1);  // every thread fetches bounds: no load under a condition
  const uint32_t* __restrict__ b = bounds + (uint64_t)m * (ntiles + 1) * batch + row;
  const int64_t base = rowbase[(uint64_t)m * batch + row];
  const bool has_row = threadIdx.x < batch;
  const float res = resid[(uint64_t)m * batch + row];
  const CsrEntries<PAIRS> e(cols[m], vals[m]);
  const void* dummy = rowbase + (uint64_t)m * batch;  // (the workspace goes on behind the last row's)
  auto stage = [&](uint32_t buf, int64_t start, uint32_t len) {
    if (threadIdx.x < (uint32_t)kCsrRows) seg[buf][threadIdx.x] = csr_segment(e, start, len, res, dummy);
  };
  {
    const uint32_t lo = b[(uint64_t)t_first * batch], hi = b[(uint64_t)(t_first + 1) * batch];
    for (uint32_t j = threadIdx.x; j < T; j += kCsrThreads) gtile[j] = 0.0;
    stage(0, base + lo, has_row ? hi - lo : 0u);
  }
  const uint32_t group = threadIdx.x / kCsrLanes, gl = threadIdx.x % kCsrLanes;
  const uint32_t j0 = group * kCsrUnroll;
  float* __restrict__ out = g + (uint64_t)m * d;
  CsrBatch<kCsrUnroll, kCsrLoads> next;
  auto request = [&](uint32_t buf) { csr_request(e, seg[buf] + j0, gl, dummy, next); };
  auto parity = [&](uint32_t t) { return ((t - t_first) / stride) & 1u; };
  auto store_maximum = [&](uint32_t t, uint32_t p) {  // by thread 0, once red[p] holds tile t's wavefront maxima
    float mx = red[p][0];
#pragma unroll
    for (int k = 1; k < kCsrThreads / kWave; ++k) mx = fmaxf(mx, red[p][k]);
    fuse.partials[(uint64_t)t * gridDim.x + m] = mx;
  };
  auto round = [&](uint32_t t) {
    const uint32_t cur = parity(t);
    const uint64_t c0 = (uint64_t)t << kCsrTileShift;
    // bounds of the workgroup's next tile (clamped: a fetch, never a branch); past its last tile the lengths become 0
    const bool more = t + stride < ntiles;
    const uint32_t tn = more ? t + stride : t;
    const uint32_t nlo = b[(uint64_t)tn * batch], nhi = b[(uint64_t)(tn + 1) * batch];
    csr_use<1>(e, seg[cur] + j0, gl, dummy, next, [&](bool in, int32_t c, float v, int u, int) {
      if (in) atomicAdd(&gtile[csr_slot((uint32_t)c)], (double)(next.r[u] * v));
    });
    stage(cur ^ 1u, base + nlo, (has_row && more) ? nhi - nlo : 0u);
    lds_barrier();  // every add of tile t has been made; the segments of tile t+1 are staged
    if (t > t_first && threadIdx.x == 0) store_maximum(t - stride, cur ^ 1u);  // older than the request below: need not be counted
    // the reference of the thread's columns for the fused scale pass, asked for ahead of the entries (loads
    // come back in order: asked for after them, its arrival would be theirs); the kind of normalisation is a
    // template argument so that no branch surrounds these loads either
    float4 r1[kPer], r2[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k)
      load_refs4_t<NORM>(fuse, c0 / 4 + (uint32_t)k * kCsrThreads + threadIdx.x, r1[k], r2[k]);
    request(cur ^ 1u);  // before the stores below
    float4* __restrict__ out4 = reinterpret_cast<float4*>(out + c0);
    float amax = 0.f;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint32_t q = (uint32_t)k * kCsrThreads + threadIdx.x;
      const float4 o = csr_take4(gtile, q);
      store_stream(out4 + q, o);
      amax = fmaxf(amax, absmax4_t<NORM>(fuse, o, r1[k], r2[k]));
    }
    amax = wave_max_nonneg(amax);
    if (threadIdx.x % kWave == 0) red[cur][threadIdx.x / kWave] = amax;
    lds_barrier();  // the tile is clear again; red is complete
  };
  lds_barrier();
  request(0);
  // The first round stands apart from the loop: at the loop's head the compiler takes the weaker of what
  // its two ways in allow to stay in flight, and only after a write-out are there stores that may.
  round(t_first);
  uint32_t t_last = t_first;
  for (uint32_t t = t_first + stride; t < ntiles; t += stride) {
    round(t);
    t_last = t;
  }
  if (threadIdx.x == 0) store_maximum(t_last, parity(t_last));
}

// The same pipeline turned by ninety degrees: a workgroup stays on ONE column tile and takes the workers
// m_first .. m_end - 1 in turn.  What a round needs of its worker -- segment bounds, row starts and
// residuals of the minibatch rows, the shard's entry array -- is fetched three rounds ahead and staged in LDS two
// ahead, its entries are asked for one ahead.  Three buffers do: what round m stages (of worker m + 2) takes the place of worker m - 1's,
// which was last read before the first barrier of round m - 1.  What belongs to the tile -- the reference of the thread's columns for the
// fused scale pass -- is fetched once and stays in registers, where the kernel above asks for it again
// every round (64 workers: the reference read 64 times over, a quarter more load instructions per round
// in a kernel bound by how fast a compute unit issues them; gradient pass 2.34 -> 2.13 ms at d = 2^24).
// Workgroups that run side by side are on adjacent tiles of the same worker, so the memory lines shared
// by the end of one tile's row segment and the start of the next tile's are still fetched once.
// FULL: d is a multiple of the tile; else rows of g start at any 4-byte boundary and the last tile reaches past their end.
// (Iterations with the tile's columns in csr_slot's order and every length of rows here, at 0.1 % density, B = 512: d = 2^24, M =
// 32 2158 -> 1941 us with the entries two to a lane; d = 2^24 - 5, which took a workgroup per tile and worker and a scale pass
// before, 2890 -> 2065; d = 5000001, M = 16 483 -> 370; d = 1000003, M = 8 75 -> 61.)
template <bool PAIRS, int NORM, bool FULL, int P>
__global__ __launch_bounds__(kCsrThreads) void csr_grad_workers_kernel(const int32_t* const* __restrict__ cols,
                                                                       const float* const* __restrict__ vals,
                                                                       const int64_t* __restrict__ rowbase,
                                                                       const uint32_t* __restrict__ bounds,
                                                                       const float* __restrict__ resid,
                                                                       float* __restrict__ g, uint64_t d, uint32_t batch,
                                                                       uint32_t ntiles, uint32_t M, uint32_t per_group,
                                                                       ScaleFusion fuse) {
  constexpr int kRows = P * (int)kCsrGroups;  // (the whole minibatch)
  extern __shared__ double gtile[];  // g over the tile's columns, accumulated in fp64
  __shared__ CsrSeg seg[3][kRows];  // of this worker, the next one and the one after it
  __shared__ float red[2][kCsrThreads / kWave];  // by parity of the round: read in the round after it was written
  constexpr uint32_t T = 1u << kCsrTileShift;
  constexpr int kPer = (int)(T / (4 * kCsrThreads));
  const uint32_t t = tile_of_workgroup(blockIdx.x, ntiles);
  const uint32_t m_first = blockIdx.y * per_group;
  const uint32_t m_end = min(m_first + per_group, M);
  const uint64_t c0 = (uint64_t)t << kCsrTileShift;
  const bool whole = FULL || c0 + T <= d;
  const uint32_t row = min(threadIdx.x, batch - 1);  // every thread fetches its row's data: no load under a condition
  const bool has_row = threadIdx.x < batch;
  // Per-worker arrays are addressed as (wavefront-uniform start of the worker's part) + (the thread's 32-bit
  // offset): no per-thread 64-bit pointer has to live across the rounds (registers are what this kernel is
  // short of, and a spilled pointer's reload at the head of a round would wait for every load in flight).
  const uint64_t per_worker = (uint64_t)(ntiles + 1) * batch;
  const uint32_t tb_row = t * batch + row;  // bounds of worker m, this tile, this row: bounds[m per_worker + tb_row]
  auto bounds_of = [&](uint32_t m) { return as_global(bounds + (uint64_t)m * per_worker); };
  auto rowbase_of = [&](uint32_t m) { return as_global(rowbase + (uint64_t)m * batch); };
  auto resid_of = [&](uint32_t m) { return as_global(resid + (uint64_t)m * batch); };
  auto dummy_of = [&](uint32_t m) { return rowbase + (uint64_t)m * batch; };
  auto stage = [&](uint32_t m, uint32_t buf, int64_t start, uint32_t len, float r) {
    if (threadIdx.x < (uint32_t)kRows) seg[buf][threadIdx.x] = csr_segment(CsrEntries<PAIRS>(cols[m], vals[m]), start, len, r, dummy_of(m));
  };
  // what a worker's round needs (worker index clamped: a fetch, never a branch)
  struct Row {
    uint32_t lo, hi;
    int64_t base;
    float res;
  };
  auto fetch = [&](uint32_t m) {
    const uint32_t mc = min(m, m_end - 1);
    return Row{bounds_of(mc)[tb_row], bounds_of(mc)[tb_row + batch], rowbase_of(mc)[row], resid_of(mc)[row]};
  };
  auto stage_fetched = [&](uint32_t m, uint32_t buf, const Row& f) {  // past the last worker the lengths are 0
    stage(min(m, m_end - 1), buf, f.base + f.lo, has_row && m < m_end ? f.hi - f.lo : 0u, f.res);
  };
  // Those of the first workers are asked for together: one after the other, each with its wait, they held up a group of two workers
  // (d = 2^20, M = 8, B = 257 13.7 -> 13.2 us).
  const Row first_worker = fetch(m_first), second_worker = fetch(m_first + 1);
  Row fetched = fetch(m_first + 2);
  for (uint32_t j = threadIdx.x; j < T; j += kCsrThreads) gtile[j] = 0.0;
  stage_fetched(m_first, 0, first_worker);
  stage_fetched(m_first + 1, 1, second_worker);
  // the reference of the thread's columns: the same for every worker
  float4 r1[kPer], r2[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k)
    if (whole)
      load_refs4_t<NORM>(fuse, c0 / 4 + (uint32_t)k * kCsrThreads + threadIdx.x, r1[k], r2[k]);
    else
      load_refs4_end<NORM>(fuse, c0 + 4 * ((uint32_t)k * kCsrThreads + threadIdx.x), d, r1[k], r2[k]);
  const uint32_t group = threadIdx.x / kCsrLanes, gl = threadIdx.x % kCsrLanes;
  // A worker's segments are taken in pieces: a piece is asked for again, of the next worker, as soon as it has been added, so that the entries
  // of all others are on their way meanwhile, behind the barriers and during the write-out.  (All of a worker's entries asked for behind
  // the barrier that ends the adds: none are on their way during the adds.  d = 2^24, M = 64, B = 512: 1900 us, of which 675 go with the stores and
  // 130 with the adds; two halves 1650, four pieces 1624.  Waiting for the stores less, by an order in which the bounds are asked for ahead of them,
  // made that form slower, 1990: reads and writes mixed cost more than apart.)
  typedef CsrBatch<1, kCsrLoads> Piece;
  Piece pieces[P];
  auto at = [&](uint32_t buf, int k) { return seg[buf] + k * (int)kCsrGroups + group; };
  auto request = [&](uint32_t m, uint32_t buf, int k) {
    const uint32_t mc = min(m, m_end - 1);
    csr_request(CsrEntries<PAIRS>(cols[mc], vals[mc]), at(buf, k), gl, dummy_of(mc), pieces[k]);
  };
  auto add = [&](uint32_t m, uint32_t buf, int k) {
    csr_use<4>(CsrEntries<PAIRS>(cols[m], vals[m]), at(buf, k), gl, dummy_of(m), pieces[k], [&](bool in, int32_t c, float v, int u, int) {
      if (in) atomicAdd(&gtile[csr_slot((uint32_t)c)], (double)(pieces[k].r[u] * v));
    });
  };
  auto store_maximum = [&](uint32_t m) {  // by thread 0, once red holds worker m's wavefront maxima
    const float* rm = red[(m - m_first) & 1u];
    float mx = rm[0];
#pragma unroll
    for (int k = 1; k < kCsrThreads / kWave; ++k) mx = fmaxf(mx, rm[k]);
    fuse.partials[(uint64_t)t * M + m] = mx;
  };
  uint32_t buf = 0;
  auto round = [&](uint32_t m) {
    const uint32_t cur = (m - m_first) & 1u, next = buf == 2 ? 0 : buf + 1, after = next == 2 ? 0 : next + 1;
#pragma unroll
    for (int k = 0; k < P; ++k) {
      add(m, buf, k);
      request(m + 1, next, k);
      if (k == 0) stage_fetched(m + 2, after, fetched);
    }
    fetched = fetch(m + 3);
    lds_barrier();  // every add of worker m has been made; the segments of worker m + 2 are staged
    if (m > m_first && threadIdx.x == 0) store_maximum(m - 1);
    buf = next;
    float* __restrict__ out = g + (uint64_t)m * d + c0;
    float4* __restrict__ out4 = reinterpret_cast<float4*>(out);
    float amax = 0.f;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
      const uint32_t q = (uint32_t)k * kCsrThreads + threadIdx.x;
      const float4 o = csr_take4(gtile, q);
      if (FULL)
        store_stream(out4 + q, o);
      else if (whole)
        store4_stream_any(out, q, o);
      else
        store4_within(out, 4 * q, d - c0, o);
      amax = fmaxf(amax, absmax4_t<NORM>(fuse, o, r1[k], r2[k]));
    }
    amax = wave_max_nonneg(amax);
    if (threadIdx.x % kWave == 0) red[cur][threadIdx.x / kWave] = amax;
    lds_barrier();  // the tile is clear again; red is complete
  };
  lds_barrier();
#pragma unroll
  for (int k = 0; k < P; ++k) request(m_first, 0, k);
  // the first round stands apart from the loop, as in the kernel above
  round(m_first);
  for (uint32_t m = m_first + 1; m < m_end; ++m) round(m);
  if (threadIdx.x == 0) store_maximum(m_end - 1);
}

// ------------------------------------------------------------------------------------------
// CSR logistic regression with few columns: two launches.
//
// With w small enough for every L2 the dot products need no column tiles: a wavefront (or sixteen, of few rows) takes a
// minibatch row, gathers w, and leaves what the gradient pass needs of the row (residual over B, start, tile bounds) -- one
// launch in place of four (row ids, bounds, dot products, their sum).  The gradient pass then has as many
// workgroups as fill the chip: each owns 2^sub_shift columns of a tile in LDS and reads the tile's whole row
// segments (out of the L2: 2^(tile_shift - sub_shift) workgroups read the same ones), adding those that are its own.
// ------------------------------------------------------------------------------------------
// WAVES: wavefronts per row.  A lane adds at most kCsrChain products in a row, as many as a running sum of the other
// dot-product passes has in a tile: a row of 2^20 entries would be chains of 2^14 otherwise.
constexpr uint32_t kCsrChain = 512;
template <bool PAIRS, bool INDEX, int WAVES>
__global__ __launch_bounds__(WAVES == 1 ? kBlock : WAVES * kWave) void csr_rows_kernel(const int64_t* const* __restrict__ rowptrs,
                                                          const int32_t* const* __restrict__ cols,
                                                          const float* const* __restrict__ vals,
                                                          const float* const* __restrict__ ys,
                                                          const uint64_t* __restrict__ n_rows,
                                                          const uint32_t* const* __restrict__ index,
                                                          const float* __restrict__ w, uint32_t* __restrict__ idx,
                                                          int64_t* __restrict__ rowbase, uint32_t* __restrict__ bounds,
                                                          float* __restrict__ resid, uint32_t batch, uint32_t ntiles,
                                                          uint32_t tile_shift, float inv_b, uint32_t k0, uint32_t k1,
                                                          uint32_t iter) {
  constexpr uint32_t kLanes = WAVES * kWave;  // lanes per row
  __shared__ float red[WAVES];
  const uint32_t m = blockIdx.y, lane = threadIdx.x % kLanes;
  const uint32_t i = WAVES == 1 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * kWavesPerBlock + threadIdx.x / kWave))
                                : blockIdx.x;
  if (i >= batch) return;  // whole wavefronts, which meet no workgroup barrier (with several per row i < batch)
  const uint32_t row = (uint32_t)__builtin_amdgcn_readfirstlane((int)minibatch_row(k0, k1, iter, m, i, n_rows[m]));
  const int64_t a = as_global(rowptrs[m])[row];
  const uint32_t nnz = (uint32_t)(as_global(rowptrs[m])[row + 1] - a);
  const float y = as_global(ys[m])[row];
  const CsrEntries<PAIRS> e(cols[m], PAIRS ? nullptr : vals[m]);
  uint32_t* __restrict__ out = bounds + (uint64_t)m * (ntiles + 1) * batch + i;
  if (INDEX) {
    const GlobalPtr<uint32_t> src = as_global(index[m]) + (uint64_t)row * (ntiles + 1);
    for (uint32_t t = lane; t <= ntiles; t += kLanes) out[(uint64_t)t * batch] = src[t];
  }
  float acc = 0.f;
  for (uint64_t first = 0; first < nnz; first += kCsrChain * kLanes) {
    const uint32_t end = (uint32_t)min((uint64_t)nnz, first + kCsrChain * kLanes);
    float part = 0.f;
#pragma unroll 4
    for (uint32_t k = (uint32_t)first + lane; k < end; k += kLanes) {
      int32_t c;
      float v;
      e.load(a + k, c, v);
      part = __builtin_fmaf(v, w[c], part);
      if (!INDEX) {  // entry k opens every tile after the tile of entry k - 1 up to its own
        const uint32_t prev = k == 0 ? 0u : ((uint32_t)e.col(a + k - 1) >> tile_shift) + 1u;
        for (uint32_t t = prev; t <= ((uint32_t)c >> tile_shift); ++t) out[(uint64_t)t * batch] = k;
      }
    }
    acc += part;
  }
  if (!INDEX) {  // and the end of the row every tile after its last entry's
    const uint32_t prev = nnz == 0 ? 0u : ((uint32_t)e.col(a + nnz - 1) >> tile_shift) + 1u;
    for (uint32_t t = prev + lane; t <= ntiles; t += kLanes) out[(uint64_t)t * batch] = nnz;
  }
  float z = wave_sum(acc);
  if (WAVES > 1) {
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = z;
    __syncthreads();
    z = red[0];
#pragma unroll
    for (int k = 1; k < WAVES; ++k) z += red[k];
  }
  if (lane == 0) {
    const uint64_t o = (uint64_t)m * batch + i;
    idx[o] = row;
    rowbase[o] = a;
    resid[o] = logistic_residual(z, y) * inv_b;
  }
}

constexpr uint32_t kCsrMinSubShift = 10;  // a column per thread
template <bool PAIRS>
__global__ __launch_bounds__(kCsrThreads) void csr_grad_sub_kernel(const int32_t* const* __restrict__ cols,
                                                                   const float* const* __restrict__ vals,
                                                                   const int64_t* __restrict__ rowbase,
                                                                   const uint32_t* __restrict__ bounds,
                                                                   const float* __restrict__ resid,
                                                                   const float* __restrict__ w, float* __restrict__ g,
                                                                   uint64_t d, uint32_t batch, uint32_t ntiles,
                                                                   uint32_t tile_shift, uint32_t sub_shift, float l2,
                                                                   bool fused, ScaleFusion fuse) {
  extern __shared__ double gtile[];  // g over the workgroup's columns, accumulated in fp64
  __shared__ CsrSeg seg[kCsrRows];
  __shared__ float red[kCsrThreads / kWave];
  const uint32_t m = blockIdx.y;
  const uint32_t T = 1u << sub_shift;
  const uint32_t c0 = blockIdx.x << sub_shift;  // (d < 2^32 here)
  const uint32_t t = blockIdx.x >> (tile_shift - sub_shift);
  for (uint32_t j = threadIdx.x; j < T; j += kCsrThreads) gtile[j] = 0.0;
  const CsrEntries<PAIRS> e(cols[m], vals[m]);
  const uint32_t group = threadIdx.x / kCsrLanes, gl = threadIdx.x % kCsrLanes;
  const void* dummy = rowbase + (uint64_t)m * batch;
  for (uint32_t first = 0; first < batch; first += kCsrRows) {
    __syncthreads();
    csr_stage_segments(e, rowbase, bounds, resid, m, batch, ntiles, t, first, seg);
    __syncthreads();
    const uint32_t j0 = group * kCsrUnroll;
    CsrBatch<kCsrUnroll, kCsrLoads> b;
    csr_request(e, seg + j0, gl, dummy, b);
    csr_use<1>(e, seg + j0, gl, dummy, b, [&](bool in, int32_t c, float v, int u, int) {
      const uint32_t at = (uint32_t)c - c0;  // (columns left of c0 wrap to far beyond T)
      if (in && at < T) atomicAdd(&gtile[at], (double)(b.r[u] * v));
    });
  }
  __syncthreads();
  float* __restrict__ out = g + (uint64_t)m * d;
  float amax = 0.f;
  for (uint32_t j = threadIdx.x; j < T; j += kCsrThreads) {
    const uint64_t c = (uint64_t)c0 + j;
    if (c < d) {
      const float o = l2 != 0.f ? __builtin_fmaf(l2, w[c], (float)gtile[j]) : (float)gtile[j];
      out[c] = o;
      if (fused) {
        const float r1 = fuse.norm != kNormNone ? fuse.gref[c] : 0.f;
        const float r2 = fuse.norm == kNormComb ? fuse.gref2[c] : 1.f;
        amax = fmaxf(amax, fabsf(normalize_dyn(fuse.norm, o, r1, r2, fuse.eps)));
      }
    }
  }
  if (fused) {
    amax = block_max(amax, red);
    if (threadIdx.x == 0) fuse.partials[(uint64_t)blockIdx.x * gridDim.y + m] = amax;
  }
}

// Chain Rosenbrock gradient ("Nonconvex Problems", d-dimensional form) plus per-worker noise.
// Fixed expression tree, one rounding per operation:
//   a = x[i+1] - x[i]*x[i];  t1 = (-400*x[i])*a;  t2 = -2*(1 - x[i])        (i < d-1)
//   b = x[i] - x[i-1]*x[i-1];  t3 = 200*b                                    (i > 0)
//   g = ((t1 + t2) + t3) + noise, absent terms left out.
__device__ __forceinline__ float rosenbrock_component(float xp, float xi, float xn, bool has_prev, bool has_next) {
  float base = 0.f;
  if (has_next) {
    const float a = xn - xi * xi;
    const float t1 = (-400.0f * xi) * a;
    const float t2 = -2.0f * (1.0f - xi);
    base = t1 + t2;
  }
  if (has_prev) {
    const float b = xi - xp * xp;
    const float t3 = 200.0f * b;
    base = has_next ? base + t3 : t3;
  }
  return base;
}

// sqrt(-2 ln u1) for u1 = ((word >> 8) + 1) 2^-24 in (0, 1]: the hardware's binary logarithm times -2 ln 2 (in two
// parts), then the square root by its reciprocal and one correction.  The argument is 0 or between 2^-23 and 34, so
// neither needs the library functions' care for subnormals, infinities and NaNs.
__device__ __forceinline__ float gaussian_radius(uint32_t word) {
  const float u = (float)((word >> 8) + 1u) * 0x1p-24f;
  const float l = __builtin_amdgcn_logf(u);
  const float x = __builtin_fmaf(l, -0x1.62e43p+0f, l * 0x1.05c61p-28f);
  const float y = __builtin_amdgcn_rsqf(x);
  const float root = x * y;
  const float r = __builtin_fmaf(__builtin_fmaf(-root, root, x), 0.5f * y, root);
  return x > 0.f ? r : 0.f;
}

// sin and cos of 2 pi u2, u2 = (word >> 8) 2^-24.  The word's top bits are the quadrant, what is left of it is t in
// [-1/2, 1/2) quarter turns, exactly; sin(pi t / 2) and cos(pi t / 2) are polynomials fitted to the least largest
// relative error, the leading term of each in two parts.  Against the library functions over all 2^24 words, in
// units of 2^-24: sine and cosine 0.75 at most, 0.25 in the mean square (0.85 and 0.25), the radius above 2.14 and
// 0.585 times its size (the same).
__device__ __forceinline__ void sincos_turn(uint32_t word, float& sine, float& cosine) {
  const float t = (float)(int32_t)((word << 2) & 0xFFFFFC00u) * 0x1p-32f;
  const float q = t * t;
  float ps = __builtin_fmaf(q, -0x1.2dc84cp-8f, 0x1.466004p-4f);
  ps = __builtin_fmaf(q, ps, -0x1.4abbbep-1f);
  ps = __builtin_fmaf(q, ps, -0x1.777a5cp-25f);
  const float s = __builtin_fmaf(t, 0x1.921fb6p+0f, t * ps);
  float pc = __builtin_fmaf(q, 0x1.d4a424p-11f, -0x1.55b1e0p-6f);
  pc = __builtin_fmaf(q, pc, 0x1.03c1b0p-2f);
  const float c0 = __builtin_fmaf(q, -0x1.3bd3ccp+0f, 1.0f);
  const float rest = __builtin_fmaf(q, -0x1.3bd3ccp+0f, 1.0f - c0);
  const float c = c0 + __builtin_fmaf(q, q * pc, rest);
  const uint32_t turn = word + 0x20000000u;  // quadrant in the top two bits
  const bool odd = (turn & 0x40000000u) != 0u;
  sine = __uint_as_float(__float_as_uint(odd ? c : s) ^ (turn & 0x80000000u));
  cosine = __uint_as_float(__float_as_uint(odd ? s : c) ^ ((turn + 0x40000000u) & 0x80000000u));
}

// Four standard normal deviates times sigma from one Philox block (Box-Muller; see NoiseGen).
__device__ __forceinline__ float4 gaussian4(const NoiseGen& gen, uint64_t block, uint32_t m) {
  const U32x4 r = philox4x32_10((uint32_t)block, m, gen.iter, 2u, gen.k0, gen.k1);
  const float ra = gaussian_radius(r.x), rb = gaussian_radius(r.z);
  float sa, ca, sb, cb;
  sincos_turn(r.y, sa, ca);
  sincos_turn(r.w, sb, cb);
  return make_float4(gen.sigma * (ra * ca), gen.sigma * (ra * sa), gen.sigma * (rb * cb), gen.sigma * (rb * sb));
}

// A thread owns 4 consecutive coordinates; the gradient is computed once and reused for all workers, the noise is
// streamed with 16-byte loads (rows of noise and g start at any 4-byte boundary when d is not a multiple of 4).  The
// last thread of such a row (TAIL) has fewer than 4: what lies beyond is read as 0, kept out of the maximum and not
// stored.  (A variant of its own: its checks cost whole rows 5 % at d = 2^20, M = 8.)  With generated noise (GEN) the
// kernel is bound by the vector unit -- Philox, logarithm, root, sine and cosine for every element -- so the kind of
// normalisation is a template argument too, and nothing in the worker loop branches.
template <int NORM, bool FUSE, bool TAIL, bool GEN>
__global__ __launch_bounds__(kBlock) void rosenbrock_vec_kernel(const float* __restrict__ x,
                                                                const float* __restrict__ noise, NoiseGen gen,
                                                                float* __restrict__ g, uint64_t d, uint32_t M,
                                                                ScaleFusion fuse) {
  constexpr int MC = 8;  // workers per trip: their noise loads are all in flight before the first is used
  __shared__ float red[kWavesPerBlock][MC];
  const uint64_t nvec = (d + 3) / 4;
  const uint64_t q = (uint64_t)blockIdx.x * kBlock + threadIdx.x;
  const bool active = q < nvec;
  const uint64_t qc = active ? q : nvec - 1;  // idle threads of the last workgroup repeat its last float4 (and store nothing)
  float4 base, r1, r2;
  {
    const float4 xv = TAIL ? load4_within(x, 4 * qc, d, 0.f) : reinterpret_cast<const float4*>(x)[qc];
    const bool first = qc == 0, last = 4 * qc + 4 >= d;
    const float xl = first ? 0.f : x[4 * qc - 1];
    const float xr = last ? 0.f : x[4 * qc + 4];
    base.x = rosenbrock_component(xl, xv.x, xv.y, !first, !TAIL || 4 * qc + 1 < d);
    base.y = rosenbrock_component(xv.x, xv.y, xv.z, true, !TAIL || 4 * qc + 2 < d);
    base.z = rosenbrock_component(xv.y, xv.z, xv.w, true, !TAIL || 4 * qc + 3 < d);
    base.w = rosenbrock_component(xv.z, xv.w, xr, true, !last);
    r1 = make_float4(0.f, 0.f, 0.f, 0.f);
    r2 = make_float4(1.f, 1.f, 1.f, 1.f);
    if (FUSE && NORM != kNormNone)
      r1 = TAIL ? load4_within(fuse.gref, 4 * qc, d, 1.f) : reinterpret_cast<const float4*>(fuse.gref)[qc];
    if (FUSE && NORM == kNormComb)
      r2 = TAIL ? load4_within(fuse.gref2, 4 * qc, d, 1.f) : reinterpret_cast<const float4*>(fuse.gref2)[qc];
  }
  const bool from_tensor = !GEN && noise != nullptr;
  for (uint32_t m0 = 0; m0 < M; m0 += MC) {
    float4 n[MC];
    if (from_tensor) {
#pragma unroll
      for (int k = 0; k < MC; ++k)  // worker index clamped: a load, never a branch
        n[k] = TAIL ? load4_within(noise + (uint64_t)min(m0 + k, M - 1) * d, 4 * qc, d, 0.f)
                    : load4_stream_any(as_global(noise) + (uint64_t)min(m0 + k, M - 1) * d, qc);
    }
    float amax[MC];
#pragma unroll
    for (int k = 0; k < MC; ++k) {
      amax[k] = 0.f;
      if (m0 + k < M) {
        float4 o = base;
        if (GEN) n[k] = gaussian4(gen, qc, m0 + k);
        if (GEN || from_tensor) {
          o.x = base.x + n[k].x;
          o.y = base.y + n[k].y;
          o.z = base.z + n[k].z;
          o.w = base.w + n[k].w;
        }
        if (active) {
          if (TAIL)
            store4_within(g + (uint64_t)(m0 + k) * d, 4 * q, d, o);
          else
            store4_any(g + (uint64_t)(m0 + k) * d, q, o);
          if (FUSE) {
            float4 v = o;
            if (TAIL && 4 * q + 4 > d) {  // 0 (or the reference itself, which the difference forms take to 0) past the end
              const float none = NORM == kNormSub || NORM == kNormComb ? 1.f : 0.f;
              if (4 * q + 1 >= d) v.y = none;
              if (4 * q + 2 >= d) v.z = none;
              v.w = none;
            }
            amax[k] = absmax4_t<NORM>(fuse, v, r1, r2);
          }
        }
      }
    }
    if (FUSE) {  // the workgroup's maxima of the trip's workers with one pair of barriers
      const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
#pragma unroll
      for (int k = 0; k < MC; ++k) {
        const float v = wave_max_nonneg(amax[k]);
        if (lane == 0) red[wave][k] = v;
      }
      __syncthreads();
      if (threadIdx.x < (uint32_t)MC && m0 + threadIdx.x < M) {
        float v = red[0][threadIdx.x];
#pragma unroll
        for (int wv = 1; wv < kWavesPerBlock; ++wv) v = fmaxf(v, red[wv][threadIdx.x]);
        fuse.partials[(uint64_t)blockIdx.x * M + m0 + threadIdx.x] = v;
      }
      __syncthreads();  // red is reused by the next trip
    }
  }
}

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

hipError_t launch_minibatch_indices(uint32_t k0, uint32_t k1, uint32_t iter, uint32_t M, uint32_t batch,
                                    const uint64_t* n_rows, uint32_t* idx, hipStream_t s) {
  dim3 grid((batch + kBlock - 1) / kBlock, M);
  hipLaunchKernelGGL(minibatch_indices_kernel, grid, dim3(kBlock), 0, s, k0, k1, iter, batch, n_rows, idx);
  return hipGetLastError();
}

uint32_t dense_row_splits(uint64_t d, uint32_t M, uint32_t batch) {
  // one pass over whole rows kept on chip by registers and LDS together: 64 K columns (between 32 K and 64 K only the full
  // width: a masked form does not fit the register file) and enough rows for two or more per workgroup
  if (d != kRowsColumns || (uint64_t)M * batch < 512) return 0;
  uint32_t S = 256 / (M < 256 ? M : 256);
  S = S < 1 ? 1 : S;
  return S < batch ? S : batch;
}

uint32_t dense_small_splits(uint64_t d, uint32_t M, uint32_t batch) {
  if (d < 4 || d > 4 * (uint64_t)kBlock || (d + 3) / 4 * M > kSmallThreads) return 0;
  const uint32_t trips = (batch + kSmallRows - 1) / kSmallRows;
  return trips < 32 ? trips : 32;
}

// Workgroups per worker: as many as the chip holds at once, fewer where the rows do not fill their trips.  Minibatches of few
// rows stay with the two passes, whose launches are as short (d = 10240, M = 8, B = 8 13.6 / 14.0 us; d = 3000, M = 8,
// B = 16 13.7 / 14.0; d = 16000, M = 32, B = 8 22.8 / 24.1; on the other side d = 5000, M = 16, B = 16 16.6 / 15.1; beyond 16 K
// columns, where the partial gradients are longer, d = 30000, M = 4, B = 100 30.5 / 31.8, d = 16385, M = 32, B = 16 26.8 / 29.1; on the
// other side d = 20000, M = 32, B = 16 37.9 / 28.5, d = 24577, M = 22, B = 24 35.6 / 34.3, d = 32768, M = 32, B = 32 53.7 / 43.4).
// At 16 K columns themselves, where the two passes cost no more than at 12 K, more rows are wanted: M = 1, B = 32 14.6 / 15.8, M = 4, B = 64
// 17.3 / 18.2, M = 8, B = 32 17.4 / 18.3; on the other side M = 9, B = 32 19.4 / 19.2, M = 2, B = 200 21.7 / 20.7, M = 8, B = 48 20.8 / 19.8.
// Whole float4 from 16 K columns on: three rows of many workers are enough.  Iterations, the two passes / this: d = 32768, M = 256,
// B = 15 220 / 150, B = 4 112 / 95.9; M = 512, B = 4 210 / 180; d = 16384, M = 512, B = 4 152 / 139; d = 20000, M = 128, B = 4 52.8 /
// 48.9; d = 24576, M = 64, B = 8 32.4 / 34.0, B = 12 40.3 / 36.8; beyond the line d = 16384, M = 512, B = 2 132 / 136, B = 1 122 / 131.
uint32_t dense_mid_splits(uint64_t d, uint32_t M, uint32_t batch) {
  if (d < 4 || d > 32 * 1024 || (M > 256 && d < kMidMostColumns) || dense_small_splits(d, M, batch) != 0) return 0;
  const uint64_t drawn = (uint64_t)M * batch;
  const bool many = d < kMidMostColumns ? batch >= 32 || (batch >= 16 && drawn >= 256) : batch >= 16 && drawn > 256;
  const bool long_rows = drawn >= 512 && batch >= (d % 4 == 0 ? 3u : 24u);  // of 16 K and more
  if (!(d <= kMidMostColumns && many) && !(d >= kMidMostColumns && long_rows)) return 0;
  const int T = dense_mid_threads(d), nv = dense_mid_columns(d);
  const uint32_t fill = 256u * (uint32_t)dense_mid_per_unit(T, nv);
  const uint64_t rows = (uint64_t)dense_mid_rows(T, nv), most = M < fill ? fill / M : 1u;
  const uint64_t trips = (batch + rows * most - 1) / (rows * most);
  return (uint32_t)((batch + rows * trips - 1) / (rows * trips));
}

size_t dense_parts_floats(uint64_t d, uint32_t M, uint32_t batch) {
  const uint32_t small = dense_small_splits(d, M, batch), mid = dense_mid_splits(d, M, batch);
  if (small + mid != 0) return (size_t)(small + mid) * M * ((d + 3) / 4 * 4);
  return (size_t)dense_row_splits(d, M, batch) * M * d;
}

namespace {
hipError_t dense_small_rows_launch(const LogregData& p, uint64_t d, uint32_t M, uint32_t batch, uint32_t k0, uint32_t k1,
                                   uint32_t iter, uint32_t* idx, float* parts, const float* w, hipStream_t s) {
  hipLaunchKernelGGL(logreg_dense_small_kernel, dim3(dense_small_splits(d, M, batch), M), dim3(kBlock), 0, s, p.X, p.y,
                     p.n_rows, idx, w, reinterpret_cast<float4*>(parts), (uint32_t)d, batch, k0, k1, iter);
  return hipGetLastError();
}
hipError_t dense_parts_launch(const float* parts, uint64_t d, uint32_t M, uint32_t batch, uint32_t S, float l2,
                                  const float* w, float* g, const ScaleFusion* fuse, uint32_t* fused_rows, hipStream_t s) {
  const uint64_t nvec = (d + 3) / 4;
  const bool by_column = d % 4 == 0 && S <= 16 && nvec * M >= 1u << 16 && aligned16(w) && aligned16(g);
  const uint32_t cols = by_column ? kBlock : kMidCols;
  const dim3 grid((uint32_t)((nvec + cols - 1) / cols), M);
  const bool fused = fuse != nullptr && fused_rows != nullptr;  // (at most 512 rows of partial maxima)
  const float inv_b = 1.0f / (float)batch;
  if (by_column) {
    auto kernel = fused ? logreg_dense_parts_kernel<true> : logreg_dense_parts_kernel<false>;
    hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, s, parts, w, g, d, S, inv_b, l2, fused ? *fuse : ScaleFusion{});
  } else {
    auto kernel = fused ? logreg_dense_mid_parts_kernel<true> : logreg_dense_mid_parts_kernel<false>;
    hipLaunchKernelGGL(kernel, grid, dim3(kBlock), 0, s, reinterpret_cast<const float4*>(parts), w, g, d, S, inv_b, l2,
                       fused ? *fuse : ScaleFusion{});
  }
  if (fused) *fused_rows = grid.x;
  return hipGetLastError();
}
}  // namespace

hipError_t launch_dense_small_step(const LogregData& p, const CodecShape& c, uint32_t batch, float l2, uint32_t iter,
                                   uint32_t* idx, float* parts, float* w, float* g, const float* gref, const float* gref2,
                                   float* scales, uint32_t* codes, float* vbar, float lr, float* ref_out, hipStream_t s) {
  const uint32_t S = dense_small_splits(c.d, c.M, batch);
  if (S == 0 || parts == nullptr || c.norm == kNormMean || c.scale_l2 != 0) return hipErrorInvalidValue;
  const hipError_t e = dense_small_rows_launch(p, c.d, c.M, batch, c.k0, c.k1, iter, idx, parts, w, s);
  if (e != hipSuccess) return e;
#define TNG_SMALL(NORM)                                                                                              \
  do {                                                                                                               \
    auto kernel = S % 8 == 0 ? c.bits == 2 ? logreg_dense_small_finish_kernel<NORM, 2, true, true>                   \
                                           : logreg_dense_small_finish_kernel<NORM, 4, true, true>                   \
                  : c.bits == 2 ? logreg_dense_small_finish_kernel<NORM, 2, true, false>                             \
                                : logreg_dense_small_finish_kernel<NORM, 4, true, false>;                            \
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kSmallThreads), 0, s, reinterpret_cast<const float4*>(parts), S, w, g,  \
                       (uint32_t)c.d, c.M, 1.0f / (float)batch, l2, gref, gref2, c.eps, scales, codes,               \
                       (uint32_t)c.words, c.k0, c.k1, iter, vbar, ref_out, 1.0f / (float)c.M, lr);                   \
  } while (0)
  switch (c.norm) {
    case kNormSub: TNG_SMALL(kNormSub); break;
    case kNormQuot: TNG_SMALL(kNormQuot); break;
    case kNormComb: TNG_SMALL(kNormComb); break;
    default: TNG_SMALL(kNormNone); break;
  }
#undef TNG_SMALL
  return hipGetLastError();
}

hipError_t launch_logreg_dense_grad(const LogregData& p, uint64_t d, uint32_t M, uint32_t batch, float l2,
                                    uint32_t k0, uint32_t k1, uint32_t iter, uint32_t* idx, float* resid,
                                    float* parts, const float* w, float* g, const ScaleFusion* fuse,
                                    uint32_t* fused_rows, hipStream_t s) {
  if (fused_rows != nullptr) *fused_rows = 0;
  const uint32_t small = parts != nullptr ? dense_small_splits(d, M, batch) : 0;
  if (small != 0) {  // the gradient that launch_dense_small_step makes, bit for bit
    const hipError_t e = dense_small_rows_launch(p, d, M, batch, k0, k1, iter, idx, parts, w, s);
    if (e != hipSuccess) return e;
    auto kernel = small % 8 == 0 ? logreg_dense_small_finish_kernel<kNormNone, 2, false, true>
                                 : logreg_dense_small_finish_kernel<kNormNone, 2, false, false>;
    hipLaunchKernelGGL(kernel, dim3(1), dim3(kSmallThreads), 0, s,
                       reinterpret_cast<const float4*>(parts), small, const_cast<float*>(w), g, (uint32_t)d, M,
                       1.0f / (float)batch, l2, nullptr, nullptr, 0.f, nullptr, nullptr, 0u, k0, k1, iter, nullptr, nullptr,
                       0.f, 0.f);
    return hipGetLastError();
  }
  const uint32_t S = parts != nullptr && aligned16(w) && aligned16(g) ? dense_row_splits(d, M, batch) : 0;
  if (S != 0) {
    constexpr int kLds = kRowsLds * kRowsThreads * (int)sizeof(float4);
    {  // 128 KiB of dynamic LDS: raised once per device
      static std::mutex attr_mutex;
      static bool attr_done[64] = {};
      int dev = -1;
      if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
      std::lock_guard<std::mutex> attr_lock(attr_mutex);
      if (!attr_done[dev]) {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(logreg_dense_rows_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, kLds);
        if (e != hipSuccess) return e;
        attr_done[dev] = true;
      }
    }
    hipLaunchKernelGGL(logreg_dense_rows_kernel, dim3(S, M), dim3(kRowsThreads), kLds, s, p.X, p.y, p.n_rows, idx, w, parts, d,
                       batch, k0, k1, iter);
    const hipError_t el = hipGetLastError();
    if (el != hipSuccess) return el;
    return dense_parts_launch(parts, d, M, batch, S, l2, w, g, fuse, fused_rows, s);
  }
  const uint32_t mid = parts != nullptr ? dense_mid_splits(d, M, batch) : 0;
  if (mid != 0) {
    const dim3 grid(mid, M);
#define TNG_MID(T, NV)                                                                                         \
  hipLaunchKernelGGL((logreg_dense_mid_kernel<T, NV>), grid, dim3(T), 0, s, p.X, p.y, p.n_rows, idx, w,        \
                     reinterpret_cast<float4*>(parts), (uint32_t)d, batch, k0, k1, iter)
    const int nv = dense_mid_columns(d);
    if (dense_mid_threads(d) == kBlock) {
      TNG_MID(kBlock, 1);
    } else if (dense_mid_threads(d) == kMidThreadsLong) {
      switch (nv) {
        case 5: TNG_MID(kMidThreadsLong, 5); break;
        case 6: TNG_MID(kMidThreadsLong, 6); break;
        case 7: TNG_MID(kMidThreadsLong, 7); break;
        default: TNG_MID(kMidThreadsLong, 8); break;
      }
    } else {
      switch (nv) {
        case 1: TNG_MID(kMidThreads, 1); break;
        case 2: TNG_MID(kMidThreads, 2); break;
        case 3: TNG_MID(kMidThreads, 3); break;
        case 4: TNG_MID(kMidThreads, 4); break;
        case 5: TNG_MID(kMidThreads, 5); break;
        case 6: TNG_MID(kMidThreads, 6); break;
        case 7: TNG_MID(kMidThreads, 7); break;
        default: TNG_MID(kMidThreads, 8); break;
      }
    }
#undef TNG_MID
    const hipError_t el = hipGetLastError();
    if (el != hipSuccess) return el;
    return dense_parts_launch(parts, d, M, batch, mid, l2, w, g, fuse, fused_rows, s);
  }
  // Rows of X and of g start at any 4-byte boundary when d is not a multiple of 4: the vector kernels
  // read and write them with 16-byte accesses that assume no more.
  const bool vec = d >= 4;
  const float inv_b = 1.0f / (float)batch;
  dim3 grid_r(batch, M);
  if (vec && (uint64_t)M * (batch / 4) >= 1024) {  // enough rows to keep the chip busy four at a time
    hipLaunchKernelGGL((logreg_dense_resid_kernel<true, 4>), dim3((batch + 3) / 4, M), dim3(kBlock), 0, s, p.X, p.y,
                       p.n_rows, idx, w, resid, d, batch, k0, k1, iter);
  } else if (vec) {
    hipLaunchKernelGGL((logreg_dense_resid_kernel<true, 1>), grid_r, dim3(kBlock), 0, s, p.X, p.y, p.n_rows, idx, w, resid,
                       d, batch, k0, k1, iter);
  }
  if (vec) {
    const uint64_t nvec = (d + 3) / 4;
    dim3 grid_g((uint32_t)((nvec + kBlock - 1) / kBlock), M);
    const bool can_fuse = fuse != nullptr && fused_rows != nullptr && grid_g.x <= kAbsmaxMaxBlocks;
    // A thread per float4 column leaves loads too few and chains of dependent rows too long where the columns of all
    // workers are few: the rows are split between row groups then, in blocks of 32, 64 or 128 columns as there are
    // more of them (few minibatch rows, or more workers or columns than the rows in registers are for).  Iterations by these
    // passes with blocks of 32 / 64 / 128 / 256 columns / unsplit: d = 1500, M = 4, B = 64 13.9 /
    // 14.7 / 14.9 / 17.1 / - us; d = 2048, M = 32, B = 256 35.8 / 34.6 / 36.9 / 45.3 / -; d = 10007, M = 8, B = 128
    // 31.4 / 28.0 / 26.5 / 31.0 / -; M = 32, B = 512 249 / 230 / 231 / 248 / 243; d = 65535, M = 16, B = 200 362 /
    // 326 / 323 / 321 / 318; few rows to split: d = 65535, M = 4, B = 16 39 / 31 / 28.0 / 27.9 / 27.2.
    const uint64_t columns = nvec * M;
    if (batch >= 16 && (columns <= (batch >= 64 ? 3u << 16 : 1u << 15) || (batch >= 64 && nvec <= 256))) {
      const uint32_t block = columns < 2048 || nvec <= 256 ? 32 : columns <= 16384 ? 64 : 128;
      const dim3 grid((uint32_t)((nvec + block - 1) / block), M);
      const bool fused = fuse != nullptr && fused_rows != nullptr && grid.x <= kAbsmaxMaxBlocks;
      const ScaleFusion f = fused ? *fuse : ScaleFusion{};
      auto kernel = block == 32   ? (fused ? logreg_dense_grad_split_kernel<32, true> : logreg_dense_grad_split_kernel<32, false>)
                    : block == 64 ? (fused ? logreg_dense_grad_split_kernel<64, true> : logreg_dense_grad_split_kernel<64, false>)
                                  : (fused ? logreg_dense_grad_split_kernel<128, true> : logreg_dense_grad_split_kernel<128, false>);
      hipLaunchKernelGGL(kernel, grid, dim3(kSplitThreads), 0, s, p.X, idx, resid, w, g, d, batch, inv_b, l2, f);
      if (fused) *fused_rows = grid.x;
      return hipGetLastError();
    }
    if (can_fuse) {
      hipLaunchKernelGGL((logreg_dense_grad_kernel<true, true>), grid_g, dim3(kBlock), 0, s, p.X, idx, resid, w, g, d,
                         batch, inv_b, l2, *fuse);
      *fused_rows = grid_g.x;
    } else {
      hipLaunchKernelGGL((logreg_dense_grad_kernel<true, false>), grid_g, dim3(kBlock), 0, s, p.X, idx, resid, w, g, d,
                         batch, inv_b, l2, ScaleFusion{});
    }
  } else {
    hipLaunchKernelGGL((logreg_dense_resid_kernel<false, 1>), grid_r, dim3(kBlock), 0, s, p.X, p.y, p.n_rows, idx, w,
                       resid, d, batch, k0, k1, iter);
    dim3 grid_g((uint32_t)((d + kBlock - 1) / kBlock), M);
    hipLaunchKernelGGL((logreg_dense_grad_kernel<false, false>), grid_g, dim3(kBlock), 0, s, p.X, idx, resid, w, g, d,
                       batch, inv_b, l2, ScaleFusion{});
  }
  return hipGetLastError();
}

uint32_t csr_tile_shift(uint64_t d) {
  uint32_t shift = kCsrTileShift;
  while (shift > 8 && (1ull << (shift - 1)) >= d) --shift;  // small problems: one tile just covering d
  return shift;
}

uint32_t csr_tiles(uint64_t d) {
  const uint32_t shift = csr_tile_shift(d);
  return (uint32_t)((d + (1ull << shift) - 1) >> shift);
}

hipError_t launch_csr_validate_rowptr(const LogregData& p, uint32_t M, uint64_t max_rows, const uint64_t* nnz,
                                      uint32_t* flag, hipStream_t s) {
  const uint64_t bx = (max_rows + kBlock - 1) / kBlock;
  hipLaunchKernelGGL(csr_validate_rowptr_kernel, dim3((uint32_t)(bx < 4096 ? bx : 4096), M), dim3(kBlock), 0, s, p.rowptr,
                     p.n_rows, nnz, flag);
  return hipGetLastError();
}

hipError_t launch_csr_validate_cols(const LogregData& p, uint64_t d, uint32_t M, uint64_t max_rows, uint32_t* flag,
                                    hipStream_t s) {
  const dim3 grid((uint32_t)(max_rows < 65535 ? max_rows : 65535), M);
  if (p.pairs)
    hipLaunchKernelGGL(csr_validate_cols_kernel<true>, grid, dim3(kBlock), 0, s, p.rowptr, p.col, p.n_rows, d, flag);
  else
    hipLaunchKernelGGL(csr_validate_cols_kernel<false>, grid, dim3(kBlock), 0, s, p.rowptr, p.col, p.n_rows, d, flag);
  return hipGetLastError();
}

hipError_t launch_csr_tile_index(const LogregData& p, uint64_t d, uint32_t M, uint64_t max_rows, hipStream_t s) {
  if (max_rows == 0 || max_rows > 0x7fffffffull || p.tile_index == nullptr) return hipErrorInvalidValue;
  const dim3 grid((uint32_t)max_rows, M);
  if (p.pairs)
    hipLaunchKernelGGL(csr_tile_index_kernel<true>, grid, dim3(kBlock), 0, s, p.rowptr, p.col, p.n_rows, p.tile_index,
                       csr_tiles(d), csr_tile_shift(d));
  else
    hipLaunchKernelGGL(csr_tile_index_kernel<false>, grid, dim3(kBlock), 0, s, p.rowptr, p.col, p.n_rows, p.tile_index,
                       csr_tiles(d), csr_tile_shift(d));
  return hipGetLastError();
}

namespace {

// Tiles per workgroup of the pipelined gradient pass: 4.89 ms per iteration at 8, 4.81 at 16, 4.78 at 32
// (d = 2^24, 64 workers, minibatch 512; 5.18 ms with one tile per workgroup).
constexpr uint32_t kCsrRun = 16;

// The two launches for few columns (see csr_rows_kernel), up to 2^21 columns of all workers.  Beyond, w no longer
// comes cheaply out of the L2 and the repeated segments cost more than the launches.  Iterations at 0.1 % density, the
// column tiles against these: d = 2^14, M = 8, B = 128 39 -> 14.6 us; d = 2^16, M = 8, B = 512 46 -> 18.5, M = 33
// 58 -> 49, M = 64 65 -> 71; d = 2^18, M = 8 55 -> 37, M = 64 110 -> 202; d = 2^19, M = 16 66 -> 113.  Denser rows are
// further ahead, though a segment is read by several workgroups (the column tiles have too few): d = 2^14, M = 8, 10 %
// 790 -> 276; d = 2^16, M = 8, 1 / 10 / 25 % 154 -> 58 / 1503 -> 410 / 3957 -> 1038; d = 2^18, M = 8, 10 % 1600 -> 1025.
bool csr_few_columns(uint64_t d, uint32_t M) { return d * M <= (1ull << 21); }

template <bool PAIRS>
hipError_t csr_few_columns_launches(const LogregData& p, uint64_t d, uint32_t M, uint32_t batch, float l2, uint32_t k0,
                                    uint32_t k1, uint32_t iter, uint32_t* idx, int64_t* rowbase, uint32_t* bounds,
                                    float* z, const float* w, float* g, const ScaleFusion* fuse, uint32_t* fused_rows,
                                    hipStream_t s) {
  const uint32_t shift = csr_tile_shift(d), ntiles = csr_tiles(d);
  const float inv_b = 1.0f / (float)batch;
  // Few rows: sixteen wavefronts take one, or the walk of a single wavefront over a long row sets the time (d = 2^21, M = 1,
  // 209715 entries a row: B = 1 776 -> 230 us, column tiles 369; B = 16 1143 -> 630; d = 2^18, M = 8, 26214 entries, B = 1
  // 132 -> 71, column tiles 98).  Short rows lose nothing by it up to 512 of them (d = 2^18, M = 8, B = 64, 262 entries 30.2
  // -> 29.6), many do: d = 2^16, M = 8, B = 512, 66 entries 18.5 -> 32.2; nor are there long rows of few columns: d = 2^14,
  // M = 8, B = 64, 16 entries 14.5 -> 15.1.
  constexpr int kFewRowsWaves = kCsrThreads / kWave;
  const bool few_rows = (uint64_t)batch * M <= 512 && d >= (1u << 16);
  const dim3 rows(few_rows ? batch : (batch + kWavesPerBlock - 1) / kWavesPerBlock, M);
  auto kernel = p.tile_index != nullptr ? (few_rows ? csr_rows_kernel<PAIRS, true, kFewRowsWaves> : csr_rows_kernel<PAIRS, true, 1>)
                                        : (few_rows ? csr_rows_kernel<PAIRS, false, kFewRowsWaves> : csr_rows_kernel<PAIRS, false, 1>);
  hipLaunchKernelGGL(kernel, rows, dim3(few_rows ? kCsrThreads : kBlock), 0, s, p.rowptr, p.col, p.val, p.y, p.n_rows, p.tile_index, w, idx,
                     rowbase, bounds, z, batch, ntiles, shift, inv_b, k0, k1, iter);
  // columns per workgroup: 2^12, halved until there is one workgroup per compute unit (twice as many: 24 against 18.5 us
  // at d = 2^16, M = 8)
  uint32_t sub = shift < 12 ? shift : 12;
  while (sub > kCsrMinSubShift && ((d + (1ull << sub) - 1) >> sub) * M < 256) --sub;
  const dim3 grid((uint32_t)((d + (1ull << sub) - 1) >> sub), M);
  const bool fused = fuse != nullptr && fused_rows != nullptr && grid.x <= kAbsmaxMaxBlocks;
  hipLaunchKernelGGL(csr_grad_sub_kernel<PAIRS>, grid, dim3(kCsrThreads), sizeof(double) << sub, s, p.col, p.val, rowbase,
                     bounds, z, w, g, d, batch, ntiles, shift, sub, l2, fused, fused ? *fuse : ScaleFusion{});
  if (fused) *fused_rows = grid.x;
  return hipGetLastError();
}

template <bool PAIRS>
hipError_t csr_grad_launches(const LogregData& p, uint64_t d, uint32_t M, uint32_t batch, float l2, const uint32_t* idx,
                             int64_t* rowbase, uint32_t* bounds, float* zpart, float* z, const float* w, float* g,
                             const ScaleFusion* fuse, uint32_t* fused_rows, hipStream_t s) {
  const float inv_b = 1.0f / (float)batch;
  const uint32_t shift = csr_tile_shift(d);
  const uint32_t ntiles = csr_tiles(d);
  const size_t lds_w = sizeof(float) << shift, lds_g = sizeof(double) << shift;
  {  // the g tile exceeds the 64 KiB default limit of dynamic LDS: raised once per device
    static std::mutex attr_mutex;
    static bool attr_done[64] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> attr_lock(attr_mutex);
    if (!attr_done[dev]) {
      const int lds_double = (int)(sizeof(double) << kCsrTileShift);
#define TNG_ALL_PIECES(P)                                                                                                            \
  reinterpret_cast<const void*>(csr_grad_workers_kernel<PAIRS, kNormNone, true, P>),                                             \
      reinterpret_cast<const void*>(csr_grad_workers_kernel<PAIRS, kNormSub, true, P>),                                              \
      reinterpret_cast<const void*>(csr_grad_workers_kernel<PAIRS, kNormQuot, true, P>),                                             \
      reinterpret_cast<const void*>(csr_grad_workers_kernel<PAIRS, kNormNone, false, P>),                                            \
      reinterpret_cast<const void*>(csr_grad_workers_kernel<PAIRS, kNormSub, false, P>),                                             \
      reinterpret_cast<const void*>(csr_grad_workers_kernel<PAIRS, kNormQuot, false, P>)
#define TNG_Z_WIDE(P, U) \
  reinterpret_cast<const void*>(csr_z_wide_kernel<PAIRS, P, U, true>), reinterpret_cast<const void*>(csr_z_wide_kernel<PAIRS, P, U, false>)
      const void* big_lds[] = {TNG_ALL_PIECES(1), TNG_ALL_PIECES(2), TNG_ALL_PIECES(3), TNG_ALL_PIECES(4),
                               TNG_Z_WIDE(1, 1), TNG_Z_WIDE(2, 1), TNG_Z_WIDE(3, 1), TNG_Z_WIDE(2, 2),
                               reinterpret_cast<const void*>(csr_grad_kernel<false, PAIRS>),
                               reinterpret_cast<const void*>(csr_grad_kernel<true, PAIRS>),
                               reinterpret_cast<const void*>(csr_grad_run_kernel<PAIRS, kNormNone>),
                               reinterpret_cast<const void*>(csr_grad_run_kernel<PAIRS, kNormSub>),
                               reinterpret_cast<const void*>(csr_grad_run_kernel<PAIRS, kNormQuot>),
                               reinterpret_cast<const void*>(csr_grad_run_kernel<PAIRS, kNormComb>)};
#undef TNG_ALL_PIECES
#undef TNG_Z_WIDE
      static_assert(2 * sizeof(float) == sizeof(double), "two tiles of w are as large as one of g");
      for (const void* kernel : big_lds) {
        const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, lds_double);
        if (e != hipSuccess) return e;
      }
      attr_done[dev] = true;
    }
  }
  if (p.tile_index != nullptr) {
    dim3 grid((ntiles + 1 + kGatherTiles - 1) / kGatherTiles, (batch + kGatherRows - 1) / kGatherRows, M);
    hipLaunchKernelGGL(csr_gather_bounds_kernel, grid, dim3(kBlock), 0, s, p.rowptr, p.tile_index, idx, rowbase, bounds,
                       batch, ntiles);
  } else {
    hipLaunchKernelGGL(csr_bounds_kernel<PAIRS>, dim3(batch, M), dim3(kBlock), 0, s, p.rowptr, p.col, idx, rowbase, bounds,
                       batch, ntiles, shift);
  }
  uint32_t nparts = ntiles;  // partial dot products per row
  if (shift == kCsrTileShift && ntiles >= 2) {
    nparts = (ntiles + 1) / 2;
    uint32_t wpb = 1;  // workers per workgroup while 1024 workgroups remain (per iteration at d = 2^24, 64 workers:
                       // 4.538 ms with 8 per workgroup, 4.531 with 16, 4.519 with 32)
    while (wpb < 32 && wpb * 2 <= M && (uint64_t)nparts * (M / (wpb * 2)) >= 1024) wpb *= 2;
    const int pieces = csr_pieces(batch);
    const bool one = wpb == 1 && batch <= (uint32_t)kCsrRows;  // one step per workgroup
#define TNG_Z_WIDE(P, U) (one ? csr_z_wide_kernel<PAIRS, P, U, true> : csr_z_wide_kernel<PAIRS, P, U, false>)
    auto kernel = pieces == 1 ? TNG_Z_WIDE(1, 1) : pieces == 2 ? TNG_Z_WIDE(2, 1) : pieces == 3 ? TNG_Z_WIDE(3, 1) : TNG_Z_WIDE(2, 2);
#undef TNG_Z_WIDE
    hipLaunchKernelGGL(kernel, dim3(nparts, (M + wpb - 1) / wpb), dim3(kCsrThreads), 2 * lds_w, s, p.col,
                       p.val, rowbase, bounds, w, zpart, d, batch, ntiles, nparts, M, wpb);
  } else {
    hipLaunchKernelGGL(csr_z_kernel<PAIRS>, dim3(M, ntiles), dim3(kCsrThreads), lds_w, s, p.col, p.val, rowbase, bounds, w,
                       zpart, d, batch, ntiles, shift);
  }
  hipLaunchKernelGGL(csr_z_reduce_kernel, dim3((batch + kReduceRows - 1) / kReduceRows, M), dim3(kBlock), 0, s, zpart, p.y, idx,
                     z, batch, nparts, inv_b);
  // The scale pass rides along when every tile is a full one and the write-out is the plain one.
  const bool full = d % (1ull << kCsrTileShift) == 0;
  // (the combined form keeps two references per column: they do not fit next to the pipeline's registers)
  const bool by_workers = fuse != nullptr && batch <= (uint32_t)kCsrRows && M >= 2 && fuse->norm != kNormComb;
  if (fuse != nullptr && fused_rows != nullptr && shift == kCsrTileShift && (full || by_workers) &&
      l2 == 0.f && ntiles <= kAbsmaxMaxBlocks && aligned16(g) && aligned16(fuse->gref) && aligned16(fuse->gref2)) {
    if (by_workers) {
      // a workgroup per tile and group of workers: groups as long as 1024 workgroups (four per compute unit)
      // remain -- per iteration at d = 2^24, 64 workers: 4.69 ms with groups of 8, 4.61 with 16, 4.57 with
      // 32, 4.54 with all 64 (4.76 with the kernel that runs over tiles)
      uint32_t per_group = 64;
      while (per_group > 2 && (uint64_t)ntiles * ((M + per_group - 1) / per_group) < 1024) per_group /= 2;
      const dim3 grid(ntiles, (M + per_group - 1) / per_group);
      const int pieces = csr_pieces(batch);
#define TNG_WORKERS_P(NORM, P) (full ? csr_grad_workers_kernel<PAIRS, NORM, true, P> : csr_grad_workers_kernel<PAIRS, NORM, false, P>)
#define TNG_WORKERS(NORM)                                                                                                \
  hipLaunchKernelGGL((pieces == 1   ? TNG_WORKERS_P(NORM, 1)                                                             \
                      : pieces == 2 ? TNG_WORKERS_P(NORM, 2)                                                             \
                      : pieces == 3 ? TNG_WORKERS_P(NORM, 3)                                                             \
                                    : TNG_WORKERS_P(NORM, 4)),                                                           \
                     grid, dim3(kCsrThreads), lds_g, s, p.col, p.val, rowbase, bounds, z, g, d, batch, ntiles, M,       \
                     per_group, *fuse)
      switch (fuse->norm) {
        case kNormSub: TNG_WORKERS(kNormSub); break;
        case kNormQuot: TNG_WORKERS(kNormQuot); break;
        default: TNG_WORKERS(kNormNone); break;
      }
#undef TNG_WORKERS
#undef TNG_WORKERS_P
    } else if (batch <= (uint32_t)kCsrRows) {
      const uint32_t run = kCsrRun;
      const dim3 grid(M, (ntiles + run - 1) / run);
#define TNG_RUN(NORM)                                                                                                   \
  hipLaunchKernelGGL((csr_grad_run_kernel<PAIRS, NORM>), grid, dim3(kCsrThreads), lds_g, s, p.col, p.val, rowbase, bounds, \
                     z, g, d, batch, ntiles, *fuse)
      switch (fuse->norm) {
        case kNormSub: TNG_RUN(kNormSub); break;
        case kNormQuot: TNG_RUN(kNormQuot); break;
        case kNormComb: TNG_RUN(kNormComb); break;
        default: TNG_RUN(kNormNone); break;
      }
#undef TNG_RUN
    } else {
      hipLaunchKernelGGL((csr_grad_kernel<true, PAIRS>), dim3(M, ntiles), dim3(kCsrThreads), lds_g, s, p.col, p.val,
                         rowbase, bounds, z, w, g, d, batch, ntiles, shift, l2, *fuse);
    }
    *fused_rows = ntiles;
  } else {
    hipLaunchKernelGGL((csr_grad_kernel<false, PAIRS>), dim3(M, ntiles), dim3(kCsrThreads), lds_g, s, p.col, p.val, rowbase,
                       bounds, z, w, g, d, batch, ntiles, shift, l2, ScaleFusion{});
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_logreg_csr_grad(const LogregData& p, uint64_t d, uint32_t M, uint32_t batch, float l2, uint32_t k0,
                                  uint32_t k1, uint32_t iter, uint32_t* idx, int64_t* rowbase, uint32_t* bounds,
                                  float* zpart, float* z, const float* w, float* g, const ScaleFusion* fuse,
                                  uint32_t* fused_rows, hipStream_t s) {
  if (fused_rows != nullptr) *fused_rows = 0;
  if (csr_few_columns(d, M))
    return p.pairs ? csr_few_columns_launches<true>(p, d, M, batch, l2, k0, k1, iter, idx, rowbase, bounds, z, w, g, fuse,
                                                    fused_rows, s)
                   : csr_few_columns_launches<false>(p, d, M, batch, l2, k0, k1, iter, idx, rowbase, bounds, z, w, g,
                                                     fuse, fused_rows, s);
  const hipError_t e = launch_minibatch_indices(k0, k1, iter, M, batch, p.n_rows, idx, s);
  if (e != hipSuccess) return e;
  return p.pairs ? csr_grad_launches<true>(p, d, M, batch, l2, idx, rowbase, bounds, zpart, z, w, g, fuse, fused_rows, s)
                 : csr_grad_launches<false>(p, d, M, batch, l2, idx, rowbase, bounds, zpart, z, w, g, fuse, fused_rows, s);
}

hipError_t launch_rosenbrock_grad(uint64_t d, uint32_t M, const float* x, const float* noise, NoiseGen gen, float* g,
                                  const ScaleFusion* fuse, uint32_t* fused_rows, hipStream_t s) {
  if (fused_rows != nullptr) *fused_rows = 0;
  const uint32_t blocks = (uint32_t)(((d + 3) / 4 + kBlock - 1) / kBlock);
  const bool fused = fuse != nullptr && fused_rows != nullptr && blocks <= kAbsmaxMaxBlocks;
  const bool generated = gen.sigma > 0.f;
  const ScaleFusion f = fused ? *fuse : ScaleFusion{};
#define TNG_ROSENBROCK(NORM, F)                                                                                       \
  do {                                                                                                                \
    auto kernel = d % 4 == 0 ? (generated ? rosenbrock_vec_kernel<NORM, F, false, true>                               \
                                          : rosenbrock_vec_kernel<NORM, F, false, false>)                             \
                             : (generated ? rosenbrock_vec_kernel<NORM, F, true, true>                                \
                                          : rosenbrock_vec_kernel<NORM, F, true, false>);                             \
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kBlock), 0, s, x, noise, gen, g, d, M, f);                          \
  } while (0)
  if (!fused) {
    TNG_ROSENBROCK(kNormNone, false);
  } else {
    switch (fuse->norm) {
      case kNormSub: TNG_ROSENBROCK(kNormSub, true); break;
      case kNormQuot: TNG_ROSENBROCK(kNormQuot, true); break;
      case kNormComb: TNG_ROSENBROCK(kNormComb, true); break;
      default: TNG_ROSENBROCK(kNormNone, true); break;
    }
  }
#undef TNG_ROSENBROCK
  if (fused) *fused_rows = blocks;
  return hipGetLastError();
}

}  // namespace tng
