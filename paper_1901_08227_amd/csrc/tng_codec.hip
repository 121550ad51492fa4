// Codec kernels of libtng: scale (max of the normalised gradient), stochastic quantise + pack,
// and decode + average + de-normalise (+ iterate / reference update), for gfx950.
//
// All three stream fp32 data once; they are bound by HBM bandwidth (and, for the quantiser, by the
// integer multiplies of the counter-based RNG), never by matrix math.  Layout choices:
//  * a workgroup owns a tile of coordinates and loops over the workers inside the kernel, so the
//    shared reference tile is fetched once and kept in registers;
//  * every global access is a coalesced 16-byte (fp32) or 4-byte (packed words) per-lane access;
//    the 2- or 4-bit codes a lane produces are transposed into whole words through LDS;
//  * Philox block j covers elements 4j..4j+3, i.e. exactly one float4.
#include "tng_device.hpp"
#include "tng_kernels.hpp"

#include <float.h>
#include <type_traits>

namespace tng {

namespace {

constexpr int kWavesPerBlock = kBlock / kWave;
constexpr uint32_t kFusedScaleRows = 256;  // at most this many rows of partial maxima are reduced by the quantiser itself,
constexpr uint64_t kFusedScaleReads = 1u << 18;  // and as many as keep it to this many reads of memory lines in all
constexpr int kLoadsPerLane = 4;  // float4 loads per lane and worker in the quantiser tile
constexpr uint64_t kWaveTileElements = (uint64_t)kWave * kLoadsPerLane * 4;  // coordinates per wavefront tile
constexpr uint32_t kMaxGridX = 1u << 20;

__global__ __launch_bounds__(kBlock) void fill_u32_kernel(uint32_t* p, uint64_t n, uint32_t v) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) p[i] = v;
}

__global__ __launch_bounds__(kBlock) void copy_f32_kernel(float* __restrict__ dst,
                                                          const float* __restrict__ src, uint64_t n) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) dst[i] = src[i];
}

// Four float4 per thread in flight and one trip per workgroup wherever the grid allows: the shape that
// measured fastest for a plain copy (1 GiB: 6.4 TB/s on read + written bytes, against 5.4 with one float4 per
// thread and 16384 workgroups striding; streaming loads and stores in both).
constexpr int kCopyPerThread = 4;
__global__ __launch_bounds__(kBlock) void copy_f32x4_kernel(float4* __restrict__ dst,
                                                            const float4* __restrict__ src, uint64_t n) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock * kCopyPerThread;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock * kCopyPerThread + threadIdx.x; i < n; i += stride) {
    float4 x[kCopyPerThread];
#pragma unroll
    for (int u = 0; u < kCopyPerThread; ++u)
      if (i + (uint64_t)u * kBlock < n) x[u] = load_stream(src + i + (uint64_t)u * kBlock);
#pragma unroll
    for (int u = 0; u < kCopyPerThread; ++u)
      if (i + (uint64_t)u * kBlock < n) store_stream(dst + i + (uint64_t)u * kBlock, x[u]);
  }
}

// Window-average reference (section "Reference Vectors"): mean of the last `window` decoded
// averages, added oldest first, one rounding per addition.
__global__ __launch_bounds__(kBlock) void window_mean_kernel(const float* __restrict__ history, uint32_t window,
                                                             uint32_t first, uint64_t d, float inv_window,
                                                             float* __restrict__ out) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x; e < d; e += stride) {
    float acc = 0.f;
    uint32_t slot = first;
    for (uint32_t k = 0; k < window; ++k) {
      acc = acc + history[(uint64_t)slot * d + e];
      slot = slot + 1 == window ? 0u : slot + 1;
    }
    out[e] = acc * inv_window;
  }
}

// The same, four coordinates per thread (d a multiple of 4, 16-byte aligned operands).
__global__ __launch_bounds__(kBlock) void window_mean_vec_kernel(const float4* __restrict__ history, uint32_t window,
                                                                 uint32_t first, uint64_t nvec, float inv_window,
                                                                 float4* __restrict__ out) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t q = (uint64_t)blockIdx.x * kBlock + threadIdx.x; q < nvec; q += stride) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    uint32_t slot = first;
    for (uint32_t k = 0; k < window; ++k) {
      const float4 h = load_stream(history + (uint64_t)slot * nvec + q);
      acc.x = acc.x + h.x;
      acc.y = acc.y + h.y;
      acc.z = acc.z + h.z;
      acc.w = acc.w + h.w;
      slot = slot + 1 == window ? 0u : slot + 1;
    }
    store_stream(out + q, make_float4(acc.x * inv_window, acc.y * inv_window, acc.z * inv_window, acc.w * inv_window));
  }
}

__global__ __launch_bounds__(kBlock) void rng_draws_kernel(uint32_t k0, uint32_t k1, uint32_t iter,
                                                           uint32_t worker, uint32_t stream,
                                                           uint64_t first, uint64_t count, uint32_t* out) {
  const uint64_t stride = (uint64_t)gridDim.x * kBlock;
  for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < count; i += stride) {
    const uint64_t j = first + i;
    const U32x4 r = philox4x32_10((uint32_t)(j >> 2), worker, iter, stream, k0, k1);
    const uint32_t lane = (uint32_t)(j & 3);
    out[i] = lane == 0 ? r.x : lane == 1 ? r.y : lane == 2 ? r.z : r.w;
  }
}

// ------------------------------------------------------------------------------------------
// Reference operands of one float4 of coordinates.
// ------------------------------------------------------------------------------------------
template <int NORM>
struct RefTile {
  float4 r1, r2;
  double inv[4];  // binary64 reciprocals of the divisor (Eq. 2: r1, combined form: r2), see reciprocals()
  // STREAM: the tile is read once by this kernel (non-temporal); otherwise it is re-read soon and
  // should stay in cache.
  template <bool STREAM = true>
  __device__ __forceinline__ void load(const float4* ref, const float4* ref2, uint64_t i, float eps) {
    r1 = make_float4(0.f, 0.f, 0.f, 0.f);
    r2 = make_float4(1.f, 1.f, 1.f, 1.f);
    if (NORM == kNormSub || NORM == kNormComb) r1 = STREAM ? load_stream(ref + i) : ref[i];
    if (NORM == kNormQuot) {
      const float4 r = STREAM ? load_stream(ref + i) : ref[i];
      r1 = make_float4(clamp_ref(r.x, eps), clamp_ref(r.y, eps), clamp_ref(r.z, eps), clamp_ref(r.w, eps));
    }
    if (NORM == kNormComb) {
      const float4 r = STREAM ? load_stream(ref2 + i) : ref2[i];
      r2 = make_float4(clamp_ref(r.x, eps), clamp_ref(r.y, eps), clamp_ref(r.z, eps), clamp_ref(r.w, eps));
    }
  }
  // The same for a float4 that may reach past the end of the row (d elements).  What lies beyond takes operands
  // under which a gradient of 0 normalises to 0 (see row_load_fill): it adds nothing to a maximum and codes to 0.
  __device__ __forceinline__ void load_ragged(const float4* ref, const float4* ref2, uint64_t i, uint64_t d, float eps) {
    if (NORM == kNormSub || NORM == kNormComb) r1 = load4_within(reinterpret_cast<const float*>(ref), 4 * i, d, 0.f);
    else if (NORM == kNormQuot) r1 = load4_within(reinterpret_cast<const float*>(ref), 4 * i, d, 1.f);
    else r1 = make_float4(0.f, 0.f, 0.f, 0.f);
    r2 = make_float4(1.f, 1.f, 1.f, 1.f);
    if (NORM == kNormComb) r2 = load4_within(reinterpret_cast<const float*>(ref2), 4 * i, d, 1.f);
    if (NORM == kNormQuot)
      r1 = make_float4(clamp_ref(r1.x, eps), clamp_ref(r1.y, eps), clamp_ref(r1.z, eps), clamp_ref(r1.w, eps));
    if (NORM == kNormComb)
      r2 = make_float4(clamp_ref(r2.x, eps), clamp_ref(r2.y, eps), clamp_ref(r2.z, eps), clamp_ref(r2.w, eps));
  }
  // Every worker divides by the same clamped reference (Eq. 2 and the combined form): the scale and the
  // quantise pass take its binary64 reciprocal once per coordinate and multiply per worker
  // (quotient_by_reciprocal), 4 operations per element instead of the 12 of a division.
  __device__ __forceinline__ void reciprocals() {
    const float4& b = NORM == kNormQuot ? r1 : r2;
    if (NORM == kNormQuot || NORM == kNormComb) {
      inv[0] = 1.0 / (double)b.x;
      inv[1] = 1.0 / (double)b.y;
      inv[2] = 1.0 / (double)b.z;
      inv[3] = 1.0 / (double)b.w;
    }
  }
};

// Worth it from four workers per reference tile on: the reciprocal itself costs about two divisions.
template <int NORM, int MC>
constexpr bool kByReciprocal = (NORM == kNormQuot || NORM == kNormComb) && MC >= 4;

// The four values one float4 of a worker's row hands to the coder, the divisions of Eq. 2 / the
// combined form done through the reciprocals; the (rare) float4 with a subnormal quotient is redone
// with the division itself, so the values are those of normalize_w bit for bit.
template <int NORM, bool RECIP>
__device__ __forceinline__ float4 normalize4(const float4& x, const RefTile<NORM>& rt, float mu) {
  if (!RECIP) {
    return make_float4(normalize_w<NORM>(x.x, rt.r1.x, rt.r2.x, mu), normalize_w<NORM>(x.y, rt.r1.y, rt.r2.y, mu),
                       normalize_w<NORM>(x.z, rt.r1.z, rt.r2.z, mu), normalize_w<NORM>(x.w, rt.r1.w, rt.r2.w, mu));
  }
  float4 n = x;  // numerators
  if (NORM == kNormComb) n = make_float4(x.x - rt.r1.x, x.y - rt.r1.y, x.z - rt.r1.z, x.w - rt.r1.w);
  float4 v = make_float4(quotient_by_reciprocal(n.x, rt.inv[0]), quotient_by_reciprocal(n.y, rt.inv[1]),
                         quotient_by_reciprocal(n.z, rt.inv[2]), quotient_by_reciprocal(n.w, rt.inv[3]));
  if ((int)is_subnormal(v.x) | (int)is_subnormal(v.y) | (int)is_subnormal(v.z) | (int)is_subnormal(v.w)) {
    const float4& b = NORM == kNormQuot ? rt.r1 : rt.r2;
    v = make_float4(n.x / b.x, n.y / b.y, n.z / b.z, n.w / b.w);
  }
  return v;
}

// max |normalize4(x)| over one float4.  The maximum is taken in binary64 and rounded once (rounding is
// monotone, so this is the maximum of the rounded quotients); it is right whenever it is 0 or at least
// 2^-125, because then the largest quotient is of normal size and every subnormal one lies below it.
template <int NORM>
__device__ __forceinline__ double absmax4_by_reciprocal(const float4& x, const RefTile<NORM>& rt) {
  float4 n = x;
  if (NORM == kNormComb) n = make_float4(x.x - rt.r1.x, x.y - rt.r1.y, x.z - rt.r1.z, x.w - rt.r1.w);
  const double q0 = fabs((double)n.x * rt.inv[0]), q1 = fabs((double)n.y * rt.inv[1]);
  const double q2 = fabs((double)n.z * rt.inv[2]), q3 = fabs((double)n.w * rt.inv[3]);
  return fmax(fmax(q0, q1), fmax(q2, q3));
}

template <int NORM>
__device__ __forceinline__ void load_ref_scalar(const float* ref, const float* ref2, uint64_t e, float eps,
                                                float& r1, float& r2) {
  r1 = 0.f;
  r2 = 1.f;
  if (NORM == kNormSub || NORM == kNormComb) r1 = ref[e];
  if (NORM == kNormQuot) r1 = clamp_ref(ref[e], eps);
  if (NORM == kNormComb) r2 = clamp_ref(ref2[e], eps);
}

// Block maximum of MC per-thread values, written to this workgroup's slot of the partial-maxima
// array (partials[blockIdx.x][m]); a second, tiny kernel reduces the slots.  Thousands of atomic
// maxima on the same few words serialise in L2 (about 10 ns each), plain stores do not.
template <int MC>
__device__ __forceinline__ void block_max_to_partials(float (&mx)[MC], uint32_t m0, uint32_t M, float* partials) {
  __shared__ float red[MC][kWavesPerBlock];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
#pragma unroll
  for (int mm = 0; mm < MC; ++mm) {
    const float v = wave_max_nonneg(mx[mm]);
    if (lane == 0) red[mm][wave] = v;
  }
  __syncthreads();
  if (threadIdx.x < MC && m0 + threadIdx.x < M) {
    float v = red[threadIdx.x][0];
#pragma unroll
    for (int k = 1; k < kWavesPerBlock; ++k) v = fmaxf(v, red[threadIdx.x][k]);
    partials[(uint64_t)blockIdx.x * M + m0 + threadIdx.x] = v;
  }
}

// scales[m] = max over the nblocks partial maxima of worker m; a maximum below the smallest normal
// number is taken as 0.  One workgroup per worker, a large one for many rows: a thread has four loads at most, all in flight together (4095
// rows of 8 workers: 7.4 us with 256 threads, 4.5 to 6.3 with 1024).
constexpr uint32_t kFinishLarge = 1024;
__host__ inline uint32_t finish_threads(uint32_t nblocks) { return nblocks > kFinishLarge ? kFinishLarge : (uint32_t)kBlock; }
template <int THREADS>
__device__ __forceinline__ float absmax_finish_worker(const float* __restrict__ partials, uint32_t nblocks, uint32_t M,
                                                      float* __restrict__ scales, uint32_t m) {
  constexpr int kWaves = THREADS / kWave;
  __shared__ float red[kWaves];
  float v = 0.f;
  for (uint32_t b0 = threadIdx.x; b0 < nblocks; b0 += 4 * THREADS) {
    float p[4];  // (past the last row the last one again)
#pragma unroll
    for (int k = 0; k < 4; ++k) p[k] = partials[(uint64_t)min(b0 + (uint32_t)(k * THREADS), nblocks - 1) * M + m];
    v = fmaxf(fmaxf(v, fmaxf(p[0], p[1])), fmaxf(p[2], p[3]));
  }
  v = wave_max_nonneg(v);
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = v;
  __syncthreads();
  if (threadIdx.x < (uint32_t)kWave) {
    v = wave_max_nonneg(red[threadIdx.x % kWaves]);
    v = v < FLT_MIN ? 0.f : v;
    if (threadIdx.x == 0) scales[m] = v;
  }
  return v;  // (the first wavefront's)
}
template <int THREADS>
__global__ __launch_bounds__(THREADS) void absmax_finish_kernel(const float* __restrict__ partials, uint32_t nblocks, uint32_t M,
                                                                float* __restrict__ scales) {
  absmax_finish_worker<THREADS>(partials, nblocks, M, scales, blockIdx.x);
}

// The M gradient rows as the vector kernels read them.  Row m starts m * pitch floats into the array;
// the pitch (= d) need not be a multiple of 4, so a row may start at any 4-byte boundary (hence the
// 16-byte loads that assume 4-byte alignment only).
struct GradRows {
  const float* base;
  uint64_t pitch;
  __device__ __forceinline__ const v4f_u_t* row(uint32_t m) const {
    return reinterpret_cast<const v4f_u_t*>(base + (uint64_t)m * pitch);
  }
};
__device__ __forceinline__ float4 load_row_stream(const v4f_u_t* p) {
  const v4f_u_t v = __builtin_nontemporal_load(p);
  return make_float4(v.x, v.y, v.z, v.w);
}
// A wavefront's tile lies inside the row (every tile but the last) or is ragged: then each float4 is checked
// against the end of the row, and what lies beyond is filled with the value that normalises to 0 -- 0 itself, and
// the worker's mean for the mean reference (RefTile::load_ragged supplies the references).  Rows whose length is
// no multiple of 4 need no launches of their own that way (they took one element-by-element launch per pass:
// scale, quantise, decode, each as long as a small kernel and one row of partial maxima more).  The ragged tile
// has workgroups of its own behind the others (tail_workgroups: one wavefront per worker, so that it is no longer
// than any other tile's work on one worker; one wavefront walking the workers one by one took 10 us at the end of
// a launch).
__device__ __forceinline__ float4 load_row_ragged(const GradRows& g, uint32_t m, uint64_t iv, uint64_t d, float fill) {
  return load4_within(g.base + (uint64_t)m * g.pitch, 4 * iv, d, fill);
}

// ------------------------------------------------------------------------------------------
// Pass 1: R_m = max_e |v_{m,e}|   (section "Gradient Compression": R = max_d |v_d|)
// ------------------------------------------------------------------------------------------
// A wavefront owns kAbsmaxLoads * 64 consecutive float4 (4 KiB) of every worker row and walks the
// workers one after the other with the next worker's four loads in flight; reading one row at a
// time (instead of all rows at once) and streaming loads measured ~20 % faster on HBM.  The
// reference tile stays in registers.
constexpr int kAbsmaxLoads = 4;

// Worker m's part of the tile.  Past the last worker (in a short group) every lane fetches the same float4 instead: a load,
// never a branch, and no memory to wait for; nothing is made of it.
__device__ __forceinline__ void absmax_load(const GradRows& g, uint32_t m, uint32_t M, const uint64_t (&iv)[kAbsmaxLoads],
                                            float4 (&x)[kAbsmaxLoads]) {
  const uint64_t keep = m < M ? ~0ull : 0ull;
  const v4f_u_t* row = g.row(min(m, M - 1));
#pragma unroll
  for (int j = 0; j < kAbsmaxLoads; ++j) x[j] = load_row_stream(row + (iv[j] & keep));
}

template <int NORM, bool RECIP>
__device__ __forceinline__ float absmax_reduce(const float4 (&x)[kAbsmaxLoads], const RefTile<NORM> (&rt)[kAbsmaxLoads],
                                               float mu) {
  if (RECIP) {
    double mx64 = 0.0;
#pragma unroll
    for (int j = 0; j < kAbsmaxLoads; ++j) mx64 = fmax(mx64, absmax4_by_reciprocal<NORM>(x[j], rt[j]));
    if (!(mx64 > 0.0 && mx64 < 0x1p-125)) return (float)mx64;
    // else (a tile whose quotients are all tiny): once more with the divisions themselves
  }
  float mx = 0.f;
#pragma unroll
  for (int j = 0; j < kAbsmaxLoads; ++j) {
    const float a0 = fabsf(normalize_w<NORM>(x[j].x, rt[j].r1.x, rt[j].r2.x, mu));
    const float a1 = fabsf(normalize_w<NORM>(x[j].y, rt[j].r1.y, rt[j].r2.y, mu));
    const float a2 = fabsf(normalize_w<NORM>(x[j].z, rt[j].r1.z, rt[j].r2.z, mu));
    const float a3 = fabsf(normalize_w<NORM>(x[j].w, rt[j].r1.w, rt[j].r2.w, mu));
    mx = fmaxf(mx, fmaxf(fmaxf(a0, a1), fmaxf(a2, a3)));
  }
  return mx;
}

template <int NORM, int MC>
__device__ __forceinline__ void absmax_rows(const GradRows& g, const RefTile<NORM> (&rt)[kAbsmaxLoads],
                                            const uint64_t (&iv)[kAbsmaxLoads], uint32_t m0, uint32_t M,
                                            const float* __restrict__ means, float (&mx)[MC]) {
  constexpr int L = kAbsmaxLoads;
  float4 xa[L], xb[L];
  auto mean_of = [&](int mm) { return NORM == kNormMean ? means[min(m0 + (uint32_t)mm, M - 1)] : 0.f; };
  absmax_load(g, m0, M, iv, xa);
#pragma unroll
  for (int mm = 0; mm < MC; mm += 2) {
    if (mm + 1 < MC) absmax_load(g, m0 + mm + 1, M, iv, xb);
    mx[mm] = fmaxf(mx[mm], absmax_reduce<NORM, kByReciprocal<NORM, MC>>(xa, rt, mean_of(mm)));
    if (mm + 1 < MC) {
      if (mm + 2 < MC) absmax_load(g, m0 + mm + 2, M, iv, xa);
      mx[mm + 1] = fmaxf(mx[mm + 1], absmax_reduce<NORM, kByReciprocal<NORM, MC>>(xb, rt, mean_of(mm + 1)));
    }
  }
}

// The maximum over the lane's part of the ragged last wavefront tile of worker m.
template <int NORM>
__device__ __forceinline__ float absmax_ragged_tile(const GradRows& g, const float4* ref4, const float4* ref24, uint32_t m,
                                                    uint64_t d, float eps, float mu) {
  constexpr int L = kAbsmaxLoads;
  RefTile<NORM> rt[L];
  float4 x[L];
#pragma unroll
  for (int j = 0; j < L; ++j) {
    const uint64_t iv = d / kWaveTileElements * (kWave * L) + (uint64_t)j * kWave + threadIdx.x % kWave;
    rt[j].load_ragged(ref4, ref24, iv, d, eps);
    x[j] = load_row_ragged(g, m, iv, d, mu);
  }
  return absmax_reduce<NORM, false>(x, rt, mu);
}

template <int NORM, int MC>
__global__ __launch_bounds__(kBlock) void absmax_vec_kernel(GradRows g, const float4* __restrict__ ref4,
                                                            const float4* __restrict__ ref24,
                                                            float* partials, uint64_t d, uint32_t main_blocks,
                                                            uint32_t M, float eps, const float* __restrict__ means) {
  constexpr int L = kAbsmaxLoads;
  constexpr uint64_t kWaveTile = (uint64_t)kWave * L;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const uint32_t m0 = blockIdx.y * MC;
  float mx[MC];
#pragma unroll
  for (int mm = 0; mm < MC; ++mm) mx[mm] = 0.f;
  const uint64_t ntiles = d / (4 * kWaveTile);  // whole wavefront tiles
  if (blockIdx.x < main_blocks) {
    for (uint64_t tile = (uint64_t)blockIdx.x * kWavesPerBlock + wave; tile < ntiles;
         tile += (uint64_t)main_blocks * kWavesPerBlock) {
      RefTile<NORM> rt[L];
      uint64_t iv[L];
#pragma unroll
      for (int j = 0; j < L; ++j) {
        iv[j] = tile * kWaveTile + (uint64_t)j * kWave + lane;
        rt[j].load(ref4, ref24, iv[j], eps);
        if (kByReciprocal<NORM, MC>) rt[j].reciprocals();
      }
      absmax_rows<NORM, MC>(g, rt, iv, m0, M, means, mx);
    }
  } else {
    if ((blockIdx.x - main_blocks) * kWavesPerBlock >= (uint32_t)MC) return;  // idle (workgroups_per_group)
    const uint32_t at = (blockIdx.x - main_blocks) * kWavesPerBlock + (uint32_t)wave, m = m0 + at;
    // (wavefronts beyond the group's workers have nothing to fetch: other workers' tiles in them were 4.6 of the pass's 11.2
    // us at d = 9000, M = 800)
    const bool mine = at < (uint32_t)MC && m < M;
    const float v = mine ? absmax_ragged_tile<NORM>(g, ref4, ref24, m, d, eps, NORM == kNormMean ? means[m] : 0.f) : 0.f;
#pragma unroll
    for (int mm = 0; mm < MC; ++mm) mx[mm] = (uint32_t)mm == at ? v : 0.f;
  }
  block_max_to_partials<MC>(mx, m0, M, partials);
}

// ------------------------------------------------------------------------------------------
// Pass 2: normalise, draw, round, sign, pack   (Algorithm 1: sample z, transmit sign (.) z and R)
//
// A wavefront owns 64 * 4 float4 = 1024 consecutive coordinates.  Load j of lane l covers
// coordinates 256 j + 4 l .. + 3, so every load instruction is one contiguous 1 KiB.  The four
// codes of a load form an 8-bit (ternary) or 16-bit (4-bit codes) fragment; fragment (j, l) is
// fragment number 64 j + l of the wavefront's packed output, so writing fragments to LDS at that
// index and reading LDS back as 32-bit words gives each lane whole words to store, contiguously.
// ------------------------------------------------------------------------------------------
// Everything a lane keeps across the worker loop of the quantiser: its four float4 positions and
// the reference operands there.
template <int NORM>
struct QuantLane {
  RefTile<NORM> rt[kLoadsPerLane];
  uint64_t iv[kLoadsPerLane];
};

template <int NORM>
__device__ __forceinline__ void load_worker_tile(const QuantLane<NORM>& q, const GradRows& g, uint32_t m,
                                                 float4 (&x)[kLoadsPerLane]) {
#pragma unroll
  for (int j = 0; j < kLoadsPerLane; ++j) x[j] = load_row_stream(g.row(m) + q.iv[j]);
}

// Codes of one worker for this lane's 16 coordinates: four fragments of 4 codes each.
template <int NORM, int BITS, bool RECIP>
__device__ __forceinline__ void quantize_worker_tile(const QuantLane<NORM>& q, const float4 (&x)[kLoadsPerLane],
                                                     float R, float mu, uint32_t m, uint32_t iter, uint32_t k0,
                                                     uint32_t k1, uint32_t (&frag)[kLoadsPerLane]) {
  if (R == 0.f) {
#pragma unroll
    for (int j = 0; j < kLoadsPerLane; ++j) frag[j] = 0u;
    return;
  }
  const float inv_r = 1.0f / R;
#pragma unroll
  for (int j = 0; j < kLoadsPerLane; ++j) {
    const U32x4 rnd = philox4x32_10((uint32_t)q.iv[j], m, iter, 0u, k0, k1);
    const float4 v = normalize4<NORM, RECIP>(x[j], q.rt[j], mu);
    frag[j] = quantize4<BITS>(v, inv_r, rnd);
  }
}

// One LDS buffer per wavefront seen as bytes, half-words or words (the types may alias each other).
typedef uint8_t __attribute__((may_alias)) lds_u8;
typedef uint16_t __attribute__((may_alias)) lds_u16;
typedef uint32_t __attribute__((may_alias)) lds_u32;
template <int WORDS, int SLOTS = 1>
union FragmentBuffer {
  lds_u8 b8[SLOTS][kWavesPerBlock][WORDS * 4];
  lds_u16 b16[SLOTS][kWavesPerBlock][WORDS * 2];
  lds_u32 b32[SLOTS][kWavesPerBlock][WORDS];
};

__device__ __forceinline__ void wave_lds_fence() {
  // Same-wavefront LDS traffic is executed in order; this only pins the compiler's order.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// A workgroup barrier behind which LDS is up to date and loads from global memory stay in flight (__syncthreads lets no
// memory operation pass, and the compiler waits for all of them).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Fragment (j, lane) is fragment number 64 j + lane of the wavefront's packed output: write the
// fragments to LDS at that index, read whole words back, store them contiguously.
// DEFER: the words stay in LDS slot `slot` (one slot per worker of the workgroup) and are written by
// flush_packed after the last worker, 16 bytes per lane.
template <int BITS, int WPW, int SLOTS, bool DEFER>
__device__ __forceinline__ void store_packed(FragmentBuffer<WPW, SLOTS>& lds, int slot, int wave, int lane,
                                             const uint32_t (&frag)[kLoadsPerLane], uint32_t* __restrict__ row,
                                             uint64_t word_base, uint64_t words) {
  if (BITS == 2) {
#pragma unroll
    for (int j = 0; j < kLoadsPerLane; ++j) lds.b8[slot][wave][j * kWave + lane] = (uint8_t)frag[j];
  } else {
#pragma unroll
    for (int j = 0; j < kLoadsPerLane; ++j) lds.b16[slot][wave][j * kWave + lane] = (uint16_t)frag[j];
  }
  if (DEFER) return;
  wave_lds_fence();
#pragma unroll
  for (int k = 0; k < WPW / kWave; ++k) {
    const uint64_t wi = word_base + (uint64_t)k * kWave + lane;
    const uint32_t word = lds.b32[slot][wave][k * kWave + lane];
    if (wi < words) store_word_through(row + wi, word);
  }
  wave_lds_fence();
}

typedef uint32_t v4u_t __attribute__((ext_vector_type(4)));

// The deferred words of `count` workers: a row of the wavefront tile is WPW words, WPW / 4 lanes
// store it 16 bytes each, so one store instruction covers 256 / WPW rows.  The store carries the
// device-coherent cache policy (sc1) like store_word_through; there is no builtin for a 16-byte store
// with that policy, hence the instruction is written out.  Nothing after it depends on the
// memory counters (the wavefront ends), and the trailing no-op covers the cycle in which the data
// registers must stay untouched.  Measured against 4-byte sc1 stores issued per worker: quantise pass
// 0.834 -> 0.806 ms; the same with non-temporal or plain 16-byte stores: 0.84 / 0.88 ms.
__device__ __forceinline__ void store4_through(uint32_t* dst, const v4u_t& w4) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" : : "v"(dst), "v"(w4) : "memory");
}
template <int WPW, int SLOTS>
__device__ __forceinline__ void flush_packed(FragmentBuffer<WPW, SLOTS>& lds, int wave, int lane,
                                             uint32_t* __restrict__ codes, uint64_t words, uint64_t word_base,
                                             uint32_t m0, uint32_t count) {
  constexpr int LPR = WPW / 4;       // lanes per row
  constexpr int RPI = kWave / LPR;   // rows per store instruction
  wave_lds_fence();
  const int quad = lane % LPR;
#pragma unroll
  for (int r0 = 0; r0 < SLOTS; r0 += RPI) {
    const uint32_t r = (uint32_t)(r0 + lane / LPR);
    if (r < count) {
      const v4u_t w4 = *reinterpret_cast<const v4u_t*>(&lds.b32[r][wave][4 * quad]);
      store4_through(codes + (uint64_t)(m0 + r) * words + word_base + 4 * quad, w4);
    }
  }
}

// Worker loop of one wavefront tile, software pipelined two workers per trip so that the two
// register sets swap roles without copies: the loads of worker m+1 are in flight while the codes
// of worker m are computed.
// Small problems: the scale pass left at most kFusedScaleRows rows of per-workgroup maxima (partials[row][m]);
// the quantiser then takes their maximum itself, a row per lane, instead of waiting for a reduction kernel of its
// own, and the first workgroup publishes scales[m].
struct FusedScale {
  const float* partials;
  uint32_t rows;
  float* out;
};

__device__ __forceinline__ float fused_scale(const FusedScale& f, uint32_t m, uint32_t M, bool publish) {
  float v = 0.f;
  for (uint32_t b = threadIdx.x % kWave; b < f.rows; b += kWave) v = fmaxf(v, f.partials[(uint64_t)b * M + m]);
  v = wave_max_nonneg(v);
  v = v < FLT_MIN ? 0.f : v;
  if (publish) f.out[m] = v;
  return v;
}

template <int NORM, int BITS, int WPW, int SLOTS, bool FUSED, bool DEFER>
__device__ __forceinline__ void quantize_rows(const QuantLane<NORM>& q, FragmentBuffer<WPW, SLOTS>& lds, int wave, int lane,
                                              const GradRows& g, const float* __restrict__ scales,
                                              uint32_t* __restrict__ codes, uint64_t words,
                                              uint64_t word_base, uint32_t m0, uint32_t m_end, uint32_t iter,
                                              uint32_t k0, uint32_t k1, const float* __restrict__ means,
                                              const FusedScale& fs, uint32_t M) {
  constexpr int L = kLoadsPerLane;
  float4 xa[L], xb[L];
  uint32_t frag[L];
  // The scale (and mean) of a worker is fetched before the tile loads that are to stay in flight
  // during the previous worker's arithmetic: loads return in order, so a scalar fetched after them
  // would make the wait for it a wait for the whole prefetch.
  auto mean_of = [&](uint32_t m) { return NORM == kNormMean ? means[m] : 0.f; };
  auto scale_of = [&](uint32_t m) {
    return FUSED ? fused_scale(fs, m, M, blockIdx.x == 0 && threadIdx.x == 0) : scales[m];
  };
  float ra = scale_of(m0), mua = mean_of(m0), rb = 0.f, mub = 0.f;
  load_worker_tile<NORM>(q, g, m0, xa);
  // Steady state: both prefetches of a trip are unconditional.  A load issued under a condition
  // makes the compiler wait for all outstanding loads where the paths join (it cannot count what
  // is in flight), which would drain the prefetch before the arithmetic it is meant to overlap.
  uint32_t m = m0;
  for (; m + 2 < m_end; m += 2) {
    rb = scale_of(m + 1);
    mub = mean_of(m + 1);
    load_worker_tile<NORM>(q, g, m + 1, xb);
    quantize_worker_tile<NORM, BITS, kByReciprocal<NORM, SLOTS>>(q, xa, ra, mua, m, iter, k0, k1, frag);
    store_packed<BITS, WPW, SLOTS, DEFER>(lds, DEFER ? (int)(m - m0) : 0, wave, lane, frag, codes + (uint64_t)m * words, word_base,
                                          words);
    ra = scale_of(m + 2);
    mua = mean_of(m + 2);
    load_worker_tile<NORM>(q, g, m + 2, xa);
    quantize_worker_tile<NORM, BITS, kByReciprocal<NORM, SLOTS>>(q, xb, rb, mub, m + 1, iter, k0, k1, frag);
    store_packed<BITS, WPW, SLOTS, DEFER>(lds, DEFER ? (int)(m + 1 - m0) : 0, wave, lane, frag,
                                          codes + (uint64_t)(m + 1) * words, word_base, words);
  }
  // one or two workers are left, the first of them already in xa
  if (m + 1 < m_end) {
    rb = scale_of(m + 1);
    mub = mean_of(m + 1);
    load_worker_tile<NORM>(q, g, m + 1, xb);
    quantize_worker_tile<NORM, BITS, kByReciprocal<NORM, SLOTS>>(q, xa, ra, mua, m, iter, k0, k1, frag);
    store_packed<BITS, WPW, SLOTS, DEFER>(lds, DEFER ? (int)(m - m0) : 0, wave, lane, frag, codes + (uint64_t)m * words, word_base,
                                          words);
    quantize_worker_tile<NORM, BITS, kByReciprocal<NORM, SLOTS>>(q, xb, rb, mub, m + 1, iter, k0, k1, frag);
    store_packed<BITS, WPW, SLOTS, DEFER>(lds, DEFER ? (int)(m + 1 - m0) : 0, wave, lane, frag,
                                          codes + (uint64_t)(m + 1) * words, word_base, words);
  } else {
    quantize_worker_tile<NORM, BITS, kByReciprocal<NORM, SLOTS>>(q, xa, ra, mua, m, iter, k0, k1, frag);
    store_packed<BITS, WPW, SLOTS, DEFER>(lds, DEFER ? (int)(m - m0) : 0, wave, lane, frag, codes + (uint64_t)m * words, word_base,
                                          words);
  }
  if (DEFER) flush_packed<WPW, SLOTS>(lds, wave, lane, codes, words, word_base, m0, m_end - m0);
}

// The ragged last wavefront tile of worker m: a wavefront of its own.
template <int NORM, int BITS, int WPW, int SLOTS>
__device__ __forceinline__ void quantize_ragged_tile(FragmentBuffer<WPW, SLOTS>& lds, int wave, int lane, const GradRows& g,
                                                     const float4* ref4, const float4* ref24, float R, float mu,
                                                     uint32_t* __restrict__ codes, uint64_t d, uint64_t words, uint32_t m,
                                                     float eps, uint32_t iter, uint32_t k0, uint32_t k1) {
  constexpr int L = kLoadsPerLane;
  const uint64_t tile = d / kWaveTileElements;
  QuantLane<NORM> q;
  float4 x[L];
  uint32_t frag[L];
#pragma unroll
  for (int j = 0; j < L; ++j) {
    q.iv[j] = tile * (kWave * L) + (uint64_t)j * kWave + lane;
    q.rt[j].load_ragged(ref4, ref24, q.iv[j], d, eps);
    x[j] = load_row_ragged(g, m, q.iv[j], d, mu);
  }
  quantize_worker_tile<NORM, BITS, false>(q, x, R, mu, m, iter, k0, k1, frag);
  store_packed<BITS, WPW, SLOTS, false>(lds, 0, wave, lane, frag, codes + (uint64_t)m * words, tile * WPW, words);
}

// skip_if_set: behind the candidate coder, all but the ragged tile's workgroups (which has no slots) return at once when
// that word says that the codes come from the slots.  (Returning from 32768 workgroups takes 9 us at d = 2^27; 4096 that
// walk the tiles return in 3, but where the rows are too dense for the slots they quantise slower: encode + decode at
// d = 2^27, M = 8, Gaussian residuals 1763 us, 1822 that way.)
// 128 registers, four wavefronts per SIMD, but for the combined form, whose two references do not fit that, and the
// quotient form in groups of 4, which takes 130: a spilled register is reloaded in the pipelined loop, where the reload
// waits for every load in flight.
template <int NORM, int BITS, int MC, bool FUSED>
__global__ __launch_bounds__(kBlock, NORM == kNormComb || (NORM == kNormQuot && MC == 4) ? 3 : 4) void quantize_pack_vec_kernel(
    GradRows g, const float4* __restrict__ ref4, const float4* __restrict__ ref24,
    const float* __restrict__ scales, uint32_t* __restrict__ codes, uint64_t d, uint64_t words, uint32_t main_blocks,
    uint32_t M, float eps, uint32_t k0, uint32_t k1, uint32_t iter, const float* __restrict__ means,
    FusedScale fs, const uint32_t* __restrict__ skip_if_set) {
  constexpr int L = kLoadsPerLane;
  constexpr int WPW = kWave * L * 4 * BITS / 32;  // packed words per wavefront tile
  __shared__ __attribute__((aligned(16))) FragmentBuffer<WPW, MC> lds;
  if (skip_if_set != nullptr && blockIdx.x < main_blocks && skip_if_set[0] != 0u) return;
  // The quotient and combined forms lack registers: there the wavefront's number is a value the compiler knows to be the
  // same in every lane, which makes row addresses scalar (encode + decode at d = 2^27, M = 8, quotient: 4-bit 1852 us with 2
  // spilled registers, 1837 this way; 2-bit 1746 / 1729).
  const int wave = kByReciprocal<NORM, MC> ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)) : (int)(threadIdx.x / kWave);
  const int lane = threadIdx.x % kWave;
  const uint64_t ntiles = d / kWaveTileElements;  // whole wavefront tiles
  const uint32_t m0 = blockIdx.y * MC;
  const uint32_t m_end = min(m0 + MC, M);
  if (blockIdx.x < main_blocks) {
    const uint64_t wave_tile = (uint64_t)blockIdx.x * kWavesPerBlock + wave;
    if (wave_tile >= ntiles) return;  // whole wavefronts of the last workgroup; nothing below meets the others
    QuantLane<NORM> q;
#pragma unroll
    for (int j = 0; j < L; ++j) {
      q.iv[j] = wave_tile * (kWave * L) + (uint64_t)j * kWave + lane;
      q.rt[j].load(ref4, ref24, q.iv[j], eps);
      if (kByReciprocal<NORM, MC>) q.rt[j].reciprocals();
    }
    // (the 16-byte stores at the end of the workgroup take words at any 4-byte boundary)
    quantize_rows<NORM, BITS, WPW, MC, FUSED, (MC > 1)>(q, lds, wave, lane, g, scales, codes, words, wave_tile * WPW, m0,
                                                        m_end, iter, k0, k1, means, fs, M);
  } else {
    const uint32_t m = m0 + (blockIdx.x - main_blocks) * kWavesPerBlock + (uint32_t)wave;
    if (m >= m_end) return;
    const float R = FUSED ? fused_scale(fs, m, M, blockIdx.x == 0 && threadIdx.x == 0) : scales[m];
    quantize_ragged_tile<NORM, BITS>(lds, wave, lane, g, ref4, ref24, R, NORM == kNormMean ? means[m] : 0.f, codes, d,
                                     words, m, eps, iter, k0, k1);
  }
}

// ------------------------------------------------------------------------------------------
// Ternary coder without a second pass over g   (section "Gradient Compression": P(z = 1) = |v| / R)
//
// In high dimension nearly every element of a row codes to 0: the largest element R is far above the
// typical |v|, and only a fraction E|v| / R of the elements -- a few percent -- draws z = 1.  Whether an
// element CAN code non-zero is decided in the scale pass, before R is known, against any lower bound
// R^ <= R at hand: fl(1 / R^) >= fl(1 / R) (the correctly rounded quotient is monotone) and
// fl(|v| x) is monotone in x, so  u >= fl(|v| fl(1 / R^))  implies  u >= fl(|v| fl(1 / R)):  level 0
// whatever R turns out to be.  The elements that fail this test -- the candidates -- are kept in a slot per
// worker and wavefront tile.  R^ is the maximum over a sample of the row taken beforehand (one tile in
// kSampleStride); a row whose sample says that its candidates will not fit the slots is left to the
// ordinary path.  The quantise pass then reads the slots instead of g.  An entry is half a word: the sign, the position within the
// 256 elements of one of the tile's four loads, and in 7 bits a bin of x = u R^ / |v|: the element codes non-zero if x is below
// rho = R^ / R, and only the few elements in the bin of rho (bin_entry below) are fetched from g and coded from the value and its
// draw.  Everything else is cleared, and the words are packed.  A slot that overflowed (a tile with more
// than 126 candidates) sends its tile through the ordinary path.  Where the sample gives no bound (its maximum is below 2^-90, zero
// included) an entry is a word: the sign, the position in 10 bits, and tau = |v| / u -- the scale up to which the element codes non-zero -- to 13 bits of its
// significand (slot_entry).  With the l2 scale a slot is per worker and chunk of
// four tiles: words of 12 bits of position and 11 of tau's significand; see l2_select_kernel.  The codes are those of the two-pass
// coder bit for bit; what changes is that g is read once: 4 + 4/M bytes per element instead of 8 + 8/M.
// Used for 2-bit codes when the row is long enough for the second read to come from
// memory; the ragged last tile of a row has no slots, the scale pass and the ordinary quantiser take it in
// workgroups of their own (encode + decode at d = 2^25 + 3, M = 5: 312 us by two passes, 238 this way; d = 2^26 + 1, M = 1:
// 255 / 208).
// ------------------------------------------------------------------------------------------
constexpr int kCandCap = 127;         // candidates a slot of words holds; word 0 of a slot is their count
constexpr int kSlotEntries = 128;     // 32-bit words per slot: 512 bytes per worker and wavefront tile
constexpr uint32_t kSlotLine = 32;    // words of its first line, which is written and read in one piece
constexpr uint32_t kSampleStride = 128;  // the sample: every 128th wavefront tile of a row
constexpr uint32_t kCandPosMask = 0x3FFu;  // low 10 bits of a candidate word: position within the tile
constexpr uint32_t kChunkPosMask = 0xFFFu;  // the l2 scale's slots are per worker and chunk of four tiles: 12 bits
constexpr int kL2SlotEntries = 448;         // 32-bit words of such a slot, all of them candidates
constexpr uint32_t kNoSlot = 255u;          // in the place of its count (a byte, in pairs): it overflowed, or the row has none
static_assert(kL2SlotEntries / 2 < (int)kNoSlot, "the count fits a byte");
constexpr float kBoundMin = 0x1p-90f;  // below, the sample gives no bound
// What a worker's slots hold: nothing (too dense), words (tau), or bins of u R^ / |v|, two to a word.
constexpr uint32_t kFormNone = 0u, kFormWords = 1u, kFormBins = 2u;

// The sample of a row taken before the scale pass: over every kSampleStride-th wavefront tile, the largest
// |v| (the lower bound R^ of the row's scale) and the sum of |v|.  Their ratio, mean |v| / R^, is the share
// of the row's elements that will be candidates -- P(u < |v| / R^) averaged over the elements -- so it tells
// beforehand whether the slots can hold them.  One worker per workgroup row (blockIdx.y); partial results per
// workgroup, reduced by the wavefronts of absmax_select_kernel that use them (for the l2 norm by sample_finish_kernel).
constexpr uint32_t kL2OverflowCounts = kBlock;  // counters that the workgroups of l2_select_kernel share
// 1024 elements x 0.10 + two standard deviations fill a slot of kCandCap, 4096 x 0.10 + two one of kL2SlotEntries
constexpr float kDenseLimit = 0.10f;
// L2: the bound is of the row's 2-norm instead, from the sum of squares over the sample in binary64 (the partial
// results are the workgroups' own norms).
constexpr int kSampleThreads = 1024, kSampleWaves = kSampleThreads / kWave;  // (few, large workgroups: few partial results)
constexpr uint32_t kSampleRows = 64;  // workgroups per worker at most
template <int NORM, bool L2>
__global__ __launch_bounds__(kSampleThreads) void sample_stats_kernel(GradRows g, const float4* __restrict__ ref4,
                                                              float* __restrict__ part_max,
                                                              float* __restrict__ part_sum, uint64_t nvec, uint32_t M) {
  constexpr int L = kAbsmaxLoads;
  constexpr uint64_t kWaveTile = (uint64_t)kWave * L;
  __shared__ float red[2][kSampleWaves];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const uint32_t m = blockIdx.y;
  const uint64_t ntiles = nvec / kWaveTile;  // whole tiles only
  const v4f_u_t* row = g.row(m);
  __shared__ double squares[kSampleWaves];
  float amax = 0.f, asum = 0.f;
  double sq = 0.0;
  for (uint64_t tile = ((uint64_t)blockIdx.x * kSampleWaves + wave) * kSampleStride; tile < ntiles;
       tile += (uint64_t)gridDim.x * kSampleWaves * kSampleStride) {
    float4 x[L], r[L];
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const uint64_t i = tile * kWaveTile + (uint64_t)(j * kWave + lane);
      x[j] = load_row_stream(row + i);
      r[j] = NORM == kNormSub ? ref4[i] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int j = 0; j < L; ++j) {
      const float a0 = fabsf(x[j].x - r[j].x), a1 = fabsf(x[j].y - r[j].y);
      const float a2 = fabsf(x[j].z - r[j].z), a3 = fabsf(x[j].w - r[j].w);
      if (L2)
        sq += ((double)a0 * a0 + (double)a1 * a1) + ((double)a2 * a2 + (double)a3 * a3);
      else
        amax = fmaxf(fmaxf(amax, fmaxf(a0, a1)), fmaxf(a2, a3));
      asum += (a0 + a1) + (a2 + a3);
    }
  }
  amax = wave_max(amax);
  asum = wave_sum(asum);
  if (L2)
    for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, kWave);
  if (lane == 0) {
    red[0][wave] = amax;
    red[1][wave] = asum;
    squares[wave] = sq;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    float mx = red[0][0], sm = red[1][0];
#pragma unroll
    for (int k = 1; k < kSampleWaves; ++k) {
      mx = fmaxf(mx, red[0][k]);
      sm += red[1][k];
      sq += squares[k];
    }
    if (L2) mx = (float)sqrt(sq);
    part_max[(uint64_t)blockIdx.x * M + m] = mx;
    part_sum[(uint64_t)blockIdx.x * M + m] = sm;
  }
}

// R^ of a row (0 when below the smallest normal number, as for a scale) from the sample's maximum, and what its slots are to hold:
// nothing where the sum of |v| over the sample says that its candidates would not fit: the scale pass then
// takes that worker's part as an ordinary scale pass and the quantise pass takes its tiles through the
// ordinary path, without the slots.  sampled = elements of a row in the sample.  (A sum that is no number compares false.  An infinite one
// compares true under an infinite maximum: the row's scale is then infinite, none of its elements is a candidate and all code to 0, as they
// do from the value.)
__device__ __forceinline__ uint32_t form_of_slots(float r_hat, float sum, float sampled) {
  return sum <= kDenseLimit * sampled * r_hat ? (r_hat < kBoundMin ? kFormWords : kFormBins) : kFormNone;
}

// The same for the l2 scale, a launch of its own, one workgroup per worker: R^ is the norm of the workgroups' norms, made smaller by 2^-10
// of itself, which is more than all roundings on the way here and in the row's own ordered sum can come to.
__global__ __launch_bounds__(kBlock) void sample_finish_kernel(const float* __restrict__ part_max,
                                                               const float* __restrict__ part_sum, uint32_t nblocks,
                                                               uint32_t M, float sampled, float* __restrict__ sample_max,
                                                               uint32_t* __restrict__ select_ok,
                                                               uint32_t* __restrict__ overflowed) {
  if (blockIdx.x == 0) overflowed[threadIdx.x] = 0u;  // l2_select_kernel adds to these
  __shared__ float red[kWavesPerBlock];
  __shared__ double squares[kWavesPerBlock];
  const uint32_t m = blockIdx.x;
  float sm = 0.f;
  double sq = 0.0;
  for (uint32_t b = threadIdx.x; b < nblocks; b += kBlock) {
    const float p = part_max[(uint64_t)b * M + m];
    sq += (double)p * p;
    sm += part_sum[(uint64_t)b * M + m];
  }
  sm = wave_sum(sm);
  for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off, kWave);
  if (threadIdx.x % kWave == 0) {
    red[threadIdx.x / kWave] = sm;
    squares[threadIdx.x / kWave] = sq;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 1; k < kWavesPerBlock; ++k) {
      sm += red[k];
      sq += squares[k];
    }
    const float mx = (float)sqrt(sq) * (1.0f - 0x1p-10f);
    sample_max[m] = mx < FLT_MIN ? 0.f : mx;
    select_ok[m] = form_of_slots(mx, sm, sampled);
  }
}

// Staging of one worker's candidates in a wavefront tile: the count and up to kCandCap candidates (value word and
// draw), one word that takes everything beyond the capacity, then a word per lane for the elements that are no
// candidates.
constexpr uint32_t kStageSink = kSlotEntries, kStageWords = kStageSink + 2 + kWave;
static_assert(kStageWords <= 255, "a candidate's two words by one instruction");
// Of the l2 scale, where candidates gather over a chunk: the staging area is written out at the end of a tile that leaves more than
// kL2FlushAt in it, so that every tile finds room for as many as a slot per tile held.  (Four workgroups a compute unit: 40.6 of
// 40.9 KB of LDS each.)
constexpr uint32_t kL2FlushAt = 48, kL2StageSink = kL2FlushAt + kSlotEntries, kL2StageWords = kL2StageSink + 2 + kWave;
static_assert(kL2StageWords % 2 == 0, "read in pairs");

// The lower bound R^ of a worker's scale, as the factor of the candidates' test
//   u < fl(|v| fl(1 / R^)),  u = (word >> 8) 2^-24,
// which is made in three operations and from above:  float(word) < |v| c1 + 258  with
// c1 = fl(fl(1 / R^) 2^32 (1 + 2^-20)).  It holds whenever the exact test does (then word < 2^32 fl(|v| / R^) + 256;
// converting the word and the two roundings on the right move either side by less than 2^-23 relatively,
// which the factor 1 + 2^-20 and the 2 added to 256 cover) and passes 2^-20 more elements than it: the
// quantise pass codes a candidate exactly, so more is harmless.  Below 2^-90 no bound is claimed (c1 would
// overflow): every non-zero element is a candidate.
__device__ __forceinline__ float candidate_factor(float r_hat) {
  return r_hat >= kBoundMin ? (1.0f / r_hat) * (0x1p32f * (1.0f + 0x1p-20f)) : INFINITY;
}

// The candidates of one float4 per lane (load j of the tile) go to number base of the staging area and behind it.  FEW: candidates
// are rare, most float4 of a whole wavefront hold none.
template <bool FEW, uint32_t POS_MASK, uint32_t SINK>
__device__ __forceinline__ void stage_candidates(uint32_t* stage, uint32_t* draws, const float4& v, const U32x4& rnd,
                                                 float c1, int j, int lane, uint32_t& base) {
  const float vv[4] = {v.x, v.y, v.z, v.w};
  const uint32_t rr[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
  bool cand[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) cand[c] = (float)rr[c] < __builtin_fmaf(fabsf(vv[c]), c1, 258.0f);
  if (FEW && __builtin_amdgcn_ballot_w64((int)cand[0] | (int)cand[1] | (int)cand[2] | (int)cand[3]) == 0ull) return;
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint64_t mask = __builtin_amdgcn_ballot_w64(cand[c]);
    const uint32_t pos = base + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32),
                                                          __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    // Every lane writes, the others into a word of their own behind the candidates': a store under a
    // condition would end the basic block at every element, and the sixteen elements of a lane could not
    // overlap.  Candidates beyond the slot's capacity (the slot is then not used) share one word.
    const uint32_t at = cand[c] ? min(pos, SINK) : SINK + 2 + (uint32_t)lane;
    stage[at] = (__float_as_uint(vv[c]) & ~POS_MASK) | (uint32_t)(256 * j + c) | 4u * (uint32_t)lane;
    draws[at] = rr[c];
    base += (uint32_t)__builtin_popcountll(mask);
  }
}

// What goes into the slot for a candidate is not v but tau = |v| / u (u its 24-bit draw), the scale up to which it codes
// non-zero, to what its position leaves of the significand: the quantise pass then compares the row's scale with tau and
// needs neither the draw nor the value.  u = 0 gives an infinite tau (or none, for v = 0), which the quantise pass takes
// as "look at the value".
template <uint32_t POS_MASK>
__device__ __forceinline__ uint32_t slot_entry(uint32_t value_word, uint32_t draw) {
  constexpr uint32_t kMagnitude = 0x7FFFFFFFu & ~POS_MASK;
  const float tau = __uint_as_float(value_word & kMagnitude) * (__builtin_amdgcn_rcpf((float)(draw >> 8)) * 0x1p24f);
  return (__float_as_uint(tau) & kMagnitude) | (value_word & (0x80000000u | POS_MASK));
}

// How it reads there.  The entry of a normal value brackets tau: its significand was cut to K = 23 - (bits of the position) bits
// twice (the value's, then tau's own) and its arithmetic is good to 2^-22, so tau lies in [lo (1 - 2^-22), hi (1 + 2^-K + 2^-21)].
// ternary_code's level [u < fl(|v| fl(1 / R))] is 1 for R <= tau (1 - 2^-21) and 0 for R >= tau (1 + 2^-21) (the two
// roundings move |v| / R by less than 2^-22 relatively, 1 / R > 2^126 included), so only a scale inside the widened bracket
// -- three candidates in ten thousand with 13 bits, a dozen with 11 -- needs the value and the draw.
// Of a value below the smallest normal number the cut may take half or all, so its tau has no such upper end, but it is below 2^-126 /
// 2^-24: only a scale of 2^-101 and more is above every such tau, and under a smaller one nothing codes 0 unseen.  (The lower
// end holds: the cut only lowers it, and a product that rounds coarsely is below every scale that is not 0.)
template <uint32_t POS_MASK>
__device__ __forceinline__ int entry_codes_one(uint32_t e, float r) {  // (false where tau is infinite or no number: not bounded)
  return (int)((e & 0x7F800000u) != 0x7F800000u) & (int)(r <= __uint_as_float(e & 0x7FFFFFFFu & ~POS_MASK) * (1.0f - 0x1p-19f));
}
template <uint32_t POS_MASK>
__device__ __forceinline__ int entry_codes_zero(uint32_t e, float r) {  // (false where tau is not bounded)
  constexpr float kAbove = POS_MASK == kCandPosMask ? 1.0f + 0x1p-12f : 1.0f + 0x1p-10f;
  return (int)(r >= 0x1p-101f) & (int)(r >= __uint_as_float((e & 0x7FFFFFFFu) | POS_MASK) * kAbove);
}
// With a bound R^ the entries are half as long.  x = u R^ / |v| is uniform on (0, 1) over the candidates, so each has the same chance to
// lie in the bin of rho and to need its value.  Bins grow with x, 208 to 1 above a half, where rho mostly is (0.8 to 0.9 in Gaussian
// rows, 0.55 to 0.9 where |v| falls off exponentially), and 44 to 1 below.  Bin 0: u = 0, or no number -- look at the value; 127 is
// none's.  The entry: the bin, the position within the tile's 256 elements of one load, the sign.
// (Writes next to the reads cost several times their bytes: at d = 2^27, M = 8 the scale pass takes 767 us without them, 831 with 8
// bytes a slot, 910 with slots of words, 200 bytes on average, 836 with one whole line of 128 bytes each.  That all of one line is
// written, and lines lie next to each other, is a part of it: half-words in slots 512 bytes apart 886.)
constexpr int kBinShift = 9;
constexpr uint32_t kNoEntry = 0xFFFFu;  // bin 127: behind the last entry
__device__ __forceinline__ uint32_t bin_of(float x) {
  const float y = fmaxf(__builtin_fmaf(x, 44.0f, 1.0f), __builtin_fmaf(x, 208.0f, -81.0f));
  return x > 0.f ? (uint32_t)fminf(y, 126.0f) : 0u;
}
__device__ __forceinline__ uint32_t bin_entry(uint32_t value_word, uint32_t draw, float c1) {
  const float a = __uint_as_float(value_word & 0x7FFFFFFFu & ~kCandPosMask);
  const float x = (float)(draw & 0xFFFFFF00u) * __builtin_amdgcn_rcpf(a * c1);
  return (bin_of(x) << kBinShift) | (__builtin_amdgcn_alignbit(value_word, value_word, 31) & 0x1FFu);
}
// The x of an entry is good to 2^-12.9 upwards (the cut of |v|) and 2^-19 downwards (c1, the reciprocal), ternary_code's roundings move its
// level by 2^-21: below the bin of rho (1 - 2^-18) the level is 1, above the bin of rho (1 + 2^-12) it is 0.
__device__ __forceinline__ uint32_t bin_limits(float r_hat, float r) {
  const float rho = r_hat / r;
  const uint32_t below = bin_of(rho * (1.0f - 0x1p-18f)), above = rho >= 0.f ? bin_of(rho * (1.0f + 0x1p-12f)) : 126u;
  return (below << 8) | (above << 16);
}
// The first lines of the slots of all of a worker's tiles lie next to each other, and behind them the rest of each.
struct Slot {
  uint32_t *line, *rest;
  __device__ __forceinline__ Slot(uint32_t* slots, uint64_t ntiles, uint32_t m, uint64_t tile) {
    uint32_t* worker = slots + (uint64_t)m * ntiles * kSlotEntries;
    line = worker + tile * kSlotLine;
    rest = worker + ntiles * kSlotLine + tile * (kSlotEntries - kSlotLine);
  }
  // half-words 64 k to 64 k + 63
  __device__ __forceinline__ uint16_t* halves(int k) const { return reinterpret_cast<uint16_t*>(k == 0 ? line : rest); }
};
__device__ __forceinline__ void store_half_through(uint16_t* p, uint32_t v) {
  __hip_atomic_store(p, (uint16_t)v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The code of element coord of worker m from its value.
template <int NORM>
__device__ __forceinline__ uint32_t code_of_element(const GradRows& g, const float4* ref4, uint64_t coord, uint32_t m, float r,
                                                    uint32_t iter, uint32_t k0, uint32_t k1) {
  const U32x4 rnd = philox4x32_10((uint32_t)(coord >> 2), m, iter, 0u, k0, k1);
  const uint32_t sel = (uint32_t)coord & 3u;
  const uint32_t word = sel == 0u ? rnd.x : sel == 1u ? rnd.y : sel == 2u ? rnd.z : rnd.w;
  float r1 = 0.f;
  if (NORM == kNormSub) r1 = reinterpret_cast<const float*>(ref4)[coord];
  return ternary_code(normalize_w<NORM>(g.base[(uint64_t)m * g.pitch + coord], r1, 1.f, 0.f), 1.0f / r, word);
}
// The codes of a wavefront's tile of worker m, which has no slot, into its 64 words of LDS.  (Two float4 at a time: all four
// need more than the 64 registers of eight wavefronts per SIMD.)
template <int NORM>
__device__ __forceinline__ void code_tile(lds_u8* bytes, const GradRows& g, const float4* ref4, const float4* ref24, uint64_t tile,
                                          uint32_t m, int lane, float r, float eps, uint32_t iter, uint32_t k0, uint32_t k1) {
  constexpr int L = kLoadsPerLane;
  const float inv_r = 1.0f / r;
#pragma unroll 1
  for (int j = 0; j < L; j += 2) {
    const uint64_t iv = tile * (kWave * L) + (uint64_t)(j * kWave + lane);
    const v4f_u_t* row = g.row(m) + iv;
    float4 v[2] = {load_row_stream(row), load_row_stream(row + kWave)};
    RefTile<NORM> rt[2];
    rt[0].load(ref4, ref24, iv, eps);
    rt[1].load(ref4, ref24, iv + kWave, eps);
#pragma unroll
    for (int k = 0; k < 2; ++k) v[k] = normalize4<NORM, false>(v[k], rt[k], 0.f);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const U32x4 rnd = philox4x32_10((uint32_t)iv + (uint32_t)(k * kWave), m, iter, 0u, k0, k1);
      bytes[(j + k) * kWave + lane] = (uint8_t)quantize4<2>(v[k], inv_r, rnd);
    }
  }
}

// The candidates of one float4 per lane as stage_candidates stages them, but for the load's place in the position, in straight
// code: a select on "candidate" becomes a branch, which ends the basic block at every element, unless the instruction is written out.
// at: LDS address of the next free word of the staging area (the draws lie kStageWords words behind); idle: a lane's own word behind it, for
// its elements that are no candidates; full: where at stops.
__device__ __forceinline__ void stage_straight(uint32_t idle, uint32_t full, const float4& v, const U32x4& rnd, float c1, int lane, uint32_t& at) {
  typedef uint32_t __attribute__((address_space(3))) lds_word;
  const float vv[4] = {v.x, v.y, v.z, v.w};
  const uint32_t rr[4] = {rnd.x, rnd.y, rnd.z, rnd.w};
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const uint64_t mask = __builtin_amdgcn_ballot_w64((float)rr[c] < __builtin_fmaf(fabsf(vv[c]), c1, 258.0f));
    const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
    const uint32_t own = (before << 2) + at;
    uint32_t to;
    asm("v_cndmask_b32 %0, %1, %2, %3" : "=v"(to) : "v"(idle), "v"(own), "s"(mask));
    lds_word* p = (lds_word*)(uintptr_t)to;
    p[0] = (__float_as_uint(vv[c]) & ~kCandPosMask) | (uint32_t)c | 4u * (uint32_t)lane;  // (the load is told by the head)
    p[kStageWords] = rr[c];
    at = min(at + 4u * (uint32_t)__builtin_popcountll(mask), full);
  }
}

// The staged candidates to their slot; false where they do not fit (only the count is written).  Words: the count, then
// an entry each.  Bins: half-words, the first two of which hold, a byte each, the number of half-words in use and how many come before
// the entries of the tile's second, third and fourth 256 elements (starts), whose positions then need 8 bits; kNoEntry behind the last.
__device__ __forceinline__ bool write_slot(const uint32_t* stage, const uint32_t* draws, uint32_t base, uint32_t starts, bool bins, float c1,
                                           int lane, const Slot& slot) {
  wave_lds_fence();
  const bool fits = base <= (uint32_t)kSlotEntries;
  if (bins) {
    const uint32_t head = min(base, 255u) | starts, e = bin_entry(stage[lane], draws[lane], c1);
    store_half_through(slot.halves(0) + (uint32_t)lane, lane < 2 ? head >> (16 * lane) : (uint32_t)lane < base ? e : kNoEntry);
    if (base > (uint32_t)kWave && fits)
      store_half_through(slot.halves(1) + (uint32_t)lane, (uint32_t)(kWave + lane) < base ? bin_entry(stage[kWave + lane], draws[kWave + lane], c1) : kNoEntry);
  } else {
#pragma unroll 1
    for (uint32_t i = (uint32_t)lane; i < (fits ? base : 1u); i += kWave)
      store_word_through((i < kSlotLine ? slot.line : slot.rest - kSlotLine) + i, i == 0u ? base - 1u : slot_entry<kCandPosMask>(stage[i], draws[i]));
  }
  wave_lds_fence();
  return fits;
}

template <int NORM, int MC>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void absmax_select_kernel(GradRows g, const float4* __restrict__ ref4,
                                                               const float4* __restrict__ ref24, float* partials,
                                                               uint64_t d, uint32_t main_blocks, uint32_t M, float eps,
                                                               const float* __restrict__ part_max, const float* __restrict__ part_sum,
                                                               uint32_t nsample, float sampled, float* __restrict__ sample_max,
                                                               uint32_t* __restrict__ select_ok,
                                                               uint32_t* __restrict__ slots,
                                                               uint32_t* __restrict__ overflowed, uint32_t k0,
                                                               uint32_t k1, uint32_t iter) {
  constexpr int L = kAbsmaxLoads;
  constexpr uint64_t kWaveTile = (uint64_t)kWave * L;
  static_assert(L == kLoadsPerLane, "the quantise pass reads the slots by the same tiles");
  static_assert(NORM == kNormNone || NORM == kNormSub, "the coder that reads g once: no divisor reference");
  // What a wavefront fetches per tile, in order: the reference, then the MC workers' parts, and nothing up to
  // a multiple of three.  The items rotate through three register buffers: while item i is worked on, items
  // i + 1 and i + 2 are on their way -- across the end of the tile as well (the next tile's reference and
  // first worker are requested during this tile's last workers).  The reference of the tile lives in LDS,
  // not in registers: three buffers then cost what two buffers and a reference did, and twice the bytes are
  // in flight per wavefront.  (Measured 2 % faster than two buffers that drained at the end of every tile:
  // the pass is bound neither by the depth of its prefetch nor by its arithmetic.)
  constexpr int kItems = (MC + 1 + 2) / 3 * 3;
  __shared__ __attribute__((aligned(16))) uint32_t stages[kWavesPerBlock][2][kStageWords];
  __shared__ __attribute__((aligned(16))) float4 refs[kWavesPerBlock][L][kWave];
  __shared__ uint32_t over[kWavesPerBlock];
  __shared__ float factor[kWavesPerBlock][MC];
  // the wavefront's number as a value the compiler knows to be the same in every lane: tile numbers, row and
  // slot addresses are then scalar, and a lane's own part of every address is one 32-bit offset
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = threadIdx.x % kWave;
  const uint32_t m0 = blockIdx.y * MC;
  const uint32_t count = min((uint32_t)MC, M - m0);
  uint32_t* stage = stages[wave][0];
  uint32_t* draws = stages[wave][1];
  uint32_t nover = 0;  // slots of this wavefront that overflowed
  float mx[MC];
#pragma unroll
  for (int mm = 0; mm < MC; ++mm) mx[mm] = 0.f;
  const uint64_t ntiles = d / kWaveTileElements;  // whole wavefront tiles
  if (blockIdx.x >= main_blocks) {  // the ragged last tile: its maximum only, the quantise pass codes it from g
    const uint32_t at = (blockIdx.x - main_blocks) * kWavesPerBlock + (uint32_t)wave;
    const float v = absmax_ragged_tile<NORM>(g, ref4, ref24, min(m0 + at, M - 1), d, eps, 0.f);
#pragma unroll
    for (int mm = 0; mm < MC; ++mm) mx[mm] = (uint32_t)mm == at ? v : 0.f;
    block_max_to_partials<MC>(mx, m0, M, partials);
    if (threadIdx.x == 0) overflowed[(uint64_t)blockIdx.y * gridDim.x + blockIdx.x] = 0u;
    return;
  }
  // A lane per worker: the factors go to LDS, and a bit tells of which the sample found the row too dense for the slots (only its
  // maximum is taken).  (A factor and a flag per worker in registers spilled to memory.)
  // The sample's partial results are reduced by every wavefront for itself, W workers side by side, all loads in flight together (a launch of its
  // own between the sample and this kernel: encode + decode d = 2^25 + 3, M = 5 2.5 us more, M = 8, no normalisation 6).
  constexpr int W = MC > 4 ? 8 : MC, kSteps = (int)kSampleRows * W / kWave;
  const uint32_t own = min(m0 + (uint32_t)min(lane % W, MC - 1), M - 1);
  float r_hat = 0.f, sum = 0.f;
  float pm[kSteps], ps[kSteps];
#pragma unroll
  for (int k = 0; k < kSteps; ++k) {
    const uint64_t at = (uint64_t)min((uint32_t)(k * (kWave / W) + lane / W), nsample - 1) * M + own;
    pm[k] = part_max[at];
    ps[k] = part_sum[at];
  }
#pragma unroll
  for (int k = 0; k < kSteps; ++k) {
    r_hat = fmaxf(r_hat, pm[k]);
    sum += (uint32_t)(k * (kWave / W) + lane / W) < nsample ? ps[k] : 0.f;
  }
#pragma unroll
  for (int off = W; off < kWave; off <<= 1) {
    r_hat = fmaxf(r_hat, __shfl_xor(r_hat, off, kWave));
    sum += __shfl_xor(sum, off, kWave);
  }
  r_hat = r_hat < FLT_MIN ? 0.f : r_hat;
  const uint32_t own_form = form_of_slots(r_hat, sum, sampled);
  if (lane < MC) factor[wave][lane] = candidate_factor(r_hat);
  if (blockIdx.x == 0 && threadIdx.x < (uint32_t)MC && m0 + threadIdx.x < M) {  // for the kernels that follow
    sample_max[own] = r_hat;
    select_ok[own] = own_form;
  }
  const uint32_t dense = (uint32_t)__builtin_amdgcn_ballot_w64(own_form == kFormNone);
  const uint32_t words = (uint32_t)__builtin_amdgcn_ballot_w64(own_form == kFormWords);
  wave_lds_fence();
  // one worker's part of the tile: its maximum, and its candidates into the slot
  auto worker = [&](const float4 (&x)[L], int mm, uint64_t tile) {
    uint32_t m = m0 + (uint32_t)mm;
    int own = lane;
    float amax = 0.f;
    if ((dense >> mm) & 1u) {  // (the same for the whole wavefront)
#pragma unroll
      for (int j = 0; j < L; ++j) {
        float4 v = x[j];
        if (NORM == kNormSub) {
          const float4 r = refs[wave][j][lane];
          v = make_float4(x[j].x - r.x, x[j].y - r.y, x[j].z - r.z, x[j].w - r.w);
        }
        amax = max3_abs(v.z, v.w, max3_abs(v.x, v.y, amax));
      }
      mx[mm] = fmaxf(mx[mm], amax);
      nover += 1u;  // counts as a slot that is not used
      return;
    }
    // what follows from m or the lane alone is made per tile: kept for all workers, or for both forms of this loop, it spilled to memory (68
    // scalar registers of groups of eight, 45 of five, 34 of four and 20 of two are kept in lanes of vector registers even so; 40, 7, 0 and 0 with
    // this form alone)
    asm volatile("" : "+s"(m), "+v"(own));
    const float c1 = factor[wave][mm];
    const bool bins = ((words >> mm) & 1u) == 0u;
    uint32_t base = bins ? 2u : 1u, starts = 0u;  // half-words 0 and 1 of the slot tell how many, or word 0
#pragma unroll
    for (int j = 0; j < L; ++j) {
      float4 v = x[j];
      if (NORM == kNormSub) {
        const float4 r = refs[wave][j][own];
        v = make_float4(x[j].x - r.x, x[j].y - r.y, x[j].z - r.z, x[j].w - r.w);
      }
      amax = max3_abs(v.z, v.w, max3_abs(v.x, v.y, amax));
      const uint64_t iv = tile * kWaveTile + (uint64_t)(j * kWave + own);
      const U32x4 rnd = philox4x32_10((uint32_t)iv, m, iter, 0u, k0, k1);
      stage_candidates<false, kCandPosMask, kStageSink>(stage, draws, v, rnd, c1, j, own, base);
      if (j + 1 < L) starts |= base << (8 * (j + 1));
    }
    static_assert(L == 4, "three starts");
    mx[mm] = fmaxf(mx[mm], amax);
    if (!write_slot(stage, draws, base, starts, bins, c1, own, Slot(slots, ntiles, m, tile))) nover += 1u;
  };
  // The same without a branch, where all workers of the group are there and have slots of bins: every item then issues the same loads and
  // stores, and the waits can be counted exactly (with a branch around the store they also waited for the store before and the
  // rows of the next item; 914 -> 900 us at d = 2^27, M = 8 with slots of words, a fifth fewer vector instructions).  Short groups, and
  // those with a row that is too dense or has no bound, keep the form above; with it the half-words still gain a little (encode + decode with
  // slots of words / now: d = 2^25, M = 3 197 / 192 us; d = 2^24, M = 6 167 / 161, M = 7 176 / 169, M = 9 212 / 206; d = 2^23, M = 11 145 / 138; one
  // of eight rows too dense, d = 2^24 265 / 261; next to d = 2^24, M = 8 184 / 173 without branches).
  const uint32_t stage_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint32_t*)stage;
  const uint32_t idle = stage_at + 4u * (kStageSink + 2 + (uint32_t)lane);
  auto worker_straight = [&](const float4 (&x)[L], int mm, uint64_t tile) {
    uint32_t m = m0 + (uint32_t)mm;
    asm volatile("" : "+s"(m));
    float amax = 0.f;
    uint32_t at = stage_at + 8u, head = 0u;
    const float c1 = factor[wave][mm];
#pragma unroll
    for (int j = 0; j < L; ++j) {
      float4 v = x[j];
      if (NORM == kNormSub) {
        const float4 r = refs[wave][j][lane];
        v = make_float4(x[j].x - r.x, x[j].y - r.y, x[j].z - r.z, x[j].w - r.w);
      }
      amax = max3_abs(v.z, v.w, max3_abs(v.x, v.y, amax));
      const U32x4 rnd = philox4x32_10((uint32_t)(tile * kWaveTile) + (uint32_t)(j * kWave + lane), m, iter, 0u, k0, k1);
      stage_straight(idle, stage_at + 4u * (kStageSink + 2), v, rnd, c1, lane, at);
      head |= ((at - stage_at) >> 2) << (j + 1 < L ? 8 * (j + 1) : 0);
    }
    mx[mm] = fmaxf(mx[mm], amax);
    const uint32_t base = (at - stage_at) >> 2;
    wave_lds_fence();
    // One store of the whole line, whatever the count (two lanes hold the head): under a condition, or of a length of its own, the waits for
    // the rows that follow could not be counted.
    const Slot slot(slots, ntiles, m, tile);
    const uint32_t e = bin_entry(stage[lane], draws[lane], c1);
    store_half_through(slot.halves(0) + (uint32_t)lane, lane < 2 ? head >> (16 * lane) : (uint32_t)lane < base ? e : kNoEntry);
    if (__builtin_expect(base > (uint32_t)kWave, 0)) {
      nover += base > (uint32_t)kSlotEntries ? 1u : 0u;
      store_half_through(slot.halves(1) + (uint32_t)lane, (uint32_t)(kWave + lane) < base ? bin_entry(stage[kWave + lane], draws[kWave + lane], c1) : kNoEntry);
    }
    wave_lds_fence();
  };
  // Every request is made whatever the tile (a load under a branch could not be counted by the waits that
  // follow it): past the wavefront's last tile all lanes read the first float4 of this tile's part again.
  auto request = [&](float4 (&b)[L], int item, uint64_t t, uint32_t keep) {
    if (item == 0) {
      if (NORM == kNormSub) {
#pragma unroll
        for (int j = 0; j < L; ++j) b[j] = load_stream(ref4 + t * kWaveTile + ((uint32_t)(j * kWave + lane) & keep));
      }
    } else if (item <= MC) {
      uint32_t m = min(m0 + (uint32_t)(item - 1), M - 1);
      asm volatile("" : "+s"(m));  // (as above)
      const v4f_u_t* row = g.row(m);
#pragma unroll
      for (int j = 0; j < L; ++j) b[j] = load_row_stream(row + t * kWaveTile + ((uint32_t)(j * kWave + lane) & keep));
    }
  };
  auto work = [&](const float4 (&b)[L], int item, uint64_t tile, bool straight) {
    if (item == 0) {
      if (NORM == kNormSub) {
#pragma unroll
        for (int j = 0; j < L; ++j) refs[wave][j][lane] = b[j];
        wave_lds_fence();
      }
    } else if (item <= MC) {
      if (straight)
        worker_straight(b, item - 1, tile);
      else if ((uint32_t)(item - 1) < count)
        worker(b, item - 1, tile);
    }
  };
  const uint64_t stride = (uint64_t)main_blocks * kWavesPerBlock;
  uint64_t tile = (uint64_t)blockIdx.x * kWavesPerBlock + wave;
  auto tiles = [&](auto STRAIGHT) {
    constexpr bool straight = decltype(STRAIGHT)::value;
    float4 b0[L], b1[L], b2[L];
    request(b0, 0, tile, ~0u);
    request(b1, 1, tile, ~0u);
    for (; tile < ntiles; tile += stride) {
      const bool more = tile + stride < ntiles;
      const uint64_t t_next = more ? tile + stride : tile;
      const uint32_t keep_next = more ? ~0u : 0u;
      // step i: request item i + 2 into the buffer that item i - 1 has just left, then work on item i
      auto step = [&](auto I, float4 (&into)[L], const float4 (&from)[L]) {
        constexpr int i = decltype(I)::value;
        constexpr bool wraps = i + 2 >= kItems;
        request(into, wraps ? i + 2 - kItems : i + 2, wraps ? t_next : tile, wraps ? keep_next : ~0u);
        work(from, i, tile, straight);
      };
      step(std::integral_constant<int, 0>{}, b2, b0);
      step(std::integral_constant<int, 1>{}, b0, b1);
      step(std::integral_constant<int, 2>{}, b1, b2);
      if constexpr (kItems > 3) {
        step(std::integral_constant<int, 3>{}, b2, b0);
        step(std::integral_constant<int, 4>{}, b0, b1);
        step(std::integral_constant<int, 5>{}, b1, b2);
      }
      if constexpr (kItems > 6) {
        step(std::integral_constant<int, 6>{}, b2, b0);
        step(std::integral_constant<int, 7>{}, b0, b1);
        step(std::integral_constant<int, 8>{}, b1, b2);
      }
    }
  };
  if (tile < ntiles) {
    if (count == (uint32_t)MC && (dense | words) == 0u)
      tiles(std::true_type{});
    else
      tiles(std::false_type{});
  }
  if (lane == 0) over[wave] = nover;
  block_max_to_partials<MC>(mx, m0, M, partials);  // has a workgroup barrier after its own LDS writes
  if (threadIdx.x == 0) {
    uint32_t total = 0;
#pragma unroll
    for (int k = 0; k < kWavesPerBlock; ++k) total += over[k];
    overflowed[(uint64_t)blockIdx.y * gridDim.x + blockIdx.x] = total;
  }
}

// Whether the slots are worth using, by one workgroup: at most one per fifty tiles may have overflowed (what they hold goes
// through a plain, unpipelined form of the ordinary path).  use_slots[0] = 1 or 0.  Of the l2 scale's slots, four tiles each, that is
// two in 25, so that tiles which overflow one here and one there still count as one in fifty: rows of M = 16, d = 2^22 (encode, us)
// whose one to three tiles in a hundred that are not zero are seldom in the sample 93 with a slot per tile, 115 with one slot in
// fifty, 86 to 92 so; d = 2^23 162 / 218 / 145; M = 64, d = 2^20 89 / 109 / 83.
struct SlotVote {
  const uint32_t* overflowed;  // n counts
  uint32_t n;
  uint64_t tiles_in_all;
  uint32_t* use_slots;
};
template <int THREADS>
__device__ __forceinline__ void vote_on_slots(const SlotVote& v) {
  __shared__ unsigned long long sum;
  if (threadIdx.x == 0) sum = 0ull;
  __syncthreads();
  unsigned long long mine = 0;
#pragma unroll 4
  for (uint32_t i = threadIdx.x; i < v.n; i += THREADS) mine += v.overflowed[i];
  atomicAdd(&sum, mine);
  __syncthreads();
  if (threadIdx.x == 0) v.use_slots[0] = sum * 50ull <= v.tiles_in_all ? 1u : 0u;
}

// The reduction of the scale pass's partial maxima (workgroups 0 .. M - 1, one per worker) and the vote.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void absmax_finish_vote_kernel(const float* __restrict__ partials, uint32_t nblocks,
                                                                    uint32_t M, float* __restrict__ scales,
                                                                    const float* __restrict__ sample_max,
                                                                    uint32_t* __restrict__ select_ok, SlotVote vote) {
  if (blockIdx.x < M) {
    const float r = absmax_finish_worker<THREADS>(partials, nblocks, M, scales, blockIdx.x);
    // for the quantise pass: the bins of the worker's slots whose elements code non-zero, and zero
    if (threadIdx.x == 0) select_ok[blockIdx.x] |= bin_limits(sample_max[blockIdx.x], r);
  } else {
    vote_on_slots<THREADS>(vote);
  }
}

// The packed codes of a tile from its slots.  A wavefront takes eight rows, a worker's tile each, eight lanes to a row; the words of a row
// are cleared in LDS, the candidates' codes are or-ed in, and all rows' words are written at the end as the quantiser writes them.
// What bounds it: slots read and codes written (0.13 + 0.27 GB at d = 2^27, M = 8: 66 us without what follows), and vector instructions for
// the elements that need their value (1.9 a wavefront there) and second lines (a fifth of the wavefronts).  So all of a wavefront's
// slots come by one load, what belongs to a row sits in its lanes, and the rare paths are behind the main one, there only once, eight
// wavefronts to a SIMD (64 registers).  At d = 2^27, M = 8 123 us with slots of words, a step per worker with all lanes on it; 173 so with
// half-words (530 vector and 640 scalar instructions a wavefront, the vector unit all but full); 98 now.  The draws of elements that need
// their value in scalar instructions: 115.
constexpr int quantize_tiles(int mc) { return 8 / mc; }  // tiles that a wavefront takes
template <int NORM, int MC>
__global__ __launch_bounds__(kBlock, 8) void quantize_candidates_kernel(
    GradRows g, const float4* __restrict__ ref4, const float4* __restrict__ ref24, const float* __restrict__ scales,
    const uint32_t* __restrict__ slots, uint32_t* __restrict__ codes, uint64_t d, uint64_t words, uint32_t M,
    float eps, uint32_t k0, uint32_t k1, uint32_t iter, const uint32_t* __restrict__ use_slots,
    const uint32_t* __restrict__ select_ok) {
  constexpr int WPW = (int)kWaveTileElements * 2 / 32;  // 64 packed words per row
  constexpr int T = quantize_tiles(MC), ROWS = MC * T;  // a row: a worker's tile
  constexpr int kLanes = 8, X = (int)kSlotLine / kLanes, E = 2 * X;  // lanes per row, words and half-words of the line in each
  static_assert(ROWS * kLanes == kWave && WPW == kWave && X == 4, "16 bytes of a row's line per lane");
  __shared__ __attribute__((aligned(16))) FragmentBuffer<WPW, ROWS> lds;
  if (use_slots[0] == 0u) return;  // too many tiles overflowed: the ordinary quantiser runs instead
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = threadIdx.x % kWave;
  const uint64_t ntiles = d / kWaveTileElements;
  const uint32_t m0 = blockIdx.y * MC, count = min((uint32_t)MC, M - m0);
  const uint64_t t0 = ((uint64_t)blockIdx.x * kWavesPerBlock + wave) * T;
  if (t0 >= ntiles) return;  // whole wavefronts; nothing below meets the other wavefronts
  auto tile_of = [&](uint32_t row) { return T == 1 ? t0 : min(t0 + row / MC, ntiles - 1); };
  auto worker_of = [&](uint32_t row) { return min(m0 + (T == 1 ? row : row % MC), M - 1); };
  auto is_live = [&](uint32_t row) { return (T == 1 ? row : row % MC) < count && (T == 1 || t0 + row / MC < ntiles); };
  auto slot_of = [&](uint32_t row) { return Slot(const_cast<uint32_t*>(slots), ntiles, worker_of(row), tile_of(row)); };
  // The first lines of all the slots (62 candidates of a row with a bound each) come by one load, and a lane has its row's limits and
  // what it needs of the head in registers of its own.
  const uint32_t row = (uint32_t)(lane / kLanes), part = (uint32_t)(lane % kLanes);
  const bool live = is_live(row);
  const v4u_t line = reinterpret_cast<const v4u_t*>(slot_of(row).line)[part];
  const float r = scales[worker_of(row)];
  const uint32_t limits = select_ok[worker_of(row)];
#pragma unroll
  for (int k = 0; k < ROWS; ++k) lds.b32[k][wave][lane] = 0u;
  wave_lds_fence();
  const uint32_t head = (uint32_t)__shfl((int)line[0], lane - (int)part), end = head & 255u;
  uint32_t x[X] = {part == 0 ? ~0u : line[0], line[1], line[2], line[3]};  // (the head is no entry)
  const bool bins = live && (limits & 255u) == kFormBins && end <= (uint32_t)kSlotEntries;
  const uint32_t below = bins ? max((limits >> 8) & 255u, 1u) - 1u : 0u, above = bins ? (limits >> 16) + 1u : 0u;
  // Codes are or-ed in as one bit, the low one of a code that is positive and the high one of a code that is negative.
  auto put = [&](uint32_t to, uint32_t pos, uint32_t code) { atomicOr(&lds.b32[to][wave][pos >> 4], code << (2u * (pos & 15u))); };
  // An element of each lane where `open`, coded from its value.
  auto settle = [&](bool open, uint32_t to, float scale, uint32_t pos) {
    const uint32_t of = worker_of(to);
    const uint64_t coord = tile_of(to) * kWaveTileElements + (open ? pos : 0u);
    const float value = g.base[(uint64_t)of * g.pitch + coord], ref = NORM == kNormSub ? reinterpret_cast<const float*>(ref4)[coord] : 0.f;
    const U32x4 rnd = philox4x32_10((uint32_t)(coord >> 2), of, iter, 0u, k0, k1);
    const uint32_t low = (pos & 1u) != 0u ? rnd.y : rnd.x, high = (pos & 1u) != 0u ? rnd.w : rnd.z;
    if (open) put(to, pos, ternary_code(normalize_w<NORM>(value, ref, 1.f, 0.f), 1.0f / scale, (pos & 2u) != 0u ? high : low));
  };
  // which of the tile's four loads half-words first to first + 7 of a slot belong to, four bits each
  auto loads_from = [](uint32_t of, uint32_t first) {
    uint32_t loads = 0u;
#pragma unroll
    for (int t = 1; t < 4; ++t) {
      const int ahead = max((int)((of >> (8 * t)) & 255u) - (int)first, 0);
      loads += ahead < 8 ? 0x11111111u << (4 * ahead) : 0u;
    }
    return loads;
  };
  const uint32_t loads = loads_from(head, E * part);
  uint64_t open[E], any = 0ull;
#pragma unroll
  for (int c = 0; c < E; ++c) {
    const uint32_t e = c % 2 == 0 ? x[c / 2] & 0xFFFFu : x[c / 2] >> 16;
    const bool one = e - (1u << kBinShift) < below << kBinShift;
    open[c] = __builtin_amdgcn_ballot_w64(e < above << kBinShift) & ~__builtin_amdgcn_ballot_w64(one);
    any |= open[c];
    if (one) atomicOr(&lds.b32[row][wave][((e >> 5) & 15u) + 16u * ((loads >> (4 * c)) & 3u)], 1u << (e & 31u));
  }
  if (any != 0ull) {  // a lane's elements one after the other, those of the other lanes at the same time
    uint32_t undecided = 0u;
#pragma unroll
    for (int c = 0; c < E; ++c) undecided |= __builtin_amdgcn_inverse_ballot_w64(open[c]) ? 1u << c : 0u;
    do {
      const uint32_t c = (uint32_t)__builtin_ctz(undecided | 256u) & 7u;
      uint32_t e = x[0];
#pragma unroll
      for (int i = 1; i < X; ++i) e = c / 2 == (uint32_t)i ? x[i] : e;
      settle(undecided != 0u, row, r, ((e >> (16 * (c & 1u) + 1)) & 255u) + 256u * ((loads >> (4 * c)) & 3u));
      undecided &= undecided - 1u;
    } while (__builtin_amdgcn_ballot_w64(undecided != 0u) != 0ull);
  }
  // The second lines, a row at a time.
  uint64_t longer = __builtin_amdgcn_ballot_w64(bins && end > (uint32_t)kWave && part == 0);
#pragma unroll 1
  for (; longer != 0ull; longer &= longer - 1ull) {
    const int l = __builtin_ctzll(longer);
    const uint32_t to = (uint32_t)l / kLanes, e = slot_of(to).halves(1)[lane];
    const uint32_t low = __builtin_amdgcn_readlane(below, l) << kBinShift, high = __builtin_amdgcn_readlane(above, l) << kBinShift;
    const uint32_t pos = ((e >> 1) & 255u) + 256u * (loads_from(__builtin_amdgcn_readlane(head, l), (uint32_t)(kWave + lane)) & 3u);
    const bool one = e - (1u << kBinShift) < low, left = !one && e < high;
    if (one) put(to, pos, 1u << (e & 1u));
    if (__builtin_amdgcn_ballot_w64(left) != 0ull) settle(left, to, scales[worker_of(to)], pos);
  }
  // Rows without a bound: slots of words.
  const bool other = live && !bins && r != 0.f;  // (R = 0: every element codes to 0)
  const bool wide = other && (limits & 255u) == kFormWords && head <= (uint32_t)kCandCap;
  if (__builtin_amdgcn_ballot_w64(wide) != 0ull) {
    auto code = [&](uint32_t to, uint32_t e, int in, float scale) {  // whether the element needs its value
      const int one = in & entry_codes_one<kCandPosMask>(e, scale);
      if (one) put(to, e & kCandPosMask, 1u | ((e >> 30) & 2u));
      return in & ~one & ~entry_codes_zero<kCandPosMask>(e, scale);
    };
    uint32_t undecided = 0u;
#pragma unroll
    for (int c = 0; c < X; ++c) undecided |= (uint32_t)code(row, x[c], (int)wide & (int)(X * part + c - 1u < head), r) << c;
    while (__builtin_amdgcn_ballot_w64(undecided != 0u) != 0ull) {
      const uint32_t c = (uint32_t)__builtin_ctz(undecided | 8u);
      uint32_t e = x[0];
#pragma unroll
      for (int i = 1; i < X; ++i) e = c == (uint32_t)i ? x[i] : e;
      settle(undecided != 0u, row, r, e & kCandPosMask);
      undecided &= undecided - 1u;
    }
    uint64_t more = __builtin_amdgcn_ballot_w64(wide && head >= kSlotLine && part == 0);
#pragma unroll 1
    for (; more != 0ull; more &= more - 1ull) {
      const int l = __builtin_ctzll(more);
      const uint32_t to = (uint32_t)l / kLanes, n = __builtin_amdgcn_readlane(head, l);
      const float scale = scales[worker_of(to)];
#pragma unroll 1
      for (uint32_t i0 = kSlotLine; i0 <= n; i0 += kWave) {
        const uint32_t i = min(i0 + (uint32_t)lane, (uint32_t)kSlotEntries - 1), e = slot_of(to).rest[i - kSlotLine];
        const int left = code(to, e, i0 + (uint32_t)lane <= n, scale);
        if (__builtin_amdgcn_ballot_w64(left != 0) != 0ull) settle(left != 0, to, scale, e & kCandPosMask);
      }
    }
  }
  // Rows too dense for slots, and slots that overflowed: the ordinary way.
  uint64_t none = __builtin_amdgcn_ballot_w64(other && !wide && part == 0);
#pragma unroll 1
  for (; none != 0ull; none &= none - 1ull) {
    const uint32_t to = (uint32_t)__builtin_ctzll(none) / kLanes;
    code_tile<NORM>(lds.b8[to][wave], g, ref4, ref24, tile_of(to), worker_of(to), lane, scales[worker_of(to)], eps, iter, k0, k1);
  }
  wave_lds_fence();
  constexpr int kStore = WPW / 4;  // lanes that store a row, 16 bytes each
#pragma unroll
  for (int k = 0; k < ROWS; k += kWave / kStore) {
    const uint32_t from = (uint32_t)(k + lane / kStore);
    if (!is_live(from)) continue;
    v4u_t w4 = *reinterpret_cast<const v4u_t*>(&lds.b32[from][wave][4 * (lane % kStore)]);
    w4 |= (w4 >> 1) & 0x55555555u;  // (leaves whole codes as they are)
    store4_through(codes + (uint64_t)worker_of(from) * words + tile_of(from) * WPW + 4 * (lane % kStore), w4);
  }
}

// ------------------------------------------------------------------------------------------
// Server: decode, average over workers in worker order, de-normalise (Eq. 1 / Eq. 2), and
// optionally w <- w - lr * v and reference <- v in the same pass.
// ------------------------------------------------------------------------------------------
// A workgroup owns a tile of kDecodeLoads * 256 float4 (4096 coordinates).  Per worker the tile's
// packed codes are 256 (ternary) or 512 (4-bit) consecutive words: each thread fetches one or two
// of them with coalesced streaming loads, kDecodeWorkers workers at a time, and the words are
// re-read from LDS as the 8- or 16-bit fragment belonging to each of the thread's float4 slots.
// A code is turned into its value by a per-worker table in LDS (2^BITS entries), which also maps
// the unused "sign with level 0" pattern to +0; two bits of long rows under finite scales are signed units times the scale
// (kUnits below).
constexpr int kDecodeLoads = 4;
constexpr int kDecodeWorkers = 8;

template <int NORM, int BITS, int V, bool STREAM_CODES>
__global__ __launch_bounds__(kBlock) void decode_vec_kernel(
    const uint32_t* __restrict__ codes, const float* __restrict__ scales, const float4* ref4,
    const float4* __restrict__ ref24, float4* __restrict__ vbar4, float4* w4, float* refout,
    uint64_t d, uint64_t words, uint32_t M, float eps, float inv_m, float lr, const float* __restrict__ means) {
  constexpr int MCH = kDecodeWorkers;
  constexpr int FPW = 32 / (4 * BITS);     // 4-code fragments per packed word: 4 (ternary) or 2
  constexpr int WPT = (V + FPW - 1) / FPW; // packed words per thread and worker (some threads idle when V < FPW)
  constexpr int WORDS = kBlock * V / FPW;  // packed words per tile and worker
  constexpr int TAB = 1 << BITS;           // table entries per worker
  constexpr uint32_t MASK = (1u << BITS) - 1u;
  constexpr float S = (float)((1 << (BITS - 1)) - 1);
  // Two bits are -1, 0 or 1 as a signed number, times R exactly: one rounding with the addition, as by the table, which is left
  // to scales that are not finite (0 times R is then no number) and to means.  Three vector instructions an element and worker instead of
  // four and a read of LDS, which shows where many workers make the pass one of arithmetic: table / units, us, each in two processes (whose times
  // differ by up to 2 us with one and the same kernel, so each is compared with its like): d = 2^23, M = 64 57.3 and 58.4 / 52.0 and
  // 53.2; d = 2^24, M = 33 58.3 and 59.7 / 54.6 and 56.2, M = 16 36.7 and 38.1 / 35.7 and 37.7; d = 2^25 + 3, M = 5 51.9 and 53.1 / 51.4 and
  // 52.8; d = 2^27, M = 8 189.8 and 191.9 / 189.0 and 189.9.
  constexpr bool kUnits = BITS == 2 && V > 1 && NORM != kNormMean;
  __shared__ union {
    lds_u32 b32[MCH][WORDS];
    lds_u8 b8[MCH][WORDS * 4];
    lds_u16 b16[MCH][WORDS * 2];
  } buf;
  __shared__ float table[MCH * TAB];
  const uint64_t vec_base = (uint64_t)blockIdx.x * (kBlock * V);
  const uint64_t word_base = (uint64_t)blockIdx.x * WORDS;
  float4 acc[V];
#pragma unroll
  for (int v = 0; v < V; ++v) acc[v] = make_float4(0.f, 0.f, 0.f, 0.f);

  // whether all scales are finite: asked for ahead of the words, the same for the whole grid
  uint32_t largest = 0u;
  bool units = false;
  for (uint32_t m = threadIdx.x % kWave; kUnits && m < M; m += kWave) largest = max(largest, __float_as_uint(scales[m]) & 0x7FFFFFFFu);
  for (uint32_t m_base = 0; m_base < M; m_base += MCH) {
    const uint32_t cnt = min((uint32_t)MCH, M - m_base);
    uint32_t wreg[MCH][WPT];
#pragma unroll
    for (int mm = 0; mm < MCH; ++mm) {
#pragma unroll
      for (int k = 0; k < WPT; ++k) {
        const uint32_t wl = k * kBlock + threadIdx.x;   // word within the tile
        const uint64_t wi = word_base + wl;
        wreg[mm][k] = 0u;
        if ((uint32_t)mm < cnt && wl < (uint32_t)WORDS && wi < words)
          wreg[mm][k] = STREAM_CODES ? __builtin_nontemporal_load(codes + (uint64_t)(m_base + mm) * words + wi)
                                     : codes[(uint64_t)(m_base + mm) * words + wi];
      }
    }
    __syncthreads();  // the previous trip's LDS reads are done
#pragma unroll
    for (int mm = 0; mm < MCH; ++mm) {
#pragma unroll
      for (int k = 0; k < WPT; ++k)
        if (k * kBlock + threadIdx.x < (uint32_t)WORDS) {
          const uint32_t level = wreg[mm][k] & 0x55555555u;  // (kUnits: a sign without a level is cleared)
          buf.b32[mm][k * kBlock + threadIdx.x] = kUnits ? wreg[mm][k] & (level | (level << 1)) : wreg[mm][k];
        }
    }
    if (m_base == 0 && kUnits) units = __builtin_amdgcn_ballot_w64(largest >= 0x7F800000u) == 0ull;
    if (units) {
      if (threadIdx.x < cnt) table[threadIdx.x] = scales[m_base + threadIdx.x];
    } else if (threadIdx.x < cnt * TAB) {
      const uint32_t mm = threadIdx.x / TAB, code = threadIdx.x % TAB;
      const float R = scales[m_base + mm];
      const float val = decode_code<BITS>(code, R, R / S);
      table[threadIdx.x] = NORM == kNormMean ? means[m_base + mm] + val : val;  // the worker's mean is added back
    }
    __syncthreads();
    if (units) {
      for (uint32_t mm = 0; mm < cnt; ++mm) {
        const float R = table[mm];
        auto unit = [](uint32_t f, int c) { return (float)((int32_t)(f << (30 - 2 * c)) >> 30); };
#pragma unroll
        for (int v = 0; v < V; ++v) {
          const uint32_t f = (uint32_t)buf.b8[mm][v * kBlock + threadIdx.x];
          acc[v].x = __builtin_fmaf(R, unit(f, 0), acc[v].x);
          acc[v].y = __builtin_fmaf(R, unit(f, 1), acc[v].y);
          acc[v].z = __builtin_fmaf(R, unit(f, 2), acc[v].z);
          acc[v].w = __builtin_fmaf(R, unit(f, 3), acc[v].w);
        }
      }
      continue;
    }
    for (uint32_t mm = 0; mm < cnt; ++mm) {
      const float* tab = table + mm * TAB;
#pragma unroll
      for (int v = 0; v < V; ++v) {
        const uint32_t f = BITS == 2 ? (uint32_t)buf.b8[mm][v * kBlock + threadIdx.x]
                                     : (uint32_t)buf.b16[mm][v * kBlock + threadIdx.x];
        acc[v].x = acc[v].x + tab[f & MASK];
        acc[v].y = acc[v].y + tab[(f >> BITS) & MASK];
        acc[v].z = acc[v].z + tab[(f >> (2 * BITS)) & MASK];
        acc[v].w = acc[v].w + tab[(f >> (3 * BITS)) & MASK];
      }
    }
  }

#pragma unroll
  for (int v = 0; v < V; ++v) {
    const uint64_t i = vec_base + (uint64_t)v * kBlock + threadIdx.x;
    if (4 * i < d) {
      const bool whole = 4 * i + 4 <= d;  // all but the last float4 of a row whose length is no multiple of 4
      RefTile<NORM> rt;
      if (whole)
        rt.load(ref4, ref24, i, eps);
      else
        rt.load_ragged(ref4, ref24, i, d, eps);
      float4 o;
      o.x = denormalize<NORM>(acc[v].x * inv_m, rt.r1.x, rt.r2.x);
      o.y = denormalize<NORM>(acc[v].y * inv_m, rt.r1.y, rt.r2.y);
      o.z = denormalize<NORM>(acc[v].z * inv_m, rt.r1.z, rt.r2.z);
      o.w = denormalize<NORM>(acc[v].w * inv_m, rt.r1.w, rt.r2.w);
      if (whole)
        store_stream(vbar4 + i, o);
      else
        store4_within(reinterpret_cast<float*>(vbar4), 4 * i, d, o);
      if (w4 != nullptr) {
        float4 w = whole ? load_stream(w4 + i) : load4_within(reinterpret_cast<const float*>(w4), 4 * i, d, 0.f);
        const float px = lr * o.x, py = lr * o.y, pz = lr * o.z, pw = lr * o.w;
        w.x = w.x - px;
        w.y = w.y - py;
        w.z = w.z - pz;
        w.w = w.w - pw;
        store4_within(reinterpret_cast<float*>(w4), 4 * i, d, w);
      }
      if (refout != nullptr) store4_within(refout, 4 * i, d, o);  // (a slot of the history ring starts at any 4-byte boundary)
    }
  }
}

// ------------------------------------------------------------------------------------------
// Workers and server in one launch (tng_step): quantise and pack every worker's part of a tile and, with the codes
// still at hand, decode, average, de-normalise and update.
//
// What bounds an iteration of a small problem is the number of its launches (2.5 to 4 us each, whatever they
// do); what a larger one saves is the second trip of the codes and the references through memory.  A thread
// owns one float4 of coordinates and walks the workers, kTailWorkers rows of loads in flight.  (Requesting the row
// eight workers further as soon as one is used measured no faster: 465 against 444 us at d = 2^24, M = 16.)
// Iterations with given gradients, the separate launches against this one: d = 10007, M = 8, 4-bit 26.4 -> 8.9 us;
// d = 2^18, M = 8 16.6 -> 9.6; d = 2^20, M = 8 24.4 -> 24.5; d = 4e6, M = 8 82.6 -> 70.8; d = 2^24, M = 64, 4-bit
// 1792 -> 1673.
// The scales come from the partial maxima of the scale pass (partials[rows][M], reduced by every workgroup for
// itself: rows * M floats out of the L2) or, rows == 0, from scales.  32 KiB of them cost a workgroup less than the
// launch that would reduce them once (about 4 us) up to 1024 workgroups of the kernel below; beyond those 8 KiB do
// (kTailPartialsLong; the scale pass then takes fewer workgroups where it can, see absmax_vec_launch).  Iterations, own
// launch / here: Rosenbrock, d = 2^20, M = 8 26.2 / 25.2 us, M = 7 23.1 / 22.8; given gradients, d = 2^20, M = 8 22.6 / 20.8, M =
// 16, 4-bit 34.5 / 33.2; d = 2^18, M = 64 29.6 / 28.5; d = 4e6, M = 8 with 8 KiB 70.0 / 65.0.
// What a wavefront waits for comes in the order in which it asked: first what makes the scales, then the reference, then the
// workers' rows, each of which is coded while the ones behind it are on their way.  (The scales behind the rows, and whole and
// ragged wavefronts in one body: every wavefront waited for all of its rows first.  This kernel, before / after: d = 2^22, M = 8,
// quotient 48.0 / 45.0 us; d = 2e6, M = 8, 4-bit 24.6 / 23.6; d = 8e6, M = 4, 4-bit 57 / 55; d = 4e6, M = 8 38.9 / 38.1.)  So too where
// the maxima are many, up to d = 2^20, eight float4 a thread (iterations, behind the rows / ahead of them: Rosenbrock chain, d = 2^20,
// M = 8 25.6 / 25.1 us, 4-bit, quotient 31.9 / 30.0; given gradients, d = 2^20, M = 16, quotient 38.5 / 37.0, combined form 42.6 / 41.1;
// d = 528384, M = 16 23.0 / 22.4), but not where they are few or would be read one by one (M no power of two: Rosenbrock, d = 2^20, M =
// 7 22.9 / 23.3).
// ------------------------------------------------------------------------------------------
constexpr int kTailWorkers = 8;
constexpr uint32_t kTailMaxWorkers = 64;
constexpr uint32_t kTailPartials = 8192, kTailPartialsLong = 2048;
constexpr uint32_t kTailFewPartials = 1024;  // up to here single loads: at a few hundred the exchange between lanes costs 0.5 us

// What the coder needs of a worker: its scale R, 1 / R and R / S, and its mean.  Of R = 0 all are 0, under which every number
// codes to level 0.  Made once per workgroup: the two divisions by every lane for every worker were a seventh of the kernel's
// instructions.  With that and the part of a draw that is the same for all workers made once (philox_block), the Rosenbrock
// iteration at d = 2^20, M = 8 went from 28.6 to 27.9 us, given gradients of d = 4e6, M = 8, quotient from 74.2 to 71.1.
struct __align__(16) TailWorker {
  float r, inv_r, step, mu;
};

// What a thread contributes to the workers' records, requested ahead of the rows of the gradients: loads return in order, so
// behind them the first worker's arithmetic would wait for the last worker's row.
constexpr int kTailLate = -1;
template <int EARLY>
struct TailOperands {
  float r, mu;  // scale and mean of worker threadIdx.x (rows == 0 or the mean reference)
  float4 top[EARLY > 0 ? EARLY : 1];  // EARLY: the thread's partial maxima, of the same four workers each
};
// EARLY: float4 a thread, where M is a power of two and kTailFewPartials < rows * M <= EARLY * 4 * kBlock, whole float4; 0: the
// scales are there; kTailLate: nothing is asked for ahead of the rows.
template <int NORM, int EARLY>
__device__ __forceinline__ void tail_request(TailOperands<EARLY>& t, const float* scales, const float* partials, uint32_t rows,
                                             uint32_t M, const float* __restrict__ means) {
  const uint32_t m = min(threadIdx.x, M - 1);
  t.r = EARLY > 0 ? 0.f : scales[m];
  t.mu = NORM == kNormMean ? means[m] : 0.f;
  static_assert(kTailFewPartials >= 4 * kBlock, "every thread has a float4");
  const uint32_t last = (rows * M / 4 - 1 - threadIdx.x) / kBlock;
  const float4* p = reinterpret_cast<const float4*>(partials) + threadIdx.x;
#pragma unroll
  for (int k = 0; k < EARLY; ++k) t.top[k] = p[min((uint32_t)k, last) * kBlock];  // past the end the last one again
}

// The M <= kTailMaxWorkers workers' records; the first workgroup publishes the scales.
template <int NORM, int BITS, int EARLY>
__device__ __forceinline__ void tail_workers(TailWorker* sWorker, uint32_t* top, float* scales, const float* partials, uint32_t rows,
                                             uint32_t M, const TailOperands<EARLY>& mine) {
  // top: as bits, non-negative floats are ordered as integers
  auto meet_here = [] {
    if (EARLY == kTailLate)
      __syncthreads();
    else
      lds_barrier();
  };
  const bool from_partials = EARLY > 0 || (EARLY < 0 && rows != 0);
  if (from_partials) {
    if (threadIdx.x < M) top[threadIdx.x] = 0u;
    meet_here();
    const uint32_t n = rows * M;
    const uint32_t apart = max(M / 4, 4u);  // lanes that far apart hold the same workers: few are left to meet in LDS
    auto meet = [&](float4 v) {
      for (uint32_t off = kWave / 2; off >= apart; off /= 2) {
        v.x = fmaxf(v.x, __shfl_xor(v.x, (int)off));
        v.y = fmaxf(v.y, __shfl_xor(v.y, (int)off));
        v.z = fmaxf(v.z, __shfl_xor(v.z, (int)off));
        v.w = fmaxf(v.w, __shfl_xor(v.w, (int)off));
      }
      if (threadIdx.x % kWave < apart) {
        const float vv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (uint32_t c = 0; c < 4; ++c)
          atomicMax(&top[(4 * threadIdx.x + c) % M], __float_as_uint(vv[c] < FLT_MIN ? 0.f : vv[c]));
      }
    };
    if (EARLY > 0) {
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < EARLY; ++k)
        v = make_float4(fmaxf(v.x, mine.top[k].x), fmaxf(v.y, mine.top[k].y), fmaxf(v.z, mine.top[k].z), fmaxf(v.w, mine.top[k].w));
      meet(v);
    } else if (n > kTailFewPartials && (M & (M - 1)) == 0 && n % 4 == 0) {  // all of a thread's float4 belong to the same four workers
      static_assert(kTailFewPartials >= 4 * kBlock, "every thread has a float4");
      const uint32_t n4 = n / 4, last = (n4 - 1 - threadIdx.x) / kBlock;
      const float4* p = reinterpret_cast<const float4*>(partials) + threadIdx.x;
      float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
      for (uint32_t k0 = 0; k0 * kBlock < n4; k0 += 4) {  // (eight at a time: a wavefront less per SIMD, by registers)
        float4 x[4];
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k) x[k] = p[min(k0 + k, last) * kBlock];  // past the end the last one again
#pragma unroll
        for (uint32_t k = 0; k < 4; ++k)
          v = make_float4(fmaxf(v.x, x[k].x), fmaxf(v.y, x[k].y), fmaxf(v.z, x[k].z), fmaxf(v.w, x[k].w));
      }
      meet(v);
    } else {
      const uint32_t used = kBlock / M * M;  // a thread stays with one worker
      if (threadIdx.x < min(used, n)) {
        float v = 0.f;
        const uint32_t last = (n - 1 - threadIdx.x) / used;
        const float* p = partials + threadIdx.x;
        for (uint32_t k0 = 0; k0 <= last; k0 += 8) {
          float x[8];
#pragma unroll
          for (uint32_t k = 0; k < 8; ++k) x[k] = p[min(k0 + k, last) * used];
#pragma unroll
          for (uint32_t k = 0; k < 8; ++k) v = fmaxf(v, x[k]);
        }
        atomicMax(&top[threadIdx.x % M], __float_as_uint(v < FLT_MIN ? 0.f : v));
      }
    }
    meet_here();
  }
  if (threadIdx.x < M) {
    const float r = from_partials ? __uint_as_float(top[threadIdx.x]) : mine.r;
    constexpr float S = (float)((1 << (BITS - 1)) - 1);
    sWorker[threadIdx.x] = TailWorker{r, r != 0.f ? 1.0f / r : 0.f, r / S, mine.mu};
    if (from_partials && blockIdx.x == 0) scales[threadIdx.x] = r;
  }
  meet_here();
}

template <int NORM, int BITS>
struct TailLds {
  FragmentBuffer<kWave * 4 * BITS / 32, kTailWorkers> fragments;
  TailWorker worker[kTailMaxWorkers];
  uint32_t top[kTailMaxWorkers];
};

// MIXED: some of the workgroup's coordinates may lie past the end of the row.  (Where whole and ragged wavefronts share one
// body, the compiler cannot count the loads in flight where their paths join, and waits for all of them before the first
// worker's arithmetic.)
template <int NORM, int BITS, bool MIXED, int EARLY>
__device__ __forceinline__ void quantize_decode_body(
    TailLds<NORM, BITS>& lds, const GradRows& g, const float4* ref4, const float4* __restrict__ ref24, float* __restrict__ scales,
    uint32_t* __restrict__ codes, uint64_t d, uint64_t words, uint32_t M, float eps, uint32_t k0, uint32_t k1, uint32_t iter,
    const float* __restrict__ means, const float* __restrict__ partials, uint32_t rows, float4* vbar4, float4* w4, float* refout, float inv_m, float lr) {
  constexpr int MC = kTailWorkers;
  constexpr int WPW = kWave * 4 * BITS / 32;  // packed words per wavefront and worker
  constexpr bool RECIP = NORM == kNormQuot || NORM == kNormComb;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const uint64_t q = (uint64_t)blockIdx.x * kBlock + threadIdx.x;  // the thread's float4
  const uint64_t wave_tile = (uint64_t)blockIdx.x * kWavesPerBlock + wave;

  const bool whole = !MIXED || (wave_tile + 1) * (kWave * 4) <= d;  // the wavefront's 256 coordinates lie inside the row

  float4 x[MC];
  auto load_rows = [&](uint32_t m0) {  // rows past M repeat the last one: no load under a condition
    if (whole) {
#pragma unroll
      for (int mm = 0; mm < MC; ++mm) x[mm] = load_row_stream(g.row(min(m0 + (uint32_t)mm, M - 1)) + q);
    } else {
#pragma unroll
      for (int mm = 0; mm < MC; ++mm) {
        const uint32_t m = min(m0 + (uint32_t)mm, M - 1);
        x[mm] = load_row_ragged(g, m, q, d, NORM == kNormMean ? means[m] : 0.f);
      }
    }
  };
  TailOperands<EARLY> mine{};
  RefTile<NORM> rt;
  if (EARLY != kTailLate)
    tail_request<NORM, EARLY>(mine, scales, partials, rows, M, means);
  else
    load_rows(0);
  if (whole)
    rt.load(ref4, ref24, q, eps);
  else
    rt.load_ragged(ref4, ref24, q, d, eps);
  if (EARLY != kTailLate) load_rows(0);
  float4 w = whole ? load_stream(w4 + q) : load4_within(reinterpret_cast<const float*>(w4), 4 * q, d, 0.f);
  if (EARLY == kTailLate && (rows == 0 || NORM == kNormMean)) tail_request<NORM, EARLY>(mine, scales, partials, rows, M, means);

  tail_workers<NORM, BITS, EARLY>(lds.worker, lds.top, scales, partials, rows, M, mine);
  rt.reciprocals();
  const PhiloxBlock block = philox_block((uint32_t)q, iter, k0, k1);

  float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
  for (uint32_t m0 = 0;;) {  // (the rows are the last loads both here and at the end of a trip: counted alike)
    const uint32_t count = min((uint32_t)MC, M - m0);
#pragma unroll
    for (int mm = 0; mm < MC; ++mm) {
      if ((uint32_t)mm < count) {
        const uint32_t m = m0 + (uint32_t)mm;
        const TailWorker wk = lds.worker[m];
        const float4 v = normalize4<NORM, RECIP>(x[mm], rt, wk.mu);
        float4 val;  // what the server decodes
        uint32_t frag = quantize4_and_values<BITS>(v, wk.inv_r, philox_draw(block, m, iter, k0, k1), wk.r, wk.step, val);
        if (BITS == 4 && wk.r == 0.f) frag = 0u;  // (a row without a number in it)
        if (BITS == 2)
          lds.fragments.b8[mm][wave][lane] = (uint8_t)frag;
        else
          lds.fragments.b16[mm][wave][lane] = (uint16_t)frag;
        if (NORM == kNormMean) val = make_float4(wk.mu + val.x, wk.mu + val.y, wk.mu + val.z, wk.mu + val.w);
        acc.x = acc.x + val.x;  // in worker order
        acc.y = acc.y + val.y;
        acc.z = acc.z + val.z;
        acc.w = acc.w + val.w;
      }
    }
    wave_lds_fence();
    for (uint32_t i = (uint32_t)lane; i < count * WPW; i += kWave) {
      const uint32_t mm = i / WPW, j = i % WPW;
      const uint64_t wi = wave_tile * WPW + j;
      if (wi < words) store_word_through(codes + (uint64_t)(m0 + mm) * words + wi, lds.fragments.b32[mm][wave][j]);
    }
    wave_lds_fence();
    m0 += MC;
    if (m0 >= M) break;
    load_rows(m0);
  }

  float4 o;
  o.x = denormalize<NORM>(acc.x * inv_m, rt.r1.x, rt.r2.x);
  o.y = denormalize<NORM>(acc.y * inv_m, rt.r1.y, rt.r2.y);
  o.z = denormalize<NORM>(acc.z * inv_m, rt.r1.z, rt.r2.z);
  o.w = denormalize<NORM>(acc.w * inv_m, rt.r1.w, rt.r2.w);
  const float px = lr * o.x, py = lr * o.y, pz = lr * o.z, pw = lr * o.w;
  w.x = w.x - px;
  w.y = w.y - py;
  w.z = w.z - pz;
  w.w = w.w - pw;
  if (whole) {
    store_stream(vbar4 + q, o);
    w4[q] = w;
  } else {
    store4_within(reinterpret_cast<float*>(vbar4), 4 * q, d, o);
    store4_within(reinterpret_cast<float*>(w4), 4 * q, d, w);
  }
  if (refout != nullptr) store4_within(refout, 4 * q, d, o);  // (a slot of the history ring starts at any 4-byte boundary)
}

template <int NORM, int BITS, int EARLY>
__global__ __launch_bounds__(kBlock, NORM == kNormQuot || NORM == kNormComb || EARLY > 2 ? 4 : 5) void quantize_decode_kernel(
    GradRows g, const float4* ref4, const float4* __restrict__ ref24, float* __restrict__ scales,
    uint32_t* __restrict__ codes, uint64_t d, uint64_t words, uint32_t M, float eps, uint32_t k0, uint32_t k1,
    uint32_t iter, const float* __restrict__ means, const float* __restrict__ partials, uint32_t rows,
    float4* __restrict__ vbar4, float4* w4, float* refout, float inv_m, float lr) {
  __shared__ __attribute__((aligned(16))) TailLds<NORM, BITS> lds;
#define TNG_BODY(MIXED, REQUESTED)                                                                                            \
  quantize_decode_body<NORM, BITS, MIXED, REQUESTED>(lds, g, ref4, ref24, scales, codes, d, words, M, eps, k0, k1, iter, means, \
                                                  partials, rows, vbar4, w4, refout, inv_m, lr)
  if (EARLY != kTailLate && (uint64_t)blockIdx.x * (4 * kBlock) + 4 * kBlock <= d)
    TNG_BODY(false, EARLY);
  else
    TNG_BODY(true, kTailLate);
#undef TNG_BODY
}

// The same where the coordinates alone leave the chip idle: a workgroup takes 256 coordinates, its wavefronts a
// worker each in turn (a wavefront of the kernel above walks all M workers, 0.6 us each), and once the codes of
// all workers are in LDS every thread decodes one coordinate, in worker order, by a table of the values.
template <int NORM, int BITS>
__global__ __launch_bounds__(kBlock) void quantize_decode_split_kernel(
    GradRows g, const float* ref, const float* __restrict__ ref2, float* __restrict__ scales,
    uint32_t* __restrict__ codes, uint64_t d, uint64_t words, uint32_t M, float eps, uint32_t k0, uint32_t k1,
    uint32_t iter, const float* __restrict__ means, const float* __restrict__ partials, uint32_t rows,
    float* __restrict__ vbar, float* w, float* refout, float inv_m, float lr) {
  constexpr int MC = 4;                       // rows of loads in flight per wavefront
  constexpr int WPW = kWave * 4 * BITS / 32;  // packed words per workgroup and worker
  constexpr int TAB = 1 << BITS;
  constexpr uint32_t MASK = (1u << BITS) - 1u;
  __shared__ union {
    lds_u8 b8[kTailMaxWorkers][kWave];
    lds_u16 b16[kTailMaxWorkers][kWave];
    lds_u32 b32[kTailMaxWorkers][WPW];
  } buf;
  __shared__ TailWorker sWorker[kTailMaxWorkers];
  __shared__ uint32_t top[kTailMaxWorkers];
  __shared__ float table[kTailMaxWorkers * TAB];
  // (the wavefront's number as a value that is the same in every lane: its workers' parts of the draws are then scalar)
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = threadIdx.x % kWave;
  const uint64_t q = (uint64_t)blockIdx.x * kWave + lane;  // the lane's float4
  const uint64_t e = (uint64_t)blockIdx.x * kBlock + threadIdx.x;  // the coordinate that the thread decodes
  const bool whole = ((uint64_t)blockIdx.x + 1) * kBlock <= d;

  float4 x[MC];
  auto load_rows = [&](uint32_t i0) {  // the wavefront's workers number i0 .. i0 + MC - 1
#pragma unroll
    for (int i = 0; i < MC; ++i) {
      const uint32_t m = min((i0 + i) * kWavesPerBlock + (uint32_t)wave, M - 1);
      x[i] = whole ? load_row_stream(g.row(m) + q) : load_row_ragged(g, m, q, d, NORM == kNormMean ? means[m] : 0.f);
    }
  };
  load_rows(0);
  RefTile<NORM> rt;
  if (whole)
    rt.load(reinterpret_cast<const float4*>(ref), reinterpret_cast<const float4*>(ref2), q, eps);
  else
    rt.load_ragged(reinterpret_cast<const float4*>(ref), reinterpret_cast<const float4*>(ref2), q, d, eps);
  const uint64_t ec = min(e, d - 1);
  float r1, r2;
  load_ref_scalar<NORM>(ref, ref2, ec, eps, r1, r2);
  const float w0 = w[ec];
  TailOperands<kTailLate> mine{};
  if (rows == 0 || NORM == kNormMean) tail_request<NORM, kTailLate>(mine, scales, partials, rows, M, means);
  tail_workers<NORM, BITS, kTailLate>(sWorker, top, scales, partials, rows, M, mine);
  for (uint32_t i = threadIdx.x; i < M * TAB; i += kBlock) {
    const TailWorker wk = sWorker[i / TAB];
    const float val = decode_code<BITS>(i % TAB, wk.r, wk.step);
    table[i] = NORM == kNormMean ? wk.mu + val : val;
  }
  const PhiloxBlock block = philox_block((uint32_t)q, iter, k0, k1);

  for (uint32_t i0 = 0; i0 * kWavesPerBlock < M; i0 += MC) {
    if (i0 != 0) load_rows(i0);
#pragma unroll
    for (int i = 0; i < MC; ++i) {
      const uint32_t m = (i0 + i) * kWavesPerBlock + (uint32_t)wave;
      if (m < M) {
        const TailWorker wk = sWorker[m];
        const float4 v = normalize4<NORM, false>(x[i], rt, wk.mu);
        uint32_t frag = quantize4<BITS>(v, wk.inv_r, philox_draw(block, m, iter, k0, k1));
        if (BITS == 4 && wk.r == 0.f) frag = 0u;  // (a row without a number in it)
        if (BITS == 2)
          buf.b8[m][lane] = (uint8_t)frag;
        else
          buf.b16[m][lane] = (uint16_t)frag;
      }
    }
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < M * WPW; i += kBlock) {
    const uint32_t m = i / WPW, j = i % WPW;
    const uint64_t wi = (uint64_t)blockIdx.x * WPW + j;
    if (wi < words) store_word_through(codes + (uint64_t)m * words + wi, buf.b32[m][j]);
  }
  float acc = 0.f;
#pragma unroll 8
  for (uint32_t m = 0; m < M; ++m) {
    const uint32_t f = BITS == 2 ? (uint32_t)buf.b8[m][threadIdx.x >> 2] : (uint32_t)buf.b16[m][threadIdx.x >> 2];
    acc = acc + table[m * TAB + ((f >> (BITS * (threadIdx.x & 3u))) & MASK)];
  }
  if (e < d) {
    const float o = denormalize<NORM>(acc * inv_m, r1, r2);
    const float p = lr * o;
    vbar[e] = o;
    w[e] = w0 - p;
    if (refout != nullptr) refout[e] = o;
  }
}

// ------------------------------------------------------------------------------------------
// One workgroup for tiny problems (d <= 4 * kBlock): scale, quantise and pack, and the server side as
// well, in one launch.
//
// A thread owns one float4 of coordinates of every worker (M <= MC rows in registers), so once the
// M scales are known -- a workgroup reduction -- it can code its values, and since it then holds all
// M codes of its coordinates it can decode, average, de-normalise and update them without reading
// anything back.  Such problems are bound by the latency of their launches (about 4 us each), not
// by bytes.
// The same kernel over several workgroups, with the maxima exchanged through device-scope atomics
// and a meeting point (bounded wait, grid checked against the occupancy), was measured too: it wins
// up to 16 workgroups (16.6 -> 15.5 us per iteration at d = 2^14, M = 8) and loses beyond (d = 2^20,
// M = 8: 32 -> 56 us): with eight compute dies, each with its own L2, every arrival and every flag
// is an access to memory-side atomics, about 25 us for a full meeting of 128 or more workgroups.
// ------------------------------------------------------------------------------------------
constexpr int kSinglePassMaxWorkers = 16;

template <int NORM, int BITS, int MC>
__global__ __launch_bounds__(kBlock) void single_pass_kernel(
    GradRows g, const float4* ref4, const float4* __restrict__ ref24, float* __restrict__ scales,
    uint32_t* __restrict__ codes, uint64_t nvec, uint64_t words, uint32_t M, float eps, uint32_t k0, uint32_t k1,
    uint32_t iter, float4* __restrict__ vbar4, float4* w4, float4* refout4, float inv_m, float lr) {
  constexpr int WPB = kBlock * 4 * BITS / 32;  // packed words per workgroup and worker
  constexpr uint32_t MASK = (1u << BITS) - 1u;
  constexpr float S = (float)((1 << (BITS - 1)) - 1);
  __shared__ float red[MC][kWavesPerBlock];
  __shared__ float sScale[MC];
  __shared__ union {
    lds_u8 b8[MC][WPB * 4];
    lds_u16 b16[MC][WPB * 2];
    lds_u32 b32[MC][WPB];
  } buf;
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const uint64_t q = threadIdx.x;  // one workgroup
  const bool active = q < nvec;

  RefTile<NORM> rt;
  rt.r1 = rt.r2 = make_float4(0.f, 0.f, 0.f, 0.f);
  float4 x[MC];
  float amax[MC];
  if (active) {
    rt.template load<false>(ref4, ref24, q, eps);
#pragma unroll
    for (int mm = 0; mm < MC; ++mm)  // rows past M repeat the last one: all loads in flight, none under a condition
      x[mm] = load_row_stream(g.row(min((uint32_t)mm, M - 1)) + q);
  }
#pragma unroll
  for (int mm = 0; mm < MC; ++mm) {
    amax[mm] = 0.f;
    if (active) {
      const float a0 = fabsf(normalize<NORM>(x[mm].x, rt.r1.x, rt.r2.x));
      const float a1 = fabsf(normalize<NORM>(x[mm].y, rt.r1.y, rt.r2.y));
      const float a2 = fabsf(normalize<NORM>(x[mm].z, rt.r1.z, rt.r2.z));
      const float a3 = fabsf(normalize<NORM>(x[mm].w, rt.r1.w, rt.r2.w));
      amax[mm] = fmaxf(fmaxf(a0, a1), fmaxf(a2, a3));
    }
    const float v = wave_max(amax[mm]);
    if (lane == 0) red[mm][wave] = v;
  }
  __syncthreads();
  if (threadIdx.x < M) {
    float v = red[threadIdx.x][0];
#pragma unroll
    for (int k = 1; k < kWavesPerBlock; ++k) v = fmaxf(v, red[threadIdx.x][k]);
    v = v < FLT_MIN ? 0.f : v;
    sScale[threadIdx.x] = v;
    scales[threadIdx.x] = v;
  }
  __syncthreads();

  uint32_t frag[MC];
#pragma unroll
  for (int mm = 0; mm < MC; ++mm) {
    frag[mm] = 0u;
    if ((uint32_t)mm < M) {
      const float R = sScale[mm];
      if (active && R != 0.f) {
        const float inv_r = 1.0f / R;
        const U32x4 rnd = philox4x32_10((uint32_t)q, (uint32_t)mm, iter, 0u, k0, k1);
        frag[mm] = quantize4<BITS>(normalize4<NORM, false>(x[mm], rt, 0.f), inv_r, rnd);
      }
      if (BITS == 2) {
        buf.b8[mm][threadIdx.x] = (uint8_t)frag[mm];
      } else {
        buf.b16[mm][threadIdx.x] = (uint16_t)frag[mm];
      }
    }
  }
  __syncthreads();
  for (uint32_t t = threadIdx.x; t < M * (uint32_t)WPB; t += kBlock) {
    const uint32_t mm = t / WPB, j = t % WPB;
    const uint64_t wi = j;
    if (wi < words) store_word_through(codes + (uint64_t)mm * words + wi, buf.b32[mm][j]);
  }

  if (active) {
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int mm = 0; mm < MC; ++mm) {
      if ((uint32_t)mm < M) {
        const float R = sScale[mm], step = R / S;
        const uint32_t f = frag[mm];
        acc.x = acc.x + decode_code<BITS>(f & MASK, R, step);
        acc.y = acc.y + decode_code<BITS>((f >> BITS) & MASK, R, step);
        acc.z = acc.z + decode_code<BITS>((f >> (2 * BITS)) & MASK, R, step);
        acc.w = acc.w + decode_code<BITS>((f >> (3 * BITS)) & MASK, R, step);
      }
    }
    float4 o;
    o.x = denormalize<NORM>(acc.x * inv_m, rt.r1.x, rt.r2.x);
    o.y = denormalize<NORM>(acc.y * inv_m, rt.r1.y, rt.r2.y);
    o.z = denormalize<NORM>(acc.z * inv_m, rt.r1.z, rt.r2.z);
    o.w = denormalize<NORM>(acc.w * inv_m, rt.r1.w, rt.r2.w);
    store_stream(vbar4 + q, o);
    float4 w = load_stream(w4 + q);
    const float px = lr * o.x, py = lr * o.y, pz = lr * o.z, pw = lr * o.w;
    w.x = w.x - px;
    w.y = w.y - py;
    w.z = w.z - pz;
    w.w = w.w - pw;
    w4[q] = w;
    if (refout4 != nullptr) refout4[q] = o;
  }
}

// ------------------------------------------------------------------------------------------
// Short rows: scale, quantise and pack in one launch.  A workgroup codes kRowTile elements of one worker, and takes the
// maximum of the worker's whole row by itself, out of the L2: at these lengths that is less than a launch between two passes
// costs.
// ------------------------------------------------------------------------------------------
constexpr int kRowThreads = 1024;
constexpr uint32_t kRowTile = 4 * kRowThreads;

template <int NORM, int BITS>
__global__ __launch_bounds__(kRowThreads) void encode_row_kernel(GradRows g, const float4* __restrict__ ref4,
                                                                 const float4* __restrict__ ref24,
                                                                 float* __restrict__ scales, uint32_t* __restrict__ codes,
                                                                 uint32_t d, uint32_t words, float eps, uint32_t k0,
                                                                 uint32_t k1, uint32_t iter) {
  constexpr uint32_t kWords = kRowTile * BITS / 32;  // packed words per workgroup
  constexpr int U = 4;
  __shared__ float red[kRowThreads / kWave];
  __shared__ union {
    lds_u8 b8[kRowThreads];
    lds_u16 b16[kRowThreads];
    lds_u32 b32[kWords];
  } buf;
  const uint32_t m = blockIdx.y, t = threadIdx.x;
  const uint32_t q = blockIdx.x * kRowThreads + t;  // the thread's float4
  const uint32_t whole = d / 4;
  RefTile<NORM> rt;
  float4 x;
  if (q < whole) {
    rt.template load<false>(ref4, ref24, q, eps);
    const v4f_u_t v = g.row(m)[q];
    x = make_float4(v.x, v.y, v.z, v.w);
  } else {  // at or past the end of the row
    rt.load_ragged(ref4, ref24, q, d, eps);
    x = load_row_ragged(g, m, q, d, 0.f);
  }
  float4 v = normalize4<NORM, false>(x, rt, 0.f);
  float amax = max3_abs(v.z, v.w, max3_abs(v.x, v.y, 0.f));
  if (gridDim.x > 1) {  // the other tiles' elements (and these again: no harm to a maximum)
    for (uint32_t i0 = t; i0 < whole; i0 += U * kRowThreads) {
      float4 xo[U];
      RefTile<NORM> ro[U];
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const uint32_t i = min(i0 + (uint32_t)k * kRowThreads, whole - 1);
        const v4f_u_t e = g.row(m)[i];
        xo[k] = make_float4(e.x, e.y, e.z, e.w);
        ro[k].template load<false>(ref4, ref24, i, eps);
      }
#pragma unroll
      for (int k = 0; k < U; ++k) {
        const float4 n = normalize4<NORM, false>(xo[k], ro[k], 0.f);
        amax = max3_abs(n.z, n.w, max3_abs(n.x, n.y, amax));
      }
    }
    const uint32_t e = 4 * whole + t;
    if (e < d) {
      float r1, r2;
      load_ref_scalar<NORM>(reinterpret_cast<const float*>(ref4), reinterpret_cast<const float*>(ref24), e, eps, r1, r2);
      amax = fmaxf(amax, fabsf(normalize<NORM>(g.base[(uint64_t)m * g.pitch + e], r1, r2)));
    }
  }
  amax = wave_max_nonneg(amax);
  if (t % kWave == 0) red[t / kWave] = amax;
  __syncthreads();
  amax = wave_max_nonneg(red[t % (kRowThreads / kWave)]);
  const float R = amax < FLT_MIN ? 0.f : amax;
  if (blockIdx.x == 0 && t == 0) scales[m] = R;
  const uint32_t frag = R != 0.f ? quantize4<BITS>(v, 1.0f / R, philox4x32_10(q, m, iter, 0u, k0, k1)) : 0u;
  if (BITS == 2)
    buf.b8[t] = (uint8_t)frag;
  else
    buf.b16[t] = (uint16_t)frag;
  __syncthreads();
  const uint32_t at = blockIdx.x * kWords + t;
  if (t < kWords && at < words) store_word_through(codes + (uint64_t)m * words + at, buf.b32[t]);
}

// ------------------------------------------------------------------------------------------
// Order-pinned float64 sums per worker: the mean of the per-worker mean reference (section
// "Reference Vectors", first option) and the l2 norm as the coder's scale.
// ------------------------------------------------------------------------------------------
// The sum of a row is defined with a fixed association so that its float32 rounding is reproducible:
// elements are cut into chunks of 4096; inside a chunk lane j (0..255) adds the elements 256 k + j,
// k = 0..15 in order, and the 256 lane sums are added in lane order; chunk sums are added in order
// inside groups of 256 chunks, group sums in order.  One wavefront owns a chunk: thread t holds
// lanes 4t..4t+3 (one float4 per k), so every load instruction covers 1 KiB of contiguous memory.
constexpr int kTreeChunk = 4096;
constexpr int kTreeLanes = 256;
constexpr int kTreeGroup = 256;

// MINMAX (mean pass only): the smallest and largest element of every chunk ride along.  Rounding is
// monotone, so max_e |fl(g_e - mu)| = max(|fl(min g - mu)|, |fl(max g - mu)|) exactly: the scale of
// the mean-referenced gradient needs no pass of its own.
template <int NORM, bool SQUARE, bool VEC, bool MINMAX>
__global__ __launch_bounds__(kBlock) void tree_chunk_kernel(const float* __restrict__ g, const float* __restrict__ ref,
                                                            const float* __restrict__ ref2,
                                                            const float* __restrict__ means,
                                                            double* __restrict__ chunk_sums,
                                                            float2* __restrict__ chunk_minmax, uint64_t d,
                                                            uint64_t first_chunk, uint64_t end_chunk,
                                                            uint64_t nchunks, float eps, uint32_t M,
                                                            uint32_t workers_per_block) {
  __shared__ double lanes[kWavesPerBlock][kTreeLanes];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const uint64_t chunk = first_chunk + (uint64_t)blockIdx.x * kWavesPerBlock + wave;
  if (chunk >= end_chunk) return;  // whole wavefront; no workgroup barrier below
  const uint64_t base = chunk * kTreeChunk + 4u * (uint32_t)lane;
  constexpr int K = kTreeChunk / kTreeLanes;
  // A wavefront takes its chunk of several workers in turn: the reference tile of the chunk is then
  // fetched from HBM once and found in cache by the following workers.
  const uint32_t m_first = blockIdx.y * workers_per_block;
  const uint32_t m_last = m_first + workers_per_block < M ? m_first + workers_per_block : M;
  for (uint32_t m = m_first; m < m_last; ++m) {
  const float* __restrict__ row = g + (uint64_t)m * d;
  const float mu = (SQUARE && NORM == kNormMean) ? means[m] : 0.f;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  float lo = INFINITY, hi = -INFINITY;
  // VEC: 16-byte loads (the row may start at any 4-byte boundary).  The caller keeps the last chunk of
  // rows whose length is not a multiple of 4 away from this variant.
  if (VEC) {
    const bool full = (chunk + 1) * kTreeChunk <= d;
    // loads in batches: all 16 rows of the chunk at once, or 8 rows plus their reference tiles
    constexpr bool kHasRef = SQUARE && (NORM == kNormSub || NORM == kNormQuot || NORM == kNormComb);
    constexpr int KB = kHasRef ? 8 : K;
#pragma unroll
    for (int k0 = 0; k0 < K; k0 += KB) {
      float4 x[KB];
      RefTile<NORM> rt[KB];
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const uint64_t e = base + (uint64_t)(k0 + k) * kTreeLanes;
        const bool in = full || e < d;
        x[k] = in ? load_row_stream(reinterpret_cast<const v4f_u_t*>(row + e)) : make_float4(0.f, 0.f, 0.f, 0.f);
        if (SQUARE && in)
          rt[k].template load<false>(reinterpret_cast<const float4*>(ref), reinterpret_cast<const float4*>(ref2), e / 4,
                                     eps);
      }
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const uint64_t e = base + (uint64_t)(k0 + k) * kTreeLanes;
        const bool in = full || e < d;
        float4 v = x[k];
        if (SQUARE && in) {
          v.x = normalize_w<NORM>(v.x, rt[k].r1.x, rt[k].r2.x, mu);
          v.y = normalize_w<NORM>(v.y, rt[k].r1.y, rt[k].r2.y, mu);
          v.z = normalize_w<NORM>(v.z, rt[k].r1.z, rt[k].r2.z, mu);
          v.w = normalize_w<NORM>(v.w, rt[k].r1.w, rt[k].r2.w, mu);
        }
        if (MINMAX && in) {
          lo = fminf(lo, fminf(fminf(v.x, v.y), fminf(v.z, v.w)));
          hi = fmaxf(hi, fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)));
        }
        const double t0 = (double)v.x, t1 = (double)v.y, t2 = (double)v.z, t3 = (double)v.w;
        acc[0] = acc[0] + (SQUARE ? t0 * t0 : t0);  // the square of a binary32 value is exact in binary64
        acc[1] = acc[1] + (SQUARE ? t1 * t1 : t1);
        acc[2] = acc[2] + (SQUARE ? t2 * t2 : t2);
        acc[3] = acc[3] + (SQUARE ? t3 * t3 : t3);
      }
    }
  } else {
    for (int k = 0; k < K; ++k) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const uint64_t e = base + (uint64_t)k * kTreeLanes + i;
        if (e < d) {
          float v = row[e];
          if (SQUARE) {
            float r1, r2;
            load_ref_scalar<NORM>(ref, ref2, e, eps, r1, r2);
            v = normalize_w<NORM>(v, r1, r2, mu);
          }
          if (MINMAX) {
            lo = fminf(lo, v);
            hi = fmaxf(hi, v);
          }
          const double t = (double)v;
          acc[i] = acc[i] + (SQUARE ? t * t : t);
        }
      }
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) lanes[wave][4 * lane + i] = acc[i];
  if (MINMAX) {
    hi = wave_max(hi);
    lo = -wave_max(-lo);
  }
  wave_lds_fence();
  if (lane == 0) {
    double total = 0.0;
#pragma unroll 16
    for (int j = 0; j < kTreeLanes; ++j) total = total + lanes[wave][j];
    chunk_sums[(uint64_t)m * nchunks + chunk] = total;
    if (MINMAX) chunk_minmax[(uint64_t)m * nchunks + chunk] = make_float2(lo, hi);
  }
  wave_lds_fence();  // the lane sums are read before the next worker overwrites them
  }
}

// Chunk sums of the squares for the normalisations with a shared reference, whole chunks only: the
// reference tile of a quarter chunk stays in registers while MC workers use it (as in the maximum
// pass), so the reference is read from memory once per MC workers.  Lane sums still add their
// elements in the order k = 0..15: the quarters and the rows inside a quarter are walked in order.
template <int NORM, int MC>
__global__ __launch_bounds__(kBlock) void l2_chunk_kernel(GradRows g, const float4* __restrict__ ref4,
                                                          const float4* __restrict__ ref24,
                                                          double* __restrict__ chunk_sums, uint64_t whole_chunks,
                                                          uint64_t nchunks, float eps, uint32_t M) {
  __shared__ double lanes[kWavesPerBlock][kTreeLanes];
  const int wave = threadIdx.x / kWave, lane = threadIdx.x % kWave;
  const uint64_t chunk = (uint64_t)blockIdx.x * kWavesPerBlock + wave;
  if (chunk >= whole_chunks) return;  // whole wavefront; no workgroup barrier below
  const uint32_t m0 = blockIdx.y * MC;
  constexpr int Q = 4;                                  // rows (k) per quarter chunk
  constexpr int K = kTreeChunk / kTreeLanes;            // 16 rows of 64 float4 per chunk
  const uint64_t v0 = chunk * (kTreeChunk / 4) + lane;  // float4 index of row k = 0
  double acc[MC][4];
#pragma unroll
  for (int mm = 0; mm < MC; ++mm) acc[mm][0] = acc[mm][1] = acc[mm][2] = acc[mm][3] = 0.0;
#pragma unroll 1
  for (int k0 = 0; k0 < K; k0 += Q) {
    RefTile<NORM> rt[Q];
#pragma unroll
    for (int k = 0; k < Q; ++k) rt[k].load(ref4, ref24, v0 + (uint64_t)(k0 + k) * kWave, eps);
#pragma unroll
    for (int mm = 0; mm < MC; ++mm) {
      // rows past M (MC not dividing M) repeat the last row; their sums are not stored
      const v4f_u_t* __restrict__ row = g.row(min(m0 + (uint32_t)mm, M - 1));
      float4 x[Q];
#pragma unroll
      for (int k = 0; k < Q; ++k) x[k] = load_row_stream(row + v0 + (uint64_t)(k0 + k) * kWave);
#pragma unroll
      for (int k = 0; k < Q; ++k) {
        const double t0 = (double)normalize<NORM>(x[k].x, rt[k].r1.x, rt[k].r2.x);
        const double t1 = (double)normalize<NORM>(x[k].y, rt[k].r1.y, rt[k].r2.y);
        const double t2 = (double)normalize<NORM>(x[k].z, rt[k].r1.z, rt[k].r2.z);
        const double t3 = (double)normalize<NORM>(x[k].w, rt[k].r1.w, rt[k].r2.w);
        acc[mm][0] = acc[mm][0] + t0 * t0;  // the square of a binary32 value is exact in binary64
        acc[mm][1] = acc[mm][1] + t1 * t1;
        acc[mm][2] = acc[mm][2] + t2 * t2;
        acc[mm][3] = acc[mm][3] + t3 * t3;
      }
    }
  }
#pragma unroll
  for (int mm = 0; mm < MC; ++mm) {
#pragma unroll
    for (int i = 0; i < 4; ++i) lanes[wave][4 * lane + i] = acc[mm][i];
    wave_lds_fence();
    if (lane == 0 && m0 + mm < M) {
      double total = 0.0;
#pragma unroll 16
      for (int j = 0; j < kTreeLanes; ++j) total = total + lanes[wave][j];
      chunk_sums[(uint64_t)(m0 + mm) * nchunks + chunk] = total;
    }
    wave_lds_fence();
  }
}

// The chunk sums of the squares and, in the same pass over g, the candidates of the ternary coder (see
// absmax_select_kernel; here hardly an element is one: the scale is sqrt(d) times the typical |v|).  A workgroup takes
// a chunk of up to kL2SelectWorkers workers, its wavefronts a worker each in turn; the chunk's reference is in LDS, and the
// lane sums of all workers are added up in order at the end, a worker per lane (by one lane per worker and wavefront, as
// above, these additions are as many instructions as all others).  A wavefront's fetches, a tile of a worker each, rotate
// through three buffers.
// A slot is per worker and chunk (its candidates gathered over the four tiles, written out earlier only where they are many),
// touched only if it holds something, and the counts of the workgroup's workers are one word: a slot per tile, its count in it, was
// a quarter of a million writes of 8 bytes among the reads at d = 2^24, M = 16, and cost this kernel 20 of its 260 us and the
// quantise pass half its time.  It holds what the slots of four tiles would, near enough: rows whose magnitude varies along them
// (log-normal by 4096 elements, M = 64, d = 2^20, sigma 0.7 / 1.0 / 1.5) encode in 96 / 96 / 97 us with a slot per tile, 97 / 101 / 121
// with one of 128 entries per chunk (their chunks overflow), 90 / 92 / 97 so.
// Encode + decode there: 500 us by two passes, 345 with a slot per tile, 306 this way (this kernel 236 to 250 for 1.14 GB: the
// vector unit's time for draws, squares and tests, 160 us, as much as memory's, 181).
constexpr int kL2SelectWorkers = 8;
template <int NORM>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(4, 4))) void l2_select_kernel(
    GradRows g, const float4* __restrict__ ref4, double* __restrict__ chunk_sums, uint64_t chunks, uint64_t nchunks,
    uint32_t M, const float* __restrict__ sample_max, const uint32_t* __restrict__ select_ok,
    uint32_t* __restrict__ slots, uint64_t* __restrict__ counts, uint32_t* __restrict__ overflowed, uint32_t k0, uint32_t k1,
    uint32_t iter) {
  static_assert(NORM == kNormNone || NORM == kNormSub, "the coder that reads g once: no divisor reference");
  constexpr int L = kLoadsPerLane;                       // rows of 64 float4 per tile
  constexpr int T = kTreeChunk / (int)kWaveTileElements;  // tiles per chunk
  constexpr int V = kTreeChunk / 4;                      // float4 per chunk
  constexpr int kSumStride = kTreeLanes + 2;             // two binary64 of padding: the lanes' reads fall on different banks
  __shared__ __attribute__((aligned(16))) uint32_t stage[kWavesPerBlock][kL2StageWords];
  __shared__ __attribute__((aligned(16))) uint32_t draws[kWavesPerBlock][kL2StageWords];
  __shared__ __attribute__((aligned(16))) float4 refs[NORM == kNormSub ? V : 1];
  __shared__ __attribute__((aligned(16))) double sums[kL2SelectWorkers][kSumStride];
  __shared__ uint8_t found[kL2SelectWorkers];  // candidates of each worker in this chunk, in pairs, or kNoSlot
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = threadIdx.x % kWave;
  const uint64_t chunk = blockIdx.x;
  const uint32_t m0 = blockIdx.y * kL2SelectWorkers;
  const uint32_t count = min((uint32_t)kL2SelectWorkers, M - m0);
  if (NORM == kNormSub) {
    float4 r[V / kBlock];
#pragma unroll
    for (int k = 0; k < V / kBlock; ++k) r[k] = load_stream(ref4 + chunk * V + k * kBlock + threadIdx.x);
#pragma unroll
    for (int k = 0; k < V / kBlock; ++k) refs[k * kBlock + threadIdx.x] = r[k];
  }
  // item i of the wavefront: tile i mod T of its worker number i / T; past the last one the last is fetched again
  const uint32_t items = count > (uint32_t)wave ? ((count - (uint32_t)wave + kWavesPerBlock - 1) / kWavesPerBlock) * T : 0u;
  auto request = [&](float4 (&b)[L], uint32_t item) {
    const uint32_t it = min(item, items - 1);
    const v4f_u_t* p = g.row(m0 + (uint32_t)wave + it / T * kWavesPerBlock) + chunk * V + (uint64_t)(it % T) * (L * kWave);
#pragma unroll
    for (int j = 0; j < L; ++j) b[j] = load_row_stream(p + (uint32_t)(j * kWave + lane));
  };
  float4 b0[L], b1[L], b2[L];
  if (items != 0) {
    request(b0, 0);
    request(b1, 1);
  }
  __syncthreads();  // the reference is in LDS
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  float c1 = 0.f;
  bool select = false, fits = false;
  uint32_t base = 0, written = 0;  // candidates of the worker in the staging area, and in its slot
  auto work = [&](const float4 (&x)[L], uint32_t item) {
    const uint32_t mm = (uint32_t)wave + item / T * kWavesPerBlock, m = m0 + mm, t = item % T;
    if (t == 0) {
      acc[0] = acc[1] = acc[2] = acc[3] = 0.0;
      c1 = candidate_factor(sample_max[m]);
      select = select_ok[m] != 0u;
      fits = select;
      base = written = 0;
    }
#pragma unroll
    for (int j = 0; j < L; ++j) {
      float4 v = x[j];
      const uint32_t at = (t * L + (uint32_t)j) * kWave + (uint32_t)lane;
      if (NORM == kNormSub) {
        const float4 r = refs[at];
        v = make_float4(x[j].x - r.x, x[j].y - r.y, x[j].z - r.z, x[j].w - r.w);
      }
      const double t0 = (double)v.x, t1 = (double)v.y, t2 = (double)v.z, t3 = (double)v.w;
      acc[0] = __builtin_fma(t0, t0, acc[0]);  // the square of a binary32 value is exact in binary64: one rounding either way
      acc[1] = __builtin_fma(t1, t1, acc[1]);
      acc[2] = __builtin_fma(t2, t2, acc[2]);
      acc[3] = __builtin_fma(t3, t3, acc[3]);
      if (select) {  // (the same for the whole wavefront)
        const U32x4 rnd = philox4x32_10((uint32_t)(chunk * V) + at, m, iter, 0u, k0, k1);
        stage_candidates<true, kChunkPosMask, kL2StageSink>(stage[wave], draws[wave], v, rnd, c1, (int)t * L + j, lane, base);
      }
    }
    // The staged candidates to the worker's slot, 8 bytes per lane, twice where there may be more than two per lane.  (Encode +
    // decode, d = 2^24, M = 16: 302.9 us with slots of 128 and no early write-out, 306.4 with a loop over the pairs, 305.7 so.)
    auto write_out = [&](bool twice) {
      const uint32_t used = (base + 1) & ~1u;
      fits = fits && base <= kL2StageSink && written + used <= (uint32_t)kL2SlotEntries;
      uint64_t* slot = reinterpret_cast<uint64_t*>(slots + ((uint64_t)m * chunks + chunk) * kL2SlotEntries + written);
      auto pair = [&](uint32_t i) {
        const uint2 vw = *reinterpret_cast<const uint2*>(&stage[wave][2 * i]);
        const uint2 dw = *reinterpret_cast<const uint2*>(&draws[wave][2 * i]);
        // (an odd one out is followed by an entry that codes nothing: tau = 0)
        const uint32_t second = 2 * i + 1 < base ? slot_entry<kChunkPosMask>(vw.y, dw.y) : 0u;
        __hip_atomic_store(slot + i, ((uint64_t)second << 32) | slot_entry<kChunkPosMask>(vw.x, dw.x), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
      };
      wave_lds_fence();
      if (fits && 2 * (uint32_t)lane < base) pair((uint32_t)lane);
      if (twice && fits && 2 * (uint32_t)(lane + kWave) < base) pair((uint32_t)(lane + kWave));
      wave_lds_fence();
      written += used;
      base = 0;
    };
    static_assert(kL2FlushAt <= 2 * kWave && kL2StageSink <= 4 * kWave, "two entries a lane, or four");
    if (__builtin_expect(base > kL2FlushAt, 0)) write_out(true);  // (the same for the whole wavefront)
    if (t == T - 1) {
      write_out(false);
      if (lane == 0) found[mm] = (uint8_t)(fits ? written / 2 : kNoSlot);
#pragma unroll
      for (int i = 0; i < 4; ++i) sums[mm][4 * lane + i] = acc[i];
    }
  };
  for (uint32_t i = 0; i < items; i += 3) {
    request(b2, i + 2);
    work(b0, i);
    request(b0, i + 3);
    if (i + 1 < items) work(b1, i + 1);
    request(b1, i + 4);
    if (i + 2 < items) work(b2, i + 2);
  }
  __syncthreads();
  if (threadIdx.x < count) {
    double total = 0.0;
#pragma unroll 16
    for (int j = 0; j < kTreeLanes; ++j) total = total + sums[threadIdx.x][j];
    chunk_sums[(uint64_t)(m0 + threadIdx.x) * nchunks + chunk] = total;
  }
  if (threadIdx.x == kWave) {  // (not the wavefront that adds the lane sums)
    uint64_t all = 0;
    uint32_t without = 0;
#pragma unroll
    for (int k = 0; k < kL2SelectWorkers; ++k) {
      const uint32_t n = (uint32_t)k < count ? found[k] : 0u;
      all |= (uint64_t)n << (8 * k);
      without += n == kNoSlot ? 1u : 0u;
    }
    __hip_atomic_store(counts + (uint64_t)blockIdx.y * chunks + chunk, all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (without != 0u) atomicAdd(&overflowed[blockIdx.x % kL2OverflowCounts], without);
  }
}

// The same for the l2 scale, whose slots are per worker and chunk of four tiles and all but empty: hardly an element is a
// candidate (a row expects at most sqrt(d) R / R^ of them, the 1-norm over the 2-norm).  The counts of eight workers lie in
// eight bytes of their own, so that nothing is written to a slot without candidates; of every slot one line is read.  A wavefront
// takes a chunk of kL2QuantWorkers workers, all their first 32 entries requested at once; tiles behind the last whole chunk (at
// most three; the ragged one is the ordinary quantiser's) have no slots and are the last row of workgroups'.
// d = 2^24, M = 16 (67 MB of codes): 28 us with a slot per tile, 16 this way (13 at the least, 5.2 TB/s).
constexpr int kL2QuantWorkers = 4;
template <int NORM>
__global__ __launch_bounds__(kBlock, 8) void quantize_l2_candidates_kernel(
    GradRows g, const float4* __restrict__ ref4, const float* __restrict__ scales, const uint32_t* __restrict__ slots,
    const uint8_t* __restrict__ counts, uint32_t* __restrict__ codes, uint64_t d, uint64_t words, uint64_t chunks, uint32_t M,
    uint32_t k0, uint32_t k1, uint32_t iter, const uint32_t* __restrict__ use_slots) {
  constexpr int MC = kL2QuantWorkers;
  constexpr int T = kTreeChunk / (int)kWaveTileElements;  // tiles per chunk
  constexpr int W = kTreeChunk / 16;                      // packed words per chunk: four a lane
  static_assert(W == 4 * kWave, "one 16-byte store per worker");
  static_assert(kL2SelectWorkers == 8 && kL2SelectWorkers % MC == 0, "the counts of eight workers are one 64-bit word");
  __shared__ __attribute__((aligned(16))) FragmentBuffer<W, MC> lds;
  if (use_slots[0] == 0u) return;  // too many slots overflowed: the ordinary quantiser runs instead
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = threadIdx.x % kWave;
  const uint32_t m0 = blockIdx.y * MC, count = min((uint32_t)MC, M - m0);
  const uint64_t chunk = (uint64_t)blockIdx.x * kWavesPerBlock + wave;
  if (chunk >= chunks) {  // (whole wavefronts; nothing below meets the others)
    const uint64_t tile = chunks * T + (chunk - chunks);
    if (tile >= d / kWaveTileElements) return;
    for (uint32_t mm = 0; mm < count; ++mm) {
      const float r = scales[m0 + mm];
      lds.b32[0][wave][lane] = 0u;
      wave_lds_fence();
      if (r != 0.f) code_tile<NORM>(lds.b8[0][wave], g, ref4, nullptr, tile, m0 + mm, lane, r, 0.f, iter, k0, k1);
      wave_lds_fence();
      store_word_through(codes + (uint64_t)(m0 + mm) * words + tile * kWave + (uint32_t)lane, lds.b32[0][wave][lane]);
      wave_lds_fence();
    }
    return;
  }
  constexpr uint32_t kGroup = kL2SelectWorkers;
  uint32_t first[MC];
  float R[MC];
#pragma unroll
  for (int mm = 0; mm < MC; ++mm) {
    const uint32_t m = min(m0 + (uint32_t)mm, M - 1);
    first[mm] = slots[((uint64_t)m * chunks + chunk) * kL2SlotEntries + ((uint32_t)lane & 31u)];
    R[mm] = scales[m];
  }
  const uint32_t four = *reinterpret_cast<const uint32_t*>(counts + ((uint64_t)(m0 / kGroup) * chunks + chunk) * kGroup + m0 % kGroup);
#pragma unroll
  for (int mm = 0; mm < MC; ++mm)
    *reinterpret_cast<v4u_t*>(&lds.b32[mm][wave][4 * lane]) = v4u_t{0u, 0u, 0u, 0u};
  wave_lds_fence();
  auto put = [&](uint32_t slot, uint32_t e, uint32_t code) {
    atomicOr(&lds.b32[slot][wave][(e & kChunkPosMask) >> 4], code << (2u * (e & 15u)));
  };
  // (rare, and behind the loop, as in quantize_candidates_kernel)
  uint32_t long_slots = 0u, no_slots = 0u, undecided = 0u;
#pragma unroll
  for (int mm = 0; mm < MC; ++mm) {
    const uint32_t e = first[mm], pairs = __builtin_amdgcn_readfirstlane(four >> (8 * mm)) & 255u;
    const bool live = (uint32_t)mm < count && R[mm] != 0.f;  // (R = 0: every element codes to 0)
    no_slots |= (live && pairs == kNoSlot ? 1u : 0u) << mm;
    long_slots |= (live && pairs != kNoSlot && pairs > 16u ? 1u : 0u) << mm;
    const int in = (uint32_t)lane < (live && pairs != kNoSlot ? min(2 * pairs, 32u) : 0u);
    const int one = in & entry_codes_one<kChunkPosMask>(e, R[mm]);
    if (one) put((uint32_t)mm, e, 1u | ((e >> 31) << 1));
    undecided |= (uint32_t)(in & ~one & ~entry_codes_zero<kChunkPosMask>(e, R[mm])) << mm;
  }
  if (long_slots != 0u || no_slots != 0u || __builtin_amdgcn_ballot_w64(undecided != 0u) != 0ull) {
#pragma unroll 1
    for (uint32_t mm = 0; mm < count; ++mm) {
      const uint32_t m = m0 + mm;
      const float r = scales[m];
      if (((no_slots >> mm) & 1u) != 0u) {
#pragma unroll 1
        for (uint32_t t = 0; t < (uint32_t)T; ++t)
          code_tile<NORM>(lds.b8[mm][wave] + t * (kWave * 4), g, ref4, nullptr, chunk * T + t, m, lane, r, 0.f, iter, k0, k1);
        continue;
      }
      const bool longer = ((long_slots >> mm) & 1u) != 0u;
      if (!longer && __builtin_amdgcn_ballot_w64((int)(undecided >> mm) & 1) == 0ull) continue;
      const uint32_t* __restrict__ sl = slots + ((uint64_t)m * chunks + chunk) * kL2SlotEntries;
      const uint32_t n = 2u * counts[((uint64_t)(m / kGroup) * chunks + chunk) * kGroup + m % kGroup];
#pragma unroll 1
      for (uint32_t i = (uint32_t)lane; i < n; i += kWave) {  // all of them once more: or-ing a code in twice changes nothing
        const uint32_t e = sl[i];
        uint32_t code = 1u | ((e >> 31) << 1);
        if (!entry_codes_one<kChunkPosMask>(e, r))
          code = entry_codes_zero<kChunkPosMask>(e, r)
                     ? 0u
                     : code_of_element<NORM>(g, ref4, chunk * kTreeChunk + (e & kChunkPosMask), m, r, iter, k0, k1);
        if (code != 0u) put(mm, e, code);
      }
    }
  }
  flush_packed<W, MC>(lds, wave, lane, codes, words, chunk * W, m0, count);
}

// One workgroup per worker: the chunk sums come to LDS GROUPS groups at a time, in whole lines (a thread per
// group that fetched its 256 chunk sums one after the other took 26 us at d = 2^24 and 39 at d = 2^27, 5 and 19 this way; 16
// groups at a time with loads under a branch, each waited for before the next, 8 and 56), a thread adds a group in
// order, and thread 0 the groups in order.  MEAN: out[m] = float(total / d), and, when chunk_minmax is
// given, scales[m] = max |g - out[m]| from the smallest and the largest element.  Otherwise
// out[m] = float(sqrt(total)), 0 when below FLT_MIN.  Division and square root of binary64 are
// correctly rounded on the device, so the float32 result is the same as on any IEEE host.
// GROUPS: 64, a lane of the first wavefront each (131 KB of LDS), or 16 or 1 where a row has no more (d = 5000, 1000 workers,
// whose workgroups then share the compute units: encode + decode 177 us; with 64 groups 4 us more).
template <bool MEAN, int GROUPS>
__global__ __launch_bounds__(kBlock) void tree_finish_kernel(const double* __restrict__ chunk_sums,
                                                             const float2* __restrict__ chunk_minmax,
                                                             uint64_t nchunks, uint64_t ngroups, uint64_t d, uint32_t M,
                                                             float* __restrict__ out, float* __restrict__ scales, SlotVote vote) {
  if (blockIdx.x >= M) {  // (behind l2_select_kernel only)
    vote_on_slots<kBlock>(vote);
    return;
  }
  constexpr int kLoads = GROUPS < 16 ? GROUPS : 16;  // in flight per thread
  __shared__ float red_lo[kWavesPerBlock], red_hi[kWavesPerBlock];
  __shared__ double part[GROUPS][kTreeGroup + 1];  // (one of padding: the groups' threads read different banks)
  __shared__ double group[GROUPS];
  const uint32_t m = blockIdx.x;
  const double* __restrict__ cs = chunk_sums + (uint64_t)m * nchunks;
  double total = 0.0;  // thread 0
  for (uint64_t q0 = 0; q0 < ngroups; q0 += GROUPS) {
    const uint64_t c0 = q0 * kTreeGroup;
    const uint32_t n = (uint32_t)min((uint64_t)(GROUPS * kTreeGroup), nchunks - c0);
    __syncthreads();  // the batch before has been added
#pragma unroll
    for (int k0 = 0; k0 < GROUPS; k0 += kLoads) {
      if ((uint32_t)k0 * kTreeGroup >= n) break;
      double v[kLoads];  // (past the end the last one again, which is not added: no load under a branch)
#pragma unroll
      for (int k = 0; k < kLoads; ++k) v[k] = cs[c0 + min((uint32_t)(k0 + k) * kTreeGroup + threadIdx.x, n - 1)];
#pragma unroll
      for (int k = 0; k < kLoads; ++k) part[k0 + k][threadIdx.x] = v[k];
    }
    __syncthreads();
    if (threadIdx.x < (uint32_t)GROUPS) {
      const uint32_t first = threadIdx.x * kTreeGroup, count = first < n ? min((uint32_t)kTreeGroup, n - first) : 0u;
      double a = 0.0;
#pragma unroll 16
      for (uint32_t c = 0; c < count; ++c) a = a + part[threadIdx.x][c];
      group[threadIdx.x] = a;
    }
    wave_lds_fence();  // (the groups' threads and thread 0 are one wavefront)
    if (threadIdx.x == 0)
      for (uint32_t q = 0; q < (uint32_t)GROUPS && q0 + q < ngroups; ++q) total = total + group[q];
  }
  if (MEAN && chunk_minmax != nullptr) {
    float lo = INFINITY, hi = -INFINITY;
    for (uint64_t c = threadIdx.x; c < nchunks; c += kBlock) {
      const float2 mm = chunk_minmax[(uint64_t)m * nchunks + c];
      lo = fminf(lo, mm.x);
      hi = fmaxf(hi, mm.y);
    }
    lo = -wave_max(-lo);
    hi = wave_max(hi);
    if (threadIdx.x % kWave == 0) {
      red_lo[threadIdx.x / kWave] = lo;
      red_hi[threadIdx.x / kWave] = hi;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    if (MEAN) {
      const float mu = (float)(total / (double)d);
      out[m] = mu;
      if (chunk_minmax != nullptr) {
        float lo = red_lo[0], hi = red_hi[0];
#pragma unroll
        for (int k = 1; k < kWavesPerBlock; ++k) {
          lo = fminf(lo, red_lo[k]);
          hi = fmaxf(hi, red_hi[k]);
        }
        const float r = fmaxf(fabsf(lo - mu), fabsf(hi - mu));
        scales[m] = r < FLT_MIN ? 0.f : r;
      }
    } else {
      const float r = (float)sqrt(total);
      out[m] = r < FLT_MIN ? 0.f : r;
    }
  }
}

// ------------------------------------------------------------------------------------------
// Launch geometry
// ------------------------------------------------------------------------------------------
inline uint32_t div_up_u32(uint64_t a, uint64_t b) {
  const uint64_t q = (a + b - 1) / b;
  return (uint32_t)(q > kMaxGridX ? kMaxGridX : q);
}

// Workers handled inside one workgroup (16, 8, 4, 2 or 1; the last group of a row of workgroups may be
// short).  A group reads the shared reference once, so fewer groups mean less traffic; a short group
// costs the scale pass repeated loads of its last row (cache hits: repeat_cost 0.3 of a row there,
// nothing in the quantiser, which stops at the last worker).  At least 2048 workgroups are kept to
// fill 256 compute units.  fives: groups of 5 as well, for the two kernels that work with candidate slots (in
// absmax_select_kernel the reference and five rows are two rounds of its three buffers); chosen for 5, 9, 10, 17 to 20 and 25 workers of long rows (encode + decode at d = 2^25: M = 5 293 us
// in a group of 8, 250 in one of 5; M = 9 450 in groups of 4, 414 in groups of 5; M = 10 476 / 433; d = 2^24: M = 20
// 425 / 411, M = 25 534 in groups of 8, 515).
inline int pick_workers_per_block(uint32_t M, uint64_t tiles, double repeat_cost, int mc_max = 8, bool fives = false) {
  int best = 1;
  double best_cost = (double)M;
  for (const int mc : {2, 4, 5, 8, 16}) {
    const uint32_t groups = (M + mc - 1) / mc;
    if (mc == 5 && !fives) continue;
    if (mc > mc_max || tiles * groups < 2048 || (mc > 8 && M <= 8)) break;
    const double cost = groups + repeat_cost * (groups * mc - M);
    if (cost <= best_cost) {
      best = mc;
      best_cost = cost;
    }
  }
  return best;
}

inline bool aligned16_or_null(const void* a, const void* b, const void* c = nullptr, const void* e = nullptr) {
  auto al = [](const void* p) { return p == nullptr || (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  return al(a) && al(b) && al(c) && al(e);
}

inline bool vec_ok(uint64_t d, const void* a, const void* b, const void* c) {
  auto al = [](const void* p) { return p == nullptr || (reinterpret_cast<uintptr_t>(p) & 15u) == 0; };
  return d % 4 == 0 && al(a) && al(b) && al(c);
}

// Workgroups behind the others that take the ragged last wavefront tile of mc workers, a worker per wavefront.
inline uint32_t tail_workgroups(uint64_t d, int mc) {
  return d % kWaveTileElements == 0 ? 0u : (uint32_t)((mc + kWavesPerBlock - 1) / kWavesPerBlock);
}

// Workgroups per group of workers where the ragged tile has some of its own.  Workgroups go to the eight compute dies in
// turn, so their number decides how many of the dies' L2s a tile's reference passes through as the groups follow one
// another: all of them if it is odd (encode + decode at 40 workers, 4-bit: d = 98 * 4096 40.0 us, 97 * 4096 42.4, 99 * 4096
// 43.1).  The ragged tile's made it odd or even as it came; idle ones behind them make it a multiple of 4: two dies per
// tile.  d = 400000, M = 40, 4-bit: as it came 44.3 us, a multiple of 2 40.1, of 4 40.1, of 8 40.7; d = 10^6 + 3, M = 16,
// quotient: 49.7 / 46.4 / 42.5 / 42.7; d = 100003, M = 33 (26 workgroups): 17.1 / 17.1 / 17.1 / 21.2, where one die in eight
// gets a third more than the others.  Below 64 the reference is too short to
// matter and the idle ones cost (d = 80000, M = 200 (21 workgroups) 61.5 us, 63.2 with 24; d = 5000, M = 1000, mean 170 with
// 2, 179 with 4).
constexpr uint32_t kGroupMultiple = 4;
inline uint32_t workgroups_per_group(uint32_t main_blocks, uint32_t tail, uint32_t groups) {
  const uint32_t n = main_blocks + tail;
  return tail == 0 || groups == 1 || n < 64 ? n : (n + kGroupMultiple - 1) / kGroupMultiple * kGroupMultiple;
}

// hold: where the one-launch tail can reduce max_left rows of partial maxima by itself, no more workgroups than leave that many, if
// these still fill the chip: a launch of its own for the reduction costs 5 us, and workgroups that walk a few tiles beat twice the
// number that take one (given gradients d = 4e6, M = 8: 980 rows of four groups and the reduction 28.8 + 4.9 us, 256 rows 26.4; d =
// 2e6, M = 8 16.4 + 4.7, 14.3).  Not for worker counts that are no power of two, whose maxima the next launch has to read one by
// one (d = 3e6, M = 7, combined form 62.1 us with the reduction's launch, 64.8 without).  With eight groups, where a few of that many
// workgroups would have a second tile, half as many with two each up to 1.6 tiles a workgroup, in whole eights (one per die; iterations
// M = 8, reduction's launch / max_left / half, us: d = 1.1e6 21.9 / 23.2 / 21.2, combined form 29.3 / 34.4 / 28.6; d = 1.5e6 27.2 / 26.7 /
// 25.6 and 35.6 / 39.0 / 34.8; at d = 1.7e6 28.6 held to max_left, 30.1 with half).  Not ahead of the
// quantiser, every wavefront of which would read all those rows (encode M = 64, d = 163840 18.4 us with the reduction's launch, 21.7
// held to 25 rows; 4-bit, quotient 21.7 / 25.6; M = 128, d = 98304 21.3 / 23.7; M = 32, d = 220004 15.7 / 16.5).
constexpr uint32_t kAbsmaxFewBlocks = 960;
// One group of workers: 1024 workgroups (four a compute unit) that walk the tiles instead of up to 4096, whose last round is
// short.  Encode + decode, before / after: d = 2^25, M = 1, 4-bit 137.8 / 133.6 us; d = 2e7, M = 2, no normalisation 71.8 / 68.5;
// d = 2^24, M = 4, 4-bit 150.6 / 148.0; d = 2^25, M = 8, combined form 546.9 / 543.9; iterations d = 2^24, M = 8 244.4 / 241.8.  Beyond
// kAbsmaxLongTiles workgroups' worth of tiles there are rounds enough (d = 2^27, M = 8, quotient 1840 / 1845); several groups
// that walk apart re-read the reference (d = 2^24, M = 9 286 / 297; d = 10^6, M = 32 65 / 68.7).
constexpr uint32_t kAbsmaxWalkers = 1024;
constexpr uint64_t kAbsmaxLongTiles = 16384;
template <int NORM, int MC>
hipError_t absmax_vec_launch(const CodecShape& c, const float* g, const float* gref, const float* gref2,
                             float* partials, uint32_t max_left, bool hold, uint32_t* nblocks, hipStream_t s) {
  const uint32_t tail = tail_workgroups(c.d, MC), groups = (c.M + MC - 1) / MC;
  const uint64_t per_y = (c.d / kWaveTileElements + kWavesPerBlock - 1) / kWavesPerBlock;
  uint32_t main_blocks = (uint32_t)(per_y < kAbsmaxMaxBlocks - tail ? per_y : kAbsmaxMaxBlocks - tail);
  const uint32_t limit = max_left > tail ? max_left - tail : 0u;
  if (hold && main_blocks > limit && limit * groups >= kAbsmaxFewBlocks && (c.M & (c.M - 1)) == 0)
    main_blocks = groups > 4 && 5 * per_y <= 8 * limit ? (((uint32_t)per_y + 1) / 2 + tail + 7) / 8 * 8 - tail : limit;
  else if (groups == 1 && main_blocks > kAbsmaxWalkers && per_y <= kAbsmaxLongTiles)
    main_blocks = kAbsmaxWalkers;
  *nblocks = main_blocks + tail;
  const dim3 grid(workgroups_per_group(main_blocks, tail, groups), groups);
  hipLaunchKernelGGL((absmax_vec_kernel<NORM, MC>), grid, dim3(kBlock), 0, s, GradRows{g, c.d}, reinterpret_cast<const float4*>(gref),
                     reinterpret_cast<const float4*>(gref2), partials, c.d, main_blocks, c.M, c.eps, c.means);
  return hipGetLastError();
}

// Scratch of the ternary coder that reads g once: the word that says whether the slots are used, the
// sample's maxima [M], the sample pass's partial maxima [kAbsmaxMaxBlocks][M], the overflow counts of the
// scale pass's workgroups (as many), the slots [M][d / 1024] of 512 bytes (of the l2 scale: [M][d / 4096] of 1792 bytes, and
// their counts).
struct CandidateScratch {
  uint32_t* use_slots;
  float* sample_max;
  uint32_t* select_ok;
  float* sample_partials;
  float* sample_sums;
  uint32_t* overflowed;
  uint32_t* slots;
};
inline size_t round_up_256(size_t v) { return (v + 255) / 256 * 256; }
inline size_t candidate_head_bytes(uint32_t M) {
  return 256 + 2 * round_up_256((size_t)M * sizeof(float)) + 3 * round_up_256((size_t)kAbsmaxMaxBlocks * M * sizeof(float));
}
inline CandidateScratch candidate_scratch(const CodecShape& c, void* scratch) {
  unsigned char* p = static_cast<unsigned char*>(scratch);
  CandidateScratch cs;
  cs.use_slots = reinterpret_cast<uint32_t*>(p);
  p += 256;
  cs.sample_max = reinterpret_cast<float*>(p);
  p += round_up_256((size_t)c.M * sizeof(float));
  cs.select_ok = reinterpret_cast<uint32_t*>(p);
  p += round_up_256((size_t)c.M * sizeof(float));
  cs.sample_partials = reinterpret_cast<float*>(p);
  p += round_up_256((size_t)kAbsmaxMaxBlocks * c.M * sizeof(float));
  cs.sample_sums = reinterpret_cast<float*>(p);
  p += round_up_256((size_t)kAbsmaxMaxBlocks * c.M * sizeof(float));
  cs.overflowed = reinterpret_cast<uint32_t*>(p);
  p += round_up_256((size_t)kAbsmaxMaxBlocks * c.M * sizeof(float));
  cs.slots = reinterpret_cast<uint32_t*>(p);
  return cs;
}

// The l2 scale's counts: a byte per worker and chunk, eight workers to a word, [ceil(M / 8)][chunks].  They lie behind its slots,
// one per worker and chunk, in the room of one per tile.
inline uint64_t* l2_slot_counts(const CodecShape& c, const CandidateScratch& cs) {
  constexpr int kTileSlots = kTreeChunk / (int)kWaveTileElements * kSlotEntries;
  static_assert(kL2SlotEntries * sizeof(uint32_t) + 8 <= kTileSlots * sizeof(uint32_t) && kL2SlotEntries % 32 == 0,
                "with 8 bytes of counts per worker it fits, and slots are whole lines of 128 bytes");
  return reinterpret_cast<uint64_t*>(cs.slots + (uint64_t)c.M * (c.d / kTreeChunk) * kL2SlotEntries);
}

// The sample: every kSampleStride-th whole wavefront tile of every row.
template <int NORM, bool L2>
hipError_t sample_launch(const CodecShape& c, const float* g, const float* gref, const CandidateScratch& cs, uint32_t* rows,
                         float* sampled, hipStream_t s) {
  const uint64_t sample_tiles = (c.d / kWaveTileElements + kSampleStride - 1) / kSampleStride;
  uint32_t nsample = div_up_u32(sample_tiles, kSampleWaves);
  if (nsample > kSampleRows) nsample = kSampleRows;
  *rows = nsample;
  *sampled = (float)(sample_tiles * kWaveTileElements);
  hipLaunchKernelGGL((sample_stats_kernel<NORM, L2>), dim3(nsample, c.M), dim3(kSampleThreads), 0, s, GradRows{g, c.d},
                     reinterpret_cast<const float4*>(gref), cs.sample_partials, cs.sample_sums, c.d / 4, c.M);
  return hipGetLastError();
}

template <int NORM>
hipError_t absmax_candidates_dispatch(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                                      const float* gref2, float* partials, const CandidateScratch& cs, float* scales,
                                      hipStream_t s) {
  const uint64_t nvec = c.d / 4;
  const int mc = pick_workers_per_block(c.M, (nvec + kBlock * kAbsmaxLoads - 1) / (kBlock * kAbsmaxLoads), 0.3, 8, true);
  uint32_t nblocks = 0;
  hipError_t e;
  uint32_t nsample = 0;
  float sampled = 0.f;
  e = sample_launch<NORM, false>(c, g, gref, cs, &nsample, &sampled, s);
  if (e != hipSuccess) return e;
  const uint64_t row_tiles = c.d / kWaveTileElements;
  const uint32_t tail = tail_workgroups(c.d, mc);
  const uint32_t per_y = div_up_u32(row_tiles, kWavesPerBlock);
  const uint32_t cap = kAbsmaxMaxBlocks - 1 - tail;
  const uint32_t main_blocks = per_y < cap ? per_y : cap;
  nblocks = main_blocks + tail;
#define TNG_SELECT(MC)                                                                                              \
  hipLaunchKernelGGL((absmax_select_kernel<NORM, MC>), dim3(nblocks, (c.M + MC - 1) / MC), dim3(kBlock), 0, s,      \
                     GradRows{g, c.d}, reinterpret_cast<const float4*>(gref), reinterpret_cast<const float4*>(gref2), \
                     partials, c.d, main_blocks, c.M, c.eps, cs.sample_partials, cs.sample_sums, nsample, sampled, cs.sample_max, cs.select_ok, cs.slots, cs.overflowed, \
                     c.k0, c.k1, iter)
  switch (mc) {
    case 8: TNG_SELECT(8); break;
    case 5: TNG_SELECT(5); break;
    case 4: TNG_SELECT(4); break;
    case 2: TNG_SELECT(2); break;
    default: TNG_SELECT(1); break;
  }
#undef TNG_SELECT
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const SlotVote vote{cs.overflowed, nblocks * ((c.M + (uint32_t)mc - 1) / (uint32_t)mc), (uint64_t)c.M * row_tiles, cs.use_slots};
  const uint32_t threads = finish_threads(nblocks);
  hipLaunchKernelGGL((threads == kFinishLarge ? absmax_finish_vote_kernel<kFinishLarge> : absmax_finish_vote_kernel<kBlock>), dim3(c.M + 1), dim3(threads), 0, s, partials, nblocks, c.M, scales, cs.sample_max,
                     cs.select_ok, vote);
  return hipGetLastError();
}

template <int NORM, int BITS>
hipError_t quantize_dispatch(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                             const float* gref2, float* scales, uint32_t* codes, const float* partials,
                             uint32_t fused_rows, hipStream_t s, const uint32_t* skip_if_set = nullptr);

template <int NORM>
hipError_t quantize_candidates_dispatch(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                                        const float* gref2, const float* scales, const CandidateScratch& cs,
                                        uint32_t* codes, hipStream_t s) {
  const uint64_t tiles = (c.d / kWaveTileElements + kWavesPerBlock - 1) / kWavesPerBlock;  // workgroups of 4 wavefront tiles
  // As absmax_select_kernel's but for the cost of a repeated row, and where that would be groups of five (5, 9 and 10 workers), tiles of one
  // worker at a time: five rows left 24 lanes of a wavefront idle (this pass at d = 2^25 + 3, M = 5 30.9 -> 26.3 us; encode + decode 246.1 ->
  // 240.6; d = 14912512, M = 9 193.8 -> 189.3; d = 13421568, M = 10 180.0 -> 178.1).  For other worker counts one at a time is 1 % ahead or
  // behind (M = 8: d = 2^27 1196 -> 1182, d = 2^23 103.0 -> 103.7; M = 33, d = 2033664 101.0 -> 102.5).
  const int fives = pick_workers_per_block(c.M, tiles, 0.01, 8, true), mc = fives == 5 ? 1 : fives;
#define TNG_QC(MC)                                                                                                   \
  hipLaunchKernelGGL((quantize_candidates_kernel<NORM, MC>),                                                           \
                     dim3((uint32_t)((tiles + quantize_tiles(MC) - 1) / quantize_tiles(MC)), (c.M + MC - 1) / MC), dim3(kBlock), 0, \
                     s, GradRows{g, c.d}, reinterpret_cast<const float4*>(gref), reinterpret_cast<const float4*>(gref2), \
                     scales, cs.slots, codes, c.d, c.words, c.M, c.eps, c.k0, c.k1, iter, cs.use_slots, cs.select_ok)
  if (c.scale_l2 != 0) {
    const uint64_t chunks = c.d / kTreeChunk, loose = c.d / kWaveTileElements % (kTreeChunk / kWaveTileElements);
    hipLaunchKernelGGL(quantize_l2_candidates_kernel<NORM>,
                       dim3((uint32_t)((chunks + loose + kWavesPerBlock - 1) / kWavesPerBlock), (c.M + kL2QuantWorkers - 1) / kL2QuantWorkers),
                       dim3(kBlock), 0, s, GradRows{g, c.d}, reinterpret_cast<const float4*>(gref), scales, cs.slots,
                       reinterpret_cast<const uint8_t*>(l2_slot_counts(c, cs)), codes, c.d, c.words, chunks, c.M, c.k0, c.k1, iter,
                       cs.use_slots);
  } else switch (mc) {
    case 8: TNG_QC(8); break;
    case 4: TNG_QC(4); break;
    case 2: TNG_QC(2); break;
    default: TNG_QC(1); break;
  }
#undef TNG_QC
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // the ordinary quantiser right behind it: one of the two returns at once, by the vote of the scale pass (the ragged
  // last tile is the ordinary one's either way: in the kernel above it cost the registers of a wavefront per SIMD)
  return quantize_dispatch<NORM, 2>(c, iter, g, gref, gref2, const_cast<float*>(scales), codes, nullptr, 0, s,
                                    cs.use_slots);
}

template <int NORM>
hipError_t absmax_dispatch(const CodecShape& c, const float* g, const float* gref, const float* gref2,
                           float* partials, float* scales, uint32_t max_left, bool hold, uint32_t* left_rows,
                           hipStream_t s) {
  uint32_t nblocks = 0;
  hipError_t e;
  switch (pick_workers_per_block(c.M, div_up_u32(c.d, (uint64_t)kBlock * kAbsmaxLoads * 4), 0.3)) {
    case 8: e = absmax_vec_launch<NORM, 8>(c, g, gref, gref2, partials, max_left, hold, &nblocks, s); break;
    case 4: e = absmax_vec_launch<NORM, 4>(c, g, gref, gref2, partials, max_left, hold, &nblocks, s); break;
    case 2: e = absmax_vec_launch<NORM, 2>(c, g, gref, gref2, partials, max_left, hold, &nblocks, s); break;
    default: e = absmax_vec_launch<NORM, 1>(c, g, gref, gref2, partials, max_left, hold, &nblocks, s); break;
  }
  if (e != hipSuccess) return e;
  if (nblocks <= max_left) {
    *left_rows = nblocks;
    return hipSuccess;
  }
  return launch_absmax_finish(partials, nblocks, c.M, scales, s);
}

template <int NORM, int BITS, int MC, bool FUSED>
hipError_t quantize_vec_launch(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                               const float* gref2, const float* scales, uint32_t* codes, const FusedScale& fs,
                               hipStream_t s, const uint32_t* skip_if_set = nullptr) {
  const uint32_t tail = tail_workgroups(c.d, MC);
  const uint32_t main_blocks = (uint32_t)((c.d / kWaveTileElements + kWavesPerBlock - 1) / kWavesPerBlock);
  const uint32_t groups = (c.M + MC - 1) / MC;
  const dim3 grid(workgroups_per_group(main_blocks, tail, groups), groups);
  hipLaunchKernelGGL((quantize_pack_vec_kernel<NORM, BITS, MC, FUSED>), grid, dim3(kBlock), 0, s, GradRows{g, c.d}, reinterpret_cast<const float4*>(gref),
                     reinterpret_cast<const float4*>(gref2), scales, codes, c.d, c.words, main_blocks, c.M, c.eps, c.k0,
                     c.k1, iter, c.means, fs, skip_if_set);
  return hipGetLastError();
}

inline int quantize_workers_per_block(const CodecShape& c) {
  constexpr uint64_t kTile = (uint64_t)kBlock * kLoadsPerLane * 4;
  return pick_workers_per_block(c.M, (c.d + kTile - 1) / kTile, 0.0, 16);
}

// Rows of partial maxima that the quantiser reduces by itself: every wavefront reads one line per row, so a launch of many
// wavefronts pays more for them than a launch of its own costs (4 us): encode + decode at d = 25000, M = 4 18.2 -> 14.9 us,
// d = 2^18, M = 8 (131072 reads) 18.1 -> 14.6, but d = 4e5, M = 40 (1.5 million) 40.7 -> 46.8.
inline uint32_t fused_scale_rows(const CodecShape& c) {
  if (quantize_workers_per_block(c) != 1) return 0;
  const uint64_t wavefronts = (c.d / kWaveTileElements + 1) * c.M, rows = kFusedScaleReads / wavefronts;
  return rows < kFusedScaleRows ? (uint32_t)rows : kFusedScaleRows;
}

// fused_rows > 0: scales is an output and the scale is taken from the first fused_rows rows of
// partials (see FusedScale); only problems small enough for one worker per workgroup go that way,
// larger ones get the reduction kernel first.
template <int NORM, int BITS>
hipError_t quantize_dispatch(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                             const float* gref2, float* scales, uint32_t* codes, const float* partials,
                             uint32_t fused_rows, hipStream_t s, const uint32_t* skip_if_set) {
  const int mc = quantize_workers_per_block(c);
  FusedScale fs{partials, fused_rows, scales};
  if (fused_rows > fused_scale_rows(c)) {
    const hipError_t e = launch_absmax_finish(partials, fused_rows, c.M, scales, s);
    if (e != hipSuccess) return e;
    fs.rows = 0;
  }
  if (fs.rows > 0) return quantize_vec_launch<NORM, BITS, 1, true>(c, iter, g, gref, gref2, scales, codes, fs, s);
#define TNG_QUANTIZE(MC) \
  return quantize_vec_launch<NORM, BITS, MC, false>(c, iter, g, gref, gref2, scales, codes, fs, s, skip_if_set)
  switch (mc) {
    case 16: TNG_QUANTIZE(16);
    case 8: TNG_QUANTIZE(8);
    case 4: TNG_QUANTIZE(4);
    case 2: TNG_QUANTIZE(2);
    default: TNG_QUANTIZE(1);
  }
#undef TNG_QUANTIZE
}

template <int NORM, int BITS>
hipError_t decode_dispatch(const CodecShape& c, const uint32_t* codes, const float* scales, const float* gref,
                           const float* gref2, float* vbar, float* w, float lr, float* ref_out,
                           hipStream_t s) {
  const float inv_m = 1.0f / (float)c.M;
  const uint64_t nvec = (c.d + 3) / 4;
  const uint64_t big_tiles = (nvec + kBlock * kDecodeLoads - 1) / (kBlock * kDecodeLoads);
  // Codes that fit the 256 MiB last-level cache were just written by the quantiser and are rewritten
  // by the next iteration: ordinary loads keep the lines resident (measured 4 % faster, and the
  // following quantise pass too); larger code arrays are streamed (measured 17 % faster at 512 MiB).
  const bool stream_codes = (uint64_t)c.M * c.words * sizeof(uint32_t) > (256ull << 20);
#define TNG_DECODE_LAUNCH(V, SC, GRID)                                                                          \
  hipLaunchKernelGGL((decode_vec_kernel<NORM, BITS, V, SC>), dim3((uint32_t)(GRID)), dim3(kBlock), 0, s, codes,  \
                     scales, reinterpret_cast<const float4*>(gref), reinterpret_cast<const float4*>(gref2),      \
                     reinterpret_cast<float4*>(vbar), reinterpret_cast<float4*>(w), ref_out, c.d, c.words, c.M,  \
                     c.eps, inv_m, lr, c.means)
  if (big_tiles >= 2048) {
    if (stream_codes) {
      TNG_DECODE_LAUNCH(kDecodeLoads, true, big_tiles);
    } else {
      TNG_DECODE_LAUNCH(kDecodeLoads, false, big_tiles);
    }
  } else {  // few coordinates: small tiles so that every compute unit still gets work
    TNG_DECODE_LAUNCH(1, false, (nvec + kBlock - 1) / kBlock);
  }
#undef TNG_DECODE_LAUNCH
  return hipGetLastError();
}

}  // namespace

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t value, hipStream_t s) {
  if (n == 0) return hipSuccess;
  const uint32_t gx = div_up_u32(n, kBlock);
  hipLaunchKernelGGL(fill_u32_kernel, dim3(gx < 8192u ? gx : 8192u), dim3(kBlock), 0, s, p, n, value);
  return hipGetLastError();
}

hipError_t launch_copy_f32(float* dst, const float* src, uint64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (vec_ok(n, dst, src, nullptr)) {
    const uint32_t gx = div_up_u32(n / 4, (uint64_t)kBlock * kCopyPerThread);
    hipLaunchKernelGGL(copy_f32x4_kernel, dim3(gx < kMaxGridX ? gx : kMaxGridX), dim3(kBlock), 0, s,
                       reinterpret_cast<float4*>(dst), reinterpret_cast<const float4*>(src), n / 4);
  } else {
    const uint32_t gx = div_up_u32(n, kBlock);
    hipLaunchKernelGGL(copy_f32_kernel, dim3(gx < 16384u ? gx : 16384u), dim3(kBlock), 0, s, dst, src, n);
  }
  return hipGetLastError();
}

hipError_t launch_window_mean(const float* history, uint32_t window, uint32_t first, uint64_t d, float* out,
                              hipStream_t s) {
  if (vec_ok(d, history, out, nullptr)) {
    const uint32_t gx = div_up_u32(d / 4, kBlock);
    hipLaunchKernelGGL(window_mean_vec_kernel, dim3(gx < 16384u ? gx : 16384u), dim3(kBlock), 0, s,
                       reinterpret_cast<const float4*>(history), window, first, d / 4, 1.0f / (float)window,
                       reinterpret_cast<float4*>(out));
  } else {
    const uint32_t gx = div_up_u32(d, kBlock);
    hipLaunchKernelGGL(window_mean_kernel, dim3(gx < 16384u ? gx : 16384u), dim3(kBlock), 0, s, history, window, first,
                       d, 1.0f / (float)window, out);
  }
  return hipGetLastError();
}

hipError_t launch_rng_draws(uint32_t k0, uint32_t k1, uint32_t iter, uint32_t worker, uint32_t stream,
                            uint64_t first, uint64_t count, uint32_t* out, hipStream_t s) {
  if (count == 0) return hipSuccess;
  const uint32_t gx = div_up_u32(count, kBlock);
  hipLaunchKernelGGL(rng_draws_kernel, dim3(gx < 8192u ? gx : 8192u), dim3(kBlock), 0, s, k0, k1, iter,
                     worker, stream, first, count, out);
  return hipGetLastError();
}

hipError_t launch_absmax_finish(const float* partials, uint32_t nblocks, uint32_t M, float* scales, hipStream_t s) {
  const uint32_t threads = finish_threads(nblocks);
  hipLaunchKernelGGL((threads == kFinishLarge ? absmax_finish_kernel<kFinishLarge> : absmax_finish_kernel<kBlock>), dim3(M), dim3(threads), 0, s, partials,
                     nblocks, M, scales);
  return hipGetLastError();
}

hipError_t launch_absmax(const CodecShape& c, const float* g, const float* gref, const float* gref2,
                         float* partials, float* scales, uint32_t max_left, bool hold, uint32_t* left_rows,
                         hipStream_t s) {
  *left_rows = 0;
  switch (c.norm) {
    case kNormNone: return absmax_dispatch<kNormNone>(c, g, nullptr, nullptr, partials, scales, max_left, hold, left_rows, s);
    case kNormSub: return absmax_dispatch<kNormSub>(c, g, gref, nullptr, partials, scales, max_left, hold, left_rows, s);
    case kNormQuot: return absmax_dispatch<kNormQuot>(c, g, gref, nullptr, partials, scales, max_left, hold, left_rows, s);
    case kNormMean: return absmax_dispatch<kNormMean>(c, g, nullptr, nullptr, partials, scales, max_left, hold, left_rows, s);
    default: return absmax_dispatch<kNormComb>(c, g, gref, gref2, partials, scales, max_left, hold, left_rows, s);
  }
}

size_t tree_sum_scratch(uint64_t d, uint32_t M) {
  const uint64_t nchunks = (d + kTreeChunk - 1) / kTreeChunk;
  const uint64_t ngroups = (nchunks + kTreeGroup - 1) / kTreeGroup;
  // chunk sums, chunk (min, max) pairs; a word per group, unused (the group sums stay on chip), keeps the workspace's size
  return (size_t)((2 * nchunks + ngroups) * M);
}

namespace {
// The ragged last chunk of every row.
template <int NORM>
hipError_t l2_last_chunk_launch(const CodecShape& c, const float* g, const float* gref, const float* gref2, double* sums,
                                uint64_t whole, uint64_t nchunks, hipStream_t s) {
  auto kernel = c.d % 4 == 0 ? tree_chunk_kernel<NORM, true, true, false> : tree_chunk_kernel<NORM, true, false, false>;
  hipLaunchKernelGGL(kernel, dim3(1, c.M), dim3(kBlock), 0, s, g, gref, gref2, c.means, sums, nullptr, c.d, whole, nchunks,
                     nchunks, c.eps, c.M, 1u);
  return hipGetLastError();
}

// The row sums from the chunk sums.
template <bool MEAN>
hipError_t tree_finish_launch(const CodecShape& c, double* sums, const float2* minmax, uint64_t nchunks, uint64_t ngroups,
                              float* out, float* scales, hipStream_t s, const SlotVote& vote = {}) {
  auto kernel = ngroups == 1   ? tree_finish_kernel<MEAN, 1>
                : ngroups <= 16 ? tree_finish_kernel<MEAN, 16>
                                : tree_finish_kernel<MEAN, 64>;
  hipLaunchKernelGGL(kernel, dim3(c.M + (vote.use_slots != nullptr ? 1u : 0u)), dim3(kBlock), 0, s, sums, minmax, nchunks,
                     ngroups, c.d, c.M, out, scales, vote);
  return hipGetLastError();
}

template <int NORM, bool SQUARE, bool MINMAX>
hipError_t tree_sum_launch(const CodecShape& c, const float* g, const float* gref, const float* gref2, double* sums,
                           float* out, float* scales, hipStream_t s) {
  const uint64_t nchunks = (c.d + kTreeChunk - 1) / kTreeChunk;
  const uint64_t ngroups = (nchunks + kTreeGroup - 1) / kTreeGroup;
  float2* minmax = reinterpret_cast<float2*>(sums + nchunks * c.M);
  const uint32_t gx = (uint32_t)((nchunks + kWavesPerBlock - 1) / kWavesPerBlock);
  constexpr bool kSharedRef = NORM == kNormSub || NORM == kNormQuot || NORM == kNormComb;
  const uint64_t whole = c.d / kTreeChunk;  // chunks that lie inside the rows entirely
  if (SQUARE && kSharedRef && whole != 0 && aligned16_or_null(gref, gref2)) {
    const uint32_t gw = (uint32_t)((whole + kWavesPerBlock - 1) / kWavesPerBlock);
    int mc = 4;  // workers per workgroup that share the reference tile in registers
    while (mc > 1 && (uint64_t)gw * ((c.M + mc - 1) / mc) < 2048) mc >>= 1;
    const GradRows rows{g, c.d};
    const float4* r4 = reinterpret_cast<const float4*>(gref);
    const float4* r24 = reinterpret_cast<const float4*>(gref2);
    dim3 grid(gw, (c.M + mc - 1) / mc);
    if (mc == 4) {
      hipLaunchKernelGGL((l2_chunk_kernel<kSharedRef ? NORM : kNormSub, 4>), grid, dim3(kBlock), 0, s, rows, r4, r24, sums,
                         whole, nchunks, c.eps, c.M);
    } else if (mc == 2) {
      hipLaunchKernelGGL((l2_chunk_kernel<kSharedRef ? NORM : kNormSub, 2>), grid, dim3(kBlock), 0, s, rows, r4, r24, sums,
                         whole, nchunks, c.eps, c.M);
    } else {
      hipLaunchKernelGGL((l2_chunk_kernel<kSharedRef ? NORM : kNormSub, 1>), grid, dim3(kBlock), 0, s, rows, r4, r24, sums,
                         whole, nchunks, c.eps, c.M);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (whole < nchunks) {  // the ragged last chunk of every row
      e = l2_last_chunk_launch<NORM>(c, g, gref, gref2, sums, whole, nchunks, s);
      if (e != hipSuccess) return e;
    }
    return tree_finish_launch<false>(c, sums, nullptr, nchunks, ngroups, out, scales, s);
  }
  // workers per workgroup: as many as leave 2048 workgroups (only worth it when a reference is shared)
  uint32_t wpb = 1;
  if (SQUARE && gref != nullptr)
    while (wpb < 8 && wpb < c.M && (uint64_t)gx * ((c.M + 2 * wpb - 1) / (2 * wpb)) >= 2048) wpb *= 2;
  dim3 grid(gx, (c.M + wpb - 1) / wpb);
  if (aligned16_or_null(gref, gref2)) {
    // the last chunk of rows whose length is not a multiple of 4 goes element by element
    const uint64_t vec_end = c.d % 4 == 0 ? nchunks : whole;
    if (vec_end != 0)
      hipLaunchKernelGGL((tree_chunk_kernel<NORM, SQUARE, true, MINMAX>), grid, dim3(kBlock), 0, s, g, gref, gref2,
                         c.means, sums, minmax, c.d, (uint64_t)0, vec_end, nchunks, c.eps, c.M, wpb);
    if (vec_end != nchunks)
      hipLaunchKernelGGL((tree_chunk_kernel<NORM, SQUARE, false, MINMAX>), dim3(1, c.M), dim3(kBlock), 0, s, g, gref,
                         gref2, c.means, sums, minmax, c.d, vec_end, nchunks, nchunks, c.eps, c.M, 1u);
  } else {
    hipLaunchKernelGGL((tree_chunk_kernel<NORM, SQUARE, false, MINMAX>), grid, dim3(kBlock), 0, s, g, gref, gref2,
                       c.means, sums, minmax, c.d, (uint64_t)0, nchunks, nchunks, c.eps, c.M, wpb);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return tree_finish_launch<!SQUARE>(c, sums, MINMAX ? minmax : nullptr, nchunks, ngroups, out, scales, s);
}

template <int NORM>
hipError_t l2_candidates_launch(const CodecShape& c, uint32_t iter, const float* g, const float* gref, double* sums,
                                const CandidateScratch& cs, float* scales, hipStream_t s) {
  const uint64_t nchunks = (c.d + kTreeChunk - 1) / kTreeChunk, ngroups = (nchunks + kTreeGroup - 1) / kTreeGroup;
  const uint64_t whole = c.d / kTreeChunk;  // chunks that lie inside the rows entirely
  uint32_t nsample = 0;
  float sampled = 0.f;
  hipError_t e = sample_launch<NORM, true>(c, g, gref, cs, &nsample, &sampled, s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(sample_finish_kernel, dim3(c.M), dim3(kBlock), 0, s, cs.sample_partials, cs.sample_sums, nsample, c.M, sampled,
                     cs.sample_max, cs.select_ok, cs.overflowed);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 grid((uint32_t)whole, (c.M + kL2SelectWorkers - 1) / kL2SelectWorkers);
  hipLaunchKernelGGL(l2_select_kernel<NORM>, grid, dim3(kBlock), 0, s, GradRows{g, c.d},
                     reinterpret_cast<const float4*>(gref), sums, whole, nchunks, c.M, cs.sample_max, cs.select_ok, cs.slots,
                     l2_slot_counts(c, cs), cs.overflowed, c.k0, c.k1, iter);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (whole < nchunks) {
    e = l2_last_chunk_launch<NORM>(c, g, gref, nullptr, sums, whole, nchunks, s);
    if (e != hipSuccess) return e;
  }
  // (and, in one more workgroup of the same launch, the vote)
  return tree_finish_launch<false>(c, sums, nullptr, nchunks, ngroups, scales, nullptr, s,
                                   SlotVote{cs.overflowed, kL2OverflowCounts,
                                            (uint64_t)c.M * whole * (kTreeChunk / kWaveTileElements), cs.use_slots});
}
}  // namespace

hipError_t launch_worker_means(const CodecShape& c, const float* g, double* sums, float* means, float* scales,
                               hipStream_t s) {
  if (scales != nullptr) return tree_sum_launch<kNormNone, false, true>(c, g, nullptr, nullptr, sums, means, scales, s);
  return tree_sum_launch<kNormNone, false, false>(c, g, nullptr, nullptr, sums, means, nullptr, s);
}

hipError_t launch_l2_scales(const CodecShape& c, const float* g, const float* gref, const float* gref2, double* sums,
                            float* scales, hipStream_t s) {
  switch (c.norm) {
    case kNormNone: return tree_sum_launch<kNormNone, true, false>(c, g, nullptr, nullptr, sums, scales, nullptr, s);
    case kNormSub: return tree_sum_launch<kNormSub, true, false>(c, g, gref, nullptr, sums, scales, nullptr, s);
    case kNormQuot: return tree_sum_launch<kNormQuot, true, false>(c, g, gref, nullptr, sums, scales, nullptr, s);
    case kNormMean: return tree_sum_launch<kNormMean, true, false>(c, g, nullptr, nullptr, sums, scales, nullptr, s);
    default: return tree_sum_launch<kNormComb, true, false>(c, g, gref, gref2, sums, scales, nullptr, s);
  }
}

size_t candidate_scratch_bytes(const CodecShape& c) {
  // 2-bit codes, a shared reference or none, and enough
  // elements (2^26: 256 MiB of gradients) for the extra launches of the sample to be noise
  // (not the quotient forms: there |v| is near 1 everywhere and a third of the elements code non-zero)
  if (c.bits != 2 || (c.norm != kNormNone && c.norm != kNormSub)) return 0;
  // (the l2 scale: nor fewer workers than a workgroup has wavefronts)
  if (c.scale_l2 != 0 && c.M < (uint32_t)kWavesPerBlock) return 0;
  // (gradients as they are, rows of any length: Gaussian ones are too dense for the slots, which is found out too late to
  // cost nothing -- d = 2^25 + 4, M = 2 117 us by two passes, 136 this way; d = 80333292, M = 13 1528 / 1731)
  if (c.scale_l2 == 0 && c.norm == kNormNone && c.d % kWaveTileElements != 0) return 0;
  // (the slots are an eighth of the gradients: up to 4 GiB for rows of any length and for the l2 scale, so that what fits the
  // card by two passes still does)
  if ((c.scale_l2 != 0 || c.d % kWaveTileElements != 0) && (uint64_t)c.M * c.d > (1ull << 33)) return 0;
  if ((uint64_t)c.M * c.d < (1ull << 26) || c.d / 1024 < 4 * (uint64_t)kSampleStride) return 0;
  return candidate_head_bytes(c.M) + (size_t)c.M * (c.d / 1024) * kSlotEntries * sizeof(uint32_t);
}

bool candidates_apply(const CodecShape& c, const float* g, const float* gref, const float* gref2,
                      const uint32_t* codes) {
  return candidate_scratch_bytes(c) != 0 && aligned16_or_null(g, gref, gref2, codes);
}

hipError_t launch_absmax_candidates(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                                    const float* gref2, float* partials, void* scratch, float* scales, hipStream_t s) {
  const CandidateScratch cs = candidate_scratch(c, scratch);
  if (c.norm == kNormSub) return absmax_candidates_dispatch<kNormSub>(c, iter, g, gref, nullptr, partials, cs, scales, s);
  return absmax_candidates_dispatch<kNormNone>(c, iter, g, nullptr, nullptr, partials, cs, scales, s);
}

hipError_t launch_l2_candidates(const CodecShape& c, uint32_t iter, const float* g, const float* gref, double* sums,
                                void* scratch, float* scales, hipStream_t s) {
  const CandidateScratch cs = candidate_scratch(c, scratch);
  if (c.norm == kNormSub) return l2_candidates_launch<kNormSub>(c, iter, g, gref, sums, cs, scales, s);
  return l2_candidates_launch<kNormNone>(c, iter, g, nullptr, sums, cs, scales, s);
}

hipError_t launch_quantize_candidates(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                                      const float* gref2, const float* scales, void* scratch, uint32_t* codes,
                                      hipStream_t s) {
  const CandidateScratch cs = candidate_scratch(c, scratch);
  if (c.norm == kNormSub) return quantize_candidates_dispatch<kNormSub>(c, iter, g, gref, nullptr, scales, cs, codes, s);
  return quantize_candidates_dispatch<kNormNone>(c, iter, g, nullptr, nullptr, scales, cs, codes, s);
}

hipError_t launch_quantize_pack(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                                const float* gref2, float* scales, uint32_t* codes, const float* partials,
                                uint32_t fused_rows, hipStream_t s) {
#define TNG_Q(NORM, R1, R2)                                                                                      \
  return c.bits == 2 ? quantize_dispatch<NORM, 2>(c, iter, g, R1, R2, scales, codes, partials, fused_rows, s)    \
                     : quantize_dispatch<NORM, 4>(c, iter, g, R1, R2, scales, codes, partials, fused_rows, s)
  switch (c.norm) {
    case kNormNone: TNG_Q(kNormNone, nullptr, nullptr);
    case kNormSub: TNG_Q(kNormSub, gref, nullptr);
    case kNormQuot: TNG_Q(kNormQuot, gref, nullptr);
    case kNormMean: TNG_Q(kNormMean, nullptr, nullptr);
    default: TNG_Q(kNormComb, gref, gref2);
  }
#undef TNG_Q
}

uint32_t quantize_fused_rows(const CodecShape& c) { return fused_scale_rows(c); }

namespace {
// A workgroup per 256 coordinates with the workers dealt to its wavefronts, or a thread per float4 that walks the
// workers?  The first up to one wavefront of coordinates per SIMD (d = 2^18; iteration with given gradients, M = 16,
// 4-bit, quotient: 14.7 against 17.9 us), and from 17 workers on at any length, where the second has too few loads
// in flight (d = 2^22, M = 32: 218 against 235 us; d = 2^24, M = 64: 1673 against 1699); the second everywhere else
// (d = 2^20, M = 8: 24.5 against 28.0 us; d = 2^24, M = 8: 247 against 275).
inline bool tail_by_wavefronts(const CodecShape& c) { return c.d <= (1u << 18) || c.M > 16; }
template <int NORM, int BITS>
hipError_t quantize_decode_dispatch(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                                    const float* gref2, float* scales, uint32_t* codes, const float* partials,
                                    uint32_t rows, float* vbar, float* w, float lr, float* ref_out, hipStream_t s) {
  if (NORM == kNormMean && rows != 0) return hipErrorInvalidValue;  // (that scale comes with the mean, complete)
  if (tail_by_wavefronts(c)) {
    hipLaunchKernelGGL((quantize_decode_split_kernel<NORM, BITS>), dim3((uint32_t)((c.d + kBlock - 1) / kBlock)),
                       dim3(kBlock), 0, s, GradRows{g, c.d}, gref, gref2, scales, codes, c.d, c.words, c.M, c.eps, c.k0,
                       c.k1, iter, c.means, partials, rows, vbar, w, ref_out, 1.0f / (float)c.M, lr);
    return hipGetLastError();
  }
  const uint32_t blocks = (uint32_t)(((c.d + 3) / 4 + kBlock - 1) / kBlock);
  const uint32_t n = rows * c.M;
  auto kernel = quantize_decode_kernel<NORM, BITS, 0>;
  if constexpr (NORM != kNormMean) {
    if (n > kTailPartials || (rows != 0 && (n <= kTailFewPartials || (c.M & (c.M - 1)) != 0 || n % 4 != 0)))
      kernel = quantize_decode_kernel<NORM, BITS, kTailLate>;
    else if (n > kTailPartialsLong)
      kernel = quantize_decode_kernel<NORM, BITS, kTailPartials / (4 * kBlock)>;
    else if (rows != 0)
      kernel = quantize_decode_kernel<NORM, BITS, kTailPartialsLong / (4 * kBlock)>;
  }
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kBlock), 0, s, GradRows{g, c.d},
                     reinterpret_cast<const float4*>(gref), reinterpret_cast<const float4*>(gref2), scales, codes, c.d,
                     c.words, c.M, c.eps, c.k0, c.k1, iter, c.means, partials, rows, reinterpret_cast<float4*>(vbar),
                     reinterpret_cast<float4*>(w), ref_out, 1.0f / (float)c.M, lr);
  return hipGetLastError();
}
}  // namespace

// Where the one launch is faster than the separate ones: while launches set the time (d <= 2^18; 2^17 with more than 16
// workers that subtract no reference); never with more workers than its table holds; beyond, the
// thread per float4 needs three workers to have loads enough in flight (iteration with given gradients, no
// normalisation, d = 2^25, M = 1 144 us apart, 185 in one launch) and takes more than eight of them in trips that drain
// (d = 2^22, M = 16 115 / 123; d = 2^24, M = 12 364 / 330), and the workers by wavefront are ahead only where the
// reference is subtracted (d = 2^23, M = 20: 308 / 297; quotient 318 / 341).  Without a reference to read again it
// saves less behind a scale pass for the largest magnitude: d = 2^20, M = 4 14.8 / 13.0, M = 8 19.8 / 21.8; d = 2^21,
// M = 3 19.2 / 21.4, M = 8 33.3 / 35.2; d = 2^23, M = 4 75 / 76, M = 8 129 / 117; d = 2^24, M = 3 118 / 123; not where the
// gradient kernel left the maxima (Rosenbrock, d = 2^20, M = 8 30.9 / 25.9; d = 2^21, M = 4 32.7 / 29.0).
bool quantize_decode_applies(const CodecShape& c, bool maxima_left) {
  if (c.M > kTailMaxWorkers) return false;
  const bool small = c.d <= (1u << 20) && c.d * c.M <= (1u << 22);
  if (c.norm == kNormNone && c.scale_l2 == 0 && !maxima_left && !small && (c.M <= 4 || c.d < (1u << 22))) return false;
  if (c.M > 16) return c.norm == kNormSub ? c.d <= (1u << 18) || c.d >= (1u << 23) : c.d <= (1u << 17);
  if (c.M > 8) return c.d <= (1u << 20) || c.d >= (1u << 23);
  return c.M > 2 || c.d <= (1u << 20);
}

uint32_t quantize_decode_rows(const CodecShape& c) {
  return (c.d <= (1u << 20) ? kTailPartials : kTailPartialsLong) / c.M;
}

hipError_t launch_quantize_decode(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                                  const float* gref2, float* scales, uint32_t* codes, const float* partials,
                                  uint32_t rows, float* vbar, float* w, float lr, float* ref_out, hipStream_t s) {
  if (c.M > kTailMaxWorkers) return hipErrorInvalidValue;
  if (rows > quantize_decode_rows(c)) {
    const hipError_t e = launch_absmax_finish(partials, rows, c.M, scales, s);
    if (e != hipSuccess) return e;
    rows = 0;
  }
#define TNG_QD(NORM, R1, R2)                                                                                          \
  return c.bits == 2 ? quantize_decode_dispatch<NORM, 2>(c, iter, g, R1, R2, scales, codes, partials, rows, vbar, w,  \
                                                         lr, ref_out, s)                                              \
                     : quantize_decode_dispatch<NORM, 4>(c, iter, g, R1, R2, scales, codes, partials, rows, vbar, w,  \
                                                         lr, ref_out, s)
  switch (c.norm) {
    case kNormNone: TNG_QD(kNormNone, nullptr, nullptr);
    case kNormSub: TNG_QD(kNormSub, gref, nullptr);
    case kNormQuot: TNG_QD(kNormQuot, gref, nullptr);
    case kNormMean: TNG_QD(kNormMean, nullptr, nullptr);
    default: TNG_QD(kNormComb, gref, gref2);
  }
#undef TNG_QD
}

namespace {
template <int NORM, int BITS>
hipError_t single_pass_dispatch(const CodecShape& c, uint32_t iter, const float* g, const float* gref,
                                const float* gref2, float* scales, uint32_t* codes, float* vbar, float* w, float lr,
                                float* ref_out, hipStream_t s) {
#define TNG_SP(MC)                                                                                                  \
  hipLaunchKernelGGL((single_pass_kernel<NORM, BITS, MC>), dim3(1), dim3(kBlock), 0, s, GradRows{g, c.d},       \
                     reinterpret_cast<const float4*>(gref), reinterpret_cast<const float4*>(gref2), scales, codes,   \
                     c.d / 4, c.words, c.M, c.eps, c.k0, c.k1, iter, reinterpret_cast<float4*>(vbar),                \
                     reinterpret_cast<float4*>(w), reinterpret_cast<float4*>(ref_out), 1.0f / (float)c.M, lr)
  if (c.M <= 8)
    TNG_SP(8);
  else
    TNG_SP(16);
#undef TNG_SP
  return hipGetLastError();
}
}  // namespace

bool single_pass_applies(const CodecShape& c, const float* g, const float* gref, const float* gref2, const float* vbar,
                         const float* w, const float* ref_out) {
  return c.scale_l2 == 0 && c.norm != kNormMean && c.d % 4 == 0 && c.d <= 4 * (uint64_t)kBlock &&
         c.M <= (uint32_t)kSinglePassMaxWorkers && aligned16_or_null(g, gref, gref2) &&
         aligned16_or_null(vbar, w, ref_out);
}

hipError_t launch_single_pass(const CodecShape& c, uint32_t iter, const float* g, const float* gref, const float* gref2,
                              float* scales, uint32_t* codes, float* vbar, float* w, float lr, float* ref_out,
                              hipStream_t s) {
  if (!single_pass_applies(c, g, gref, gref2, vbar, w, ref_out)) return hipErrorInvalidValue;
#define TNG_SPD(NORM, R1, R2)                                                                                        \
  return c.bits == 2 ? single_pass_dispatch<NORM, 2>(c, iter, g, R1, R2, scales, codes, vbar, w, lr, ref_out, s) \
                     : single_pass_dispatch<NORM, 4>(c, iter, g, R1, R2, scales, codes, vbar, w, lr, ref_out, s)
  switch (c.norm) {
    case kNormNone: TNG_SPD(kNormNone, nullptr, nullptr);
    case kNormSub: TNG_SPD(kNormSub, gref, nullptr);
    case kNormQuot: TNG_SPD(kNormQuot, gref, nullptr);
    default: TNG_SPD(kNormComb, gref, gref2);
  }
#undef TNG_SPD
}

// Rows of one tile; longer rows while the workgroups, each of which reads its whole row, are one round of the compute units, up to
// 2^16 elements, half as many where each is divided by a reference.  Encode + decode, two passes against this one: d = 1000, M =
// 64 17.7 -> 14.5 us; d = 4096, M = 8 12.6 -> 10.0; d = 25000, M = 4, 4-bit 12.7 -> 10.2; d = 25001, M = 7, quotient 12.7 -> 10.1; d =
// 65536, M = 8 12.5 -> 10.3; d = 32768, M = 8, combined form 12.8 -> 11.0, M = 32 12.8 -> 12.5; beyond the line d = 65536, M = 32 (512
// workgroups) 13.4 -> 21.0, d = 131072, M = 8 12.7 -> 16.3.
// A workgroup costs the same however much of its tile the row fills (4.6 ns of the chip), so many rows have to fill it.  Encode of
// two bits / four with the quotient, two passes against this one: d = 4096, M = 2048 13.4 -> 10.9 / 18.0 -> 13.3, M = 16384 95.9 ->
// 82.6 / 110 -> 95.5; d = 1000, M = 1024 9.4 -> 7.0 / 10.1 -> 8.5; d = 4, M = 1024 8.8 -> 7.6 / 8.8 -> 9.0; beyond the line d = 4,
// M = 2048 9.7 -> 12.5 / 11.5 -> 15.3, M = 65535 118 -> 305 / 158 -> 383; d = 2048, M = 2048 9.9 -> 11.5 / 13.6 -> 13.8, M = 16384
// 58.7 -> 74.0 / 75.9 -> 93.5; d = 1000, M = 16384 72.2 -> 77.1 / 70.8 -> 96.9.
constexpr uint64_t kRowMax = 1u << 16;
constexpr uint64_t kRowGroups = 256;
constexpr uint32_t kRowFew = 1024;
bool encode_row_applies(const CodecShape& c) {
  if (c.norm == kNormMean || c.scale_l2) return false;
  if (c.d <= kRowTile) return c.M <= kRowFew || c.d > kRowTile / 4 * 3;
  const bool divides = c.norm == kNormQuot || c.norm == kNormComb;
  return c.d <= (divides ? kRowMax / 2 : kRowMax) && (c.d + kRowTile - 1) / kRowTile * c.M <= kRowGroups;
}

hipError_t launch_encode_row(const CodecShape& c, uint32_t iter, const float* g, const float* gref, const float* gref2,
                             float* scales, uint32_t* codes, hipStream_t s) {
  const dim3 grid((uint32_t)((c.d + kRowTile - 1) / kRowTile), c.M);
#define TNG_ROW(NORM)                                                                                                        \
  hipLaunchKernelGGL((c.bits == 2 ? encode_row_kernel<NORM, 2> : encode_row_kernel<NORM, 4>), grid, dim3(kRowThreads), 0, s, \
                     GradRows{g, c.d}, reinterpret_cast<const float4*>(gref), reinterpret_cast<const float4*>(gref2),        \
                     scales, codes, (uint32_t)c.d, (uint32_t)c.words, c.eps, c.k0, c.k1, iter)
  switch (c.norm) {
    case kNormNone: TNG_ROW(kNormNone); break;
    case kNormSub: TNG_ROW(kNormSub); break;
    case kNormQuot: TNG_ROW(kNormQuot); break;
    default: TNG_ROW(kNormComb); break;
  }
#undef TNG_ROW
  return hipGetLastError();
}

hipError_t launch_decode(const CodecShape& c, const uint32_t* codes, const float* scales, const float* gref,
                         const float* gref2, float* vbar, float* w, float lr, float* ref_out, hipStream_t s) {
#define TNG_D(NORM, R1, R2)                                                                          \
  return c.bits == 2 ? decode_dispatch<NORM, 2>(c, codes, scales, R1, R2, vbar, w, lr, ref_out, s)   \
                     : decode_dispatch<NORM, 4>(c, codes, scales, R1, R2, vbar, w, lr, ref_out, s)
  switch (c.norm) {
    case kNormNone: TNG_D(kNormNone, nullptr, nullptr);
    case kNormSub: TNG_D(kNormSub, gref, nullptr);
    case kNormQuot: TNG_D(kNormQuot, gref, nullptr);
    case kNormMean: TNG_D(kNormMean, nullptr, nullptr);
    default: TNG_D(kNormComb, gref, gref2);
  }
#undef TNG_D
}

}  // namespace tng
