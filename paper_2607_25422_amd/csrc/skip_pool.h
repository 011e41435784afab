// Float64 means of row ranges of a [rows][d] matrix (internal to libskip.so):
// the mean-pooled question (paper Sec. 3.3, Def. B.2; Def. B.1 scoring
// vector) and the pooled passage keys (Def. B.3).
#pragma once

#include "skip_common.h"

namespace skip {

// Workgroup = (column slice of 64 lanes x CH x 16 bytes, range); wave w sums
// rows w, w+4, ... (Q rows, CH 16-byte chunks each, in flight per lane); the
// four partial sums are combined in wave order through LDS (CH and Q do not
// change the order of a column's sum).
// Questions are written as the scoring vector u = mean / sqrt(d) + w, passage
// keys as their mean.  The same workgroup body runs in the pooling launch and
// in the prune launch (passage keys beside the scoring).
constexpr int kPoolChunks = 2;      // beside the scoring: CH = 2, Q = 4
constexpr int kPoolRows = 4;

template <typename T>
struct PoolRanges {
  const T* src;
  const int32_t* offsets;
  int n;            // ranges
  int total;        // rows of src
  double* out;      // [n][d]
};

// Bytes of LDS one pooling workgroup uses (four waves' partial sums).
template <typename T>
constexpr size_t pool_lds_bytes(int chunks = kPoolChunks) {
  return 4 * 64 * chunks * Vec16<T>::n * sizeof(double);
}

// One pooling workgroup (256 threads): range j of rg, column slice `slice`;
// `question` ranges are written as the scoring vector (mean / sqrt(d) + w).
// part: pool_lds_bytes<T>(CH) of LDS.  Contains one __syncthreads().
template <typename T, int CH = kPoolChunks, int Q = kPoolRows>
__device__ __forceinline__ void pool_block(const PoolRanges<T>& rg, int j, int slice,
                                           bool question, const T* __restrict__ w, int d,
                                           double* part) {
  constexpr int VEC = Vec16<T>::n;
  const T* __restrict__ src = rg.src;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  int cc[CH];                            // first column of each chunk
  bool ok[CH];
#pragma unroll
  for (int h = 0; h < CH; ++h) {
    cc[h] = ((slice * CH + h) * 64 + lane) * VEC;
    ok[h] = cc[h] < d;
  }
  int t0, t1;
  range_of(rg.offsets, j, rg.total, t0, t1);
  double acc[CH][VEC];
#pragma unroll
  for (int h = 0; h < CH; ++h)
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc[h][e] = 0.0;
  int t = t0 + wave;
  for (; t + 4 * (Q - 1) < t1; t += 4 * Q) {
    u32x4 x[Q][CH];
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int h = 0; h < CH; ++h)
        x[q][h] = ok[h] ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(
                              src + (size_t)(t + 4 * q) * d + cc[h]))
                        : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        double v[VEC];
        unpack16_f64<T>(x[q][h], v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[h][e] += v[e];
      }
  }
  if constexpr (Q > kPoolRows) {
    if (t < t1) {
      // the wave's last rows (fewer than Q), in flight together (rows past
      // the range are read as its last row and not added)
      u32x4 x[Q - 1][CH];
#pragma unroll
      for (int q = 0; q < Q - 1; ++q)
#pragma unroll
        for (int h = 0; h < CH; ++h)
          x[q][h] = *reinterpret_cast<const u32x4*>(src + (size_t)min(t + 4 * q, t1 - 1) * d +
                                                    (ok[h] ? cc[h] : 0));
#pragma unroll
      for (int q = 0; q < Q - 1; ++q)
#pragma unroll
        for (int h = 0; h < CH; ++h) {
          double v[VEC];
          unpack16_f64<T>(t + 4 * q < t1 ? x[q][h] : u32x4{0u, 0u, 0u, 0u}, v);
#pragma unroll
          for (int e = 0; e < VEC; ++e) acc[h][e] += v[e];
        }
    }
  } else {
    // (beside the scoring the registers are the scoring's)
    for (; t < t1; t += 4) {
#pragma unroll
      for (int h = 0; h < CH; ++h) {
        if (!ok[h]) continue;
        u32x4 x = *reinterpret_cast<const u32x4*>(src + (size_t)t * d + cc[h]);
        double v[VEC];
        unpack16_f64<T>(x, v);
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc[h][e] += v[e];
      }
    }
  }
  // part[wave][lane][CH * VEC]
  double* mine = part + ((size_t)wave * 64 + lane) * (CH * VEC);
#pragma unroll
  for (int h = 0; h < CH; ++h)
#pragma unroll
    for (int e = 0; e < VEC; ++e) mine[h * VEC + e] = acc[h][e];
  __syncthreads();
  if (wave != 0) return;
  const int L = t1 - t0;
  const double rsd = 1.0 / sqrt((double)d);
  const size_t wstride = (size_t)64 * (CH * VEC);
#pragma unroll
  for (int h = 0; h < CH; ++h) {
    if (!ok[h]) continue;
    double wv[VEC];
    if (question && w) {
      unpack16_f64<T>(*reinterpret_cast<const u32x4*>(w + cc[h]), wv);
    } else {
#pragma unroll
      for (int e = 0; e < VEC; ++e) wv[e] = 0.0;
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const int i = h * VEC + e;
      const double s = ((mine[i] + mine[wstride + i]) + mine[2 * wstride + i]) +
                       mine[3 * wstride + i];
      double m = (L > 0) ? s / (double)L : 0.0;
      if (question) m = m * rsd + wv[e];
      rg.out[(size_t)j * d + cc[h] + e] = m;
    }
  }
}

// One launch serves two independent sets of ranges: the questions (ranges
// 0..nq-1 of Qtok, written as the scoring vector) and the passages (the
// following ranges of Kh, written as their mean).  counters (or NULL): the
// per-question completion counters of the scoring launch, cleared here.
template <typename T, int CH, int Q>
__global__ void __launch_bounds__(256)
pool_kernel(PoolRanges<T> qr, const T* __restrict__ w, PoolRanges<T> pr, int d,
            int32_t* __restrict__ counters) {
  __shared__ double part[4 * 64 * CH * Vec16<T>::n];
  const bool question = (int)blockIdx.y < qr.n;
  const int j = question ? (int)blockIdx.y : (int)blockIdx.y - qr.n;
  if (counters && question && blockIdx.x == 0 && threadIdx.x == 0) counters[j] = 0;
  pool_block<T, CH, Q>(question ? qr : pr, j, blockIdx.x, question, w, d, part);
}

// Few ranges (fewer than kPoolFew workgroups of the form beside the scoring):
// CH = 1, Q = 8, twice the workgroups and a question of up to 32 tokens in one
// round of loads, a latency each: 16 questions of 32 tokens, d = 4096, 8.2 ->
// 5.5 us; 19 tokens of d = 1024, 4.9 -> 3.2 us (its last rows came one after
// another); 45 passages of 37..301 tokens, d = 2048, and 6 questions, 15.6 ->
// 9.1 us each.  Many ranges are bound by HBM and keep the longer runs of a row:
// 160 passages of 256 tokens, d = 4096 (640 workgroups), 60 us against 70.
// Between 256 and 512 workgroups the first form wins by 0.77-0.98 over d = 256 ..
// 8192 and 4 .. 1024 rows, except on ranges that start 2 MiB apart and meet in
// the memory channels (256 rows of 8 KiB: 1.07-1.14 of a call that pools and
// scores) and on 4 rows of one slice (1.03-1.08).
constexpr long long kPoolFew = 512;

// Questions (Qtok by q_offsets -> u, nq ranges) and passages (Kh by
// passage_offsets -> kbar, np ranges); either set may be empty.
inline hipError_t launch_pools(int dtype, int d, const void* Qtok, const int32_t* q_offsets,
                               int nq, int total_qtok, const void* w, double* u,
                               const void* Kh, const int32_t* passage_offsets, int np,
                               int total_tokens, double* kbar, hipStream_t s,
                               int32_t* counters = nullptr) {
  if (nq + np <= 0) return hipSuccess;
  auto slices = [&](int chunks) {
    const int cols = 64 * chunks * (dtype == SKIP_F32 ? Vec16<float>::n : Vec16<bf16_t>::n);
    return (d + cols - 1) / cols;
  };
  auto go = [&](auto tag, auto kernel, int chunks) -> hipError_t {
    using T = decltype(tag);
    hipLaunchKernelGGL(kernel, dim3(slices(chunks), nq + np), dim3(256), 0, s,
                       PoolRanges<T>{(const T*)Qtok, q_offsets, nq, total_qtok, u}, (const T*)w,
                       PoolRanges<T>{(const T*)Kh, passage_offsets, np, total_tokens, kbar}, d,
                       counters);
    return hipGetLastError();
  };
  if ((long long)slices(kPoolChunks) * (nq + np) < kPoolFew)
    return dtype == SKIP_F32 ? go(float{}, pool_kernel<float, 1, 8>, 1)
                             : go(bf16_t{}, pool_kernel<bf16_t, 1, 8>, 1);
  return dtype == SKIP_F32
             ? go(float{}, pool_kernel<float, kPoolChunks, kPoolRows>, kPoolChunks)
             : go(bf16_t{}, pool_kernel<bf16_t, kPoolChunks, kPoolRows>, kPoolChunks);
}

}  // namespace skip
