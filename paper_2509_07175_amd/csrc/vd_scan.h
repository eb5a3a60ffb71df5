// vd_scan.h -- device-wide exclusive prefix sum (three launches, no host sync; up
// to kOne elements one launch, in which one block walks over them: 4.6 us at
// 4,000 and 14 us at 16,000 elements, against 8 us and two launches more; a clip
// has two lists scanned by one launch of two blocks).
//
// Tile = 1024 elements per 256-thread block.  Pass 1 scans each tile in LDS and
// writes the tile total; pass 2 scans the tile totals in one block (looping over
// chunks of 1024); pass 3 adds the tile offsets.  out[n] receives the grand
// total, so out has n+1 entries.  Used for counting-sort offsets and CSR
// offsets; it is bandwidth-bound and far from the hot path.
#pragma once
#include <hip/hip_runtime.h>

namespace vdscan {

constexpr int kThreads = 256;
constexpr int kTile = 1024;

template <typename TIn, typename TOut>
__global__ void __launch_bounds__(kThreads) tile_scan(const TIn *in, long long n, TOut *out,
                                                      TOut *tile_sum) {
  __shared__ TOut s[kTile];
  const long long base = (long long)blockIdx.x * kTile;
  for (int k = threadIdx.x; k < kTile; k += kThreads) {
    const long long i = base + k;
    s[k] = i < n ? (TOut)in[i] : (TOut)0;
  }
  __syncthreads();
  // each thread owns 4 consecutive elements
  TOut loc[4];
  TOut run = 0;
  for (int j = 0; j < 4; j++) { loc[j] = run; run += s[threadIdx.x * 4 + j]; }
  __syncthreads();
  __shared__ TOut t[kThreads];
  t[threadIdx.x] = run;
  __syncthreads();
  for (int d = 1; d < kThreads; d <<= 1) {
    TOut v = threadIdx.x >= (unsigned)d ? t[threadIdx.x - d] : (TOut)0;
    __syncthreads();
    t[threadIdx.x] += v;
    __syncthreads();
  }
  const TOut off = t[threadIdx.x] - run;
  for (int j = 0; j < 4; j++) {
    const long long i = base + threadIdx.x * 4 + j;
    if (i < n) out[i] = off + loc[j];
  }
  if (threadIdx.x == kThreads - 1) tile_sum[blockIdx.x] = t[kThreads - 1];
}

template <typename T>
__global__ void __launch_bounds__(kThreads) sums_scan(T *tile_sum, long long ntiles, T *total_out) {
  __shared__ T t[kThreads];
  T carry = 0;
  for (long long b = 0; b < ntiles; b += kThreads) {
    const long long i = b + threadIdx.x;
    const T v = i < ntiles ? tile_sum[i] : (T)0;
    t[threadIdx.x] = v;
    __syncthreads();
    for (int d = 1; d < kThreads; d <<= 1) {
      T u = threadIdx.x >= (unsigned)d ? t[threadIdx.x - d] : (T)0;
      __syncthreads();
      t[threadIdx.x] += u;
      __syncthreads();
    }
    if (i < ntiles) tile_sum[i] = carry + t[threadIdx.x] - v;
    const T last = t[kThreads - 1];
    __syncthreads();
    carry += last;
  }
  if (threadIdx.x == 0) *total_out = carry;
}

template <typename T>
__global__ void __launch_bounds__(kThreads) add_offsets(T *out, long long n, const T *tile_sum) {
  const long long base = (long long)blockIdx.x * kTile;
  const T off = tile_sum[blockIdx.x];
  for (int k = threadIdx.x; k < kTile; k += kThreads) {
    const long long i = base + k;
    if (i < n) out[i] += off;
  }
}

constexpr long long kOne = 16384;
constexpr int kOneThreads = 1024;

// One job of one_scan: out[0..n] from in[0..n); `zero` (nullable): n ints cleared.
template <typename TIn, typename TOut>
struct ScanJob {
  const TIn *in;
  TOut *out;
  int *zero;
};

// block b scans job b
template <typename TIn, typename TOut>
__global__ void __launch_bounds__(kOneThreads) one_scan(long long n, ScanJob<TIn, TOut> j0, ScanJob<TIn, TOut> j1) {
  const ScanJob<TIn, TOut> j = blockIdx.x ? j1 : j0;
  __shared__ TOut t[kOneThreads / 64];
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  TOut carry = 0;
  for (long long b = 0; b < n; b += 4 * kOneThreads) {
    const long long i = b + 4 * threadIdx.x;
    TOut v[4], run = 0;
    for (int k = 0; k < 4; k++) {
      v[k] = run;
      run += i + k < n ? (TOut)j.in[i + k] : (TOut)0;
    }
    TOut inc = run;
    for (int d = 1; d < 64; d <<= 1) {
      const TOut u = __shfl_up(inc, d, 64);
      inc += l >= d ? u : (TOut)0;
    }
    if (l == 63) t[w] = inc;
    __syncthreads();
    TOut off = carry, all = 0;
    for (int k = 0; k < kOneThreads / 64; k++) {
      off += k < w ? t[k] : (TOut)0;
      all += t[k];
    }
    for (int k = 0; k < 4; k++)
      if (i + k < n) {
        j.out[i + k] = off + inc - run + v[k];
        if (j.zero) j.zero[i + k] = 0;
      }
    carry += all;
    __syncthreads();
  }
  if (threadIdx.x == 0) j.out[n] = carry;
}

inline long long tiles(long long n) { return (n + kTile - 1) / kTile; }

// out[0..n] = exclusive scan of in[0..n), out[n] = total.
// tmp must hold tiles(n) elements of TOut.
template <typename TIn, typename TOut>
inline void exclusive_scan(const TIn *in, long long n, TOut *out, TOut *tmp, hipStream_t st) {
  if (n <= kOne) {
    const ScanJob<TIn, TOut> j{in, out, nullptr};
    hipLaunchKernelGGL((one_scan<TIn, TOut>), dim3(1), dim3(kOneThreads), 0, st, n, j, j);
    return;
  }
  const long long nt = tiles(n) > 0 ? tiles(n) : 1;
  hipLaunchKernelGGL((tile_scan<TIn, TOut>), dim3((unsigned)nt), dim3(kThreads), 0, st, in, n, out, tmp);
  hipLaunchKernelGGL((sums_scan<TOut>), dim3(1), dim3(kThreads), 0, st, tmp, nt, out + n);
  hipLaunchKernelGGL((add_offsets<TOut>), dim3((unsigned)nt), dim3(kThreads), 0, st, out, n, tmp);
}

}  // namespace vdscan
