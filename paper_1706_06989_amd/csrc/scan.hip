// Device-wide exclusive prefix sums of one or several arrays of one length, in
// one launch up to kChunk values and two beyond (block sums, then every block
// adds up the block sums before its own: at most a few hundred loads a thread
// at 10^8 values).  Launches are what bounds it at the walk's sizes (about 3 us
// each): a walk level scans six arrays at once, in 2 launches where it took 18.
// Deterministic: integer sums in a fixed order.  In place is allowed.
#include "internal.h"

namespace amfmm {
namespace {

constexpr int kBS = 256;  // threads per block (4 waves of 64)
constexpr int kIT = 8;    // consecutive items per thread
constexpr int kChunk = kBS * kIT;

template <typename T>
__device__ T wave_incl_scan(T v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    T o = __shfl_up(v, d, 64);
    if (lane >= d) v += o;
  }
  return v;
}

// exclusive scan of one value per thread across the block; block total in *tot
template <typename T>
__device__ T block_excl_scan(T v, T* tot) {
  __shared__ T wsum[kBS / 64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  T inc = wave_incl_scan(v);
  if (lane == 63) wsum[w] = inc;
  __syncthreads();
  T off = 0, all = 0;
#pragma unroll
  for (int i = 0; i < kBS / 64; ++i) {
    if (i < w) off += wsum[i];
    all += wsum[i];
  }
  __syncthreads();
  *tot = all;
  return off + inc - v;
}

// block sums of every array of the set (blockIdx.y)
template <typename T>
__global__ void __launch_bounds__(kBS) k_reduce(ScanSet<T> set, int64_t n, T* __restrict__ bsum,
                                                unsigned long long* clock) {
  take_time(clock);
  const T* __restrict__ in = set.in[blockIdx.y];
  const int64_t base = (int64_t)blockIdx.x * kChunk;
  T s = 0;
#pragma unroll
  for (int i = 0; i < kIT; ++i) {
    int64_t idx = base + i * kBS + threadIdx.x;
    if (idx < n) s += in[idx];
  }
  T tot;
  block_excl_scan(s, &tot);
  if (threadIdx.x == 0) bsum[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = tot;
}

// scans one chunk per block of every array of the set; the block's offset is
// the sum of the block sums before it; writes out[0..n) and out[n] = total
template <typename T>
__global__ void __launch_bounds__(kBS) k_scan_chunk(ScanSet<T> set, int64_t n, const T* __restrict__ bsum,
                                                    unsigned long long* clock) {
  take_time(clock);
  __shared__ T tile[kChunk];
  const T* in = set.in[blockIdx.y];
  T* out = set.out[blockIdx.y];
  const int64_t base = (int64_t)blockIdx.x * kChunk;
#pragma unroll
  for (int i = 0; i < kIT; ++i) {
    int64_t idx = base + i * kBS + threadIdx.x;
    tile[i * kBS + threadIdx.x] = idx < n ? in[idx] : T(0);
  }
  T before = 0;
  for (unsigned b = threadIdx.x; b < blockIdx.x; b += kBS) before += bsum[(int64_t)blockIdx.y * gridDim.x + b];
  T offset;
  block_excl_scan(before, &offset);
  __syncthreads();
  T v[kIT];
  T s = 0;
#pragma unroll
  for (int i = 0; i < kIT; ++i) {
    v[i] = tile[threadIdx.x * kIT + i];
    s += v[i];
  }
  T tot;
  T ex = block_excl_scan(s, &tot) + offset;
#pragma unroll
  for (int i = 0; i < kIT; ++i) {
    tile[threadIdx.x * kIT + i] = ex;
    if (base + threadIdx.x * kIT + i == n - 1) out[n] = ex + v[i];
    ex += v[i];
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kIT; ++i) {
    int64_t idx = base + i * kBS + threadIdx.x;
    if (idx < n) out[idx] = tile[i * kBS + threadIdx.x];
  }
}

template <typename T>
__global__ void k_zero_heads(ScanSet<T> set) {
  set.out[threadIdx.x][0] = 0;
}

template <typename T>
void scan_impl(Ctx& c, const ScanSet<T>& set, int count, int64_t n, unsigned long long* clock = nullptr) {
  if (n <= 0) {
    hipLaunchKernelGGL(k_zero_heads<T>, dim3(1), dim3(count), 0, c.stream, set);
    AMFMM_HIP(hipGetLastError());
    return;
  }
  const int64_t nb = (n + kChunk - 1) / kChunk;
  T* bsum = (T*)ensure(c, c.scratch, sizeof(T) * (size_t)(nb * count));
  const dim3 grid((unsigned)nb, (unsigned)count);
  if (nb > 1) hipLaunchKernelGGL(k_reduce<T>, grid, dim3(kBS), 0, c.stream, set, n, bsum, clock);
  hipLaunchKernelGGL(k_scan_chunk<T>, grid, dim3(kBS), 0, c.stream, set, n, (const T*)bsum,
                     nb > 1 ? nullptr : clock);
  AMFMM_HIP(hipGetLastError());
}

}  // namespace

void scan_i32(Ctx& c, const int32_t* in, int32_t* out, int64_t n) {
  scan_impl<int32_t>(c, ScanSet<int32_t>{{in}, {out}}, 1, n);
}
void scan_i64(Ctx& c, const ScanSet<int64_t>& set, int count, int64_t n, unsigned long long* clock) {
  scan_impl<int64_t>(c, set, count, n, clock);
}

}  // namespace amfmm
