// Stable LSD radix sort of (uint64 key, int32 value) pairs, 8-bit digits.
//
// Per pass: per-tile digit histograms (LDS atomics; counts are order-free), the
// offsets of every (digit, tile), and a stable scatter.  In the scatter a wave
// takes 64 kItems consecutive elements, ranks equal digits with 8 ballots (match
// mask) against its own running counts in LDS, and only then meets the
// workgroup's other waves: two barriers a tile, where ranking slab by slab
// across the workgroup took three for each of 16 slabs (302 us a pass at 16.8M
// elements, 13 us at 4096).  Up to kDirect tiles the scatter adds up the
// histograms itself, which saves the scan's launches.  Up to kSmall elements one
// workgroup sorts in LDS, all passes in one launch (the 24 launches of 4096
// elements took 165 us).
#include "device_math.h"
#include "internal.h"

namespace amfmm {
namespace {

constexpr int kBS = 256;
constexpr int kWaves = kBS / 64;
constexpr int kBins = 256;
constexpr int kDirect = 128;

// hist[digit * sd + tile * sb]
template <int kItems>
__global__ void __launch_bounds__(kBS) k_hist(const uint64_t* __restrict__ keys, int64_t n, int shift,
                                              int32_t* __restrict__ hist, int sd, int sb) {
  __shared__ int32_t h[kBins];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int64_t base = (int64_t)blockIdx.x * (kBS * kItems);
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t e = base + j * kBS + threadIdx.x;
    if (e < n) atomicAdd(&h[(keys[e] >> shift) & 0xFF], 1);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * sd + (int64_t)blockIdx.x * sb] = h[threadIdx.x];
}

// lanes of this wave with the same digit among the valid ones
__device__ inline uint64_t match_digit(int d, bool valid) {
  uint64_t mask = __ballot(valid);
#pragma unroll
  for (int b = 0; b < 8; ++b) {
    const bool bit = (d >> b) & 1;
    const uint64_t bb = __ballot(bit);
    mask &= bit ? bb : ~bb;
  }
  return mask;
}

// exclusive prefix over the first 256 threads' values (ws: a word per wave)
__device__ inline int32_t scan256(int32_t v, int32_t* ws) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int32_t inc = v;
#pragma unroll
  for (int d = 1; d < 64; d <<= 1) {
    const int32_t o = __shfl_up(inc, d, 64);
    if (lane >= d) inc += o;
  }
  if (w < 4 && lane == 63) ws[w] = inc;
  __syncthreads();
  int32_t off = 0;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    if (q < w) off += ws[q];
  return off + inc - v;
}

// DIRECT: hist holds the tiles' counts, tile-major, summed here; else their
// scanned offsets, digit-major
template <int kItems, bool DIRECT>
__global__ void __launch_bounds__(kBS) k_scatter(const uint64_t* __restrict__ kin, const int32_t* __restrict__ vin,
                                                 uint64_t* __restrict__ kout, int32_t* __restrict__ vout, int64_t n,
                                                 int shift, const int32_t* __restrict__ hist, int nblk) {
  __shared__ int32_t cnt[kWaves][kBins];
  __shared__ int32_t ws[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) cnt[q][tid] = 0;
  // where this tile's elements of digit tid go
  int32_t to;
  if (DIRECT) {
    int32_t all = 0, before = 0;
#pragma unroll 8
    for (int b = 0; b < nblk; ++b) {
      const int32_t v = hist[b * kBins + tid];
      all += v;
      before += b < (int)blockIdx.x ? v : 0;
    }
    to = scan256(all, ws) + before;
  } else {
    to = hist[(int64_t)tid * nblk + blockIdx.x];
  }
  __syncthreads();
  const uint64_t lt = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
  const int64_t base = (int64_t)blockIdx.x * (kBS * kItems) + w * (64 * kItems) + lane;
  uint64_t key[kItems];
  int32_t val[kItems], rank[kItems];
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const int64_t e = base + j * 64;
    key[j] = e < n ? kin[e] : 0;
    val[j] = e < n ? vin[e] : 0;
  }
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    const bool valid = base + j * 64 < n;
    const int d = (int)((key[j] >> shift) & 0xFF);
    const uint64_t m = match_digit(d, valid);
    const int below = __popcll(m & lt);
    // every lane reads before the first of a digit adds, and the next slab
    // reads after
    const int32_t run = cnt[w][d];
    rank[j] = run + below;
    wave_sync();
    if (valid && below == 0) cnt[w][d] = run + __popcll(m);
    wave_sync();
  }
  __syncthreads();
  {
    int32_t at = to;
#pragma unroll
    for (int q = 0; q < kWaves; ++q) {
      const int32_t v = cnt[q][tid];
      cnt[q][tid] = at;
      at += v;
    }
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < kItems; ++j) {
    if (base + j * 64 < n) {
      const int32_t dst = cnt[w][(key[j] >> shift) & 0xFF] + rank[j];
      kout[dst] = key[j];
      vout[dst] = val[j];
    }
  }
}

// One workgroup, everything in LDS: kSmallItems elements per thread in
// registers (wave w holds elements w 64 kSmallItems + 64 j + lane), written to
// their places in LDS and read back each pass.
constexpr int kSmallBS = 1024;
constexpr int kSmallWaves = kSmallBS / 64;
constexpr int kSmallItems = 8;
constexpr int kSmall = kSmallBS * kSmallItems;

__global__ void __launch_bounds__(kSmallBS) k_sort_small(uint64_t* __restrict__ keys, int32_t* __restrict__ vals, int n,
                                                         int passes) {
  __shared__ uint64_t sk[kSmall];
  __shared__ int32_t sv[kSmall];
  __shared__ int32_t cnt[kSmallWaves][kBins];
  __shared__ int32_t ws[kSmallWaves];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint64_t lt = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
  // waves share the elements evenly, in slabs of 64
  const int slabs = (n + 63) / 64, per = (slabs + kSmallWaves - 1) / kSmallWaves;
  const int base = w * per * 64 + lane;
  uint64_t key[kSmallItems];
  int32_t val[kSmallItems], rank[kSmallItems];
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const int e = base + j * 64;
    const bool valid = j < per && e < n;
    key[j] = valid ? keys[e] : 0;
    val[j] = valid ? vals[e] : 0;
  }
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
    for (int q = tid; q < kSmallWaves * kBins; q += kSmallBS) (&cnt[0][0])[q] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      if (j >= per) break;
      const bool valid = base + j * 64 < n;
      const int d = (int)((key[j] >> shift) & 0xFF);
      const uint64_t m = match_digit(d, valid);
      const int below = __popcll(m & lt);
      const int32_t run = cnt[w][d];
      rank[j] = run + below;
      wave_sync();
      if (valid && below == 0) cnt[w][d] = run + __popcll(m);
      wave_sync();
    }
    __syncthreads();
    int32_t all = 0;
    if (tid < kBins)
      for (int q = 0; q < kSmallWaves; ++q) all += cnt[q][tid];
    int32_t at = scan256(all, ws);
    if (tid < kBins)
      for (int q = 0; q < kSmallWaves; ++q) {
        const int32_t v = cnt[q][tid];
        cnt[q][tid] = at;
        at += v;
      }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      if (j < per && base + j * 64 < n) {
        const int32_t dst = cnt[w][(key[j] >> shift) & 0xFF] + rank[j];
        sk[dst] = key[j];
        sv[dst] = val[j];
      }
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kSmallItems; ++j) {
      const int e = base + j * 64;
      if (j < per && e < n) {
        key[j] = sk[e];
        val[j] = sv[e];
      }
    }
  }
#pragma unroll
  for (int j = 0; j < kSmallItems; ++j) {
    const int e = base + j * 64;
    if (j < per && e < n) {
      keys[e] = key[j];
      vals[e] = val[j];
    }
  }
}

template <int kItems>
void sort_passes(Ctx& c, uint64_t* ka, int32_t* va, uint64_t* kb, int32_t* vb, int64_t n, int passes) {
  const int nblk = (int)((n + kBS * kItems - 1) / (kBS * kItems));
  const int64_t nh = (int64_t)kBins * nblk;
  int32_t* hist = (int32_t*)ensure(c, c.hist, sizeof(int32_t) * (nh + 1));
  const bool direct = nblk <= kDirect;
  for (int p = 0; p < passes; ++p) {
    const int shift = 8 * p;
    hipLaunchKernelGGL(k_hist<kItems>, dim3(nblk), dim3(kBS), 0, c.stream, ka, n, shift, hist, direct ? 1 : nblk,
                       direct ? kBins : 1);
    if (!direct) scan_i32(c, hist, hist, nh);
    hipLaunchKernelGGL((direct ? k_scatter<kItems, true> : k_scatter<kItems, false>), dim3(nblk), dim3(kBS), 0,
                       c.stream, ka, va, kb, vb, n, shift, (const int32_t*)hist, nblk);
    AMFMM_HIP(hipGetLastError());
    std::swap(ka, kb);
    std::swap(va, vb);
  }
}

}  // namespace

void radix_sort(Ctx& c, uint64_t* keys, int32_t* vals, uint64_t* keys_alt, int32_t* vals_alt,
                int64_t n, int bits) {
  if (n <= 1) return;
  int passes = (bits + 7) / 8;
  if (passes & 1) ++passes;  // even count: result lands back in keys/vals
  if (n <= kSmall) {
    hipLaunchKernelGGL(k_sort_small, dim3(1), dim3(kSmallBS), 0, c.stream, keys, vals, (int)n, passes);
    AMFMM_HIP(hipGetLastError());
  } else if (n <= 4 * kBS * kDirect) {
    // tiles of 1024, as many as the scatter sums by itself
    sort_passes<4>(c, keys, vals, keys_alt, vals_alt, n, passes);
  } else {
    sort_passes<16>(c, keys, vals, keys_alt, vals_alt, n, passes);
  }
}

}  // namespace amfmm
