// Octree build (Sec. 2): validation + bounding cube, Morton keys, stable sort,
// gather into sorted double4 particles, and the cells of all levels at once.
//
// Cells are numbered in (level, first particle) order: cells of one level are
// contiguous and sorted by their key prefix, children of a cell are
// contiguous and in octant order.  A cell splits into its non-empty octants
// iff it holds more than n_crit particles and sits above level 21.
//
// Compiled with -ffp-contract=off: the key arithmetic must round exactly as
// written so that keys (and hence the tree) are reproducible bit for bit.
#include "internal.h"

namespace amfmm {
namespace {

constexpr int kBS = 256;
constexpr int kBBoxBlocks = 1024;

__device__ inline bool finite(double v) { return __builtin_isfinite(v); }

// Per block: min of (x, y, z, -x, -y, -z) over the finite particles and, in
// the last two of its eight words, whether it met a non-finite value or a
// mass that is not positive (one pass over the inputs for both).
__global__ void __launch_bounds__(kBS) k_bbox_partial(const double* __restrict__ x, const double* __restrict__ y,
                                                      const double* __restrict__ z, const double* __restrict__ m,
                                                      int64_t n, double* __restrict__ part,
                                                      unsigned long long* clock) {
  take_time(clock);
  double v6[6] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY};
  int bad = 0, badm = 0;
  for (int64_t i = (int64_t)blockIdx.x * kBS + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBS) {
    const double v[3] = {x[i], y[i], z[i]}, mi = m[i];
    if (!(finite(v[0]) && finite(v[1]) && finite(v[2]) && finite(mi))) {
      bad = 1;
      continue;
    }
    if (!(mi > 0.0)) badm = 1;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
      v6[d] = fmin(v6[d], v[d]);
      v6[3 + d] = fmin(v6[3 + d], -v[d]);
    }
  }
  __shared__ double s[6][kBS];
  for (int q = 0; q < 6; ++q) s[q][threadIdx.x] = v6[q];
  const int anyb = __syncthreads_or(bad), anym = __syncthreads_or(badm);
  for (int w = kBS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w)
      for (int q = 0; q < 6; ++q) s[q][threadIdx.x] = fmin(s[q][threadIdx.x], s[q][threadIdx.x + w]);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double* o = part + (int64_t)blockIdx.x * 8;
    for (int q = 0; q < 6; ++q) o[q] = s[q][0];
    o[6] = anyb ? 1.0 : 0.0;
    o[7] = anym ? 1.0 : 0.0;
  }
}

// the box on the device, and box and flags in the host's words (pinned)
__global__ void __launch_bounds__(kBS) k_bbox_final(const double* __restrict__ part, int nb, double* __restrict__ box,
                                                    double* __restrict__ host) {
  __shared__ double s[8][kBS];
  double v[8] = {INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, INFINITY, 0.0, 0.0};
  for (int b = threadIdx.x; b < nb; b += kBS) {
    for (int q = 0; q < 6; ++q) v[q] = fmin(v[q], part[(int64_t)b * 8 + q]);
    for (int q = 6; q < 8; ++q) v[q] = fmax(v[q], part[(int64_t)b * 8 + q]);
  }
  for (int q = 0; q < 8; ++q) s[q][threadIdx.x] = v[q];
  __syncthreads();
  for (int w = kBS / 2; w > 0; w >>= 1) {
    if ((int)threadIdx.x < w) {
      for (int q = 0; q < 6; ++q) s[q][threadIdx.x] = fmin(s[q][threadIdx.x], s[q][threadIdx.x + w]);
      for (int q = 6; q < 8; ++q) s[q][threadIdx.x] = fmax(s[q][threadIdx.x], s[q][threadIdx.x + w]);
    }
    __syncthreads();
  }
  if (threadIdx.x < 8) {
    const double r = threadIdx.x < 3 || threadIdx.x > 5 ? s[threadIdx.x][0] : -s[threadIdx.x][0];
    box[threadIdx.x] = r;
    host[threadIdx.x] = r;
  }
}

// spread the low 21 bits of v so that bit b lands on bit 3b
__device__ inline uint64_t spread3(uint64_t v) {
  v &= 0x1fffffull;
  v = (v | (v << 32)) & 0x1f00000000ffffull;
  v = (v | (v << 16)) & 0x1f0000ff0000ffull;
  v = (v | (v << 8)) & 0x100f00f00f00f00full;
  v = (v | (v << 4)) & 0x10c30c30c30c30c3ull;
  v = (v | (v << 2)) & 0x1249249249249249ull;
  return v;
}

__global__ void __launch_bounds__(kBS) k_keys(const double* __restrict__ x, const double* __restrict__ y,
                                              const double* __restrict__ z, int64_t n, const double* __restrict__ box,
                                              uint64_t* __restrict__ keys, int32_t* __restrict__ idx,
                                              unsigned long long* clock) {
  take_time(clock);
  int64_t i = (int64_t)blockIdx.x * kBS + threadIdx.x;
  if (i >= n) return;
  const double lo[3] = {box[0], box[1], box[2]};
  double side = 0.0;
  for (int d = 0; d < 3; ++d) side = fmax(side, box[3 + d] - lo[d]);
  if (side == 0.0) side = 1.0;
  const double scale = (double)(1ull << kMaxLevel) / side;
  const uint64_t qmax = (1ull << kMaxLevel) - 1;
  const double v[3] = {x[i], y[i], z[i]};
  uint64_t q[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    double f = floor((v[d] - lo[d]) * scale);
    uint64_t qi = f <= 0.0 ? 0ull : (uint64_t)f;
    q[d] = qi > qmax ? qmax : qi;
  }
  keys[i] = (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
  idx[i] = (int32_t)i;
}

__global__ void __launch_bounds__(kBS) k_gather(const double* __restrict__ x, const double* __restrict__ y,
                                                const double* __restrict__ z, const double* __restrict__ m,
                                                int64_t n, const int32_t* __restrict__ perm, double4* __restrict__ pos) {
  int64_t s = (int64_t)blockIdx.x * kBS + threadIdx.x;
  if (s >= n) return;
  int32_t i = perm[s];
  pos[s] = make_double4(x[i], y[i], z[i], m[i]);
}

// Cells from the sorted keys, all levels at once.  Two particles share their
// cells down to level shared(k, k'), the number of leading octant digits their
// keys have in common.  A cell of level l holds more than n_crit particles iff
// n_crit + 1 consecutive particles inside it share level l, so the leaf level
// of particle i is 1 + the largest shared(key[j], key[j + n_crit]) over the
// windows [j, j + n_crit] that contain i (0 without any, at most kMaxLevel).
// The cells that start at particle i are those of levels c + 1 .. leaf(i),
// c = shared(key[i-1], key[i]), and a cell's rank in its level is the number
// of particles before i that start one there: per-tile counts of every level,
// one scan, and an emitting pass that ranks inside the tile with ballots.
// What bounds it is launches and read-backs, not bytes (2 B written, 10 B read
// a particle): the level-by-level build it replaces took two kernels, a scan
// and a read-back per level (1.2 ms at 4.2M particles and 12 levels; 0.21 ms
// at 4096 and 4 levels).
constexpr int kTile = 1024;       // particles (and threads) per block
constexpr int kTW = kTile / 64;   // waves per block
constexpr int kLev = kMaxLevel + 1;

__device__ inline int shared_levels(uint64_t a, uint64_t b) {
  const uint64_t x = a ^ b;
  return x == 0 ? kMaxLevel : (kMaxLevel - 1) - (63 - __builtin_clzll(x)) / 3;
}

// info[i] = (c + 1) | leaf level << 8; hist[(2 l) * nblk + blk] the internal
// cells of level l that start in the tile, hist[(2 l + 1) * nblk + blk] the leaves
__global__ void __launch_bounds__(kTile) k_tree_levels(const uint64_t* __restrict__ keys, int32_t n, int n_crit,
                                                       uint16_t* __restrict__ info, int32_t* __restrict__ hist,
                                                       int nblk, unsigned long long* clock) {
  take_time(clock);
  // windows' levels + 1 of particles [tile - n_crit, tile + kTile) (0: none),
  // then their running maxima; n_crit is at most 4096
  __shared__ uint8_t w[2][kTile + 4096];
  __shared__ int32_t cnt[2 * kLev];
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t base = (int64_t)blockIdx.x * kTile;
  const int len = kTile + n_crit;
  if (tid < 2 * kLev) cnt[tid] = 0;
  for (int t = tid; t < len; t += kTile) {
    const int64_t j = base - n_crit + t;
    w[0][t] = j >= 0 && j + n_crit < n ? (uint8_t)(shared_levels(keys[j], keys[j + n_crit]) + 1) : (uint8_t)0;
  }
  __syncthreads();
  // w[cur][t] becomes the maximum over [t - span + 1, t]
  int cur = 0, span = 1;
  for (; 2 * span <= n_crit + 1; span *= 2, cur ^= 1) {
    for (int t = tid; t < len; t += kTile) {
      const uint8_t a = w[cur][t], b = t >= span ? w[cur][t - span] : (uint8_t)0;
      w[cur ^ 1][t] = a > b ? a : b;
    }
    __syncthreads();
  }
  const int64_t i = base + tid;
  const bool valid = i < n;
  const int t = tid + n_crit;
  const uint8_t wa = w[cur][t], wb = w[cur][t - (n_crit + 1 - span)];
  const int leaf = min(kMaxLevel, (int)(wa > wb ? wa : wb));
  const int c = valid && i > 0 ? shared_levels(keys[i - 1], keys[i]) : -1;
  if (valid) info[i] = (uint16_t)((c + 1) | (leaf << 8));
  for (int l = 0; l < kLev; ++l) {
    const uint64_t bi = __ballot(valid && c < l && l < leaf), bl = __ballot(valid && c < l && l == leaf);
    if (lane == 0 && bi) atomicAdd(&cnt[2 * l], __popcll(bi));
    if (lane == 0 && bl) atomicAdd(&cnt[2 * l + 1], __popcll(bl));
  }
  __syncthreads();
  if (tid < 2 * kLev) hist[(int64_t)tid * nblk + blockIdx.x] = cnt[tid];
}

// one block per row of hist: its exclusive prefix sums in place, the total in
// tot[row] and in the host's word
__global__ void __launch_bounds__(kTile) k_tree_scan(int32_t* __restrict__ hist, int nblk, int32_t* __restrict__ tot,
                                                     int64_t* __restrict__ host) {
  __shared__ int32_t ws[kTW];
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int32_t* row = hist + (int64_t)blockIdx.x * nblk;
  int32_t carry = 0;
  for (int b = 0; b < nblk; b += kTile) {
    const int32_t v = b + tid < nblk ? row[b + tid] : 0;
    int32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int32_t o = __shfl_up(inc, d, 64);
      if (lane >= d) inc += o;
    }
    if (lane == 63) ws[wv] = inc;
    __syncthreads();
    int32_t off = carry, all = 0;
#pragma unroll
    for (int q = 0; q < kTW; ++q) {
      if (q < wv) off += ws[q];
      all += ws[q];
    }
    __syncthreads();
    if (b + tid < nblk) row[b + tid] = off + inc - v;
    carry += all;
  }
  if (tid == 0) {
    tot[blockIdx.x] = carry;
    host[blockIdx.x] = carry;
  }
}

__global__ void __launch_bounds__(kTile) k_tree_emit(int32_t n, const uint16_t* __restrict__ info,
                                                     const int32_t* __restrict__ hist, int nblk,
                                                     const int32_t* __restrict__ tot, int32_t* __restrict__ beg,
                                                     int32_t* __restrict__ par, int32_t* __restrict__ ch0,
                                                     int32_t* __restrict__ nch, int8_t* __restrict__ lev,
                                                     int32_t* __restrict__ leaves, int32_t* __restrict__ leafof) {
  __shared__ int32_t pc[kLev][kTW], pl[kLev][kTW];  // starts per wave: cells, leaves; then their prefixes
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  const uint64_t lt = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
  const int64_t i = (int64_t)blockIdx.x * kTile + tid;
  const bool valid = i < n;
  const int v = valid ? info[i] : 0;
  const int c = (v & 0xff) - 1, leaf = v >> 8;
  for (int l = 0; l < kLev; ++l) {
    const uint64_t bc = __ballot(valid && c < l && l <= leaf), bl = __ballot(valid && c < l && l == leaf);
    if (lane == 0) {
      pc[l][wv] = __popcll(bc);
      pl[l][wv] = __popcll(bl);
    }
  }
  __syncthreads();
  if (tid < kLev) {
    // first cell and leaf of this tile on level tid, then wave by wave
    int32_t sc = 0, sl = 0;
    for (int l = 0; l < tid; ++l) {
      sc += tot[2 * l] + tot[2 * l + 1];
      sl += tot[2 * l + 1];
    }
    const int32_t hi = hist[(int64_t)(2 * tid) * nblk + blockIdx.x], hl = hist[(int64_t)(2 * tid + 1) * nblk + blockIdx.x];
    sc += hi + hl;
    sl += hl;
    for (int q = 0; q < kTW; ++q) {
      const int32_t a = pc[tid][q], b = pl[tid][q];
      pc[tid][q] = sc;
      pl[tid][q] = sl;
      sc += a;
      sl += b;
    }
  }
  __syncthreads();
  // R: cells of level l that start before particle i (its own cell's index
  // when it starts one); a cell that starts inside its parent finds it as the
  // last one that started before i
  int32_t prev = 0;
  bool prev_starts = false;
  for (int l = 0; l < kLev; ++l) {
    if (!__ballot(valid && ((l >= c && l <= leaf) || l == leaf))) continue;  // no lane on this level
    const bool starts = valid && c < l && l <= leaf;
    const uint64_t bc = __ballot(starts), bl = __ballot(starts && l == leaf);
    const int32_t R = pc[l][wv] + __popcll(bc & lt);
    if (starts) {
      beg[R] = (int32_t)i;
      lev[R] = (int8_t)l;
      par[R] = l == 0 ? -1 : (prev_starts ? prev : prev - 1);
      if (prev_starts) ch0[prev] = R;
      if (l == leaf) {
        ch0[R] = -1;
        nch[R] = 0;
        leaves[pl[l][wv] + __popcll(bl & lt)] = R;
      }
    }
    if (valid && l == leaf) leafof[i] = starts ? R : R - 1;
    prev = R;
    prev_starts = starts;
  }
}

// particle and child counts: siblings are contiguous and tile their parent,
// so a cell ends where its next sibling begins, or with its parent
__global__ void __launch_bounds__(kBS) k_tree_counts(int32_t nc, int32_t n, const int32_t* __restrict__ beg,
                                                     const int32_t* __restrict__ par, const int32_t* __restrict__ ch0,
                                                     int32_t* __restrict__ cnt, int32_t* __restrict__ nch) {
  const int32_t c = blockIdx.x * kBS + threadIdx.x;
  if (c >= nc) return;
  int32_t a = c, end = n;
  while (a > 0) {
    const int32_t p = par[a];
    if (a + 1 < nc && par[a + 1] == p) {
      end = beg[a + 1];
      break;
    }
    a = p;
  }
  cnt[c] = end - beg[c];
  int32_t q = ch0[c];
  if (q >= 0) {
    int32_t k = 1;
    while (q + k < nc && par[q + k] == c) ++k;
    nch[c] = k;
  }
}

}  // namespace

void bbox_start(Ctx& c, const double* x, const double* y, const double* z, const double* m, int64_t n) {
  int nb = (int)std::min<int64_t>(kBBoxBlocks, (n + kBS - 1) / kBS);
  double* part = (double*)ensure(c, c.scratch2, sizeof(double) * 8 * (size_t)nb);
  double* box = (double*)ensure(c, c.bbox, sizeof(double) * 8);
  hipLaunchKernelGGL(k_bbox_partial, dim3(nb), dim3(kBS), 0, c.stream, x, y, z, m, n, part,
                     clock_word(c));
  hipLaunchKernelGGL(k_bbox_final, dim3(1), dim3(kBS), 0, c.stream, (const double*)part, nb, box,
                     (double*)(c.pinned + kPinBox));
  AMFMM_HIP(hipGetLastError());
}

void build_keys_sort(Ctx& c, const double* x, const double* y, const double* z, const double* m,
                     int64_t n) {
  uint64_t* keys = (uint64_t*)ensure(c, c.keys, sizeof(uint64_t) * n);
  int32_t* perm = (int32_t*)ensure(c, c.perm, sizeof(int32_t) * n);
  uint64_t* k2 = (uint64_t*)ensure(c, c.keys2, sizeof(uint64_t) * n);
  int32_t* p2 = (int32_t*)ensure(c, c.perm2, sizeof(int32_t) * n);
  double4* pos = (double4*)ensure(c, c.pos4, sizeof(double4) * n);
  hipLaunchKernelGGL(k_keys, dim3(blocks_for(n, kBS)), dim3(kBS), 0, c.stream, x, y, z, n,
                     (const double*)c.bbox.p, keys, perm, clock_word(c));
  AMFMM_HIP(hipGetLastError());
  radix_sort(c, keys, perm, k2, p2, n, 3 * kMaxLevel);
  hipLaunchKernelGGL(k_gather, dim3(blocks_for(n, kBS)), dim3(kBS), 0, c.stream, x, y, z, m, n,
                     perm, pos);
  AMFMM_HIP(hipGetLastError());
  c.n = n;
}

int input_status(Ctx& c) {
  sync(c);
  const double* box = (const double*)(c.pinned + kPinBox);
  return box[6] != 0.0 ? AMFMM_E_NONFINITE : (box[7] != 0.0 ? AMFMM_E_INVALID : AMFMM_OK);
}

int build_levels(Ctx& c) {
  const int32_t n = (int32_t)c.n;
  const int nblk = (int)blocks_for(n, kTile);
  const size_t rows = 2 * kLev;
  int32_t* hist = (int32_t*)ensure(c, c.scratch2, sizeof(int32_t) * (rows * nblk + rows) + sizeof(uint16_t) * (size_t)n);
  int32_t* tot = hist + rows * nblk;
  uint16_t* info = (uint16_t*)(tot + rows);
  int64_t* host = c.pinned + kPinTree;
  hipLaunchKernelGGL(k_tree_levels, dim3(nblk), dim3(kTile), 0, c.stream, (const uint64_t*)c.keys.p, n, c.opt.n_crit,
                     info, hist, nblk, clock_word(c));
  hipLaunchKernelGGL(k_tree_scan, dim3((unsigned)rows), dim3(kTile), 0, c.stream, hist, nblk, tot, host);
  AMFMM_HIP(hipGetLastError());
  const int st = input_status(c);
  if (st != AMFMM_OK) return st;
  const double* box = (const double*)(c.pinned + kPinBox);
  std::copy(box, box + 6, c.box);
  c.level_start.assign(1, 0);
  int32_t nc = 0, nleaves = 0;
  for (int l = 0; l < kLev && host[2 * l] + host[2 * l + 1] > 0; ++l) {
    nc += (int32_t)(host[2 * l] + host[2 * l + 1]);
    nleaves += (int32_t)host[2 * l + 1];
    c.level_start.push_back(nc);
  }
  int32_t* beg = (int32_t*)ensure(c, c.c_begin, sizeof(int32_t) * (size_t)nc);
  int32_t* cnt = (int32_t*)ensure(c, c.c_count, sizeof(int32_t) * (size_t)nc);
  int32_t* par = (int32_t*)ensure(c, c.c_parent, sizeof(int32_t) * (size_t)nc);
  int32_t* ch0 = (int32_t*)ensure(c, c.c_child0, sizeof(int32_t) * (size_t)nc);
  int32_t* nch = (int32_t*)ensure(c, c.c_nchild, sizeof(int32_t) * (size_t)nc);
  int8_t* lev = (int8_t*)ensure(c, c.c_level, (size_t)nc);
  int32_t* leaves = (int32_t*)ensure(c, c.leaves, sizeof(int32_t) * (size_t)nleaves);
  int32_t* leafof = (int32_t*)ensure(c, c.leafof, sizeof(int32_t) * (size_t)n);
  hipLaunchKernelGGL(k_tree_emit, dim3(nblk), dim3(kTile), 0, c.stream, n, (const uint16_t*)info, (const int32_t*)hist,
                     nblk, (const int32_t*)tot, beg, par, ch0, nch, lev, leaves, leafof);
  hipLaunchKernelGGL(k_tree_counts, dim3(blocks_for(nc, kBS)), dim3(kBS), 0, c.stream, nc, n, (const int32_t*)beg,
                     (const int32_t*)par, (const int32_t*)ch0, cnt, nch);
  AMFMM_HIP(hipGetLastError());
  c.ncells = nc;
  c.depth = (int32_t)c.level_start.size() - 2;
  c.nleaves = nleaves;
  return AMFMM_OK;
}

}  // namespace amfmm
