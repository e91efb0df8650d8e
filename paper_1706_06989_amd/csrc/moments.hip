// Upward pass (Sec. 2): mass M (eq. 1), centre of mass Z, quadrupole M_ij
// (eq. quad) and octupole M_ijk about Z, and R_max.
//
//  * leaves: one thread per leaf, sequential over its particles in key order;
//  * parents: 8 lanes per cell, level by level, summing the children in
//    octant order (mass and first moment), then shifting the children's M_ij,
//    M_ijk to the parent's centre (exact for moments about a centre of mass);
//  * R_max: exact largest distance to Z over the cell's particles; every
//    particle visits its ancestors level by level, lanes holding the same
//    ancestor reduce within the wave first, and a wave carries the run at
//    the end of one 64-particle slab into the next before its atomic max.
//
// Compiled with -ffp-contract=off: the centres of mass and R_max must round
// exactly as written (they decide the walk, which is reproduced bit for bit).
#include "internal.h"

namespace amfmm {
namespace {

constexpr int kBS = 256;

// packed mom layout: [0]=M, [1..6]=M_ij (xx xy xz yy yz zz), [7..16]=M_ijk
// (xxx xxy xxz xyy xyz xzz yyy yyz yzz zzz), [17] pad
__device__ inline void add_about(double* M2, double* M3, double mu, double x, double y, double z) {
  // mu x_i x_j and mu x_i x_j x_k, multiplied left to right
  double mx = mu * x, my = mu * y, mz = mu * z;
  M2[0] += mx * x;
  M2[1] += mx * y;
  M2[2] += mx * z;
  M2[3] += my * y;
  M2[4] += my * z;
  M2[5] += mz * z;
  M3[0] += mx * x * x;
  M3[1] += mx * x * y;
  M3[2] += mx * x * z;
  M3[3] += mx * y * y;
  M3[4] += mx * y * z;
  M3[5] += mx * z * z;
  M3[6] += my * y * y;
  M3[7] += my * y * z;
  M3[8] += my * z * z;
  M3[9] += mz * z * z;
}

__global__ void __launch_bounds__(kBS) k_leaf_moments(const double4* __restrict__ pos, const int32_t* __restrict__ leaves,
                                                      int32_t nleaves, const int32_t* __restrict__ beg,
                                                      const int32_t* __restrict__ cnt, double4* __restrict__ geo,
                                                      double* __restrict__ mom, double4* __restrict__ msum,
                                                      unsigned long long* clock) {
  take_time(clock);
  int32_t i = blockIdx.x * kBS + threadIdx.x;
  if (i >= nleaves) return;
  int32_t c = leaves[i];
  int32_t b = beg[c], e = b + cnt[c];
  double M = 0.0, Sx = 0.0, Sy = 0.0, Sz = 0.0;
  for (int32_t p = b; p < e; ++p) {
    double4 q = pos[p];
    M += q.w;
    Sx += q.w * q.x;
    Sy += q.w * q.y;
    Sz += q.w * q.z;
  }
  double Zx = Sx / M, Zy = Sy / M, Zz = Sz / M;
  double M2[6] = {}, M3[10] = {};
  for (int32_t p = b; p < e; ++p) {
    double4 q = pos[p];
    add_about(M2, M3, q.w, q.x - Zx, q.y - Zy, q.z - Zz);
  }
  geo[c] = make_double4(Zx, Zy, Zz, 0.0);
  msum[c] = make_double4(Sx, Sy, Sz, M);
  double* o = mom + (int64_t)c * kMom;
  o[0] = M;
  for (int q = 0; q < 6; ++q) o[1 + q] = M2[q];
  for (int q = 0; q < 10; ++q) o[7 + q] = M3[q];
  o[17] = 0.0;
}

// One parent from its children, 8 lanes per parent (lane q of the group holds
// child q).  The sums over the children run in octant order: mass and first
// moment by passing the children's values through the group, the shifted
// M_ij and M_ijk through the group's rows of LDS, summed by 8 lanes two
// components each.  One thread per parent took 8 dependent rounds of loads
// (12-15 us a level however small); this takes one.
constexpr int kM2MGroup = 8;
constexpr int kM2MPad = 17;  // LDS row of one child: 6 + 10 values, padded

__device__ inline void m2m_parent(int32_t c, int lane8, double (*rows)[kM2MPad], const int32_t* __restrict__ ch0,
                                  const int32_t* __restrict__ nch, double4* geo, double* mom, double4* msum,
                                  bool valid) {
  const int32_t k = valid ? nch[c] : 0;
  const int32_t q = (k ? ch0[c] : 0) + lane8;
  const bool has = lane8 < k;
  double4 s = make_double4(0.0, 0.0, 0.0, 0.0), g = s;
  double cm[17];
#pragma unroll
  for (int u = 0; u < 17; ++u) cm[u] = 0.0;
  if (has) {
    s = msum[q];
    g = geo[q];
#pragma unroll
    for (int u = 0; u < 17; ++u) cm[u] = mom[(int64_t)q * kMom + u];
  }
  double M = 0.0, Sx = 0.0, Sy = 0.0, Sz = 0.0;
#pragma unroll
  for (int j = 0; j < kM2MGroup; ++j) {
    const double w = __shfl(s.w, j, kM2MGroup), x = __shfl(s.x, j, kM2MGroup);
    const double y = __shfl(s.y, j, kM2MGroup), z = __shfl(s.z, j, kM2MGroup);
    if (j < k) {
      M += w;
      Sx += x;
      Sy += y;
      Sz += z;
    }
  }
  const double Zx = Sx / M, Zy = Sy / M, Zz = Sz / M;
  if (has) {
    const double mc = cm[0];
    const double d[3] = {g.x - Zx, g.y - Zy, g.z - Zz};
    const double* a = cm + 1;  // child M_ij
    const double* t = cm + 7;  // child M_ijk
    // M_ij += Mc_ij + Mc d_i d_j
    const int I2[6][2] = {{0, 0}, {0, 1}, {0, 2}, {1, 1}, {1, 2}, {2, 2}};
#pragma unroll
    for (int u = 0; u < 6; ++u) rows[lane8][u] = a[u] + mc * d[I2[u][0]] * d[I2[u][1]];
    // M_ijk += Mc_ijk + Mc_ij d_k + Mc_jk d_i + Mc_ik d_j + Mc d_i d_j d_k
    const int I3[10][3] = {{0, 0, 0}, {0, 0, 1}, {0, 0, 2}, {0, 1, 1}, {0, 1, 2},
                           {0, 2, 2}, {1, 1, 1}, {1, 1, 2}, {1, 2, 2}, {2, 2, 2}};
    auto p2 = [&](int x, int y) {
      int lo = x < y ? x : y, hi = x < y ? y : x;
      return a[lo == 0 ? hi : (lo == 1 ? 2 + hi : 5)];
    };
#pragma unroll
    for (int u = 0; u < 10; ++u) {
      int ii = I3[u][0], jj = I3[u][1], kk = I3[u][2];
      rows[lane8][6 + u] = t[u] + p2(ii, jj) * d[kk] + p2(jj, kk) * d[ii] + p2(ii, kk) * d[jj] +
                           mc * d[ii] * d[jj] * d[kk];
    }
  }
  __syncthreads();
  if (k) {
    double* o = mom + (int64_t)c * kMom;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int u = 2 * lane8 + h;
      double v = 0.0;
      for (int j = 0; j < k; ++j) v += rows[j][u];
      o[1 + u] = v;
    }
    if (lane8 == 0) {
      geo[c] = make_double4(Zx, Zy, Zz, 0.0);
      msum[c] = make_double4(Sx, Sy, Sz, M);
      o[0] = M;
      o[17] = 0.0;
    }
  }
}

__global__ void __launch_bounds__(kBS) k_m2m(int32_t c0, int32_t nl, const int32_t* __restrict__ ch0,
                                             const int32_t* __restrict__ nch, double4* geo, double* mom,
                                             double4* msum) {
  __shared__ double rows[kBS / kM2MGroup][kM2MGroup][kM2MPad];
  const int32_t i = (blockIdx.x * kBS + threadIdx.x) / kM2MGroup;
  m2m_parent(c0 + i, threadIdx.x % kM2MGroup, rows[threadIdx.x / kM2MGroup], ch0, nch, geo, mom, msum, i < nl);
}

// The top levels (those of at most kTopCells cells), bottom-up, in one block:
// a launch each costs more than their work.
constexpr int kTopBS = 1024;
constexpr int kTopCells = 2 * kTopBS / kM2MGroup;
struct TopLevels {
  int32_t n;                         // levels 0 .. n-1
  int32_t start[kMaxLevel + 2];
};

__global__ void __launch_bounds__(kTopBS) k_m2m_top(TopLevels t, const int32_t* __restrict__ ch0,
                                                    const int32_t* __restrict__ nch, double4* geo, double* mom,
                                                    double4* msum) {
  __shared__ double rows[kTopBS / kM2MGroup][kM2MGroup][kM2MPad];
  for (int l = t.n - 1; l >= 0; --l) {
    for (int32_t b = t.start[l]; b < t.start[l + 1]; b += kTopBS / kM2MGroup) {
      const int32_t c = b + threadIdx.x / kM2MGroup;
      m2m_parent(c, threadIdx.x % kM2MGroup, rows[threadIdx.x / kM2MGroup], ch0, nch, geo, mom, msum,
                 c < t.start[l + 1]);
      __syncthreads();  // the parents written, the rows read
    }
  }
}

__global__ void __launch_bounds__(kBS) k_zero_u64(unsigned long long* p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * kBS + threadIdx.x;
  if (i < n) p[i] = 0ull;
}

// 64-particle slabs one wave of k_rmax takes, in key order: as many as leave
// kRmaxWaves waves to fill the chip, at most kRmaxSlabs (a fixed 32 left
// 100003 particles on 49 waves: 269 us).
constexpr int kRmaxSlabs = 32;
constexpr int64_t kRmaxWaves = 8192;

// R_max^2 of every ancestor of every particle, by atomic max on the bit
// pattern (order-preserving for non-negative doubles).  A wave takes
// `slabs` consecutive slabs of 64 particles; on each level, lanes with
// the same ancestor (contiguous, as cells are) reduce to the run's first
// lane, and the run that reaches the slab's end stays pending in the wave
// and joins the next slab's first run when that has the same cell.  A cell
// of many particles so gets one atomic per wave that touches it rather than
// one per slab (all waves otherwise meet on the same few top cells).
__global__ void __launch_bounds__(kBS) k_rmax(const double4* __restrict__ pos, int64_t n, int slabs,
                                              const int32_t* __restrict__ leafof, const int32_t* __restrict__ par,
                                              const int8_t* __restrict__ lev, const double4* __restrict__ geo,
                                              unsigned long long* __restrict__ r2max) {
  const int lane = threadIdx.x & 63;
  const int64_t p0 = (((int64_t)blockIdx.x * kBS + threadIdx.x) >> 6) * (64 * (int64_t)slabs);
  // per level, the pending run (wave-uniform): its cell (-1: none) and max
  int32_t pend_id[kMaxLevel + 1];
  double pend_r2[kMaxLevel + 1];
#pragma unroll
  for (int l = 0; l <= kMaxLevel; ++l) {
    pend_id[l] = -1;
    pend_r2[l] = -1.0;
  }
  for (int s = 0; s < slabs; ++s) {
    const int64_t p = p0 + (int64_t)s * 64 + lane;
    if (p0 + (int64_t)s * 64 >= n) break;  // wave-uniform
    const bool valid = p < n;
    int32_t anc[kMaxLevel + 1];
    const double4 q = valid ? pos[p] : make_double4(0, 0, 0, 0);
    {
      int32_t a = valid ? leafof[p] : -1;
      int L = valid ? (int)lev[a] : -1;
#pragma unroll
      for (int l = kMaxLevel; l >= 0; --l) {
        if (l > L) {
          anc[l] = -1;
        } else {
          anc[l] = a;
          a = par[a];
        }
      }
    }
#pragma unroll
    for (int l = 0; l <= kMaxLevel; ++l) {
      const int32_t id = anc[l];
      // no particle of the slab below this level: deeper runs stay pending
      if (!__any(id >= 0)) break;
      double r2 = -1.0;
      if (id >= 0) {
        const double4 g = geo[id];
        const double dx = q.x - g.x, dy = q.y - g.y, dz = q.z - g.z;
        r2 = (dx * dx + dy * dy) + dz * dz;
      }
      // segmented max over contiguous lanes with the same ancestor
#pragma unroll
      for (int off = 1; off < 64; off <<= 1) {
        const double o = __shfl_down(r2, off, 64);
        const int32_t oid = __shfl_down(id, off, 64);
        if (lane + off < 64 && oid == id && o > r2) r2 = o;
      }
      const int32_t prev = __shfl_up(id, 1, 64);
      const bool head = id >= 0 && (lane == 0 || prev != id);
      const unsigned long long hm = __ballot(head);  // nonzero: some lane has an ancestor here
      const int last = 63 - __clzll(hm);
      const bool joins = __shfl(id, 0, 64) == pend_id[l];
      if (lane == 0 && joins) r2 = fmax(r2, pend_r2[l]);
      if (lane == 0 && !joins && pend_id[l] >= 0)
        atomicMax(&r2max[pend_id[l]], (unsigned long long)__double_as_longlong(pend_r2[l]));
      if (head && lane != last) atomicMax(&r2max[id], (unsigned long long)__double_as_longlong(r2));
      pend_id[l] = __shfl(id, last, 64);
      pend_r2[l] = __shfl(r2, last, 64);
    }
  }
  if (lane == 0) {
#pragma unroll
    for (int l = 0; l <= kMaxLevel; ++l)
      if (pend_id[l] >= 0) atomicMax(&r2max[pend_id[l]], (unsigned long long)__double_as_longlong(pend_r2[l]));
  }
}

__global__ void __launch_bounds__(kBS) k_rmax_final(int32_t nc, const unsigned long long* __restrict__ r2max,
                                                    double4* __restrict__ geo) {
  int32_t c = blockIdx.x * kBS + threadIdx.x;
  if (c >= nc) return;
  geo[c].w = sqrt(__longlong_as_double((long long)r2max[c]));
}

}  // namespace

void upward_pass(Ctx& c) {
  const int32_t nc = c.ncells;
  double4* geo = (double4*)ensure(c, c.geo, sizeof(double4) * nc);
  double* mom = (double*)ensure(c, c.mom, sizeof(double) * kMom * (size_t)nc);
  double4* msum = (double4*)ensure(c, c.msum, sizeof(double4) * nc);
  const int32_t* beg = as<int32_t>(c.c_begin);
  const int32_t* cnt = as<int32_t>(c.c_count);
  hipLaunchKernelGGL(k_leaf_moments, dim3(blocks_for(c.nleaves, kBS)), dim3(kBS), 0, c.stream,
                     (const double4*)c.pos4.p, as<int32_t>(c.leaves), c.nleaves, beg, cnt, geo, mom, msum,
                     clock_word(c));
  AMFMM_HIP(hipGetLastError());
  TopLevels top{};
  while (top.n <= c.depth && c.level_start[top.n + 1] - c.level_start[top.n] <= kTopCells) ++top.n;
  std::copy(c.level_start.begin(), c.level_start.end(), top.start);
  for (int l = c.depth - 1; l >= top.n; --l) {
    int32_t c0 = c.level_start[l], nl = c.level_start[l + 1] - c0;
    hipLaunchKernelGGL(k_m2m, dim3(blocks_for((int64_t)nl * kM2MGroup, kBS)), dim3(kBS), 0, c.stream, c0, nl,
                       as<int32_t>(c.c_child0), as<int32_t>(c.c_nchild), geo, mom, msum);
    AMFMM_HIP(hipGetLastError());
  }
  hipLaunchKernelGGL(k_m2m_top, dim3(1), dim3(kTopBS), 0, c.stream, top, as<int32_t>(c.c_child0),
                     as<int32_t>(c.c_nchild), geo, mom, msum);
  // R_max
  unsigned long long* r2 = (unsigned long long*)ensure(c, c.scratch2, sizeof(unsigned long long) * (size_t)nc);
  hipLaunchKernelGGL(k_zero_u64, dim3(blocks_for(nc, kBS)), dim3(kBS), 0, c.stream, r2, (int64_t)nc);
  const int slabs = (int)std::max<int64_t>(1, std::min<int64_t>(kRmaxSlabs, c.n / (64 * kRmaxWaves)));
  const int64_t rmax_waves = (c.n + 64 * slabs - 1) / (64 * slabs);
  hipLaunchKernelGGL(k_rmax, dim3(blocks_for(rmax_waves * 64, kBS)), dim3(kBS), 0, c.stream, (const double4*)c.pos4.p,
                     c.n, slabs, as<int32_t>(c.leafof), as<int32_t>(c.c_parent), as<int8_t>(c.c_level),
                     (const double4*)geo, r2);
  hipLaunchKernelGGL(k_rmax_final, dim3(blocks_for(nc, kBS)), dim3(kBS), 0, c.stream, nc,
                     (const unsigned long long*)r2, geo);
  AMFMM_HIP(hipGetLastError());
  c.have_moments = true;
}

}  // namespace amfmm
