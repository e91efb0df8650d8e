// Evaluation: far field per target cell, push-down to the leaves, and the
// near field fused with the evaluation at the particles and the unsort.
//
// Far field (eqs. 2-4, dipoles dropped, octupole constant dropped): for the
// target X and a source Y with R = Z_X - Z_Y, the Taylor coefficients of the
// potential about Z_X are
//   C    += M_Y D + 1/2 M_Y,lm D_lm          C_k   += M_Y D_k + 1/2 M_Y,lm D_klm
//   C_kl += M_Y D_kl                          C_klm += M_Y D_klm
// (eq. 2 read as a polynomial in x; eq. 4 for the other cell of a pair is the
// same expression with R -> -R, so directed evaluation per target reproduces
// the symmetric pair exactly up to summation order).  The correction of eq. 7
// (prefactor 1/6, see the appendix at P = 3) adds F_c/M_X to X with
//   F_c,i = -(1/6) Q_jkl D_ijkl,  Q = M_X,jkl M_Y - M_X M_Y,jkl,
// contracted in closed form: Q_jkl D_ijkl = t4 R_i (Q.RRR) + 3 t3 (Q_ikl R_k
// R_l + R_i Q_jkk R_j) + 3 t2 Q_ikk with t2 = -3/R^5, t3 = 15/R^7, t4 =
// -105/R^9.  Eq. 8 keeps only 3 t3 Q_ikl R_k R_l + 3 t2 Q_ikk.
//
// One wave per target cell, lanes over its sources, fixed-order reduction
// (deterministic).  Mixed precision: R = Z_X - Z_Y is formed in FP64
// and rounded, the coefficient terms are FP32 and each lane adds at most
// kFarFlush of them in FP32 before an FP64 flush; the correction (which
// cancels M_X,jkl M_Y against M_X M_Y,jkl) stays FP64.  UC and TC of the plain
// -1/R read each source from one 128-byte record (k_far_rec), the rest from the
// cells' arrays (k_far).
#include <cmath>
#include <type_traits>

#include "device_math.h"
#include "internal.h"

namespace amfmm {
namespace {

constexpr int kBS = 256;

// sources per lane summed in FP32 before an FP64 flush (mixed path)
constexpr int kFarFlush = 8;

// Far-field source records of UC and TC at the plain -1/R: 128 bytes, one cache
// line.  The derivatives are traceless in every index pair, so the traceless
// octupole (7 components: xxx xxy xxz xyy xyz yyy yyz; xzz, yzz, zzz follow) is
// all the correction needs, here over the cell's mass (masses are positive).  At FP64 the quadrupole is traceless too (5
// components: xx xy xz yy yz); mixed precision keeps all six, rounded to FP32
// as they are used.  FP64 records are in units of powers of two near the box's
// side and the total mass (FarUnit), which changes no rounding: in the caller's
// units M / R^7 leaves the exponent range long before the results do (lengths of
// 10^18 with masses of 10^-192, say).  FP32 has no range to spare for a unit that
// fits the box rather than the distances within it.
struct alignas(128) FarRec {
  double z[3], m;
  double o[7];
  float q[6];
  float pad[4];
};
struct alignas(128) FarRec64 {
  double z[3], m;
  double o[7];
  double q[5];
};
static_assert(sizeof(FarRec) == 128 && sizeof(FarRec64) == 128, "far record");

template <bool MIXED>
__global__ void __launch_bounds__(kBS) k_pack_far(int32_t nc, const double4* __restrict__ geo,
                                                  const double* __restrict__ mom, int el, void* __restrict__ out) {
  const int32_t c = blockIdx.x * kBS + threadIdx.x;
  if (c >= nc) return;
  const double4 g = geo[c];
  const double* mo = mom + (int64_t)c * kMom;
  double T[10];
  octupole_traceless(mo + 7, T);
  const double M = mo[0];
  const double o[7] = {T[0] / M, T[1] / M, T[2] / M, T[3] / M, T[4] / M, T[6] / M, T[7] / M};
  auto common = [&](auto& r) {
    r.z[0] = g.x;
    r.z[1] = g.y;
    r.z[2] = g.z;
    r.m = M;
#pragma unroll
    for (int u = 0; u < 7; ++u) r.o[u] = o[u];
  };
  if (MIXED) {
    FarRec r;
    common(r);
#pragma unroll
    for (int u = 0; u < 6; ++u) r.q[u] = (float)mo[1 + u];
#pragma unroll
    for (int u = 0; u < 4; ++u) r.pad[u] = 0.0f;
    ((FarRec*)out)[c] = r;
  } else {
    FarRec64 r;
    common(r);
    const double tr = (mo[1] + mo[4] + mo[6]) / 3.0;
    r.q[0] = mo[1] - tr;
    r.q[1] = mo[2];
    r.q[2] = mo[3];
    r.q[3] = mo[4] - tr;
    r.q[4] = mo[5];
    const FarUnit unit(el, mom);
#pragma unroll
    for (int u = 0; u < 3; ++u) r.z[u] = unit.length(r.z[u]);
    r.m = unit.moment(r.m, 0);
#pragma unroll
    for (int u = 0; u < 7; ++u) r.o[u] = unit.length(r.o[u], 3);
#pragma unroll
    for (int u = 0; u < 5; ++u) r.q[u] = unit.moment(r.q[u], 2);
    ((FarRec64*)out)[c] = r;
  }
}

// Sums of 24 values over the wave: each exchange sends the half of the values
// that the other lane goes on with, 24 -> 12 -> 6 -> 3, so 21 exchanges and nine
// plain ones take the place of 144.  Lane l ends with the totals of values
// first, first + 1, first + 2, first = 12 bit5 + 6 bit4 + 3 bit3 of l.  The
// additions of one value pair lanes as a butterfly over 32, 16, ..., 1 does.
__device__ inline void wave_sum24(double v[24], int lane, double out[3]) {
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int off = 32 >> s, half = 12 >> s;
    const bool hi = lane & off;
#pragma unroll
    for (int k = 0; k < half; ++k) {
      const double send = hi ? v[k] : v[k + half], keep = hi ? v[k + half] : v[k];
      v[k] = keep + __shfl_xor(send, off, 64);
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    out[k] = v[k];
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) out[k] += __shfl_xor(out[k], off, 64);
  }
}

// a target's coefficients and corrections (F: times cf) from every lane's sums,
// out of the unit they were made in
__device__ inline void store_local(double* __restrict__ o, const double acc[20], const double F[3], double cf, int lane,
                                   const FarUnit& unit) {
  double v[24], t[3];
#pragma unroll
  for (int u = 0; u < 20; ++u) v[u] = acc[u];
#pragma unroll
  for (int i = 0; i < 3; ++i) v[20 + i] = F[i];
  v[23] = 0.0;
  wave_sum24(v, lane, t);
  const int first = 12 * ((lane >> 5) & 1) + 6 * ((lane >> 4) & 1) + 3 * ((lane >> 3) & 1), k = lane & 7;
  if (k < 3) {
    const double s = k == 0 ? t[0] : (k == 1 ? t[1] : t[2]);
    const int i = first + k, order = i >= 20 ? 1 : (i >= 10 ? 3 : (i >= 4 ? 2 : (i >= 1 ? 1 : 0)));
    o[i] = unit.coefficient(i >= 20 ? cf * s : s, order);
  }
}

// Far field of UC and TC from the records (see k_far).  What bounds it is the
// vector cache, which answers one 64-byte request a cycle: a lane loading its
// own record takes eight requests (0.93 a cycle measured; at FP64, from two
// arrays, eleven).  Eight neighbouring lanes fetch one record instead, straight
// to the wave's 8 KB of LDS (16 bytes a lane, two requests a record), and each
// lane reads its own there, slot q of record r holding piece q ^ (r mod 8)
// (conflict-free); the next 64 records travel while this lane computes.
// 4M two spheres at theta 0.35, FP64: 13.3 -> 5.7 ms; 16.8M at the benchmark's
// tolerance, mixed: 256 -> 155 ms.  One wave per workgroup, so that none waits
// for a neighbour's longer list, and octupoles per mass: 5.2 and 145 ms.
// (mixed TC at four waves a SIMD spills a register, whose reload waits for the
// records on their way as well: 228 ms)
template <int VARIANT, bool MIXED>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(MIXED && VARIANT ? 3 : 4)))
k_far_rec(int32_t c_lo, const void* __restrict__ recs, const int64_t* __restrict__ fstart,
          const int32_t* __restrict__ fcount, const int32_t* __restrict__ fsrc, const double* __restrict__ mom, int el,
          double* __restrict__ loc, unsigned long long* clock) {
  take_time(clock);
  using Rec = typename std::conditional<MIXED, FarRec, FarRec64>::type;
  const Rec* __restrict__ rec = (const Rec*)recs;
  __shared__ double2 buf[64 * 8];
  const int lane = threadIdx.x;
  const int32_t Xi = (int32_t)xcd_block(blockIdx.x, gridDim.x);
  const int32_t X = c_lo + Xi;
  const int32_t cnt = uniform(fcount[X]);
  const int32_t* __restrict__ src = fsrc + fstart[X];
  const FarUnit unit = MIXED ? FarUnit() : FarUnit(el, mom);
  const Rec& rx = rec[X];
  // the target's side in scalar registers
  const double gx[3] = {uniform_f64(rx.z[0]), uniform_f64(rx.z[1]), uniform_f64(rx.z[2])};
  double oX[7];
#pragma unroll
  for (int u = 0; u < 7; ++u) oX[u] = VARIANT ? uniform_f64(rx.o[u]) : 0.0;
  double acc[20], F[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < 20; ++u) acc[u] = 0.0;
  // lanes past the end fetch the target's own record and do not use it
  auto fetch = [&](int32_t y) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = 8 * i + (lane >> 3);
      const double2* from = (const double2*)(rec + __shfl(y, r, 64)) + ((lane & 7) ^ (r & 7));
      __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)from,
                                       (__attribute__((address_space(3))) void*)(buf + 64 * i), 16, 0, 0);
    }
  };
  int32_t ahead = lane + 64 < cnt ? src[lane + 64] : X;
  if (cnt > 0) fetch(lane < cnt ? src[lane] : X);
  float a32[20];
#pragma unroll
  for (int u = 0; u < 20; ++u) a32[u] = 0.0f;
  int batch = 0;
  for (int32_t j0 = 0; j0 < cnt; j0 += 64) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    double2 p[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) p[q] = buf[8 * lane + (q ^ (lane & 7))];
    // every lane's record is in registers before the next ones arrive
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (j0 + 64 < cnt) {
      fetch(ahead);
      const int32_t j2 = j0 + 128 + lane;
      ahead = j2 < cnt ? src[j2] : X;
    }
    if (j0 + lane < cnt) {
      const double R[3] = {gx[0] - p[0].x, gx[1] - p[0].y, gx[2] - p[1].x};
      const double M = p[1].y;
      const double o7[7] = {p[2].x, p[2].y, p[3].x, p[3].y, p[4].x, p[4].y, p[5].x};
      if (MIXED) {
        const float2 q01 = __builtin_bit_cast(float2, p[5].y), q23 = __builtin_bit_cast(float2, p[6].x),
                     q45 = __builtin_bit_cast(float2, p[6].y);
        const float Rf[3] = {(float)R[0], (float)R[1], (float)R[2]};
        const float Q2f[6] = {q01.x, q01.y, q23.x, q23.y, q45.x, q45.y};
        far_coeffs<float>(Rf, (float)M, Q2f, a32, 0.0f);
      } else {
        const double Q2[6] = {p[5].y, p[6].x, p[6].y, p[7].x, p[7].y, -p[5].y - p[7].x};
        far_coeffs_traceless(R, M, Q2, acc);
      }
      if (VARIANT) far_correction_traceless(R, oX, M, o7, F);
    }
    if (MIXED && ++batch == kFarFlush) {
      batch = 0;
#pragma unroll
      for (int u = 0; u < 20; ++u) {
        acc[u] += (double)a32[u];
        a32[u] = 0.0f;
      }
    }
  }
  if (MIXED) {
#pragma unroll
    for (int u = 0; u < 20; ++u) acc[u] += (double)a32[u];
  }
  store_local(loc + (int64_t)X * kLoc, acc, F, VARIANT ? -45.0 / 6.0 : 0.0, lane, unit);
}

template <int VARIANT, bool MIXED>
__global__ void __launch_bounds__(64) k_far(int32_t c_lo, const double4* __restrict__ geo, const double* __restrict__ mom,
                                             const int64_t* __restrict__ fstart, const int32_t* __restrict__ fcount,
                                             const int32_t* __restrict__ fsrc, double* __restrict__ loc, double eps2,
                                             unsigned long long* clock) {
  take_time(clock);
  const int lane = threadIdx.x;
  const int32_t Xi = (int32_t)xcd_block(blockIdx.x, gridDim.x);
  const int32_t X = c_lo + Xi;
  const int32_t cnt = fcount[X];
  const int64_t st = fstart[X];
  const double4 gx = geo[X];
  const double* mx = mom + (int64_t)X * kMom;
  const double MX = mx[0];
  double OX[10];
#pragma unroll
  for (int u = 0; u < 10; ++u) OX[u] = VARIANT ? mx[7 + u] : 0.0;
  double acc[20], F[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int u = 0; u < 20; ++u) acc[u] = 0.0;
  const int64_t step = MIXED ? 64 * kFarFlush : (int64_t)cnt + 64;
  for (int64_t j0 = lane; j0 < cnt; j0 += step) {
    float a32[20];
#pragma unroll
    for (int u = 0; u < 20; ++u) a32[u] = 0.0f;
    const int64_t j1 = j0 + step < cnt ? j0 + step : cnt;
    for (int64_t j = j0; j < j1; j += 64) {
      const int32_t Y = fsrc[st + j];
      const double4 gy = geo[Y];
      const double* my = mom + (int64_t)Y * kMom;
      const double M = my[0];
      const double R[3] = {gx.x - gy.x, gx.y - gy.y, gx.z - gy.z};
      if (MIXED) {
        const float Rf[3] = {(float)R[0], (float)R[1], (float)R[2]};
        float Q2f[6];
#pragma unroll
        for (int u = 0; u < 6; ++u) Q2f[u] = (float)my[1 + u];
        far_coeffs<float>(Rf, (float)M, Q2f, a32, (float)eps2);
      } else {
        double Q2[6];
#pragma unroll
        for (int u = 0; u < 6; ++u) Q2[u] = my[1 + u];
        far_coeffs<double>(R, M, Q2, acc, eps2);
      }
      if (VARIANT) {
        double O3[10];
#pragma unroll
        for (int u = 0; u < 10; ++u) O3[u] = my[7 + u];
        far_correction<VARIANT>(R, MX, OX, M, O3, F, eps2);
      }
    }
    if (MIXED) {
#pragma unroll
      for (int u = 0; u < 20; ++u) acc[u] += (double)a32[u];
    }
  }
  store_local(loc + (int64_t)X * kLoc, acc, F, VARIANT ? -1.0 / (6.0 * MX) : 0.0, lane, FarUnit());
}

// loc[c] += Taylor shift of its parent's coefficients to its centre
__device__ inline void l2l_cell(int32_t c, const int32_t* __restrict__ par, const double4* __restrict__ geo,
                                double* loc) {
  const int32_t P = par[c];
  const double4 gc = geo[c], gp = geo[P];
  const double d[3] = {gc.x - gp.x, gc.y - gp.y, gc.z - gp.z};
  const double* L = loc + (int64_t)P * kLoc;
  double* o = loc + (int64_t)c * kLoc;
  double C1[3] = {L[1], L[2], L[3]};
  double C2[6], C3[10];
#pragma unroll
  for (int u = 0; u < 6; ++u) C2[u] = L[4 + u];
#pragma unroll
  for (int u = 0; u < 10; ++u) C3[u] = L[10 + u];
  const double dd[6] = {d[0] * d[0], d[0] * d[1], d[0] * d[2], d[1] * d[1], d[1] * d[2], d[2] * d[2]};
  const double mult[6] = {1.0, 2.0, 2.0, 1.0, 2.0, 1.0};
  // (C3 dd)_k and (C2 d)_k
  double C3dd[3], C2d[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double s = 0.0;
#pragma unroll
    for (int p = 0; p < 6; ++p) s = fma(mult[p] * C3[kT3[p][k]], dd[p], s);
    C3dd[k] = s;
  }
  C2d[0] = fma(C2[0], d[0], fma(C2[1], d[1], C2[2] * d[2]));
  C2d[1] = fma(C2[1], d[0], fma(C2[3], d[1], C2[4] * d[2]));
  C2d[2] = fma(C2[2], d[0], fma(C2[4], d[1], C2[5] * d[2]));
  double c0v = L[0];
#pragma unroll
  for (int k = 0; k < 3; ++k) c0v += d[k] * (C1[k] + 0.5 * C2d[k] + (1.0 / 6.0) * C3dd[k]);
  o[0] += c0v;
#pragma unroll
  for (int k = 0; k < 3; ++k) o[1 + k] += C1[k] + C2d[k] + 0.5 * C3dd[k];
#pragma unroll
  for (int p = 0; p < 6; ++p) {
    double s = C2[p];
#pragma unroll
    for (int m = 0; m < 3; ++m) s = fma(C3[kT3[p][m]], d[m], s);
    o[4 + p] += s;
  }
#pragma unroll
  for (int u = 0; u < 10; ++u) o[10 + u] += C3[u];
#pragma unroll
  for (int i2 = 0; i2 < 3; ++i2) o[20 + i2] += L[20 + i2];
}

__global__ void __launch_bounds__(kBS) k_l2l(int32_t c0, int32_t nl, const int32_t* __restrict__ par,
                                             const double4* __restrict__ geo, double* loc, unsigned long long* clock) {
  take_time(clock);
  const int32_t i = blockIdx.x * kBS + threadIdx.x;
  if (i < nl) l2l_cell(c0 + i, par, geo, loc);
}

// The top levels, downwards, in one block: a launch each (3 us) costs as much
// as their work while a level is at most a few hundred cells.
constexpr int kTopBS = 512;
struct TopLevels {
  int32_t n;  // levels 1 .. n-1
  int32_t start[kMaxLevel + 2];
};

__global__ void __launch_bounds__(kTopBS) k_l2l_top(TopLevels t, const int32_t* __restrict__ par,
                                                    const double4* __restrict__ geo, double* loc,
                                                    unsigned long long* clock) {
  take_time(clock);
  for (int l = 1; l < t.n; ++l) {
    for (int32_t c = t.start[l] + threadIdx.x; c < t.start[l + 1]; c += kTopBS) l2l_cell(c, par, geo, loc);
    __syncthreads();
  }
}

__global__ void k_zero_u64_n(unsigned long long* p, int n, unsigned long long* clock) {
  take_time(clock);
  if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

}  // namespace

void zero_u64(Ctx& c, unsigned long long* p, int n, unsigned long long* clock) {
  hipLaunchKernelGGL(k_zero_u64_n, dim3(1), dim3(64), 0, c.stream, p, n, clock);
  AMFMM_HIP(hipGetLastError());
}

// the 128-byte records carry traceless moments, enough for UC and TC of the
// plain -1/R (the derivatives of a softened one, and eq. 8's tensor, are not
// traceless)
static bool has_records(const Ctx& c) {
  return c.opt.variant != AMFMM_TCO && c.opt.softening == 0.0 && c.opt.order == 3;
}

int length_exponent(const Ctx& c) {
  double v = c.opt.softening;
  for (int d = 0; d < 3; ++d) v = std::max(v, c.box[3 + d] - c.box[d]);
  return v > 0.0 && std::isfinite(v) ? std::ilogb(v) : 0;
}

void far_prepare(Ctx& c) {
  if (c.opt.order != 3 && c.ncells > 0) order_pack(c);
  if (!has_records(c) || c.ncells <= 0) return;
  void* rec = ensure_if_room(c, c.farrec, sizeof(FarRec) * (size_t)c.ncells);
  if (!rec) return;
  hipLaunchKernelGGL(c.opt.precision == AMFMM_MIXED ? k_pack_far<true> : k_pack_far<false>, dim3(blocks_for(c.ncells, kBS)), dim3(kBS), 0, c.stream, c.ncells,
                     (const double4*)c.geo.p, (const double*)c.mom.p, length_exponent(c), rec);
  AMFMM_HIP(hipGetLastError());
}

void far_field(Ctx& c, int32_t c_lo, int32_t c_hi) {
  const int32_t nc = c_hi - c_lo;
  if (nc <= 0) return;
  double* loc = (double*)ensure_keep(c, c.loc, sizeof(double) * kLoc * (size_t)c.ncells,
                                     sizeof(double) * kLoc * (size_t)c.ncells);
  if (c.opt.order != 3) {
    ++c.far_launches;
    order_far(c, c_lo, c_hi, loc);
    return;
  }
  if (has_records(c) && c.farrec.p) {
    ++c.far_launches;
    const bool tc = c.opt.variant == AMFMM_TC;
    auto kern = c.opt.precision == AMFMM_MIXED ? (tc ? k_far_rec<AMFMM_TC, true> : k_far_rec<AMFMM_UC, true>)
                                               : (tc ? k_far_rec<AMFMM_TC, false> : k_far_rec<AMFMM_UC, false>);
    hipLaunchKernelGGL(kern, dim3(nc), dim3(64), 0, c.stream, c_lo, (const void*)c.farrec.p,
                       (const int64_t*)c.far_start.p, (const int32_t*)c.far_count.p, (const int32_t*)c.far_src.p,
                       (const double*)c.mom.p, length_exponent(c), loc, clock_word(c));
    AMFMM_HIP(hipGetLastError());
    return;
  }
  auto args = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(nc), dim3(64), 0, c.stream, c_lo, (const double4*)c.geo.p, (const double*)c.mom.p,
                       (const int64_t*)c.far_start.p, (const int32_t*)c.far_count.p, (const int32_t*)c.far_src.p, loc,
                       c.opt.softening * c.opt.softening, clock_word(c));
  };
  ++c.far_launches;
  const bool mixed = c.opt.precision == AMFMM_MIXED;
  switch (c.opt.variant) {
    case AMFMM_UC: mixed ? args(k_far<AMFMM_UC, true>) : args(k_far<AMFMM_UC, false>); break;
    case AMFMM_TC: mixed ? args(k_far<AMFMM_TC, true>) : args(k_far<AMFMM_TC, false>); break;
    default: mixed ? args(k_far<AMFMM_TCO, true>) : args(k_far<AMFMM_TCO, false>); break;
  }
  AMFMM_HIP(hipGetLastError());
}

void push_down_all(Ctx& c) {
  int l = 1;
  if (c.opt.order == 3 && c.depth >= 1) {
    TopLevels top{};
    for (top.n = 1; top.n <= c.depth && c.level_start[top.n + 1] - c.level_start[top.n] <= kTopBS;) ++top.n;
    std::copy(c.level_start.begin(), c.level_start.end(), top.start);
    hipLaunchKernelGGL(k_l2l_top, dim3(1), dim3(kTopBS), 0, c.stream, top, as<int32_t>(c.c_parent),
                       (const double4*)c.geo.p, as<double>(c.loc), clock_word(c));
    AMFMM_HIP(hipGetLastError());
    l = top.n;
  }
  for (; l <= c.depth; ++l) push_down(c, c.level_start[l], c.level_start[l + 1]);
}

void push_down(Ctx& c, int32_t c_lo, int32_t c_hi) {
  const int32_t nl = c_hi - c_lo;
  if (nl <= 0) return;
  if (c.opt.order != 3) {  // the order-3 records hold zeros
    order_push_down(c, c_lo, c_hi);
    return;
  }
  hipLaunchKernelGGL(k_l2l, dim3(blocks_for(nl, kBS)), dim3(kBS), 0, c.stream, c_lo, nl, as<int32_t>(c.c_parent),
                     (const double4*)c.geo.p, as<double>(c.loc), clock_word(c));
  AMFMM_HIP(hipGetLastError());
}

}  // namespace amfmm
