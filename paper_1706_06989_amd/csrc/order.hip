// The appendix's general expansion order on the GPU, P = 4, in FP64: the
// Green's function G(R + x - y) (R = Z_X - Z_Y, x and y the offsets from the
// two centres of mass) expanded to order P in both offsets, and the
// corrective force of that order that cancels each pair's torque.
//
// Multi-indices alpha = (a, b, c) stand for index tuples (x^alpha = x^a y^b
// z^c, alpha! = a! b! c!).  Per cell: moments M_alpha = sum mu x^alpha about
// the centre of mass (|alpha| <= P, leaves from their particles, parents by
// shifting their children's); per target cell X the local coefficients
//   L_alpha = sum_Y sum_beta (-1)^|beta| / beta! D_(alpha+beta)(R) M_Y,beta
// over |alpha| + |beta| <= P, dipole terms (|beta| = 1) and the constant
// |alpha| = 0, |beta| = P dropped (as at P = 3), and with the correction
// (TC) the acceleration g_c = F_c / M_X,
//   F_c,k = -sum_n (-1)^n sum_{|alpha| = P-n, |beta| = n} M_X,alpha M_Y,beta
//           D_(alpha+beta+e_k)(R) / (alpha! beta!)
// (evaluated as one symmetric order-P tensor of moment products against D)
// (at P = 3 this is eq. 7; the mirrored pair gives -F_c, since D of odd order
// changes sign with R).  The derivatives D_gamma of g(R) = -1/sqrt(R^2 +
// eps^2) come from f_k = (1/R d/dR)^k g by pairing equal indices.  Push-down
// shifts L to each child's centre; at a particle the acceleration is minus
// the gradient of sum_alpha x^alpha / alpha! L_alpha, plus g_c.
//
// Evaluated per directed pair (each target its own sources), one wave per
// target cell, lanes over its sources, fixed-order butterfly sums: the same
// organisation as the order-3 far field.
#include <cmath>

#include "device_math.h"
#include "internal.h"

namespace amfmm {
namespace {

constexpr int kBS = 256;
constexpr int kP = 4;

// multi-indices of order <= n
constexpr int num_mi(int n) { return (n + 1) * (n + 2) * (n + 3) / 6; }
constexpr int kNL = num_mi(kP);  // moments, local coefficients, derivatives
static_assert(kNL + 3 <= kLocGen, "local record");

// graded enumeration: order n, then a from n down, then b from n - a down
struct MITable {
  int a[kNL], b[kNL], c[kNL], n[kNL];
  double fact[kNL];
};
constexpr MITable make_mi() {
  MITable t{};
  int k = 0;
  for (int n = 0; n <= kP; ++n)
    for (int a = n; a >= 0; --a)
      for (int b = n - a; b >= 0; --b) {
        const int c = n - a - b;
        t.a[k] = a;
        t.b[k] = b;
        t.c[k] = c;
        t.n[k] = n;
        double f = 1.0;
        for (int i = 2; i <= a; ++i) f *= i;
        for (int i = 2; i <= b; ++i) f *= i;
        for (int i = 2; i <= c; ++i) f *= i;
        t.fact[k] = f;
        ++k;
      }
  return t;
}
constexpr MITable kMI = make_mi();

__host__ __device__ constexpr int mi_id(int a, int b, int c) {
  return num_mi(a + b + c - 1) + (b + c) * (b + c + 1) / 2 + c;
}
static_assert(mi_id(0, 0, 0) == 0 && mi_id(0, 0, 1) == 3 && mi_id(2, 0, 0) == 4 && mi_id(0, 0, 4) == kNL - 1,
              "multi-index numbering");

// ways to pair p of g equal indices: g! / (p! (g - 2p)! 2^p)
constexpr double pair_ways(int g, int p) {
  double v = 1.0;
  for (int i = 2; i <= g; ++i) v *= i;
  for (int i = 2; i <= p; ++i) v /= i;
  for (int i = 2; i <= g - 2 * p; ++i) v /= i;
  for (int i = 0; i < p; ++i) v /= 2.0;
  return v;
}

// binomial coefficient
constexpr double binom(int n, int k) {
  double v = 1.0;
  for (int i = 1; i <= k; ++i) v = v * (n - k + i) / i;
  return v;
}

// The terms of the far field, the correction and the moment shift, listed
// once at compile time (every index a constant after unrolling).
// local coefficients: L[al] += coef D[g] M_source[be], coef = (-1)^|be| / be!
struct Term {
  int al, be, g;
  double coef;
};
constexpr bool local_term(int al, int be) {
  return kMI.n[al] + kMI.n[be] <= kP && kMI.n[be] != 1 && !(kMI.n[al] == 0 && kMI.n[be] == kP);
}
constexpr int count_local() {
  int k = 0;
  for (int al = 0; al < kNL; ++al)
    for (int be = 0; be < kNL; ++be) k += local_term(al, be);
  return k;
}
constexpr int kNLocal = count_local();
struct LocalTerms {
  Term t[kNLocal];
};
// (source moment outer: each is loaded once and used at once)
constexpr LocalTerms make_local() {
  LocalTerms r{};
  int k = 0;
  for (int be = 0; be < kNL; ++be)
    for (int al = 0; al < kNL; ++al)
      if (local_term(al, be)) {
        const int sb = kMI.n[be] % 2 ? -1 : 1;
        r.t[k++] = {al, be, mi_id(kMI.a[al] + kMI.a[be], kMI.b[al] + kMI.b[be], kMI.c[al] + kMI.c[be]),
                    sb / kMI.fact[be]};
      }
  return r;
}
constexpr LocalTerms kLocal = make_local();

// one value per multi-index; kSign: (-1)^|be| / be!, the factor of the source
// moment be in every term above
struct PerIndex {
  double c[kNL];
};
constexpr PerIndex make_signs() {
  PerIndex r{};
  for (int be = 0; be < kNL; ++be) r.c[be] = (kMI.n[be] % 2 ? -1.0 : 1.0) / kMI.fact[be];
  return r;
}
constexpr PerIndex kSign = make_signs();
// 1 / al!
constexpr PerIndex make_inv_fact() {
  PerIndex r{};
  for (int al = 0; al < kNL; ++al) r.c[al] = 1.0 / kMI.fact[al];
  return r;
}
constexpr PerIndex kInvFact = make_inv_fact();
// lanes of the evaluation kernel per leaf
constexpr int kL2PLanes = 8;
constexpr bool local_coef_check() {
  for (int i = 0; i < kNLocal; ++i)
    if (kLocal.t[i].coef != kSign.c[kLocal.t[i].be]) return false;
  return true;
}
static_assert(local_coef_check(), "local term coefficients are (-1)^|be| / be!");

// correction: the moment products gathered into one symmetric order-P tensor,
// q[g] += coef M_target[al] M_source[be] (g = al + be), coef = (-1)^|be| g! /
// (al! be!), over |al| + |be| = P with neither a dipole; its component g
// stands for the P! / g! index tuples of g, so that (with the P! that F is
// divided by at the end) s_k = 1/P! sum over tuples q_ijlm D_ijlmk
constexpr bool corr_term(int al, int be) {
  return kMI.n[al] + kMI.n[be] == kP && kMI.n[al] != 1 && kMI.n[be] != 1;
}
constexpr int count_corr() {
  int k = 0;
  for (int al = 0; al < kNL; ++al)
    for (int be = 0; be < kNL; ++be) k += corr_term(al, be);
  return k;
}
constexpr int kNCorr = count_corr();
struct CorrTerm {
  int al, be, q;
  double coef;
};
struct CorrTerms {
  CorrTerm t[kNCorr];
};
// (source moment outer, as for the local terms)
constexpr CorrTerms make_corr() {
  CorrTerms r{};
  int k = 0;
  for (int be = 0; be < kNL; ++be)
    for (int al = 0; al < kNL; ++al)
      if (corr_term(al, be)) {
        const int a = kMI.a[al] + kMI.a[be], b = kMI.b[al] + kMI.b[be], c = kMI.c[al] + kMI.c[be];
        const int sb = kMI.n[be] % 2 ? -1 : 1;
        const int g = mi_id(a, b, c);
        r.t[k++] = {al, be, g - num_mi(kP - 1), sb * kMI.fact[g] / (kMI.fact[al] * kMI.fact[be])};
      }
  return r;
}
constexpr CorrTerms kCorr = make_corr();

// moment shift: M_parent[be] += coef M_child[ga] s^[d], coef = C(be, ga)
constexpr bool shift_term(int be, int ga) {
  return kMI.a[ga] <= kMI.a[be] && kMI.b[ga] <= kMI.b[be] && kMI.c[ga] <= kMI.c[be];
}
constexpr int count_shift() {
  int k = 0;
  for (int be = 0; be < kNL; ++be)
    for (int ga = 0; ga < kNL; ++ga) k += shift_term(be, ga);
  return k;
}
constexpr int kNShift = count_shift();
struct ShiftTerms {
  Term t[kNShift];  // al: the parent's moment, be: the child's, g: the power of s
};
constexpr ShiftTerms make_shift() {
  ShiftTerms r{};
  int k = 0;
  for (int be = 0; be < kNL; ++be)
    for (int ga = 0; ga < kNL; ++ga)
      if (shift_term(be, ga))
        r.t[k++] = {be, ga, mi_id(kMI.a[be] - kMI.a[ga], kMI.b[be] - kMI.b[ga], kMI.c[be] - kMI.c[ga]),
                    binom(kMI.a[be], kMI.a[ga]) * binom(kMI.b[be], kMI.b[ga]) * binom(kMI.c[be], kMI.c[ga])};
  return r;
}
constexpr ShiftTerms kShift = make_shift();
static_assert(kNLocal == 135 && kNCorr == 66, "term counts at P = 4");

// Derivative terms: D_gamma = sum over the pairings (p, q, r pairs among the
// x, y and z indices of gamma) of f_(|gamma| - p - q - r) times the number of
// such pairings times R^(gamma - 2 (p, q, r)).
struct DerivTerm {
  int g, f, e0, e1, e2;
  double coef;
};
constexpr int count_deriv() {
  int k = 0;
  for (int g = 0; g < kNL; ++g) k += (kMI.a[g] / 2 + 1) * (kMI.b[g] / 2 + 1) * (kMI.c[g] / 2 + 1);
  return k;
}
constexpr int kNDeriv = count_deriv();
struct DerivTerms {
  DerivTerm t[kNDeriv];
};
constexpr DerivTerms make_deriv() {
  DerivTerms r{};
  int k = 0;
  for (int g = 0; g < kNL; ++g)
    for (int p = 0; 2 * p <= kMI.a[g]; ++p)
      for (int q = 0; 2 * q <= kMI.b[g]; ++q)
        for (int u = 0; 2 * u <= kMI.c[g]; ++u)
          r.t[k++] = {g, kMI.n[g] - p - q - u, kMI.a[g] - 2 * p, kMI.b[g] - 2 * q, kMI.c[g] - 2 * u,
                      pair_ways(kMI.a[g], p) * pair_ways(kMI.b[g], q) * pair_ways(kMI.c[g], u)};
  return r;
}
constexpr DerivTerms kDeriv = make_deriv();

// The radial factors f_k = (1/R d/dR)^k g of g = -1/sqrt(R^2 + eps^2),
// f_0 = -1/sqrt(s), f_(k+1) = -(2k+1) f_k / s (1/s = f_0^2)
__device__ inline void radial(const double R[3], double eps2, double f[kP + 2]) {
  f[0] = -rsqrt_f64(((R[0] * R[0] + R[1] * R[1]) + R[2] * R[2]) + eps2);
  const double is = f[0] * f[0];
#pragma unroll
  for (int k = 0; k <= kP; ++k) f[k + 1] = (-(2.0 * k + 1.0) * f[k]) * is;
}

// the radial factors and the powers R_i^k, k <= P
__device__ inline void radial_and_powers(const double R[3], double eps2, double f[kP + 2], double pw[3][kP + 1]) {
  radial(R, eps2, f);
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    pw[i][0] = 1.0;
#pragma unroll
    for (int k = 0; k < kP; ++k) pw[i][k + 1] = pw[i][k] * R[i];
  }
}

// D_gamma(R) for |gamma| <= P
__device__ inline void derivatives(const double R[3], double eps2, double D[kNL]) {
  double f[kP + 2], pw[3][kP + 1];
  radial_and_powers(R, eps2, f, pw);
#pragma unroll
  for (int g = 0; g < kNL; ++g) D[g] = 0.0;
#pragma unroll
  for (int i = 0; i < kNDeriv; ++i) {
    const DerivTerm& t = kDeriv.t[i];
    D[t.g] = fma(f[t.f], t.coef * ((pw[0][t.e0] * pw[1][t.e1]) * pw[2][t.e2]), D[t.g]);
  }
}

// push-down shift: L'[al] += L[g] d^[ga] / ga!, g = al + ga, |al| + |ga| <= P
constexpr int count_l2l() {
  int k = 0;
  for (int al = 0; al < kNL; ++al)
    for (int ga = 0; ga < kNL; ++ga) k += kMI.n[al] + kMI.n[ga] <= kP;
  return k;
}
constexpr int kNL2L = count_l2l();
struct L2LTerms {
  Term t[kNL2L];  // al: the child's coefficient, be: the power of d, g: the parent's coefficient
};
constexpr L2LTerms make_l2l() {
  L2LTerms r{};
  int k = 0;
  for (int al = 0; al < kNL; ++al)
    for (int ga = 0; ga < kNL; ++ga)
      if (kMI.n[al] + kMI.n[ga] <= kP)
        r.t[k++] = {al, ga, mi_id(kMI.a[al] + kMI.a[ga], kMI.b[al] + kMI.b[ga], kMI.c[al] + kMI.c[ga]),
                    1.0 / kMI.fact[ga]};
  return r;
}
constexpr L2LTerms kL2L = make_l2l();

// x^alpha, |alpha| <= P
__device__ inline void monomials(const double x[3], double X[kNL]) {
  double pw[3][kP + 1];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    pw[i][0] = 1.0;
#pragma unroll
    for (int k = 0; k < kP; ++k) pw[i][k + 1] = pw[i][k] * x[i];
  }
#pragma unroll
  for (int g = 0; g < kNL; ++g) X[g] = (pw[0][kMI.a[g]] * pw[1][kMI.b[g]]) * pw[2][kMI.c[g]];
}

__device__ inline double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// leaf moments from the particles, in key order (one thread per leaf)
__global__ void __launch_bounds__(kBS) k_mono_leaves(const double4* __restrict__ pos,
                                                     const int32_t* __restrict__ leaves, int32_t nleaves,
                                                     const int32_t* __restrict__ beg, const int32_t* __restrict__ cnt,
                                                     const double4* __restrict__ geo, double* __restrict__ mono) {
  const int32_t i = blockIdx.x * kBS + threadIdx.x;
  if (i >= nleaves) return;
  const int32_t c = leaves[i];
  const double4 z = geo[c];
  double acc[kNL];
#pragma unroll
  for (int g = 0; g < kNL; ++g) acc[g] = 0.0;
  for (int32_t p = beg[c]; p < beg[c] + cnt[c]; ++p) {
    const double4 q = pos[p];
    const double x[3] = {q.x - z.x, q.y - z.y, q.z - z.z};
    double X[kNL];
    monomials(x, X);
#pragma unroll
    for (int g = 0; g < kNL; ++g) acc[g] += q.w * X[g];
  }
  double* o = mono + (int64_t)c * kNL;
#pragma unroll
  for (int g = 0; g < kNL; ++g) o[g] = acc[g];
}

// parent moments: each child's shifted by s = Z_child - Z_parent,
// M_beta += sum_{gamma <= beta} C(beta, gamma) M_child,gamma s^(beta-gamma),
// children in octant order (one thread per parent)
__global__ void __launch_bounds__(kBS) k_mono_up(int32_t c0, int32_t nl, const int32_t* __restrict__ ch0,
                                                 const int32_t* __restrict__ nch, const double4* __restrict__ geo,
                                                 double* __restrict__ mono) {
  const int32_t i = blockIdx.x * kBS + threadIdx.x;
  if (i >= nl) return;
  const int32_t c = c0 + i;
  if (nch[c] == 0) return;
  const double4 zp = geo[c];
  double acc[kNL];
#pragma unroll
  for (int g = 0; g < kNL; ++g) acc[g] = 0.0;
  for (int32_t k = ch0[c]; k < ch0[c] + nch[c]; ++k) {
    const double4 zc = geo[k];
    const double s[3] = {zc.x - zp.x, zc.y - zp.y, zc.z - zp.z};
    double S[kNL];
    monomials(s, S);
    const double* m = mono + (int64_t)k * kNL;
    double mc[kNL];
#pragma unroll
    for (int g = 0; g < kNL; ++g) mc[g] = m[g];
#pragma unroll
    for (int i = 0; i < kNShift; ++i) acc[kShift.t[i].al] += kShift.t[i].coef * mc[kShift.t[i].be] * S[kShift.t[i].g];
  }
  double* o = mono + (int64_t)c * kNL;
#pragma unroll
  for (int g = 0; g < kNL; ++g) o[g] = acc[g];
}

// Source records of the far field and the correction, kRec doubles a cell: the
// order-4 moments, centre, mass, the order-2 moments, which both need, and the
// order-3 ones times their factor (kSign: each has one use), placed so that the
// correction reads the first kCorrPieces times 16 bytes and the far field
// the last kFarPieces (dipole moments enter neither).
constexpr int kRecH = 0, kRecZ = 16, kRecQ = 20, kRecO = 26, kRec = 36;
constexpr int kMiQ = num_mi(1), kMiO = num_mi(2), kMiH = num_mi(3);
constexpr int kCorrPieces = kRecO / 2, kFarPieces = (kRec - kRecZ) / 2;
static_assert(kRecH + kNL - kMiH <= kRecZ && kRecQ + kMiO - kMiQ == kRecO && kRecO + kMiH - kMiO == kRec && kP == 4,
              "source record");

// value i of a cell's record, in powers of two of the box's side and the total
// mass (see FarUnit: in the caller's units the correction's M^2 R^8 leaves the
// exponent range at lengths of 10^18 with masses of 10^96)
__device__ inline double record_value(int i, const double4* __restrict__ z, const double* __restrict__ m,
                                      const FarUnit& unit) {
  if (i < kRecZ) return i - kRecH < kNL - kMiH ? unit.moment(m[kMiH + i - kRecH], 4) : 0.0;
  if (i < kRecZ + 3) return unit.length(((const double*)z)[i - kRecZ]);
  if (i < kRecQ) return unit.moment(m[0], 0);
  if (i < kRecO) return unit.moment(m[kMiQ + i - kRecQ], 2);
  return kSign.c[kMiO + i - kRecO] * unit.moment(m[kMiO + i - kRecO], 3);
}

// (one thread per 16 bytes)
__global__ void __launch_bounds__(kBS) k_pack_order(int32_t nc, const double4* __restrict__ geo,
                                                    const double* __restrict__ mono, int el,
                                                    double2* __restrict__ out) {
  const int64_t t = (int64_t)blockIdx.x * kBS + threadIdx.x;
  const int64_t c = t / (kRec / 2);
  if (c >= nc) return;
  const int p = 2 * (int)(t - c * (kRec / 2));
  const FarUnit unit(el, mono);
  const double* m = mono + c * kNL;
  out[t] = make_double2(record_value(p, geo + c, m, unit), record_value(p + 1, geo + c, m, unit));
}

// PIECES times 16 bytes of the record of cell y, from value FROM on, without the
// records: where they have no room (the same values, so the same results)
template <int FROM, int PIECES>
__device__ __forceinline__ void gather_record(const double4* __restrict__ geo, const double* __restrict__ mono,
                                              int32_t y, const FarUnit& unit, double v[2 * PIECES]) {
#pragma unroll
  for (int i = 0; i < 2 * PIECES; ++i) v[i] = record_value(FROM + i, geo + y, mono + (int64_t)y * kNL, unit);
}

// 64 records (PIECES times 16 bytes of each, from `from` on) to the wave's LDS,
// record after record: lane l takes pieces l, l + 64, ... of the row, so that
// neighbouring lanes read neighbouring bytes.  What bounded both kernels was the
// vector cache, which answers one request of up to 64 bytes a cycle: a lane that
// loads its own source takes one for every 16 bytes (12 and 15 a source), this
// way it is 3 and 4.  4M particles: 3.4 -> 2.6 and 3.7 -> 2.3 ms (of the latter 0.5 by
// corr_force); now 290 and 225 FP64 instructions a source bound them.
template <int PIECES>
__device__ __forceinline__ void fetch_records(const double2* __restrict__ from, int32_t y, int lane, double2* buf) {
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    const int q = 64 * i + lane, r = q / PIECES;
    const double2* src = from + (int64_t)__shfl(y, r, 64) * (kRec / 2) + (q - r * PIECES);
    __builtin_amdgcn_global_load_lds((__attribute__((address_space(1))) void*)src,
                                     (__attribute__((address_space(3))) void*)(buf + 64 * i), 16, 0, 0);
  }
}

// This lane's record out of LDS, then the next 64 on their way (lanes past the
// end fetch the target's and do not use it).
template <int PIECES>
__device__ __forceinline__ void take_record(const double2* __restrict__ from, const int32_t* __restrict__ src,
                                            int32_t j0, int32_t cnt, int32_t X, int lane, double2* buf, int32_t& ahead,
                                            double v[2 * PIECES]) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int q = 0; q < PIECES; ++q) {
    const double2 w = buf[PIECES * lane + q];
    v[2 * q] = w.x;
    v[2 * q + 1] = w.y;
  }
  // every lane's record is in registers before the next ones arrive
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  if (j0 + 64 < cnt) {
    fetch_records<PIECES>(from, ahead, lane, buf);
    const int32_t j2 = j0 + 128 + lane;
    ahead = j2 < cnt ? src[j2] : X;
  }
}

// Sums of 40 values over the wave, halved between exchanges (40 -> 20 -> 10 ->
// 5 in each lane): 35 and 15 exchanges instead of 240.  Lane l ends with the
// totals of values 20 bit5 + 10 bit4 + 5 bit3 of l, and the four after it; the
// additions of one value pair lanes as a butterfly over 32, 16, ..., 1 does.
__device__ inline int wave_sum40(double v[40], int lane, double out[5]) {
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    const int off = 32 >> s, half = 20 >> s;
    const bool hi = lane & off;
#pragma unroll
    for (int k = 0; k < half; ++k) {
      const double send = hi ? v[k] : v[k + half], keep = hi ? v[k + half] : v[k];
      v[k] = keep + __shfl_xor(send, off, 64);
    }
  }
#pragma unroll
  for (int k = 0; k < 5; ++k) {
    out[k] = v[k];
#pragma unroll
    for (int off = 4; off > 0; off >>= 1) out[k] += __shfl_xor(out[k], off, 64);
  }
  return 20 * ((lane >> 5) & 1) + 10 * ((lane >> 4) & 1) + 5 * ((lane >> 3) & 1);
}

// Far field of one target cell per wave: its local coefficients (locg: kNL
// coefficients, then g_c, zero here: k_corr_order sets it for TC) and, for
// the order-3 kernels that run after it, zeros in its loc record (the
// evaluation at the particles adds this expansion separately).  One wave per
// workgroup here and in k_corr_order (4M particles, both: 7.8 -> 6.9 ms).
template <bool REC>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(2))) k_far_order(
    int32_t c_lo, const double2* __restrict__ rec, const double4* __restrict__ geo, const double* __restrict__ mono,
    const int64_t* __restrict__ fstart, const int32_t* __restrict__ fcount, const int32_t* __restrict__ fsrc, int el,
    double* __restrict__ locg, double* __restrict__ loc, double eps2, unsigned long long* clock) {
  take_time(clock);
  __shared__ double2 buf[REC ? 64 * kFarPieces : 1];
  const int lane = threadIdx.x;
  const int32_t X = c_lo + (int32_t)xcd_block(blockIdx.x, gridDim.x);
  const int32_t cnt = uniform(fcount[X]);
  const int32_t* __restrict__ src = fsrc + fstart[X];
  const double2* __restrict__ from = rec + kRecZ / 2;
  const FarUnit unit(el, mono);
  const double* zx = REC ? (const double*)(from + (int64_t)X * (kRec / 2)) : (const double*)(geo + X);
  const double gx[3] = {REC ? zx[0] : unit.length(zx[0]), REC ? zx[1] : unit.length(zx[1]),
                        REC ? zx[2] : unit.length(zx[2])};
  double L[kNL];
#pragma unroll
  for (int g = 0; g < kNL; ++g) L[g] = 0.0;
  int32_t ahead = REC && lane + 64 < cnt ? src[lane + 64] : X;
  if (REC && cnt > 0) fetch_records<kFarPieces>(from, lane < cnt ? src[lane] : X, lane, buf);
  for (int32_t j0 = 0; j0 < cnt; j0 += 64) {
    double v[2 * kFarPieces];
    if (REC) take_record<kFarPieces>(from, src, j0, cnt, X, lane, buf, ahead, v);
    else gather_record<kRecZ, kFarPieces>(geo, mono, j0 + lane < cnt ? src[j0 + lane] : X, unit, v);
    if (j0 + lane < cnt) {
      const double R[3] = {gx[0] - v[0], gx[1] - v[1], gx[2] - v[2]};
      double D[kNL];
      derivatives(R, eps2, D);
      // source moments times their factor, then one fma per term
      auto cm = [&](int be) {
        return be == 0 ? kSign.c[0] * v[3]
                       : (be < kMiO ? kSign.c[be] * v[kRecQ - kRecZ + be - kMiQ] : v[kRecO - kRecZ + be - kMiO]);
      };
#pragma unroll
      for (int i = 0; i < kNLocal; ++i)
        L[kLocal.t[i].al] = fma(D[kLocal.t[i].g], cm(kLocal.t[i].be), L[kLocal.t[i].al]);
    }
  }
  double v[40], t[5];
#pragma unroll
  for (int g = 0; g < 40; ++g) v[g] = g < kNL ? L[g] : 0.0;
  static_assert(kNL <= 40 && kLocGen == 40, "sums of 40");
  const int first = wave_sum40(v, lane, t), k = lane & 7;
  if (k < 5) {
    const int i = first + k, order = i >= kMiH ? 4 : (i >= kMiO ? 3 : (i >= kMiQ ? 2 : (i >= 1 ? 1 : 0)));
    const double s = k == 0 ? t[0] : (k == 1 ? t[1] : (k == 2 ? t[2] : (k == 3 ? t[3] : t[4])));
    locg[(int64_t)X * kLocGen + i] = unit.coefficient(s, order);
  }
  if (lane < kLoc) loc[(int64_t)X * kLoc + lane] = 0.0;
  static_assert(kLoc <= 64, "one lane a coefficient");
}

// F_k -= sum over index tuples of q_ijlm D_ijlmk, without the 21 derivatives:
// pairing the equal indices of D = f_5 RRRRR + f_4 sum_10 delta RRR + f_3 sum_15
// delta delta R inside the symmetric tensor q leaves, with q3_k = q_kijl R_i R_j
// R_l, q4 = q3 R, the trace t_kl = q_iikl, t1 = t R, t2 = t1 R and t0 = tr t,
//   (f_5 q4 + 6 f_4 t2 + 3 f_3 t0) R_k + 4 f_4 q3_k + 12 f_3 t1_k
// (202 instead of 301 instructions a source; 2.8 -> 2.3 ms at 4M particles).
__device__ inline void corr_force(const double R[3], double eps2, const double* q, double F[3]) {
  constexpr int kQ0 = num_mi(kP - 1);
  double f[kP + 2], X[kNL];
  radial(R, eps2, f);
  monomials(R, X);
  double q3[3] = {0.0, 0.0, 0.0}, t1[3] = {0.0, 0.0, 0.0}, t[6];
#pragma unroll
  for (int b = num_mi(2); b < num_mi(3); ++b) {
    const double w = (6.0 / kMI.fact[b]) * X[b];
#pragma unroll
    for (int k = 0; k < 3; ++k)
      q3[k] = fma(q[mi_id(kMI.a[b] + (k == 0), kMI.b[b] + (k == 1), kMI.c[b] + (k == 2)) - kQ0], w, q3[k]);
  }
#pragma unroll
  for (int d = num_mi(1); d < num_mi(2); ++d) {
    const int a = kMI.a[d], b = kMI.b[d], c = kMI.c[d];
    t[d - num_mi(1)] = (q[mi_id(a + 2, b, c) - kQ0] + q[mi_id(a, b + 2, c) - kQ0]) + q[mi_id(a, b, c + 2) - kQ0];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int i = 0; i < 3; ++i)
      t1[k] = fma(t[mi_id((k == 0) + (i == 0), (k == 1) + (i == 1), (k == 2) + (i == 2)) - num_mi(1)], R[i], t1[k]);
  const double q4 = fma(q3[0], R[0], fma(q3[1], R[1], q3[2] * R[2]));
  const double t2 = fma(t1[0], R[0], fma(t1[1], R[1], t1[2] * R[2]));
  const double t0 = (t[mi_id(2, 0, 0) - num_mi(1)] + t[mi_id(0, 2, 0) - num_mi(1)]) + t[mi_id(0, 0, 2) - num_mi(1)];
  const double a = fma(f[5], q4, fma(6.0 * f[4], t2, (3.0 * f[3]) * t0));
#pragma unroll
  for (int k = 0; k < 3; ++k) F[k] -= fma(a, R[k], fma(4.0 * f[4], q3[k], (12.0 * f[3]) * t1[k]));
}

// The correction (TC) of one target cell per wave over the same sources:
// g_c = F_c / M_X into locg (after k_far_order).  Only the order-(P+1)
// derivatives and the moments of orders 0, 2 and P enter.
template <bool REC>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3))) k_corr_order(
    int32_t c_lo, const double2* __restrict__ rec, const double4* __restrict__ geo, const double* __restrict__ mono,
    const int64_t* __restrict__ fstart, const int32_t* __restrict__ fcount, const int32_t* __restrict__ fsrc, int el,
    double* __restrict__ locg, double eps2) {
  constexpr int kNQ = num_mi(kP) - num_mi(kP - 1);  // order-P components
  __shared__ double2 buf[REC ? 64 * kCorrPieces : 1];
  const int lane = threadIdx.x;
  const int32_t X = c_lo + (int32_t)xcd_block(blockIdx.x, gridDim.x);
  const int32_t cnt = uniform(fcount[X]);
  const int32_t* __restrict__ src = fsrc + fstart[X];
  const FarUnit unit(el, mono);
  // the target's record in scalar registers
  double own[2 * kCorrPieces];
  if (REC) {
#pragma unroll
    for (int i = 0; i < 2 * kCorrPieces; ++i) own[i] = ((const double*)(rec + (int64_t)X * (kRec / 2)))[i];
  } else {
    gather_record<0, kCorrPieces>(geo, mono, X, unit, own);
  }
#pragma unroll
  for (int i = 0; i < 2 * kCorrPieces; ++i) own[i] = uniform_f64(own[i]);
  const double gx[3] = {own[kRecZ], own[kRecZ + 1], own[kRecZ + 2]};
  const double MX = own[kRecZ + 3];
  double F[3] = {0.0, 0.0, 0.0};
  int32_t ahead = REC && lane + 64 < cnt ? src[lane + 64] : X;
  if (REC && cnt > 0) fetch_records<kCorrPieces>(rec, lane < cnt ? src[lane] : X, lane, buf);
  for (int32_t j0 = 0; j0 < cnt; j0 += 64) {
    double v[2 * kCorrPieces];
    if (REC) take_record<kCorrPieces>(rec, src, j0, cnt, X, lane, buf, ahead, v);
    else gather_record<0, kCorrPieces>(geo, mono, j0 + lane < cnt ? src[j0 + lane] : X, unit, v);
    if (j0 + lane < cnt) {
      const double R[3] = {gx[0] - v[kRecZ], gx[1] - v[kRecZ + 1], gx[2] - v[kRecZ + 2]};
      double Q[kNQ];
#pragma unroll
      for (int q = 0; q < kNQ; ++q) Q[q] = 0.0;
      // (the constant goes with the source moment: products shared between terms)
      auto moment = [](const double* r, int be) {
        return be == 0 ? r[kRecZ + 3] : (be < kMiO ? r[kRecQ + be - kMiQ] : r[kRecH + be - kMiH]);
      };
#pragma unroll
      for (int i = 0; i < kNCorr; ++i) {
        const CorrTerm& c = kCorr.t[i];
        Q[c.q] = fma(moment(own, c.al), c.coef * moment(v, c.be), Q[c.q]);
      }
      corr_force(R, eps2, Q, F);
    }
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) F[k] = wave_sum(F[k]);
  if (lane == 0) {
    double* o = locg + (int64_t)X * kLocGen;
#pragma unroll
    for (int k = 0; k < 3; ++k) o[kNL + k] = unit.coefficient(F[k] / (24.0 * MX), 1);  // P! M_X
  }
}

// locg[child] += the parent's expansion shifted to the child's centre,
// L'_alpha = sum_gamma L_(alpha+gamma) d^gamma / gamma!, d = Z_child - Z_parent;
// g_c adds (one thread per child)
__global__ void __launch_bounds__(kBS) k_l2l_order(int32_t c0, int32_t nl, const int32_t* __restrict__ par,
                                                   const double4* __restrict__ geo, double* __restrict__ locg,
                                                   unsigned long long* clock) {
  take_time(clock);
  const int32_t i = blockIdx.x * kBS + threadIdx.x;
  if (i >= nl) return;
  const int32_t c = c0 + i;
  const int32_t P = par[c];
  const double4 gc = geo[c], gp = geo[P];
  const double d[3] = {gc.x - gp.x, gc.y - gp.y, gc.z - gp.z};
  double Dm[kNL];
  monomials(d, Dm);
  const double* L = locg + (int64_t)P * kLocGen;
  double* o = locg + (int64_t)c * kLocGen;
  double Lp[kNL], acc[kNL];
#pragma unroll
  for (int g = 0; g < kNL; ++g) {
    Lp[g] = L[g];
    acc[g] = 0.0;
  }
#pragma unroll
  for (int i = 0; i < kNL2L; ++i) acc[kL2L.t[i].al] += Lp[kL2L.t[i].g] * (Dm[kL2L.t[i].be] * kL2L.t[i].coef);
#pragma unroll
  for (int g = 0; g < kNL; ++g) o[g] += acc[g];
#pragma unroll
  for (int k = 0; k < 3; ++k) o[kNL + k] += L[kNL + k];
}

// At every particle of the target leaves: G times minus the gradient of the
// leaf's expansion, plus g_c, added to the near field's outputs (caller
// order); the potential likewise (kL2PLanes lanes per leaf, over its particles).
// leaves == nullptr: the leaves among cells [c_lo, c_lo + count).
__global__ void __launch_bounds__(kBS) k_l2p_order(int32_t count, const int32_t* __restrict__ leaves, int32_t c_lo,
                                                   const int32_t* __restrict__ nch, const int32_t* __restrict__ beg,
                                                   const int32_t* __restrict__ cnt, const double4* __restrict__ pos,
                                                   const double4* __restrict__ geo, const double* __restrict__ locg,
                                                   const int32_t* __restrict__ perm, double G,
                                                   double* __restrict__ ax, double* __restrict__ ay,
                                                   double* __restrict__ az, double* __restrict__ pot) {
  // kL2PLanes lanes per leaf (leaves hold a few particles each)
  const int64_t li = ((int64_t)blockIdx.x * kBS + threadIdx.x) / kL2PLanes;
  const int sl = (int)(threadIdx.x % kL2PLanes);
  if (li >= count) return;
  const int32_t X = leaves ? leaves[li] : c_lo + (int32_t)li;
  if (!leaves && nch[X] != 0) return;
  const double4 z = geo[X];
  const double* L = locg + (int64_t)X * kLocGen;
  for (int32_t p = beg[X] + sl; p < beg[X] + cnt[X]; p += kL2PLanes) {
    const double4 q = pos[p];
    const double x[3] = {q.x - z.x, q.y - z.y, q.z - z.z};
    double Xm[kNL];
    monomials(x, Xm);
    // x^al / al!, the reciprocal factorials as constants
#pragma unroll
    for (int al = 0; al < kNL; ++al) Xm[al] *= kInvFact.c[al];
    double phi = 0.0;
#pragma unroll
    for (int al = 0; al < kNL; ++al) phi = fma(Xm[al], L[al], phi);
    double g[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      double s = 0.0;
#pragma unroll
      for (int al = 0; al < kNL; ++al) {
        if (kMI.n[al] >= kP) continue;
        s = fma(Xm[al], L[mi_id(kMI.a[al] + (k == 0), kMI.b[al] + (k == 1), kMI.c[al] + (k == 2))], s);
      }
      g[k] = -s + L[kNL + k];
    }
    const int32_t o = perm[p];
    ax[o] += G * g[0];
    ay[o] += G * g[1];
    az[o] += G * g[2];
    if (pot) pot[o] += G * phi;
  }
}

}  // namespace

void order_upward(Ctx& c) {
  const int32_t nc = c.ncells;
  double* mono = (double*)ensure(c, c.mono, sizeof(double) * kNL * (size_t)nc);
  hipLaunchKernelGGL(k_mono_leaves, dim3(blocks_for(c.nleaves, kBS)), dim3(kBS), 0, c.stream,
                     (const double4*)c.pos4.p, as<int32_t>(c.leaves), c.nleaves, as<int32_t>(c.c_begin),
                     as<int32_t>(c.c_count), (const double4*)c.geo.p, mono);
  AMFMM_HIP(hipGetLastError());
  for (int l = c.depth - 1; l >= 0; --l) {
    const int32_t c0 = c.level_start[l], nl = c.level_start[l + 1] - c0;
    hipLaunchKernelGGL(k_mono_up, dim3(blocks_for(nl, kBS)), dim3(kBS), 0, c.stream, c0, nl,
                       as<int32_t>(c.c_child0), as<int32_t>(c.c_nchild), (const double4*)c.geo.p, mono);
    AMFMM_HIP(hipGetLastError());
  }
}

void order_pack(Ctx& c) {
  double2* rec = (double2*)ensure_if_room(c, c.farrec, sizeof(double) * kRec * (size_t)c.ncells);
  if (!rec) return;
  hipLaunchKernelGGL(k_pack_order, dim3(blocks_for((int64_t)c.ncells * (kRec / 2), kBS)), dim3(kBS), 0, c.stream,
                     c.ncells, (const double4*)c.geo.p, (const double*)c.mono.p, length_exponent(c), rec);
  AMFMM_HIP(hipGetLastError());
}

void order_far(Ctx& c, int32_t c_lo, int32_t c_hi, double* loc) {
  const int32_t nc = c_hi - c_lo;
  if (nc <= 0) return;
  double* locg = (double*)ensure_keep(c, c.locg, sizeof(double) * kLocGen * (size_t)c.ncells,
                                      sizeof(double) * kLocGen * (size_t)c.ncells);
  const bool recs = c.farrec.p != nullptr;
  const int el = length_exponent(c);
  const double eps = std::ldexp(c.opt.softening, -el), eps2 = eps * eps;
  hipLaunchKernelGGL(recs ? k_far_order<true> : k_far_order<false>, dim3(nc), dim3(64), 0, c.stream, c_lo,
                     (const double2*)c.farrec.p, (const double4*)c.geo.p, (const double*)c.mono.p,
                     (const int64_t*)c.far_start.p, (const int32_t*)c.far_count.p, (const int32_t*)c.far_src.p, el,
                     locg, loc, eps2, clock_word(c));
  AMFMM_HIP(hipGetLastError());
  if (c.opt.variant != AMFMM_UC) {
    hipLaunchKernelGGL(recs ? k_corr_order<true> : k_corr_order<false>, dim3(nc), dim3(64), 0, c.stream, c_lo,
                       (const double2*)c.farrec.p, (const double4*)c.geo.p, (const double*)c.mono.p,
                       (const int64_t*)c.far_start.p, (const int32_t*)c.far_count.p, (const int32_t*)c.far_src.p, el,
                       locg, eps2);
    AMFMM_HIP(hipGetLastError());
  }
}

void order_push_down(Ctx& c, int32_t c_lo, int32_t c_hi) {
  const int32_t nl = c_hi - c_lo;
  if (nl <= 0) return;
  hipLaunchKernelGGL(k_l2l_order, dim3(blocks_for(nl, kBS)), dim3(kBS), 0, c.stream, c_lo, nl,
                     as<int32_t>(c.c_parent), (const double4*)c.geo.p, as<double>(c.locg), clock_word(c));
  AMFMM_HIP(hipGetLastError());
}

void order_l2p(Ctx& c, const int32_t* leaves, int32_t c_lo, int32_t count, double* ax, double* ay, double* az,
               double* pot) {
  if (count <= 0) return;
  hipLaunchKernelGGL(k_l2p_order, dim3(blocks_for((int64_t)count * kL2PLanes, kBS)), dim3(kBS), 0, c.stream, count,
                     leaves, c_lo,
                     as<int32_t>(c.c_nchild), as<int32_t>(c.c_begin), as<int32_t>(c.c_count),
                     (const double4*)c.pos4.p, (const double4*)c.geo.p, (const double*)c.locg.p, as<int32_t>(c.perm),
                     c.opt.G, ax, ay, az, pot);
  AMFMM_HIP(hipGetLastError());
}

}  // namespace amfmm
