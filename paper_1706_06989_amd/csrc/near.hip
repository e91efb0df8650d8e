// Near field (direct summation between particles of non-accepted leaf pairs),
// fused with the evaluation of the far-field coefficients at each particle and
// the scatter back to caller order.
//
// One wave per target leaf, and per workgroup: lists differ, and four waves in
// a workgroup hold its LDS and registers until the longest is done (one instead
// of four: 262144 particles at the benchmark's tolerance 17.0 -> 12.8 ms, 16.8M
// 196 -> 165, 4M two spheres at FP64 11.6 -> 10.2).  Each lane holds K targets in registers
// (register blocking: one source load feeds K interactions) and a slice of
// the sources; lanes = (target group g, slice s), 64 / groups slices per group
// (any count: the partial sums of a group reduce over a fixed tree into its
// first lane, deterministic).  K is 1, 2 or 4, chosen per leaf to waste the
// fewest lanes (leaves hold a few particles: 7 on average at n_crit = 25).
// The leaf's source entries are staged in LDS a bufferful at a time,
// consecutive lanes copying consecutive particles.
//
// A leaf in the outskirts can face a whole core: its list is hundreds of
// times the average and one wave's run over it was most of the phase (2.3 of
// 2.4 ms at 100003 particles, theta 0.5).  Lists that cost more than twice a
// share of the phase's total are cut into segments of whole buffer fills, one
// wave each, which run first; k_near_join adds up their partial sums in segment
// order.  The fills, and so the FP32 blocks, are those of the uncut list.  (One
// kernel with the last segment to end adding them up needs a device-wide fence
// per segment: 0.99 instead of 0.33 ms for a pilot solve at 262144.)
//
// Mixed precision: targets and staged sources are FP32 offsets from the
// target leaf's centre of mass (each difference taken in FP64, then rounded),
// the pair terms are FP32 (hardware reciprocal square root), and each lane's
// FP32 sums run over at most kFlush sources before they are flushed into a
// compensated FP64 sum per target and component: an FP64 accumulator plus the
// rounding error of every addition to it (TwoSum, Knuth), collected in an
// FP32 compensation term (the errors are below 2^-53 of the sum, so FP32
// holds them to far below FP64 resolution).  The slices of a target are
// reduced the same way; the compensation is added back once, before L2P.
// L2P and the output stay FP64.
#include <cstdio>
#include <cstdlib>

#include "device_math.h"
#include "internal.h"

namespace amfmm {
namespace {

constexpr int kBS = 256;
constexpr int kWaves = kBS / 64;
constexpr int kTGMax = 4; // targets per lane: 1, 2 or 4
// source particles staged in LDS: 10 KB a workgroup of one wave, so 16 of them fit
// a CU's 160 KB, the four waves a SIMD that the registers allow
constexpr int kCap = 320;

__device__ inline int pow2floor(int v) { return 1 << (31 - __builtin_clz(v)); }

constexpr int kFlush = 32;  // FP32 terms per lane and target before an FP64 flush

// s + b = s' + e exactly (TwoSum: six operations, no condition on the
// magnitudes; the library is built without contraction, so no step fuses);
// s <- s', the rounding error e goes to the compensation term c
__device__ inline void comp_add(double& s, float& c, double b) {
  const double t = s + b;
  const double bp = t - s;
  const double e = (s - (t - bp)) + (b - bp);
  s = t;
  c += (float)e;
}

// One source and this lane's kTG targets in FP32.  MASK: a pair at r = 0 is
// skipped; without it such a pair makes gp infinite or NaN (the root's estimate
// is infinite there).  SOFT: the softened kernel, 1/(r^2 + eps2)^{1/2} and
// ^{3/2} (Sec. 4).
template <int kTG, bool SOFT, bool MASK>
__device__ __forceinline__ void pairs_f32(const float4 q, const float* tx, const float* ty, const float* tz, float* gx,
                                          float* gy, float* gz, float* gp, float eps2) {
#pragma unroll
  for (int u = 0; u < kTG; ++u) {
    const float dx = q.x - tx[u], dy = q.y - ty[u], dz = q.z - tz[u];
    const float r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
    float y = __builtin_amdgcn_rsqf(SOFT ? r2 + eps2 : r2);
    if (MASK) y = r2 > 0.0f ? y : 0.0f;
    const float my = q.w * y;
    const float my3 = my * (y * y);
    gx[u] = fmaf(my3, dx, gx[u]);
    gy[u] = fmaf(my3, dy, gy[u]);
    gz[u] = fmaf(my3, dz, gz[u]);
    gp[u] -= my;
  }
}

// FP32 interactions of this lane's targets (offsets t*) with sources
// p[0], p[nsl], ...: `n` of them for every lane, and one more where `extra`.
template <int kTG, bool SOFT, bool MASK>
__device__ __forceinline__ void near_run_f32(const float4* p, int n, bool extra, int nsl, const float* tx,
                                             const float* ty, const float* tz, float* gx, float* gy, float* gz,
                                             float* gp, float eps2) {
#pragma unroll
  for (int u = 0; u < kTG; ++u) gx[u] = gy[u] = gz[u] = gp[u] = 0.0f;
#pragma unroll(kTG == 4 ? 1 : 4 / kTG)
  for (int i = 0; i < n; ++i, p += nsl) pairs_f32<kTG, SOFT, MASK>(*p, tx, ty, tz, gx, gy, gz, gp, eps2);
  if (extra) pairs_f32<kTG, SOFT, MASK>(*p, tx, ty, tz, gx, gy, gz, gp, eps2);
}

// A buffer of `fill` sources, this lane taking s, s + nsl, ...; FP32 sums of at
// most kFlush terms flushed into the compensated FP64 sums (f*, compensation
// terms c*).  All lanes run the same count (fill / nsl, one more for the first
// fill % nsl lanes), so the loop's counter is scalar.  Coincident pairs are rare
// (a leaf meets itself once): blocks run without the test, and one whose
// potential is not finite afterwards runs again with it; softened pairs have no
// such mark and are always tested.  What bounds this loop is instruction issue:
// 15.5 instead of 23 vector instructions a pair at one target per lane, 14.3
// instead of 18.8 at four (with the copy by entry masks below: 262144 particles
// at the benchmark's tolerance, evaluation 19.2 -> 17.0 ms, 16.8M 220 -> 196 ms).
template <int kTG, bool SOFT>
__device__ __forceinline__ void near_tile_f32(const float4* buf, int fill, int s, int nsl, float inv_nsl, const float* tx,
                                     const float* ty, const float* tz, double* fx, double* fy, double* fz, double* ph,
                                     float* cx, float* cy, float* cz, float* cp, float eps2) {
  const int full = uniform((int)(((float)fill + 0.5f) * inv_nsl));  // fill / nsl (both below 1024)
  const int rem = fill - full * nsl;
  const float4* p = buf + s;
  for (int b = 0; b < full + (rem > 0); b += kFlush) {
    const int n = min(kFlush, full - b);
    const bool extra = n < kFlush && s < rem;
    float gx[kTG], gy[kTG], gz[kTG], gp[kTG];
    near_run_f32<kTG, SOFT, SOFT>(p, n, extra, nsl, tx, ty, tz, gx, gy, gz, gp, eps2);
    if (!SOFT) {
      bool odd = false;
#pragma unroll
      for (int u = 0; u < kTG; ++u) odd = odd || !(fabsf(gp[u]) < INFINITY);
      if (__builtin_expect(__ballot(odd) != 0, 0))
        near_run_f32<kTG, SOFT, true>(p, n, extra, nsl, tx, ty, tz, gx, gy, gz, gp, eps2);
    }
    p += n * nsl;
#pragma unroll
    for (int u = 0; u < kTG; ++u) {
      comp_add(fx[u], cx[u], (double)gx[u]);
      comp_add(fy[u], cy[u], (double)gy[u]);
      comp_add(fz[u], cz[u], (double)gz[u]);
      comp_add(ph[u], cp[u], (double)gp[u]);
    }
  }
}

// one source and this lane's kTG targets in FP64 (a pair at r = 0 skipped)
template <int kTG, bool SOFT>
__device__ __forceinline__ void pairs_f64(const double4 q, const double* tx, const double* ty, const double* tz,
                                          double* fx, double* fy, double* fz, double* ph, double eps2) {
#pragma unroll
  for (int u = 0; u < kTG; ++u) {
    const double dx = q.x - tx[u], dy = q.y - ty[u], dz = q.z - tz[u];
    const double r2 = fma(dx, dx, fma(dy, dy, dz * dz));
    double y;
    if (SOFT) {
      y = rsqrt_f64_1nr(r2 + eps2);
      y = r2 > 0.0 ? y : 0.0;
    } else {
      y = rsqrt_f64_1nr_or_zero(r2);
    }
    const double my = q.w * y;
    const double my3 = my * (y * y);
    fx[u] = fma(my3, dx, fx[u]);
    fy[u] = fma(my3, dy, fy[u]);
    fz[u] = fma(my3, dz, fz[u]);
    ph[u] -= my;
  }
}

// interactions of this lane's kTG targets with sources buf[s], buf[s+nsl], ...
// (4M two spheres at theta 0.35, evaluation: 13.2 -> 11.6 ms with the scalar
// counter and half of the root's register masked instead of all of it)
template <int kTG, bool SOFT>
__device__ __forceinline__ void near_tile(const double4* buf, int fill, int s, int nsl, float inv_nsl, const double* tx,
                                 const double* ty, const double* tz, double* fx, double* fy, double* fz, double* ph,
                                 double eps2) {
  const int full = uniform((int)(((float)fill + 0.5f) * inv_nsl));
  const int rem = fill - full * nsl;
  const double4* p = buf + s;
#pragma unroll(kTG == 4 ? 1 : 2)
  for (int i = 0; i < full; ++i, p += nsl) pairs_f64<kTG, SOFT>(*p, tx, ty, tz, fx, fy, fz, ph, eps2);
  if (s < rem) pairs_f64<kTG, SOFT>(*p, tx, ty, tz, fx, fy, fz, ph, eps2);
}

// FP32 offset of a particle from a centre (difference in FP64, then rounded)
__device__ inline float4 offset32(const double4 p, const double4 c) {
  return make_float4((float)(p.x - c.x), (float)(p.y - c.y), (float)(p.z - c.z), (float)p.w);
}

// Targets per lane (1, 2 or 4) for a block of ntc <= 64 targets: the fewest
// lane steps, a step over one source costing 19 units per target and 3 of its own
// (ties: more targets per lane).  A fixed rule, one for both precisions: the
// weights are those of an earlier pair loop (23 instructions at one target per
// lane, 18.8 at four; now 15.5 and 14.3), and since they order sums of FP32 terms
// they stay.
__host__ __device__ constexpr int targets_per_lane(int ntc) {
  int best = kTGMax, bnsl = 64 / ((ntc + kTGMax - 1) / kTGMax);
  for (int k = 2; k >= 1; k >>= 1) {
    const int nsl = 64 / ((ntc + k - 1) / k);
    if ((19 * k + 3) * bnsl < (19 * best + 3) * nsl) {
      best = k;
      bnsl = nsl;
    }
  }
  return best;
}

// Partial sums of one segment's targets: four components and (mixed) their
// compensation terms.
struct NearPart {
  double f[4];
  float c[4];
};

// A wave's share of a list: the buffer fills that start at positions [lo, hi)
// of the list's particles, and where its sums go (part: one per target of the
// block, or nullptr: the wave has the whole list and finishes the targets).
struct NearShare {
  int64_t lo, hi;
  NearPart* part;
};

// What every target of the phase needs to end: its cell's expansion and outputs.
struct NearOut {
  const int32_t* perm;
  double G;
  double *ax, *ay, *az, *pot;
};

__device__ inline void near_finish(const double4 pt, const double4 gx, const double* L, int32_t o, const NearOut& out,
                                   double sx, double sy, double sz, double sp) {
  const double x[3] = {pt.x - gx.x, pt.y - gx.y, pt.z - gx.z};
  double gl[3], phi;
  eval_local(L, x, gl, phi);
  out.ax[o] = out.G * (sx + gl[0]);
  out.ay[o] = out.G * (sy + gl[1]);
  out.az[o] = out.G * (sz + gl[2]);
  if (out.pot) out.pot[o] = out.G * (sp + phi);
}

// Skips the fills of a list that start before position lo: k and pos become
// the first entry and position not skipped, off (a multiple of cap) the part
// of an oversized entry k that is.  The entries' counts are fetched kSkip at a
// time into the wave's staging buffer, so that a skipped fill costs an LDS
// read and a scan, not two dependent loads from memory.
constexpr int kSkip = 2048;

__device__ inline void near_skip(int lane, int64_t st, int32_t nsc, int cap, int64_t lo, int32_t* cbuf,
                                 const int32_t* __restrict__ nsrc, const int32_t* __restrict__ cnt, int32_t& k,
                                 int64_t& pos, int32_t& off) {
  while (k < nsc && pos < lo) {
    const int32_t k0 = k, m = min(kSkip, nsc - k0);
    for (int32_t i = lane; i < m; i += 64) cbuf[i] = cnt[nsrc[st + k0 + i]];
    wave_sync();
    while (pos < lo && k < nsc && (k - k0 + 64 <= m || k0 + m == nsc)) {
      const int32_t i = k - k0 + lane;
      const int32_t cl = i < m ? cbuf[i] : 0;
      const int32_t inc = wave_incl_scan(cl);
      const int take = __popcll(__ballot(i < m && inc <= cap));
      if (take > 0) {
        pos += __shfl(inc, take - 1, 64);
        k += take;
      } else {
        const int32_t c0 = __shfl(cl, 0, 64);
        if (pos + (int64_t)((c0 - 1) / cap) * cap < lo) {
          pos += c0;
          k += 1;
        } else {
          off = (int32_t)((lo - pos + cap - 1) / cap) * cap;
          wave_sync();
          return;
        }
      }
    }
    wave_sync();  // counts read before the next are fetched
  }
}

// One block of ntc <= 64 targets starting at tb, kTG per lane, against this
// wave's share of the leaf's near list.
template <int kTG, bool MIXED, bool SOFT>
__device__ __forceinline__ void near_block(int lane, int32_t tb, int ntc, int64_t st, int32_t nsc, const double4 gx,
                                     const double* L, double4* buf, const NearShare& share,
                                     const int32_t* __restrict__ nsrc, const int32_t* __restrict__ beg,
                                     const int32_t* __restrict__ cnt, const double4* __restrict__ pos,
                                     const NearOut& out, double eps2) {
  float4* buf32 = reinterpret_cast<float4*>(buf);
  constexpr int cap = MIXED ? 2 * kCap : kCap;
  int64_t at = 0;    // position of the next fill in the list's particles
  int32_t off0 = 0;  // particles of entry k that belong to other waves
  const int ng = (ntc + kTG - 1) / kTG;
  const int nsl = 64 / ng;  // slices per group: as many lanes as the groups leave
  const int g = lane / nsl, s = lane % nsl;
  const float inv_nsl = 1.0f / (float)nsl;
  const bool active = g < ng;
  double tx[kTG], ty[kTG], tz[kTG];
  float ux[kTG], uy[kTG], uz[kTG];  // mixed: FP32 offsets from the leaf centre
  double fx[kTG], fy[kTG], fz[kTG], ph[kTG];
  float cx[kTG], cy[kTG], cz[kTG], cp[kTG];  // mixed: compensation terms
#pragma unroll
  for (int q = 0; q < kTG; ++q) {
    cx[q] = cy[q] = cz[q] = cp[q] = 0.0f;
    const int t = g * kTG + q;
    const double4 p = pos[tb + ((active && t < ntc) ? t : 0)];
    tx[q] = p.x;
    ty[q] = p.y;
    tz[q] = p.z;
    ux[q] = (float)(p.x - gx.x);
    uy[q] = (float)(p.y - gx.y);
    uz[q] = (float)(p.z - gx.z);
    fx[q] = fy[q] = fz[q] = ph[q] = 0.0;
  }
  // The near list is consumed 64 entries at a time: every lane fetches one
  // source leaf (index, first particle, count), an in-wave prefix sum places
  // each leaf in this wave's LDS buffer, and the wave copies them.  Leaves are
  // taken while they fit.  The next round's entries are fetched while this
  // round copies and computes.
  int32_t k = 0;
  if (share.lo > 0) near_skip(lane, st, nsc, cap, share.lo, reinterpret_cast<int32_t*>(buf), nsrc, cnt, k, at, off0);
  int32_t Yl = k + lane < nsc ? nsrc[st + k + lane] : -1;
  int32_t bl = Yl >= 0 ? beg[Yl] : 0;
  int32_t cl = Yl >= 0 ? cnt[Yl] : 0;
  while (k < nsc && at < share.hi) {
    const int32_t inc = wave_incl_scan(cl);  // inclusive prefix over lanes
    const uint64_t fits = __ballot(Yl >= 0 && inc <= cap);
    const int take = __popcll(fits);  // prefix is monotone: leading lanes fit
    const int adv = take > 0 ? take : 1;
    const int32_t kn = k + adv + lane;
    const int32_t Yn = kn < nsc ? nsrc[st + kn] : -1;
    int fill = 0;
    if (take > 0) {
      fill = __shfl(inc, take - 1, 64);
      // Cooperative copy: buffer slot v belongs to the last entry that starts
      // at or before v, so consecutive lanes copy consecutive particles.  The
      // entries' starts become one 64-bit mask per 64 slots (set in the
      // buffer's first words and taken into lanes before the copy overwrites
      // them), and a slot's entry is a count of the bits up to its own.  (A
      // search over the lanes' prefix sums took six dependent exchanges a
      // slot.)  Slots past the fill, up to the next multiple of 64, get its
      // last particle again: no lane is masked off (165 -> 154 ms at 16.8M
      // particles).  Two slots per lane and iteration, both loads in flight.
      static_assert(cap % 64 == 0, "whole groups of slots");
      const int32_t startx = inc - cl, delta = bl - startx;
      uint64_t* words = reinterpret_cast<uint64_t*>(buf);
      if (lane < cap / 64) words[lane] = 0ull;
      wave_sync();
      if (lane < take) atomicOr((unsigned long long*)&words[startx >> 6], 1ull << (startx & 63));
      wave_sync();
      const uint64_t mine = words[lane < cap / 64 ? lane : 0];
      wave_sync();
      const uint32_t mine_lo = (uint32_t)mine, mine_hi = (uint32_t)(mine >> 32);
      int32_t before = -1;  // entries that start before the group, less one
      auto source = [&](int32_t v0) {
        const uint32_t lo = __builtin_amdgcn_readlane(mine_lo, v0 >> 6), hi = __builtin_amdgcn_readlane(mine_hi, v0 >> 6);
        const uint64_t m = ((uint64_t)hi << 32) | lo, up = m >> 1;
        // bits 0 .. lane of m
        const int32_t e = (int32_t)__builtin_amdgcn_mbcnt_hi(
            (uint32_t)(up >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)up, before + (int32_t)(m & 1)));
        before += __popcll(m);
        return (uint32_t)(__shfl(delta, e, 64) + min(v0 + lane, fill - 1));
      };
      auto put = [&](int32_t v, const double4 q) {
        if (MIXED) buf32[v] = offset32(q, gx);
        else buf[v] = q;
      };
      int32_t v0 = 0;
      for (; v0 + 64 < fill; v0 += 128) {
        const uint32_t fa = source(v0), fb = source(v0 + 64);
        const double4 pa = pos[fa], pb = pos[fb];
        put(v0 + lane, pa);
        put(v0 + 64 + lane, pb);
      }
      if (v0 < fill) put(v0 + lane, pos[source(v0)]);
      at += fill;
    } else {
      // a single leaf larger than the buffer (coincident points at the
      // deepest level): stream it in buffer-sized pieces
      const int32_t b0 = __shfl(bl, 0, 64), c0 = __shfl(cl, 0, 64);
      for (int32_t off = off0; off < c0 && at + off < share.hi; off += cap) {
        const int part = min(cap, c0 - off);
        if (MIXED) {
          for (int i = lane; i < part; i += 64) buf32[i] = offset32(pos[b0 + off + i], gx);
        } else {
          for (int i = lane; i < part; i += 64) buf[i] = pos[b0 + off + i];
        }
        wave_sync();
        if (active) {
          if (MIXED) near_tile_f32<kTG, SOFT>(buf32, part, s, nsl, inv_nsl, ux, uy, uz, fx, fy, fz, ph, cx, cy, cz, cp, (float)eps2);
          else near_tile<kTG, SOFT>(buf, part, s, nsl, inv_nsl, tx, ty, tz, fx, fy, fz, ph, eps2);
        }
        wave_sync();
      }
      at += c0;
      off0 = 0;
    }
    // the next round's extents load while this round computes
    const int32_t bn = Yn >= 0 ? beg[Yn] : 0;
    const int32_t cn = Yn >= 0 ? cnt[Yn] : 0;
    if (take > 0) {
      wave_sync();
      if (active) {
        if (MIXED) near_tile_f32<kTG, SOFT>(buf32, fill, s, nsl, inv_nsl, ux, uy, uz, fx, fy, fz, ph, cx, cy, cz, cp, (float)eps2);
        else near_tile<kTG, SOFT>(buf, fill, s, nsl, inv_nsl, tx, ty, tz, fx, fy, fz, ph, eps2);
      }
      wave_sync();
    }
    Yl = Yn;
    bl = bn;
    cl = cn;
    k += adv;
  }
  // sum the slices of each group into its first lane (a fixed tree: at
  // step off, slice s adds slice s + off of its own group)
  for (int off = nsl > 1 ? pow2floor(nsl - 1) : 0; off > 0; off >>= 1) {
    const bool take = s + off < nsl;
#pragma unroll
    for (int u = 0; u < kTG; ++u) {
      const double vx = __shfl(fx[u], lane + off, 64), vy = __shfl(fy[u], lane + off, 64);
      const double vz = __shfl(fz[u], lane + off, 64), vp = __shfl(ph[u], lane + off, 64);
      if (MIXED) {
        const float wx = __shfl(cx[u], lane + off, 64), wy = __shfl(cy[u], lane + off, 64);
        const float wz = __shfl(cz[u], lane + off, 64), wp = __shfl(cp[u], lane + off, 64);
        if (take) {
          comp_add(fx[u], cx[u], vx);
          comp_add(fy[u], cy[u], vy);
          comp_add(fz[u], cz[u], vz);
          comp_add(ph[u], cp[u], vp);
          cx[u] += wx;
          cy[u] += wy;
          cz[u] += wz;
          cp[u] += wp;
        }
      } else if (take) {
        fx[u] += vx;
        fy[u] += vy;
        fz[u] += vz;
        ph[u] += vp;
      }
    }
  }
  if (share.part) {
    if (active && s == 0) {
#pragma unroll
      for (int u = 0; u < kTG; ++u) {
        const int t = g * kTG + u;
        if (t < ntc) {
          NearPart& o = share.part[t];
          o.f[0] = fx[u];
          o.f[1] = fy[u];
          o.f[2] = fz[u];
          o.f[3] = ph[u];
          if (MIXED) {
            o.c[0] = cx[u];
            o.c[1] = cy[u];
            o.c[2] = cz[u];
            o.c[3] = cp[u];
          }
        }
      }
    }
    return;
  }
  if (MIXED) {
    // the compensated sums, rounded once to FP64
#pragma unroll
    for (int u = 0; u < kTG; ++u) {
      fx[u] += (double)cx[u];
      fy[u] += (double)cy[u];
      fz[u] += (double)cz[u];
      ph[u] += (double)cp[u];
    }
  }
  // lane s < kTG of group g finishes target g kTG + s with the sums of the
  // group's first lane
  const int t = g * kTG + s;
  double sx = 0.0, sy = 0.0, sz = 0.0, sp = 0.0;
#pragma unroll
  for (int u = 0; u < kTG; ++u) {
    const double vx = __shfl(fx[u], g * nsl, 64), vy = __shfl(fy[u], g * nsl, 64);
    const double vz = __shfl(fz[u], g * nsl, 64), vp = __shfl(ph[u], g * nsl, 64);
    if (s == u) {
      sx = vx;
      sy = vy;
      sz = vz;
      sp = vp;
    }
  }
  if (active && s < kTG && t < ntc)  // (reloaded: the mixed path keeps no FP64 copy)
    near_finish(pos[tb + t], gx, L, out.perm[tb + t], out, sx, sy, sz, sp);
}

template <bool MIXED, bool SOFT>
__device__ __forceinline__ void near_targets(int lane, int32_t tb, int ntc, int64_t st, int32_t nsc, const double4 gx,
                                             const double* L, double4* buf, const NearShare& share,
                                             const int32_t* __restrict__ nsrc, const int32_t* __restrict__ beg,
                                             const int32_t* __restrict__ cnt, const double4* __restrict__ pos,
                                             const NearOut& out, double eps2) {
  const int K = targets_per_lane(ntc);
  if (K == 1)
    near_block<1, MIXED, SOFT>(lane, tb, ntc, st, nsc, gx, L, buf, share, nsrc, beg, cnt, pos, out, eps2);
  else if (K == 2)
    near_block<2, MIXED, SOFT>(lane, tb, ntc, st, nsc, gx, L, buf, share, nsrc, beg, cnt, pos, out, eps2);
  else
    near_block<kTGMax, MIXED, SOFT>(lane, tb, ntc, st, nsc, gx, L, buf, share, nsrc, beg, cnt, pos, out, eps2);
}

// Lane steps (in instructions) one wave takes over nsp sources with ntc targets.
__host__ __device__ constexpr int64_t near_cost(int ntc, int64_t nsp) {
  const int K = targets_per_lane(ntc);
  const int nsl = 64 / ((ntc + K - 1) / K);
  return nsp * (19 * K + 3) / nsl;
}

// 64 targets cost the least a target, and what one target and source cost at most
constexpr int64_t kCostUnit = 64 * 63 * 61 * 60;  // sources, to see past near_cost's rounding
constexpr bool full_blocks_cost_least() {
  for (int t = 1; t <= 64; ++t)
    if (t * near_cost(64, kCostUnit) > 64 * near_cost(t, kCostUnit) + 64) return false;
  return true;
}
static_assert(full_blocks_cost_least(), "room for partial sums");
constexpr double most_cost() {
  double v = 0.0;
  for (int t = 1; t <= 64; ++t) {
    const double w = (double)(near_cost(t, kCostUnit) + 1) / ((double)t * (double)kCostUnit);
    v = w > v ? w : v;
  }
  return v;
}
constexpr double kMostCost = most_cost();

// The targets of a phase: the leaves of a list, or of up to kMaxLevel + 1 ranges
// of cells (unused: first is beyond all).  A phase per range took five launches
// on each level of every batch of subtrees: 131072 particles at theta 0.7 in
// batches of 1 MB of lists 1.10 ms in 28 phases, now 0.69 in 11.
struct NearRanges {
  int32_t first[kMaxLevel + 1];  // targets before the range
  int32_t off[kMaxLevel + 1];    // its first cell, less those
};
struct NearTargets {
  const int32_t* leaves;
  const NearRanges* ranges;  // (in memory: as kernel arguments every wave would load them)
  int32_t count;
  // target li's cell
  __device__ int32_t cell(int32_t li) const {
    if (leaves) return leaves[li];
    int32_t o = ranges->off[0];
#pragma unroll
    for (int r = 1; r <= kMaxLevel; ++r) o = li >= ranges->first[r] ? ranges->off[r] : o;
    return li + o;
  }
};
__global__ void k_near_ranges(NearRanges v, NearRanges* out) { *out = v; }

// One segment of one target block's list; the block itself has seg = 0.
struct NearUnit {
  int32_t X, tb, seg, nseg;
  int32_t slot;  // first partial sum of the block (segment-major, ntc each)
};

// Cutting the long lists.  A list is cut when it costs more than two shares, a
// share being the phase's whole cost over NearPlan::shares (a quarter of what one of
// 4096 waves in flight gets at 16384) and at least kMinShare, below which a
// segment's own start and end outweigh its work (about 3000 instructions, 5 us).
// A block of c > 2 shares gets at most 3/2 c segments, and a leaf's blocks (all
// cut like its first, the dearest) cost at least half of what that counts, so
// there are at most 3 shares' worth of segments.  A leaf's targets cost at least
// as much each as those of a full block, so a leaf of t targets, cut like a block
// of c, costs c t / 64 and gets 3/2 c t / share partial sums: 64 times 3/2 hold
// the whole phase's (while no leaf holds more than n_crit particles, as above the
// deepest level, n_crit of them do).  near_room adds what rounding down in the
// costs and the share takes away, so that no request is refused: which lists are
// cut, and with it how they are summed, depends on the lists alone.
constexpr int64_t kMinShare = 4000;
struct NearPlan {
  NearUnit* units;
  NearUnit* groups;    // the cut blocks
  uint8_t* cut;        // per leaf: its blocks are in units
  NearPart* parts;
  unsigned long long* words;  // [0] interactions, [2] cost, [3] units, [4] groups, [5] partial sums
  int64_t shares, max_parts;
};

__device__ inline int64_t wave_total(int64_t v) {
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d, 64);
  return v;
}

// one thread per target leaf: interactions and cost of the phase
__global__ void __launch_bounds__(kBS) k_near_cost(NearTargets tg, const int32_t* __restrict__ nch,
                                                   const int32_t* __restrict__ cnt, const int64_t* __restrict__ parts,
                                                   unsigned long long* __restrict__ words) {
  const int32_t li = blockIdx.x * kBS + threadIdx.x;
  int64_t inter = 0, cost = 0;
  if (li < tg.count) {
    const int32_t X = tg.cell(li);
    if (tg.leaves || nch[X] == 0) {
      const int32_t nt = cnt[X];
      const int64_t nsp = parts[X];
      inter = nt * (nsp - 1);
      for (int32_t b = 0; b < nt; b += 64) cost += near_cost(min(64, nt - b), nsp);
    }
  }
  inter = wave_total(inter);
  cost = wave_total(cost);
  __shared__ int64_t s[2][kWaves];
  if ((threadIdx.x & 63) == 0) {
    s[0][threadIdx.x >> 6] = inter;
    s[1][threadIdx.x >> 6] = cost;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    int64_t v = 0;
    for (int q = 0; q < kWaves; ++q) v += s[threadIdx.x][q];
    if (v) atomicAdd(&words[2 * threadIdx.x], (unsigned long long)v);
  }
}

// one thread per target leaf: cut or not; the wave writes its leaves' units
__global__ void __launch_bounds__(kBS) k_near_cut(NearTargets tg, const int32_t* __restrict__ nch, const int32_t* __restrict__ beg,
                                                  const int32_t* __restrict__ cnt, const int64_t* __restrict__ parts,
                                                  NearPlan plan) {
  const int32_t li = blockIdx.x * kBS + threadIdx.x;
  const int lane = threadIdx.x & 63;
  const int64_t share = max(kMinShare, (int64_t)plan.words[2] / plan.shares);
  int32_t X = 0, nt = 0, nblk = 0, unit0 = 0, group0 = 0, slot0 = 0;
  bool cut = false;
  if (li < tg.count) {
    X = tg.cell(li);
    if (tg.leaves || nch[X] == 0) {
      nt = cnt[X];
      const int64_t nsp = parts[X];
      nblk = (nt + 63) / 64;
      // one length for all blocks of a leaf: the first is the largest
      const int64_t c0 = near_cost(min(64, nt), nsp);
      if (c0 > 2 * share) {
        const int64_t nseg = (c0 + share - 1) / share;
        const int64_t np = nseg * nt;
        // (always room: see near_room)
        const unsigned long long at = atomicAdd(&plan.words[5], (unsigned long long)np);
        if ((int64_t)at + np <= plan.max_parts) {
          cut = true;
          slot0 = (int32_t)at;
          unit0 = (int32_t)atomicAdd(&plan.words[3], (unsigned long long)(nseg * nblk));
          group0 = (int32_t)atomicAdd(&plan.words[4], (unsigned long long)nblk);
        }
      }
      plan.cut[li] = cut ? 1 : 0;
    }
  }
  for (uint64_t m = __ballot(cut); m; m &= m - 1) {
    const int o = __ffsll((unsigned long long)m) - 1;
    const int32_t x = __shfl(X, o, 64), n = __shfl(nt, o, 64), nb = __shfl(nblk, o, 64), u0 = __shfl(unit0, o, 64),
                  g0 = __shfl(group0, o, 64), s0 = __shfl(slot0, o, 64);
    const int64_t c0 = near_cost(min(64, n), parts[x]);
    const int32_t nseg = (int32_t)((c0 + share - 1) / share);
    for (int32_t j = lane; j < nseg * nb; j += 64) {
      const int32_t b = j / nseg;
      const NearUnit u{x, beg[x] + 64 * b, j % nseg, nseg, s0 + 64 * b * nseg};
      plan.units[u0 + j] = u;
      if (u.seg == 0) plan.groups[g0 + b] = u;
    }
  }
}

// Room for the cut lists' segments and partial sums (the bounds above), shares
// at most all / kMinShare of them for a phase that costs `all`: no target meets
// more than the n particles.
struct NearRoom {
  size_t units, parts;
};
NearRoom near_room(const Ctx& c, int64_t shares) {
  const double all = kMostCost * (double)c.n * (double)c.n;
  const double s = std::min((double)shares, all / (double)kMinShare) * (1.0 + 1.0 / 512.0);
  const int targets = c.depth < kMaxLevel ? std::min(64, c.opt.n_crit) : 64;
  return NearRoom{(size_t)(3.0 * s) + 64, (size_t)(1.5 * targets * s) + 64};
}

// blocks that run segments, ahead of the blocks of whole leaves
constexpr int kUnitBlocks = 4096;

template <bool MIXED, bool SOFT>
__global__ void __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(4))) k_near(NearTargets tg,
                                              const int32_t* __restrict__ nch,
                                              const int32_t* __restrict__ beg, const int32_t* __restrict__ cnt,
                                              const double4* __restrict__ pos, const double4* __restrict__ geo,
                                              const double* __restrict__ loc, const int64_t* __restrict__ nstart,
                                              const int32_t* __restrict__ ncount, const int32_t* __restrict__ nsrc,
                                              const int64_t* __restrict__ parts, NearOut out, NearPlan plan,
                                              double eps2) {
  const int lane = threadIdx.x;
  // FP64 staging holds kCap double4 per wave; the mixed path puts 2 kCap
  // float4 offsets in the same bytes
  __shared__ double4 buf[kCap];
  static_assert(kSkip * sizeof(int32_t) <= kCap * sizeof(double4), "skip buffer");
  // this wave's work: segments u, u + kUnitBlocks, ... or the target
  // blocks of one leaf (one call site for both: the code is the same)
  const bool seg = blockIdx.x < kUnitBlocks;
  int32_t u = 0, nu = 0, X = 0, tb = 0;
  if (seg) {
    u = (int32_t)blockIdx.x;
    nu = uniform((int32_t)plan.words[3]);
  } else {
    const int32_t li = (int32_t)xcd_block(blockIdx.x - kUnitBlocks, gridDim.x - kUnitBlocks);
    if (li >= tg.count) return;
    X = uniform(tg.cell(li));
    if (!tg.leaves && uniform(nch[X]) != 0) return;
    if (plan.cut && uniform((int32_t)plan.cut[li])) return;
    tb = uniform(beg[X]);
  }
  for (;;) {
    NearShare share{0, INT64_MAX, nullptr};
    if (seg) {
      if (u >= nu) return;
      const NearUnit& un = plan.units[u];
      X = uniform(un.X);
      tb = uniform(un.tb);
      const int64_t nsp = parts[X], q = uniform(un.seg), nseg = uniform(un.nseg);
      share.lo = nsp * q / nseg;
      share.hi = nsp * (q + 1) / nseg;
    }
    const int32_t end = uniform(beg[X]) + uniform(cnt[X]);
    const int ntc = min(64, end - tb);
    if (seg) share.part = plan.parts + uniform(plan.units[u].slot) + (int64_t)uniform(plan.units[u].seg) * ntc;
    const double4 gx = geo[X];
    const double* L = loc + (int64_t)X * kLoc;
    near_targets<MIXED, SOFT>(lane, tb, ntc, nstart[X], uniform(ncount[X]), gx, L, buf, share, nsrc, beg, cnt, pos, out,
                              eps2);
    if (!seg) {
      tb += 64;
      if (tb >= end) return;
      continue;
    }
    u += kUnitBlocks;
  }
}

// One wave per cut target block: lanes (target t, row j) add segments j, j +
// nj, ..., then the rows in order, and end the targets.
constexpr int kJoinBlocks = 256;
template <bool MIXED>
__global__ void __launch_bounds__(kBS) k_near_join(const int32_t* __restrict__ beg, const int32_t* __restrict__ cnt,
                                                   const double4* __restrict__ pos, const double4* __restrict__ geo,
                                                   const double* __restrict__ loc, NearOut out, NearPlan plan) {
  const int lane = threadIdx.x & 63;
  const int32_t ng = (int32_t)plan.words[4];
  for (int32_t g = uniform((int32_t)(blockIdx.x * kWaves + (threadIdx.x >> 6))); g < ng; g += kJoinBlocks * kWaves) {
    const NearUnit un = plan.groups[g];
    const int32_t X = uniform(un.X), tb = uniform(un.tb), nseg = uniform(un.nseg);
    const int ntc = min(64, uniform(beg[X]) + uniform(cnt[X]) - tb);
    const NearPart* __restrict__ part = plan.parts + uniform(un.slot);
    const int nj = 64 / ntc, t = lane % ntc, j = lane / ntc;
    double f[4] = {0.0, 0.0, 0.0, 0.0};
    float c[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (j < nj) {
#pragma unroll 4
      for (int32_t q = j; q < nseg; q += nj) {
        const NearPart& p = part[(int64_t)q * ntc + t];
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          if (MIXED) {
            comp_add(f[d], c[d], p.f[d]);
            c[d] += p.c[d];
          } else {
            f[d] += p.f[d];
          }
        }
      }
    }
    for (int r = 1; r < nj; ++r) {
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const double v = __shfl(f[d], t + r * ntc, 64);
        const float w = MIXED ? __shfl(c[d], t + r * ntc, 64) : 0.0f;
        if (j == 0) {
          if (MIXED) {
            comp_add(f[d], c[d], v);
            c[d] += w;
          } else {
            f[d] += v;
          }
        }
      }
    }
    if (MIXED) {
#pragma unroll
      for (int d = 0; d < 4; ++d) f[d] += (double)c[d];
    }
    if (j == 0)
      near_finish(pos[tb + t], geo[X], loc + (int64_t)X * kLoc, out.perm[tb + t], out, f[0], f[1], f[2], f[3]);
  }
}

}  // namespace

void near_field(Ctx& c, const CellRanges* ranges, double* ax, double* ay, double* az, double* pot) {
  NearTargets tg{ranges ? nullptr : (const int32_t*)c.leaves.p, nullptr, ranges ? 0 : c.nleaves};
  if (ranges) {
    NearRanges v{};
    std::fill(v.first, v.first + kMaxLevel + 1, INT32_MAX);
    for (int r = 0; r < ranges->n; ++r) {
      v.first[r] = tg.count;
      v.off[r] = ranges->lo[r] - tg.count;
      tg.count += ranges->hi[r] - ranges->lo[r];
    }
    if (tg.count <= 0) return;
    NearRanges* dev = (NearRanges*)((char*)c.counters.p + kCounterBytes);
    static_assert(sizeof(NearRanges) <= kRangeBytes, "room behind the counters");
    hipLaunchKernelGGL(k_near_ranges, dim3(1), dim3(1), 0, c.stream, v, dev);
    tg.ranges = dev;
  }
  const int32_t count = tg.count;
  if (count <= 0) return;
  ++c.near_launches;
  const bool mixed = c.opt.precision == AMFMM_MIXED, soft = c.opt.softening > 0.0;
  // room for the cut lists' segments and partial sums (fewer shares where
  // memory is the caller's arena); without it every list stays whole
  NearPlan plan{};
  plan.shares = c.arena ? 2048 : 16384;
  const NearRoom room = near_room(c, plan.shares);
  plan.max_parts = (int64_t)room.parts;
  const size_t pb = sizeof(NearPart) * room.parts;
  const size_t ub = sizeof(NearUnit) * room.units, gb = ub;
  if (char* w = (char*)ensure_if_room(c, c.near_plan, pb + ub + gb + (size_t)count)) {
    plan.parts = (NearPart*)w;
    plan.units = (NearUnit*)(w + pb);
    plan.groups = (NearUnit*)(w + pb + ub);
    plan.cut = (uint8_t*)(w + pb + ub + gb);
  }
  plan.words = (unsigned long long*)c.counters.p;
  const int32_t* nch = as<int32_t>(c.c_nchild);
  const int32_t* beg = as<int32_t>(c.c_begin);
  const int32_t* cnt = as<int32_t>(c.c_count);
  const int64_t* parts = (const int64_t*)c.near_parts.p;
  zero_u64(c, plan.words + 2, 4, clock_word(c));
  hipLaunchKernelGGL(k_near_cost, dim3(blocks_for(count, kBS)), dim3(kBS), 0, c.stream, tg, nch, cnt, parts, plan.words);
  if (plan.cut)
    hipLaunchKernelGGL(k_near_cut, dim3(blocks_for(count, kBS)), dim3(kBS), 0, c.stream, tg, nch, beg, cnt, parts, plan);
  auto kern = mixed ? (soft ? k_near<true, true> : k_near<true, false>)
                    : (soft ? k_near<false, true> : k_near<false, false>);
  const NearOut out{as<int32_t>(c.perm), c.opt.G, ax, ay, az, pot};
  hipLaunchKernelGGL(kern, dim3(kUnitBlocks + count), dim3(64), 0, c.stream, tg, nch, beg, cnt,
                     (const double4*)c.pos4.p, (const double4*)c.geo.p, (const double*)c.loc.p,
                     (const int64_t*)c.near_start.p, (const int32_t*)c.near_count.p, (const int32_t*)c.near_src.p,
                     parts, out, plan, c.opt.softening * c.opt.softening);
  if (plan.cut)
    hipLaunchKernelGGL(mixed ? k_near_join<true> : k_near_join<false>, dim3(kJoinBlocks), dim3(kBS), 0, c.stream, beg,
                       cnt, (const double4*)c.pos4.p, (const double4*)c.geo.p, (const double*)c.loc.p, out, plan);
  AMFMM_HIP(hipGetLastError());
  if (getenv("AMFMM_DEBUG_NEAR") && !c.arena) {
    unsigned long long h[6];
    AMFMM_HIP(hipMemcpyAsync(h, plan.words, sizeof(h), hipMemcpyDeviceToHost, c.stream));
    sync(c);
    fprintf(stderr, "near field: targets %d cut blocks %llu segments %llu of %zu partial sums %llu of %zu\n", count,
            h[4], h[3], plan.cut ? room.units : 0, h[5], plan.cut ? room.parts : 0);
  }
  if (c.opt.order == 3) return;
  if (!ranges) order_l2p(c, tg.leaves, 0, count, ax, ay, az, pot);
  for (int r = 0; ranges && r < ranges->n; ++r)
    order_l2p(c, nullptr, ranges->lo[r], ranges->hi[r] - ranges->lo[r], ax, ay, az, pot);
}

}  // namespace amfmm
