// gauss.h -- the Edwards-Anderson model with Gaussian couplings (Sec. 2.1:
// couplings drawn from a standard normal distribution; the 2D Gaussian
// workload of Sec. 4.2), device side shared by the Gaussian kernels.
//
// Couplings live on a fixed-point grid, J = n 2^-16 with |n| <= 2^19 (the
// float32 values the caller passes must lie on it), and are held as the
// integers n.  Local fields and energies are then exact integers of 2^-16
// units whatever the summation order, and the chain is decided by integer
// data plus one real comparison per move: a Metropolis flip with energy
// change dE > 0 (or an exchange with D > 0) is accepted iff the move's 32-bit
// Philox word r satisfies r < 2^32 exp(-beta dE 2^-16) (Eq. (5) and the
// Metropolis rule of Sec. 2.2, with beta the inverse temperature or the
// difference of the two inverse temperatures).  That comparison is decided
// exactly, in three tiers: float32 with a certified error margin, then
// double, then double-double (about 2^-98 relative), each tier deciding only
// where its error bound cannot change the answer.
//
// Per-site coupling data, grouped by the four same-colour sites of one
// Philox call (group gi of colour c: word w = gi mod NW, field f and group q
// of that field from gi / NW = f Gp + q, sites b = 4q + j, j < 4, of field f;
// Gp = ceil(H/4)): int4 Jg[S][2][2d+1][NGc], entry k < 2d the value -2 n of
// the bond in direction k (+x0, -x0, +x1, -x1, +x2, -x2) of each of the four
// sites, entry 2d the sum of the site's 2d couplings.  With a_k = 1 where
// the site and its neighbour in direction k are antiparallel,
// x = s_i h_i = sum_k n_k (1 - 2 a_k) = Hs + sum_k a_k (-2 n_k).
#pragma once
#include "device.h"

namespace ptsg {

constexpr int kGaussUnitBits = 16;       // J = n 2^-16
constexpr int32_t kGaussMaxUnits = 1 << 19;  // |J| <= 8
// What 32 bits have to hold: twice a local field exactly as a float (the
// acceptance tiers), a wavefront's local fields of a group of four sites a lane
// (the sweep's energies), the boundary bonds of a 2D row, each -2n (Houdayer moves).
static_assert(2ll * 6 * kGaussMaxUnits < 1ll << 24, "local fields as floats");
static_assert(64ll * 4 * 6 * kGaussMaxUnits < 1ll << 31, "wavefront sums of local fields");
static_assert(32ll * 4 * (2ll * kGaussMaxUnits + 1) < 1ll << 31, "a row's energy change");

// Groups of four same-colour sites per colour of a lattice.
__host__ __device__ constexpr int gauss_groups(const Geo& g) {
  return g.NW * g.P * ((g.H + 3) / 4);
}

// ---------------------------------------------------------------------------
// Double-double arithmetic (Dekker's error-free sum and product; the product
// through a fused multiply-add).
// ---------------------------------------------------------------------------
struct dd {
  double hi, lo;
};
__host__ __device__ inline dd dd_two_sum(double a, double b) {
  const double s = a + b, bb = s - a;
  return dd{s, (a - (s - bb)) + (b - bb)};
}
__host__ __device__ inline dd dd_fast_sum(double a, double b) {  // |a| >= |b|
  const double s = a + b;
  return dd{s, b - (s - a)};
}
__host__ __device__ inline dd dd_two_prod(double a, double b) {
  const double p = a * b;
  return dd{p, fma(a, b, -p)};
}
__host__ __device__ inline dd dd_add(dd a, dd b) {
  dd s = dd_two_sum(a.hi, b.hi);
  const dd t = dd_two_sum(a.lo, b.lo);
  s.lo += t.hi;
  s = dd_fast_sum(s.hi, s.lo);
  s.lo += t.lo;
  return dd_fast_sum(s.hi, s.lo);
}
__host__ __device__ inline dd dd_mul(dd a, dd b) {
  dd p = dd_two_prod(a.hi, b.hi);
  p.lo += a.hi * b.lo + a.lo * b.hi;
  return dd_fast_sum(p.hi, p.lo);
}
__host__ __device__ inline dd dd_mul_d(dd a, double b) {
  dd p = dd_two_prod(a.hi, b);
  p.lo += a.lo * b;
  return dd_fast_sum(p.hi, p.lo);
}
// a / b for a double b: the quotient's leading part, then the exact remainder
// divided once more.
__host__ __device__ inline dd dd_div_d(dd a, double b) {
  const double q1 = a.hi / b;
  const dd p = dd_two_prod(q1, b);
  const double r = ((a.hi - p.hi) - p.lo) + a.lo;
  return dd_fast_sum(q1, r / b);
}

// ln 2 as a double-double (the double nearest ln 2 and the remainder).
constexpr double kLn2Hi = 0x1.62e42fefa39efp-1;
constexpr double kLn2Lo = 0x1.abc9e3b39803fp-56;

// r < 2^32 exp(-b u 2^-16) for b > 0 and u > 0, in double-double: y = b u
// 2^-16 exactly (an error-free product, then a power-of-two scale), reduced
// as y = k ln 2 + f with |f| <= ln(2)/2 + 2^-40, exp(-f) by its Taylor series
// (24 terms, Horner form; the remainder is below 2^-110), and t = exp(-f)
// 2^(32 - k).  r = 0 is always accepted (t > 0); for r >= 1 acceptance needs
// t > 1, i.e. y < 32 ln 2 = 22.18...
__host__ __device__ inline bool gauss_accept_dd(uint32_t r, double b, int64_t u) {
  if (r == 0u) return true;
  dd y = dd_two_prod(b, (double)u);
  y.hi *= 0x1p-16;
  y.lo *= 0x1p-16;
  if (y.hi > 22.25) return false;
  const int k = (int)rint(y.hi / kLn2Hi);
  const dd f = dd_add(y, dd_mul_d(dd{-kLn2Hi, -kLn2Lo}, (double)k));
  const dd mf{-f.hi, -f.lo};
  dd s{1.0, 0.0};
  for (int n = 24; n >= 1; --n) s = dd_add(dd{1.0, 0.0}, dd_div_d(dd_mul(s, mf), (double)n));
  s.hi = ldexp(s.hi, 32 - k);
  s.lo = ldexp(s.lo, 32 - k);
  // r < s.hi + s.lo  <=>  r - s.hi < s.lo; the difference is exact where it
  // matters (Sterbenz) and has the right sign elsewhere.
  return (double)r - s.hi < s.lo;
}

// The float32 tier's per-temperature constant, b log2(e) 2^-15 rounded to
// float (host and device compute it with the same double operations): cz x is
// the log2 of the inverse acceptance probability of a flip with local field x
// (energy change 2x units).  Capped so that its product with any x is finite
// (beyond the cap no x >= 1 is accepted by a word r >= 1 anyway).
__host__ __device__ inline float gauss_cz(double b) {
  const double c = b * 1.4426950408889634 / 32768.0;
  return c < 0x1p100 ? (float)c : 0x1p100f;
}

// The double tier: y = b u 2^-16 rounded once (relative error 2^-53), exp in
// double (within a few ulp); together well inside the 2^-40 margin.  Cases
// inside the margin go to the double-double tier.
__device__ inline bool gauss_accept_d(uint32_t r, double b, int64_t u) {
  const double y = b * (double)u * 0x1p-16;
  if (y > 22.25) return r == 0u;
  const double t = ldexp(exp(-y), 32);
  const double rd = (double)r;
  if (rd < t * (1.0 - 0x1p-40)) return true;
  if (rd > t * (1.0 + 0x1p-40)) return false;
  return gauss_accept_dd(r, b, u);
}

// The Metropolis decision for local field x (u = 2x < 2^24 energy units, any
// sign), in base-2 logarithms: d = log2 r - 32 + cz x, accepted iff d < 0.  The
// logarithm of the word does not wait for the local field, one fma forms d,
// and the decision is its sign bit; the threshold form 2^32 2^-z needs two
// more multiplies and two compares per site.  Errors: r to float 2^-24
// relative (2^-23.5 in log2), v_log_f32 2^-19 (one ulp below 32), the
// difference 2^-20, cz x 2^-24 relative (2^-18.9 where cz x <= 33), the sum
// below 2^-19: under 2^-17 in all, so a |d| above 2^-15 is decided here.  Where
// cz x > 33 every r >= 1 gives d > 1/2 and is rejected, rightly (the threshold
// is below 1/2); r = 0 gives d = -inf and is accepted, rightly; x <= 0 gives
// d <= 0 up to those errors.  Words inside the band (4e-5 of the threshold)
// go to the double tier, which decides x <= 0 too.
constexpr float kMetroBand = 0x1p-15f;
__device__ __forceinline__ float gauss_metro_log(uint32_t r, float cz, int x) {
  return __builtin_fmaf((float)x, cz, __builtin_amdgcn_logf((float)r) - 32.0f);
}
__device__ inline bool gauss_accept_metro(uint32_t r, float cz, double b, uint32_t u) {
  // (test entry: u may be odd; u cz / 2 is as exact as x cz)
  const float d = __builtin_fmaf((float)u, 0.5f * cz, __builtin_amdgcn_logf((float)r) - 32.0f);
  return fabsf(d) > kMetroBand ? d < 0.0f : gauss_accept_d(r, b, (int64_t)u);
}

// ---------------------------------------------------------------------------
// Site groups of the Gaussian kernels.
// ---------------------------------------------------------------------------
// Decodes group gi of a colour: word w, field f, group q.
struct GroupPos {
  int w, f, q, shift, nv;
};
__device__ __forceinline__ GroupPos group_pos(const Geo& g, int gi) {
  const int Gp = (g.H + 3) / 4;
  GroupPos p;
  p.w = gi % g.NW;
  const int fg = gi / g.NW;
  p.f = fg / Gp;
  p.q = fg - p.f * Gp;
  p.shift = p.f * g.H + 4 * p.q;
  p.nv = min(4, g.H - 4 * p.q);
  return p;
}

__device__ __forceinline__ int lane_of(const int4& v, int j) {
  return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w;
}
__device__ __forceinline__ uint32_t word_of(const Ctr4& v, int j) {
  return j == 0 ? v.x : j == 1 ? v.y : j == 2 ? v.z : v.w;
}

// Bit `at` of a sign-extended to a mask (0 or -1), one v_bfe_i32.  Written as
// an instruction so that the compiler keeps the mask-and-add form (its own
// canonical form, a compare and a select per term, costs one more).
__device__ __forceinline__ int bit_mask(uint32_t a, int at) {
  int r;
  asm("v_bfe_i32 %0, %1, %2, 1" : "=v"(r) : "v"(a), "v"(at));
  return r;
}

// x = s_i h_i of the four sites of a group (bits sh .. sh + 3) from the
// antiparallel words a[k] and the group's coupling data: the site's bit of
// a[k] as a mask selects the term.
template <int D>
__device__ __forceinline__ void group_fields(const uint32_t (&a)[2 * D], int sh, const int4 (&m)[2 * D],
                                             const int4& hs, int (&x)[4]) {
  x[0] = hs.x;
  x[1] = hs.y;
  x[2] = hs.z;
  x[3] = hs.w;
#pragma unroll
  for (int k = 0; k < 2 * D; k += 2) {
    // two terms at a time: one three-input add
    x[0] += (m[k].x & bit_mask(a[k], sh)) + (m[k + 1].x & bit_mask(a[k + 1], sh));
    x[1] += (m[k].y & bit_mask(a[k], sh + 1)) + (m[k + 1].y & bit_mask(a[k + 1], sh + 1));
    x[2] += (m[k].z & bit_mask(a[k], sh + 2)) + (m[k + 1].z & bit_mask(a[k + 1], sh + 2));
    x[3] += (m[k].w & bit_mask(a[k], sh + 3)) + (m[k + 1].w & bit_mask(a[k + 1], sh + 3));
  }
}

// The Metropolis decisions of one group of four same-colour sites whose
// Philox words are r, in two parts so that a caller can interleave two groups:
// gauss_group_fast computes the local fields and the float32 tier without
// branches: the flip bits F and `sure`, whether all four are decided (for
// lanes of a part group, the unused sites' too: x = 0 there);
// gauss_group_finish decides the rare undecided sites by the exact tiers.
// F keeps the valid sites (vmask).
template <int D>
__device__ __forceinline__ void gauss_group_fast(const uint32_t (&a)[2 * D], int sh,
                                                 const int4 (&m)[2 * D], const int4& hs, const Ctr4& r,
                                                 float cz, int (&x)[4], uint32_t& F, bool& sure) {
  group_fields<D>(a, sh, m, hs, x);
  const float d0 = gauss_metro_log(r.x, cz, x[0]), d1 = gauss_metro_log(r.y, cz, x[1]);
  const float d2 = gauss_metro_log(r.z, cz, x[2]), d3 = gauss_metro_log(r.w, cz, x[3]);
  // sign bits, the last site's first
  F = __float_as_uint(d3) >> 31;
  F = __builtin_amdgcn_alignbit(F, __float_as_uint(d2), 31);
  F = __builtin_amdgcn_alignbit(F, __float_as_uint(d1), 31);
  F = __builtin_amdgcn_alignbit(F, __float_as_uint(d0), 31);
  sure = fminf(fminf(fabsf(d0), fabsf(d1)), fminf(fabsf(d2), fabsf(d3))) > kMetroBand;
}
__device__ __forceinline__ uint32_t gauss_group_finish(const int (&x)[4], const Ctr4& r, float cz,
                                                       double beta, uint32_t F, bool sure,
                                                       uint32_t vmask) {
  if (!sure) {
    for (int j = 0; j < 4; ++j) {
      const int xj = j == 0 ? x[0] : j == 1 ? x[1] : j == 2 ? x[2] : x[3];
      const uint32_t rj = word_of(r, j);
      if (fabsf(gauss_metro_log(rj, cz, xj)) > kMetroBand) continue;
      const bool acc = gauss_accept_d(rj, beta, 2 * (int64_t)xj);
      F = (F & ~(1u << j)) | ((uint32_t)acc << j);
    }
  }
  return F & vmask;
}
// Energy change of the group's flips F.
__device__ __forceinline__ int gauss_flip_energy(const int (&x)[4], uint32_t F) {
  int s = (x[0] & bit_mask(F, 0)) + (x[1] & bit_mask(F, 1));
  s += (x[2] & bit_mask(F, 2)) + (x[3] & bit_mask(F, 3));
  return 2 * s;
}
template <int D>
__device__ __forceinline__ uint32_t gauss_group_flips(const uint32_t (&a)[2 * D], int sh,
                                                      const int4 (&m)[2 * D], const int4& hs,
                                                      uint32_t vmask, const Ctr4& r, float cz,
                                                      double beta, int (&x)[4]) {
  uint32_t F;
  bool sure;
  gauss_group_fast<D>(a, sh, m, hs, r, cz, x, F, sure);
  return gauss_group_finish(x, r, cz, beta, F, sure, vmask);
}

// Energy change of replica a when the cluster C (both colours' words) is
// exchanged with replica b: the sum over bonds leaving C of 2 n s_i^a s_j^a,
// taken from the colour-0 end of every bond (with m = -2n, m (2 a - 1) where a
// = 1 if the bond's two spins of replica a are antiparallel).  Threads t of T
// share the groups; each returns its part.
template <int D>
__device__ inline int64_t gauss_cluster_delta(const Geo& g, const uint32_t* C, const uint32_t* A,
                                              const int4* __restrict__ J0, int t, int T) {
  const int NW = g.NW, NGc = gauss_groups(g);
  int64_t dl = 0;
  for (int gi = t; gi < NGc; gi += T) {
    const GroupPos gp = group_pos(g, gi);
    const WordNb nb = word_nb(g, gp.w);
    const uint32_t vmask = (1u << gp.nv) - 1u;
    uint32_t nc[2 * D], X[2 * D];
    neighbour_words<D>(g, C + NW, gp.w, nb, nb.par, nc);
    const uint32_t C0 = C[gp.w];
    uint32_t any = 0;
#pragma unroll
    for (int k = 0; k < 2 * D; ++k) {
      X[k] = ((C0 ^ nc[k]) >> gp.shift) & vmask;
      any |= X[k];
    }
    if (!any) continue;
    uint32_t na[2 * D];
    neighbour_words<D>(g, A + NW, gp.w, nb, nb.par, na);
    const uint32_t A0 = A[gp.w];
#pragma unroll
    for (int k = 0; k < 2 * D; ++k) {
      if (!X[k]) continue;
      const uint32_t a = (A0 ^ na[k]) >> gp.shift;
      const int4 m = J0[(size_t)k * NGc + gi];
      for (int j = 0; j < 4; ++j)
        if ((X[k] >> j) & 1u) dl += ((a >> j) & 1u) ? lane_of(m, j) : -lane_of(m, j);
    }
  }
  return dl;
}

// (hi, lo) += (vhi, vlo) as one 128-bit integer held in two int64 words.
__device__ __forceinline__ void add128(int64_t* lo, int64_t* hi, uint64_t vlo, uint64_t vhi) {
  const uint64_t l = (uint64_t)*lo + vlo;
  *lo = (int64_t)l;
  *hi = (int64_t)((uint64_t)*hi + vhi + (l < vlo ? 1u : 0u));
}

}  // namespace ptsg
