// fused_device.h -- whole Monte Carlo steps (Sec. 2.4: Metropolis sweep, Houdayer
// move per same-temperature pair, replica-exchange pass, measurement) in one
// persistent kernel.  A workgroup holds one disorder sample (or one replica
// set of it, or one part of a sample too large for a workgroup) resident in
// LDS as colour-split row words for all steps of the launch; HBM is touched
// only to load the configurations at the start and store them at the end.
//
// Results are bit-identical to the per-step kernels: the same row update
// (rowops.h), the same Philox counters, exchange decisions taken in ascending
// k with the updated map, Houdayer seeds chosen in increasing site order.
#pragma once
#include <utility>

#include "device.h"
#include "kernels.h"
#include "exchange_ops.h"
#include "houdayer_ops.h"
#include "multicluster.h"
#include "rowops.h"

namespace ptsg {


// 2D samples get the in-register Houdayer move (one row per lane: L <= 64).
__host__ __device__ inline bool rows_houdayer(const Geo& g) { return g.d == 2; }

// ---------------------------------------------------------------------------
// Wave-level helpers.  Lanes of one wavefront exchange data through LDS; the
// wavefront issues its LDS instructions in order, so a compiler fence plus a
// wait for outstanding LDS operations orders one lane's writes before
// another lane's later reads.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------------------
// Replica exchange for both sets of the resident sample.  The pass is
// sequential in k, but every decision depends only on which configuration is
// carried up from below: with the pre-pass map m0, the configuration at
// position k before step k is m0[j] for some j <= k, and b = m0[k+1].  All
// candidate decisions (c, k, j) are evaluated in parallel and kept as bits
// (exchange_decide: half a wavefront per row (c, k) up to 32 temperatures, a
// wavefront above), then a wavefront per set follows the chain by ballots
// (exchange_chain: one lane per set above 64 temperatures).
// ---------------------------------------------------------------------------
// The inputs of pass u that the step's sweep and Houdayer move do not change:
// the map before the pass and one Philox word per (set, k).  Written before
// the sweep, so that the sweep's closing barrier orders them before the
// decisions.
__device__ __forceinline__ void exchange_prepare(const FusedArgs& A, uint32_t* lds, int s,
                                                 uint32_t u, int c_lo, int nsets) {
  const Geo& g = A.g;
  const int NT = g.NT, tid = threadIdx.x, T = blockDim.x;
  const int32_t* sotl = reinterpret_cast<const int32_t*>(lds + A.lay.sot);
  int32_t* sot0 = reinterpret_cast<int32_t*>(lds + A.lay.sot0);
  uint32_t* rpt = lds + A.lay.rpt;
  for (int i = tid; i < 2 * NT; i += T) sot0[i] = sotl[i];
  for (int i = tid; i < nsets * (NT - 1); i += T) {
    const int c = c_lo + i / (NT - 1), k = i - (c - c_lo) * (NT - 1);
    rpt[c * NT + k] =
        philox10(Ctr4{(uint32_t)k, u, (uint32_t)c, (kTagPT << 28) | (uint32_t)s}, g.key0, g.key1).x;
  }
}

// The pass itself, after exchange_prepare and a workgroup barrier; with WALK
// and `walk`, pass m (counted from 1) of the replica walk, with round trips
// summed in LDS (`walk` is false where the job does not track the walk or
// another workgroup of the sample keeps it).
template <bool WALK>
__device__ __forceinline__ void exchange_resident(const FusedArgs& A, uint32_t* lds, int c_lo,
                                                  int nsets, uint32_t m, bool walk) {
  const Geo& g = A.g;
  const int NT = g.NT;
  const int32_t* El = reinterpret_cast<const int32_t*>(lds + A.lay.E);
  const int32_t* sot0 = reinterpret_cast<const int32_t*>(lds + A.lay.sot0);
  const uint32_t* rpt = lds + A.lay.rpt;
  uint32_t* acc = lds + A.lay.acc;
  exchange_decide(NT, c_lo, nsets, acc, [&](int c, int k, int j) {
    const int a = sot0[c * NT + j], b = sot0[c * NT + k + 1];
    const int32_t D = El[c * NT + b] - El[c * NT + a];
    if (D <= 0) return true;
    const int md = D >> 1;
    return md < A.M && rpt[c * NT + k] < A.thrpt[(size_t)k * A.M + md];
  });
  __syncthreads();
  exchange_chain<WALK>(NT, c_lo, nsets, reinterpret_cast<int32_t*>(lds + A.lay.sot),
                       reinterpret_cast<int32_t*>(lds + A.lay.tos), sot0, acc,
                       WALK && walk ? reinterpret_cast<int32_t*>(lds + A.lay.walk) : nullptr,
                       WALK && walk ? reinterpret_cast<uint64_t*>(lds + A.lay.trip) : nullptr, m);
  __syncthreads();
}

// ---------------------------------------------------------------------------
// Moments of one temperature from the energies of its two replicas and the
// number of sites where they differ: sum E (both replicas), sum E^2, q, |q|,
// q^2 and q^4 as a 128-bit (lo, hi) pair, with Q = N q = N - 2 neg.  Each
// word is added in place with a 64-bit LDS atomic (one thread per
// temperature, so the atomics only keep the compiler from holding all eight
// words in registers at once); the carry out of the low q^4 word comes from
// the value it replaced.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void add_moments(const Geo& g, int64_t* m, int32_t ea, int32_t eb, int neg) {
  const int64_t Q = (int64_t)g.N - 2 * (int64_t)neg;
  const int64_t Ea = ea, Eb = eb;
  unsigned long long* u = reinterpret_cast<unsigned long long*>(m);
  atomicAdd(u + 0, (unsigned long long)(Ea + Eb));
  atomicAdd(u + 1, (unsigned long long)(Ea * Ea + Eb * Eb));
  atomicAdd(u + 2, (unsigned long long)Q);
  atomicAdd(u + 3, (unsigned long long)(Q < 0 ? -Q : Q));
  const uint64_t q2 = (uint64_t)(Q * Q);
  atomicAdd(u + 4, (unsigned long long)q2);
  const uint64_t q4lo = q2 * q2, q4hi = __umul64hi(q2, q2);
  const uint64_t old = atomicAdd(u + 5, (unsigned long long)q4lo);
  atomicAdd(u + 6, (unsigned long long)(q4hi + (old + q4lo < old ? 1u : 0u)));
}

// ---------------------------------------------------------------------------
// Measurement of every temperature of the resident sample: one wavefront per
// temperature counts the sites where its two replicas differ and adds the
// moments.
// ---------------------------------------------------------------------------
typedef short __attribute__((ext_vector_type(2))) Short2;

// How many lanes have a bit of `mask` set, each bit counted by itself: in XE
// for an even lane, in XO for an odd one.  The lanes' words are added as
// bit-sliced numbers (plane b: bit b of the count of every bit position), the
// 32 lanes of each half summing one of the two words.
__device__ __forceinline__ int column_counts(uint32_t XE, uint32_t XO, int lane, uint32_t mask) {
  const auto h = __builtin_amdgcn_permlane32_swap(XE, XO, false, false);
  uint32_t p[7] = {h[0] ^ h[1], h[0] & h[1], 0, 0, 0, 0, 0};
  auto add = [&](auto move, int planes) {
    uint32_t t = move(p[0]), c = p[0] & t;
    p[0] ^= t;
#pragma unroll
    for (int b = 1; b < planes; ++b) {
      t = move(p[b]);
      const uint32_t x = p[b];
      p[b] = bop3<kXor3>(x, t, c);
      c = bop3<kMaj3>(x, t, c);
    }
    p[planes] = c;
  };
  add([](uint32_t v) { return dpp_zero<kRowShr1>(v); }, 2);
  add([](uint32_t v) { return dpp_zero<kRowShr2>(v); }, 3);
  add([](uint32_t v) { return dpp_zero<kRowShr4>(v); }, 4);
  add([](uint32_t v) { return dpp_zero<kRowShr8>(v); }, 5);
  add([](uint32_t v) { return dpp_zero<kBcast15, 0xA>(v); }, 6);
  int n = 0;
#pragma unroll
  for (int b = 6; b >= 0; --b) {
    const uint32_t even = __builtin_amdgcn_readlane(p[b], 31), odd = __builtin_amdgcn_readlane(p[b], 63);
    n = 2 * n + __popc((lane & 1 ? odd : even) & mask);
  }
  return n;
}

// The two-replica modes of temperature k (mode_autocorr) by one wavefront,
// from the resident words of its two replicas: plane counts of the differing
// sites in the wavefront's LDS counters (slow axes by LDS atomics per word
// field, in 3D after the neighbouring lanes of the same plane have been added
// up: 16 lanes otherwise meet on one address at L = 16; the fast axis x0, whose
// sites interleave inside a field, by column_counts: bit j of a colour-c word
// is the site x0 = 2 (j mod H) + ((c + par) & 1) of its field's row), then
// A(delta) for delta <= L/2 added to the item's LDS sums.  Bound by instruction
// issue.  What the modes add to a measured step (us): 3D L = 16, 500 samples x
// 32 temperatures 10.9, against 19.7 with a ballot per bit position and one
// lane per delta for all axes; 3D L = 24, 100 x 16: 11.9 against 18.9; 2D
// L = 64, 500 x 24: 17 against 23.
__device__ __forceinline__ void modes_resident(const Geo& g, const FusedLayout& lay, uint32_t* lds,
                                               const uint32_t* Wa, const uint32_t* Wb, int k,
                                               int wave, int lane) {
  const int L = g.L, NW = g.NW, MH = L / 2 + 1;
  int32_t* cnt = reinterpret_cast<int32_t*>(lds + lay.mcnt) + wave * 3 * L;
  int64_t* acc = reinterpret_cast<int64_t*>(lds + lay.modes) + (size_t)k * MH;
  for (int i = lane; i < 3 * L; i += 64) cnt[i] = 0;
  wave_lds_sync();
  const int team = g.d == 3 ? min(L & -L, 16) : 1;
  uint32_t col0 = 0;  // the first bit of every row field
  for (int f = 0; f < g.P; ++f) col0 |= 1u << (f * g.H);
  int col = 0;  // lane x < L: differing sites at x0 = x
  for (int base = 0; base < NW; base += 64) {
    const int w = base + lane;
    uint32_t X0 = 0, X1 = 0;
    int par = 0, xs = 0;
    if (w < NW) {
      X0 = (Wa[w] ^ Wb[w]) & g.maskW;
      X1 = (Wa[NW + w] ^ Wb[NW + w]) & g.maskW;
      const WordNb q = word_nb(g, w);
      par = q.par;
      if (g.d == 3) {
        const int n = __popc(X0) + __popc(X1);
        if (n) atomicAdd(&cnt[L + q.x1], n);
      }
      xs = q.xs;
    }
    for (int f = 0; f < g.P; ++f) {
      const uint32_t m = g.maskH << (f * g.H);
      int n = __popc(X0 & m) + __popc(X1 & m);
      if (g.d == 3) {  // lanes of equal xs first
        n += (int)dpp_zero<kRowShr1>((uint32_t)n);
        if (team > 2) n += (int)dpp_zero<kRowShr2>((uint32_t)n);
        if (team > 4) n += (int)dpp_zero<kRowShr4>((uint32_t)n);
        if (team > 8) n += (int)dpp_zero<kRowShr8>((uint32_t)n);
      }
      if (w < NW && ((lane + 1) & (team - 1)) == 0 && n) atomicAdd(&cnt[(g.d - 1) * L + f * g.B + xs], n);
    }
    // colour-0 words hold the sites of x0 parity par, colour-1 words the other
    const uint32_t XE = par ? X1 : X0, XO = par ? X0 : X1;
    col += column_counts(XE, XO, lane, col0 << (lane >> 1));
  }
  if (lane < L) cnt[lane] = col;
  wave_lds_sync();
  // Plane sums P = L^(d-1) - 2 cnt (|P| <= 2^12) packed in 16-bit pairs, in
  // place: per axis the L/2 even-aligned pairs (P(2i), P(2i+1)), then the L/2
  // odd-aligned ones (P(2i+1), P(2i+2 mod L)).  sum_x P(x) P(x + delta) is then
  // L/2 two-way dot products of pair i with the pair starting at 2i + delta,
  // an even- or odd-aligned one as delta is even or odd.
  const int half = L / 2, plane = g.N / L;
  uint32_t pe[2], po[2];  // lane q and q + 64 of the d * half pairs (at most 96)
  int32_t* at[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const int q = lane + 64 * u;
    at[u] = nullptr;
    if (q < g.d * half) {
      const int mu = (q >= half ? 1 : 0) + (q >= 2 * half ? 1 : 0), i = q - mu * half;
      int32_t* c = cnt + mu * L;
      const int x = plane - 2 * c[2 * i], y = plane - 2 * c[2 * i + 1];
      const int z = plane - 2 * c[i + 1 == half ? 0 : 2 * i + 2];
      pe[u] = ((uint32_t)x & 0xFFFFu) | ((uint32_t)y << 16);
      po[u] = ((uint32_t)y & 0xFFFFu) | ((uint32_t)z << 16);
      at[u] = c + i;
    }
  }
  wave_lds_sync();
#pragma unroll
  for (int u = 0; u < 2; ++u)
    if (at[u]) {
      at[u][0] = (int32_t)pe[u];
      at[u][half] = (int32_t)po[u];
    }
  wave_lds_sync();
  // delta < L/2: one delta a lane, all axes' pairs in a row cut over the
  // 64 >> sh (at least two) copies of that lane range: 48 of the 96 pairs at most
  // in a copy's sum.
  constexpr long long kPair = 2ll * (1 << 12) * (1 << 12);  // L <= 64: |P| <= 2^12
  static_assert(48 * kPair < 1ll << 31 && 96 * (kPair / 4) < 1ll << 31, "mode sums in 32 bits");
  const Short2* pairs = reinterpret_cast<const Short2*>(cnt);
  const int sh = 32 - __clz(half - 1), dl = lane & ((1 << sh) - 1), all = g.d * half;
  const int chunk = (all + (64 >> sh) - 1) >> (6 - sh);
  const int q0 = (lane >> sh) * chunk, q1 = min(all, q0 + chunk);
  if (dl < half && q0 < all) {
    const int mu = (q0 >= half ? 1 : 0) + (q0 >= 2 * half ? 1 : 0), j0 = dl >> 1;
    const int other = (dl & 1) ? half : 0;
    int i = q0 - mu * half, j = i + j0, base = mu * L, sum = 0;
    if (j >= half) j -= half;
    for (int q = q0; q < q1; ++q) {
      sum = __builtin_amdgcn_sdot2(pairs[base + i], pairs[base + other + j], sum, false);
      if (++j == half) j = 0;
      if (++i == half) {
        i = 0;
        j = j0;
        base += L;
      }
    }
    atomicAdd(reinterpret_cast<unsigned long long*>(acc + dl), (unsigned long long)(int64_t)sum);
  }
  // delta = L/2: a pair a lane.  The plane sums are even, so every dot product
  // is a multiple of four.
  int far = 0;
  for (int q = lane; q < all; q += 64) {
    const int mu = (q >= half ? 1 : 0) + (q >= 2 * half ? 1 : 0), i = q - mu * half, j = i + (half >> 1);
    const Short2* E = pairs + mu * L;
    far += __builtin_amdgcn_sdot2(E[i], E[((half & 1) ? half : 0) + (j >= half ? j - half : j)], 0, false) >> 2;
  }
  far = wave_total(far);
  if (lane == 0) atomicAdd(reinterpret_cast<unsigned long long*>(acc + half), (unsigned long long)((int64_t)far * 4));
  wave_lds_sync();
}

template <bool MODES>
__device__ __forceinline__ void measure_resident(const FusedArgs& A, uint32_t* lds) {
  const Geo& g = A.g;
  const int NT = g.NT, NW = g.NW, tid = threadIdx.x, T = blockDim.x;
  const uint32_t* W = lds + A.lay.W;
  const int32_t* El = reinterpret_cast<const int32_t*>(lds + A.lay.E);
  const int32_t* sotl = reinterpret_cast<const int32_t*>(lds + A.lay.sot);
  int64_t* mom = reinterpret_cast<int64_t*>(lds + A.lay.mom);
  const int wave = tid >> 6, lane = tid & 63, nwave = T >> 6;
  for (int k = wave; k < NT; k += nwave) {
    const int a = sotl[k], b = NT + sotl[NT + k];
    const uint32_t* Wa = W + (size_t)a * 2 * NW;
    const uint32_t* Wb = W + (size_t)b * 2 * NW;
    int neg = 0;
    for (int w = lane; w < 2 * NW; w += 64) neg += __popc(Wa[w] ^ Wb[w]);
    neg = wave_total(neg);
    if (lane == 0) add_moments(g, mom + (size_t)k * 8, El[a], El[b], neg);
    if (MODES && A.modes) modes_resident(g, A.lay, lds, Wa, Wb, k, wave, lane);
  }
  __syncthreads();
}


// ---------------------------------------------------------------------------
// Column fills for a square lattice held one row per lane (2D: L <= 64 rows).
// The even sites of row r have colour r & 1, and the site above bit b of row
// r's even-site word is bit b of row r + 1's even-site word (likewise for the
// odd sites), so the chain X_r = even-site word of row r (and Y, the odd-site
// words) links equal bits of consecutive lanes, periodically (lane L - 1 to
// lane 0).  The lanes past the last row take part as transparent ones (every
// bit of q set, none of c): what reaches lane L - 1 passes through them to
// lane 63 and wraps, so that every L runs the same 64-lane scans.  Filling a
// chain from its cluster bits through its q bits is a scan with the associative
// operator (q1, c1) then (q2, c2) -> (q1 & q2, c2 | (q2 & c1)).  Upward it
// runs over rows of 16 lanes by DPP row shifts and then across rows by the
// DPP broadcasts of lanes 15 and 31; downward by row shifts and then across
// rows through the four row totals read back as wavefront constants.  The
// AND-of-q half of every step depends on q alone and is computed once per
// pair; each fill then costs one DPP move and one AND-OR per step.
// ---------------------------------------------------------------------------
struct ColumnChain {
  uint32_t q;
  uint32_t p1, p2, p3, p4, p5, p6;  // upward: AND of q over the lanes each step has joined
  uint32_t d1, d2, d3;              // downward, within the row
  uint32_t m0, m1, m2, m3;          // AND of q from the lane to the top of its row, row r only
  uint32_t t0, t1, t2, t3;          // AND of q over all of row r (wavefront constants)
};

__device__ __forceinline__ ColumnChain column_chain(uint32_t q, int lane) {
  ColumnChain h;
  h.q = q;
  uint32_t p = q;
  h.p1 = p = p & dpp_ones<kRowShr1>(p);
  h.p2 = p = p & dpp_ones<kRowShr2>(p);
  h.p3 = p = p & dpp_ones<kRowShr4>(p);
  h.p4 = p = p & dpp_ones<kRowShr8>(p);
  h.p5 = p = p & dpp_ones<kBcast15, 0xA>(p);
  h.p6 = p & dpp_ones<kBcast31, 0xC>(p);
  uint32_t d = q;
  h.d1 = d = d & dpp_ones<kRowShl1>(d);
  h.d2 = d = d & dpp_ones<kRowShl2>(d);
  h.d3 = d = d & dpp_ones<kRowShl4>(d);
  d &= dpp_ones<kRowShl8>(d);
  const int row = lane >> 4;
  h.m0 = row == 0 ? d : 0u;
  h.m1 = row == 1 ? d : 0u;
  h.m2 = row == 2 ? d : 0u;
  h.m3 = row == 3 ? d : 0u;
  h.t0 = (uint32_t)__builtin_amdgcn_readlane((int)d, 0);
  h.t1 = (uint32_t)__builtin_amdgcn_readlane((int)d, 16);
  h.t2 = (uint32_t)__builtin_amdgcn_readlane((int)d, 32);
  h.t3 = (uint32_t)__builtin_amdgcn_readlane((int)d, 48);
  return h;
}

// Every q bit of the chain connected along it (periodically) to a bit of c,
// for c a subset of q.
__device__ __forceinline__ uint32_t column_fill(const ColumnChain& h, uint32_t c) {
  // upward; then what reaches lane 63 continues from lane 0
  uint32_t u = c;
  u |= dpp_zero<kRowShr1>(u) & h.q;
  u |= dpp_zero<kRowShr2>(u) & h.p1;
  u |= dpp_zero<kRowShr4>(u) & h.p2;
  u |= dpp_zero<kRowShr8>(u) & h.p3;
  u |= dpp_zero<kBcast15, 0xA>(u) & h.p4;
  u |= dpp_zero<kBcast31, 0xC>(u) & h.p5;
  u |= h.p6 & (uint32_t)__builtin_amdgcn_readlane((int)u, 63);
  // downward within rows, then across rows from the reach at each row's
  // lowest lane: r0 (lane 0, without the wrap) goes on from lane 63
  uint32_t d = c;
  d |= dpp_zero<kRowShl1>(d) & h.q;
  d |= dpp_zero<kRowShl2>(d) & h.d1;
  d |= dpp_zero<kRowShl4>(d) & h.d2;
  d |= dpp_zero<kRowShl8>(d) & h.d3;
  const uint32_t c0 = (uint32_t)__builtin_amdgcn_readlane((int)d, 0);
  const uint32_t c1 = (uint32_t)__builtin_amdgcn_readlane((int)d, 16);
  const uint32_t c2 = (uint32_t)__builtin_amdgcn_readlane((int)d, 32);
  const uint32_t c3 = (uint32_t)__builtin_amdgcn_readlane((int)d, 48);
  const uint32_t r0 = c0 | (h.t0 & (c1 | (h.t1 & (c2 | (h.t2 & c3)))));
  const uint32_t r48 = c3 | (h.t3 & r0);
  const uint32_t r32 = c2 | (h.t2 & r48);
  const uint32_t r16 = c1 | (h.t1 & r32);
  d |= (h.m0 & r16) | (h.m1 & r32) | (h.m2 & r48) | (h.m3 & r0);
  return u | d;
}

// x as a value that the compiler cannot hoist: what derives from it (masks,
// addresses) is recomputed where it is used instead of staying live in
// registers through the rest of the step loop.
__device__ __forceinline__ int recomputed(int x) {
  asm volatile("" : "+v"(x));
  return x;
}

// The Houdayer cluster of pair k grown by one wavefront in LDS words (Qw, Cw:
// 2 NW words each), for lattices of more words than lanes.  False if the pair
// has no q = -1 site; else Cw holds the cluster's colour words.
template <int D>
__device__ __forceinline__ bool lds_cluster(const Geo& g, const uint32_t* Wa, const uint32_t* Wb,
                                            uint32_t* Qw, uint32_t* Cw, int s, int k, uint32_t v,
                                            int lane) {
  const int NW = g.NW;
  for (int w = lane; w < NW; w += 64) {
    const uint32_t q0 = Wa[w] ^ Wb[w], q1 = Wa[NW + w] ^ Wb[NW + w];
    const bool par = word_nb(g, w).par;
    Qw[w] = par ? q1 : q0;
    Qw[NW + w] = par ? q0 : q1;
    Cw[w] = Cw[NW + w] = 0u;
  }
  wave_lds_sync();
  if (!seed_words(g, Qw, Cw, s, k, v, lane)) return false;
  wave_lds_sync();
  for (bool first = true;; first = false) {
    bool changed = false;
    for (int w = lane; w < NW; w += 64) changed |= grow_rows<D>(g, Cw, Qw, w, first);
    wave_lds_sync();
    if (!__any(changed)) break;
  }
  for (int w = lane; w < NW; w += 64)
    if (word_nb(g, w).par) {  // colour form
      const uint32_t e = Cw[w];
      Cw[w] = Cw[NW + w];
      Cw[NW + w] = e;
    }
  wave_lds_sync();
  return true;
}

// Geometry of a 2D row held by itself in a word's low H bits.
__device__ __forceinline__ Geo row_geo(const Geo& g) {
  Geo r = g;
  r.P = 1;
  r.B = g.L;
  r.LB = 1u;
  r.HB = 1u << (g.H - 1);
  r.maskW = g.maskH;
  return r;
}

// A lane's row of a 2D lattice (lanes past the last row hold none): its word
// and field shift, whether it exists, and the lanes of the next and previous
// rows (periodic).  LS = 64: row = word = lane.
struct LaneRow {
  int w, sh, next, prev;
  bool valid;
};
template <int LS>
__device__ __forceinline__ LaneRow lane_row(const Geo& g, int lane) {
  LaneRow r;
  if constexpr (LS == 64) {
    r.w = lane;
    r.sh = 0;
    r.next = r.prev = lane;  // unused: the wavefront rotates
    r.valid = true;
  } else {
    r.valid = lane < g.L;
    const int R = r.valid ? lane : 0, f = R / g.B;
    r.w = R - f * g.B;
    r.sh = f * g.H;
    r.next = !r.valid ? lane : lane == g.L - 1 ? 0 : lane + 1;
    r.prev = !r.valid ? lane : lane == 0 ? g.L - 1 : lane - 1;
  }
  return r;
}
// The row's field of word x (0 for a lane without a row).
template <int LS>
__device__ __forceinline__ uint32_t row_field(const Geo& g, const LaneRow& r, uint32_t x) {
  if constexpr (LS == 64) return x;
  return r.valid ? (x >> r.sh) & g.maskH : 0u;
}
// The next / previous row's value of x.
template <int LS>
__device__ __forceinline__ uint32_t row_next(const LaneRow& r, uint32_t x) {
  if constexpr (LS == 64) return dpp_ones<kWaveRol1>(x);  // lane 63 takes lane 0
  return (uint32_t)__builtin_amdgcn_ds_bpermute(4 * r.next, (int)x);
}
template <int LS>
__device__ __forceinline__ uint32_t row_prev(const LaneRow& r, uint32_t x) {
  if constexpr (LS == 64) return dpp_ones<kWaveRor1>(x);
  return (uint32_t)__builtin_amdgcn_ds_bpermute(4 * r.prev, (int)x);
}

// The Houdayer cluster of pair k of a 2D sample, one row per lane, everything
// in registers: overlap, seed (the m-th q = -1 site in site order, by a scan
// over lanes), flood fill alternating column fills and row closures until one
// of them adds nothing.  g is the row geometry.  False (for the whole
// wavefront) if the pair has no q = -1 site; else c0, c1 are the cluster's
// colour-0 and colour-1 fields of this lane's row.
template <int LS>
__device__ __forceinline__ bool rows_cluster(const Geo& g, const LaneRow& lr, int NW, const uint32_t* Wa,
                                             const uint32_t* Wb, int s, int k, uint32_t v, int lane,
                                             uint32_t& c0, uint32_t& c1) {
  const bool odd = lane & 1;  // parity of the row = colour of its even sites
  const uint32_t q0 = row_field<LS>(g, lr, Wa[lr.w] ^ Wb[lr.w]);
  const uint32_t q1 = row_field<LS>(g, lr, Wa[NW + lr.w] ^ Wb[NW + lr.w]);
  const uint32_t qx = odd ? q1 : q0, qy = odd ? q0 : q1;
  // q = -1 sites up to and including this row (a DPP scan over the rows)
  const uint32_t lc = __popc(q0) + __popc(q1);
  const uint32_t incl = wave_scan(lc);
  const uint32_t n = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  if (n == 0) return false;
  // seed: the m-th q = -1 site in increasing site order (row by row)
  const uint32_t m = seed_rank(g, s, k, v, n);
  uint32_t X = 0, Y = 0;  // cluster: even-site and odd-site words of the row
  if (m >= incl - lc && m < incl) rank_in_row64(qx, qy, m - (incl - lc), X, Y);
  const uint32_t rqx = __builtin_bitreverse32(qx), rqy = __builtin_bitreverse32(qy);
  row_closure(g, X, Y, qx, qy, rqx, rqy);
  const uint32_t clear = lr.valid ? 0u : ~0u;  // transparent lanes of the column scans
  const ColumnChain hx = column_chain(qx | clear, lane), hy = column_chain(qy | clear, lane);
  for (;;) {
    uint32_t nx = column_fill(hx, X), ny = column_fill(hy, Y);
    if constexpr (LS != 64) {
      nx &= ~clear;
      ny &= ~clear;
    }
    if (!__any(nx != X || ny != Y)) break;
    X = nx;
    Y = ny;
    row_closure(g, nx, ny, qx, qy, rqx, rqy);
    if (!__any(nx != X || ny != Y)) break;
    X = nx;
    Y = ny;
  }
  c0 = odd ? Y : X;
  c1 = odd ? X : Y;
  return true;
}

// Exchanges the pair's replicas on the cluster fields c0, c1 of this lane's
// row; ab: the row's words before the move (replica a's colours, then b's;
// read by the whole-word form only).
template <int LS>
__device__ __forceinline__ void rows_exchange(const LaneRow& lr, int NW, uint32_t* Wa, uint32_t* Wb,
                                              const uint32_t (&ab)[4], uint32_t c0, uint32_t c1) {
  if constexpr (LS == 64) {
    Wa[lr.w] = ab[0] ^ c0;
    Wa[64 + lr.w] = ab[1] ^ c1;
    Wb[lr.w] = ab[2] ^ c0;
    Wb[64 + lr.w] = ab[3] ^ c1;
  } else {
    // rows that share a word write only their own bits
    if (c0) {
      atomicXor(&Wa[lr.w], c0 << lr.sh);
      atomicXor(&Wb[lr.w], c0 << lr.sh);
    }
    if (c1) {
      atomicXor(&Wa[NW + lr.w], c1 << lr.sh);
      atomicXor(&Wb[NW + lr.w], c1 << lr.sh);
    }
  }
}

// The next pair of the Houdayer phase for this wavefront, from the hottest
// down (clusters grow larger and take more passes at high temperature), each
// to the next free wavefront; -1 when none is left.  Every lane adds 1 (one
// 64-count LDS atomic per take) and all read lane 0's result: a take under a
// lane-0 branch would let the compiler run the other lanes on into the next
// pair without it.  The counter is cleared after each Houdayer phase.
__device__ __forceinline__ int take_pair_hottest(uint32_t* hctr, int NT) {
  const uint32_t i = (uint32_t)__builtin_amdgcn_readfirstlane((int)atomicAdd(hctr, 1u)) >> 6;
  return i >= (uint32_t)NT ? -1 : NT - 1 - (int)i;
}

// Houdayer moves of a 2D sample, one wavefront per pair at a time and one row
// per lane (rows_cluster), then the energy change from the bonds leaving the
// cluster (vertical neighbours taken from the adjacent rows' lanes) and the
// exchange on the cluster.  gw is the sample's geometry (LS = 64: folded).
// Any L <= 64 has at most one row per lane, so no 2D shape needs LDS for its
// cluster; bound by the VALU work of the fills (about 8 rounds of two column
// fills and a closure per hot pair).  Against the flood fill through LDS words
// that every L < 64 took before, whole steps: L = 50, 77 samples x 2 x 13:
// 62.6 -> 21.4 us; L = 50, 500 x 2 x 24: 172 -> 63 us; L = 32, 77 x 2 x 13:
// 38.4 -> 14.8 us.
template <int LS>
__device__ __forceinline__ void houdayer_rows(const Geo& gw, uint32_t* W, const uint32_t* Jl, int32_t* El,
                                              const int32_t* sotl, int s, uint32_t v, uint32_t* hctr,
                                              int lane) {
  const Geo g = LS == 64 ? gw : row_geo(gw);
  const int NT = g.NT, NW = gw.NW;
  const bool odd = lane & 1;
  const LaneRow lr = lane_row<LS>(gw, lane);
  for (;;) {
    const int k = take_pair_hottest(hctr, NT);
    if (k < 0) break;
    const int a = sotl[k], b = NT + sotl[NT + k];
    uint32_t* Wa = W + (size_t)a * 2 * NW;
    uint32_t* Wb = W + (size_t)b * 2 * NW;
    uint32_t c0, c1;
    if (!rows_cluster<LS>(g, lr, NW, Wa, Wb, s, k, v, lane, c0, c1)) continue;
    uint32_t ab[4] = {Wa[lr.w], Wa[NW + lr.w], 0u, 0u};
    if constexpr (LS == 64) {
      ab[2] = Wb[lr.w];
      ab[3] = Wb[NW + lr.w];
    }
    const uint32_t a0 = row_field<LS>(g, lr, ab[0]), a1 = row_field<LS>(g, lr, ab[1]);
    // energy change of replica a over the bonds of the colour-0 sites (each
    // bond has one): +x0, -x0 in the row, +x1, -x1 in the next/previous row
    uint32_t nc[4], na[4];
    x0_neighbours(g, c1, odd, nc[0], nc[1]);
    x0_neighbours(g, a1, odd, na[0], na[1]);
    nc[2] = row_next<LS>(lr, c1);
    nc[3] = row_prev<LS>(lr, c1);
    na[2] = row_next<LS>(lr, a1);
    na[3] = row_prev<LS>(lr, a1);
    int cross = 0, cross_u = 0;
#pragma unroll
    for (int dir = 0; dir < 4; ++dir) {
      const uint32_t X = c0 ^ nc[dir];
      const uint32_t U = a0 ^ na[dir] ^ (LS == 64 ? Jl[dir * NW + lr.w] : Jl[dir * NW + lr.w] >> lr.sh);
      cross += __popc(X);
      cross_u += __popc(X & U);
    }
    const int delta = wave_total(2 * (cross - 2 * cross_u));
    rows_exchange<LS>(lr, NW, Wa, Wb, ab, c0, c1);
    if (lane == 0) {
      El[a] += delta;
      El[b] -= delta;
    }
  }
}

// ---------------------------------------------------------------------------
// The same move for a 3D sample with at most 64 words per colour, one word
// index (P rows of one x1) per lane, everything in registers.  The cluster is
// kept in row form (even and odd sites of each row field), in which the
// neighbours along x1 and x2 of a lane's even word are the even words of four
// other lanes.
// ---------------------------------------------------------------------------
__host__ __device__ inline bool words_houdayer(const Geo& g) { return g.d == 3 && g.NW <= 64; }

// A lane's word: whether it exists, its neighbour geometry, and the lanes (as
// ds_bpermute byte indices) holding the words next to it.  LS = 16: rows of 16
// lanes are the x1 chains, so x1 neighbours are DPP row rotations.
struct LaneWord {
  WordNb nb;
  int w, up1, dn1, ups, dns;
  bool valid;
};
__device__ __forceinline__ LaneWord lane_word(const Geo& g, int lane) {
  LaneWord r;
  r.valid = lane < g.NW;
  r.w = r.valid ? lane : 0;
  r.nb = word_nb(g, r.w);
  r.up1 = 4 * (r.valid ? r.nb.w1p : lane);
  r.dn1 = 4 * (r.valid ? r.nb.w1m : lane);
  r.ups = 4 * (r.valid ? r.nb.wsp : lane);
  r.dns = 4 * (r.valid ? r.nb.wsm : lane);
  return r;
}
constexpr int kRowRor1 = 0x121, kRowRor15 = 0x12F;  // lane i takes i - 1 / i + 1 (mod 16)
template <int LS>
__device__ __forceinline__ uint32_t word_up1(const LaneWord& r, uint32_t x) {
  if constexpr (LS == 16) return dpp_zero<kRowRor15>(x);
  return (uint32_t)__builtin_amdgcn_ds_bpermute(r.up1, (int)x);
}
template <int LS>
__device__ __forceinline__ uint32_t word_dn1(const LaneWord& r, uint32_t x) {
  if constexpr (LS == 16) return dpp_zero<kRowRor1>(x);
  return (uint32_t)__builtin_amdgcn_ds_bpermute(r.dn1, (int)x);
}
__device__ __forceinline__ uint32_t word_ups(const Geo& g, const LaneWord& r, uint32_t x) {
  const uint32_t y = (uint32_t)__builtin_amdgcn_ds_bpermute(r.ups, (int)x);
  return r.nb.crp ? rot_fields_down(g, y) : y;
}
__device__ __forceinline__ uint32_t word_dns(const Geo& g, const LaneWord& r, uint32_t x) {
  const uint32_t y = (uint32_t)__builtin_amdgcn_ds_bpermute(r.dns, (int)x);
  return r.nb.crm ? rot_fields_up(g, y) : y;
}

// The Houdayer cluster of pair k: as rows_cluster, with the fill advancing one
// word along x1 and x2 per round and a whole run along x0.  c0, c1: the
// cluster's colour-0 and colour-1 bits of this lane's word.
template <int LS>
__device__ __forceinline__ bool words_cluster(const Geo& g, const LaneWord& lw, const uint32_t* Wa,
                                              const uint32_t* Wb, int s, int k, uint32_t v, uint32_t& c0,
                                              uint32_t& c1) {
  const int NW = g.NW;
  const bool par = lw.nb.par;
  uint32_t q0 = Wa[lw.w] ^ Wb[lw.w], q1 = Wa[NW + lw.w] ^ Wb[NW + lw.w];
  if (!lw.valid) q0 = q1 = 0u;
  const uint32_t ME = par ? q1 : q0, MO = par ? q0 : q1;
  const uint32_t n = (uint32_t)wave_total(__popc(ME) + __popc(MO));
  if (n == 0) return false;
  uint32_t m = seed_rank(g, s, k, v, n);
  // site order is field by field, then lane by lane (x2 = f B + xs', then x1)
  uint32_t E = 0, O = 0;
  for (int f = 0;; ++f) {
    const uint32_t fe = (ME >> (f * g.H)) & g.maskH, fo = (MO >> (f * g.H)) & g.maskH;
    const uint32_t lc = __popc(fe) + __popc(fo), incl = wave_scan(lc);
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    if (m >= tot) {
      m -= tot;
      continue;
    }
    if (m >= incl - lc && m < incl) {
      rank_in_row64(fe, fo, m - (incl - lc), E, O);
      E <<= f * g.H;
      O <<= f * g.H;
    }
    break;
  }
  const uint32_t rME = __builtin_bitreverse32(ME), rMO = __builtin_bitreverse32(MO);
  row_fill(g, E, O, ME, MO, rME, rMO);
  for (;;) {
    const uint32_t xe = word_up1<LS>(lw, E) | word_dn1<LS>(lw, E) | word_ups(g, lw, E) | word_dns(g, lw, E);
    const uint32_t xo = word_up1<LS>(lw, O) | word_dn1<LS>(lw, O) | word_ups(g, lw, O) | word_dns(g, lw, O);
    uint32_t nE = E | (ME & (xe | ((O & g.HB) >> (g.H - 1))));
    uint32_t nO = O | (MO & (xo | ((E & g.LB) << (g.H - 1))));
    if (!__any(nE != E || nO != O)) break;
    E = nE;
    O = nO;
    row_fill(g, E, O, ME, MO, rME, rMO);
  }
  c0 = par ? O : E;
  c1 = par ? E : O;
  return true;
}

// Houdayer moves of such a sample, one wavefront per pair at a time.  Bound by
// the rounds of the fill (a round waits for its cross-lane moves); 3D L = 12,
// 256 samples x 2 x 20: 30 -> 15 us of a 49 -> 34 us step against the fill
// through LDS words; L = 16: 34 -> 12 us.
template <int LS>
__device__ __forceinline__ void houdayer_words(const Geo& g, uint32_t* W, const uint32_t* Jl, int32_t* El,
                                               const int32_t* sotl, int s, uint32_t v, uint32_t* hctr,
                                               int lane) {
  const int NT = g.NT, NW = g.NW;
  const LaneWord lw = lane_word(g, lane);
  for (;;) {
    const int k = take_pair_hottest(hctr, NT);
    if (k < 0) break;
    const int a = sotl[k], b = NT + sotl[NT + k];
    uint32_t* Wa = W + (size_t)a * 2 * NW;
    uint32_t* Wb = W + (size_t)b * 2 * NW;
    uint32_t c0, c1;
    if (!words_cluster<LS>(g, lw, Wa, Wb, s, k, v, c0, c1)) continue;
    // energy change of replica a over the bonds of the colour-0 sites
    uint32_t nc[6], na[6];
    x0_neighbours(g, c1, lw.nb.par, nc[0], nc[1]);
    nc[2] = word_up1<LS>(lw, c1);
    nc[3] = word_dn1<LS>(lw, c1);
    nc[4] = word_ups(g, lw, c1);
    nc[5] = word_dns(g, lw, c1);
    neighbour_words<3>(g, Wa + NW, lw.w, lw.nb, lw.nb.par, na);
    const uint32_t a0 = Wa[lw.w];
    int cross = 0, cross_u = 0;
#pragma unroll
    for (int dir = 0; dir < 6; ++dir) {
      const uint32_t X = c0 ^ nc[dir];
      const uint32_t U = a0 ^ na[dir] ^ Jl[dir * NW + lw.w];
      cross += __popc(X);
      cross_u += __popc(X & U);
    }
    const int delta = wave_total(lw.valid ? 2 * (cross - 2 * cross_u) : 0);
    wave_lds_sync();  // every lane has read its neighbours' words
    if (lw.valid) {
      Wa[lw.w] ^= c0;
      Wa[NW + lw.w] ^= c1;
      Wb[lw.w] ^= c0;
      Wb[NW + lw.w] ^= c1;
    }
    if (lane == 0) {
      El[a] += delta;
      El[b] -= delta;
    }
  }
}

// ---------------------------------------------------------------------------
// Houdayer moves for all NT pairs of the resident sample: each wavefront
// takes one pair at a time and grows its cluster alone, so clusters of very
// different size (cold versus hot pairs) do not wait for one another.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void houdayer_resident(const FusedArgs& A, uint32_t* lds, int s,
                                                  uint32_t v) {
  const Geo& g = A.g;
  const int NT = g.NT, NW = g.NW, tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  uint32_t* W = lds + A.lay.W;
  const uint32_t* Jl = lds + A.lay.J;  // colour-0 direction words first
  int32_t* El = reinterpret_cast<int32_t*>(lds + A.lay.E);
  const int32_t* sotl = reinterpret_cast<const int32_t*>(lds + A.lay.sot);
  uint32_t* hctr = lds + A.lay.hq;
  if constexpr (D == 2) {
    if (g.L == 64)
      houdayer_rows<64>(fixed_shape<2, 64>(g), W, Jl, El, sotl, s, v, hctr, recomputed(lane));
    else
      houdayer_rows<0>(g, W, Jl, El, sotl, s, v, hctr, recomputed(lane));
  } else if (g.L == 16) {
    houdayer_words<16>(fixed_shape<3, 16>(g), W, Jl, El, sotl, s, v, hctr, recomputed(lane));
  } else if (words_houdayer(g)) {
    houdayer_words<0>(g, W, Jl, El, sotl, s, v, hctr, recomputed(lane));
  } else {
    const int W2 = 2 * NW;
    uint32_t* Qw = lds + A.lay.Qs + (size_t)wave * 2 * W2;  // row form
    uint32_t* Cw = Qw + W2;
    for (;;) {
      const int k = take_pair_hottest(hctr, NT);
      if (k < 0) break;
      const int a = sotl[k], b = NT + sotl[NT + k];
      uint32_t* Wa = W + (size_t)a * W2;
      uint32_t* Wb = W + (size_t)b * W2;
      if (!lds_cluster<D>(g, Wa, Wb, Qw, Cw, s, k, v, lane)) continue;
      // energy change of replica a, then exchange the replicas on the cluster
      int dl = 0;
      for (int w = lane; w < NW; w += 64) dl += cluster_delta_word<D>(g, Cw, Wa, Jl, w);
      const int delta = wave_total(dl);
      for (int i = lane; i < W2; i += 64) {
        const uint32_t cw = Cw[i];
        if (cw) {
          Wa[i] ^= cw;
          Wb[i] ^= cw;
        }
      }
      if (lane == 0) {
        El[a] += delta;
        El[b] -= delta;
      }
      wave_lds_sync();
    }
  }
  __syncthreads();
  if (tid == 0) *hctr = 0u;  // the next use is behind the step's barriers
}

// ---------------------------------------------------------------------------
// Multi-cluster Houdayer moves for all NT pairs of the resident sample: the
// first PC wavefronts (those with a scratch area) take the pairs, hottest first,
// each finding the exchanged clusters of its pair (multi_cluster_words),
// then applying them as the single-cluster move applies its cluster.
// ---------------------------------------------------------------------------
template <int D>
__device__ __forceinline__ void houdayer_multi_resident(const FusedArgs& A, uint32_t* lds, int s,
                                                        uint32_t v) {
  const Geo& g = A.g;
  const int NT = g.NT, NW = g.NW, W2 = 2 * NW, tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63, PC = A.lay.PC;
  uint32_t* W = lds + A.lay.W;
  const uint32_t* Jl = lds + A.lay.J;
  int32_t* El = reinterpret_cast<int32_t*>(lds + A.lay.E);
  const int32_t* sotl = reinterpret_cast<const int32_t*>(lds + A.lay.sot);
  if (wave < PC) {
    const int stride = (multi_scratch_words(g) + 1) & ~1;
    uint32_t* Qw = lds + A.lay.Qs + (size_t)wave * stride;
    uint32_t* Cw = Qw + W2;
    for (;;) {
      const int k = take_pair_hottest(lds + A.lay.hq, NT);
      if (k < 0) break;
      const int a = sotl[k], b = NT + sotl[NT + k];
      uint32_t* Wa = W + (size_t)a * W2;
      uint32_t* Wb = W + (size_t)b * W2;
      for (int i = lane; i < W2; i += 64) Qw[i] = Wa[i] ^ Wb[i];
      wave_lds_sync();
      multi_cluster_words<D>(
          g, Qw, Cw, Cw + W2, s, k, v, lane, 64, [] { wave_lds_sync(); },
          [](bool b) {
            wave_lds_sync();
            return (bool)__any(b);
          });
      int dl = 0;
      for (int w = lane; w < NW; w += 64) dl += cluster_delta_word<D>(g, Cw, Wa, Jl, w);
      const int delta = wave_total(dl);
      for (int i = lane; i < W2; i += 64) {
        const uint32_t cw = Cw[i];
        if (cw) {
          Wa[i] ^= cw;
          Wb[i] ^= cw;
        }
      }
      if (lane == 0) {
        El[a] += delta;
        El[b] -= delta;
      }
      wave_lds_sync();
    }
  }
  __syncthreads();
  if (tid == 0) lds[A.lay.hq] = 0u;  // the next use is behind the step's barriers
}

// ---------------------------------------------------------------------------
// One Metropolis sweep (colour 0, then colour 1) of the resident
// configurations ls in [0, nres): configuration ls is slot slot0 + ls, its
// words at W + ls * 2 NW, its couplings J (colour-c direction words at
// J + c * 2 D NW).  A configuration's colour-1 update reads only its own
// colour-0 words, so when each configuration's words fall to one wavefront
// (NW a multiple or a divisor of 64: the 64-item units of a configuration,
// or the whole configurations of a unit, all go to the same wavefront) every
// wavefront runs both half-sweeps of its configurations back to back,
// ordered by a wavefront-level LDS fence, as long as that spreads the words
// over the wavefronts as evenly as the flat loop; otherwise the workgroup
// meets between the colours.  Ends with a workgroup barrier.
// ---------------------------------------------------------------------------
template <int D, int LS>
__device__ __forceinline__ void sweep_resident_shape(const Geo& g, const FusedArgs& A,
                                                     const uint32_t* J, uint32_t* W, int32_t* El,
                                                     const int32_t* tosl, const uint32_t* thrl,
                                                     int slot0, int nres, int s, uint32_t t) {
  const int NW = g.NW, W2 = 2 * NW, items = nres * NW, tid = threadIdx.x, T = blockDim.x;
  auto update = [&](int it, int c) {
    const int ls = LS ? it / NW : (int)__umulhi((uint32_t)it, A.magicNW), w = it - ls * NW;
    const int slot = slot0 + ls;
    const int k = tosl[slot];
    int dE = 0;
    sweep_word<D>(g, W + ls * W2, J + c * 2 * D * NW, c, w, slot, s, t, thrl[k * 4 + 0],
                  thrl[k * 4 + 1], thrl[k * 4 + 2], dE);
    if (dE) atomicAdd(&El[slot], dE);
  };
  // whole configurations per wavefront only where that loads the wavefronts
  // as evenly as the flat loop (a split part can hold fewer configurations
  // than there are wavefronts)
  const int nwave = T >> 6;
  const bool owned =
      64 % NW == 0 ||
      (NW % 64 == 0 && (nres + nwave - 1) / nwave * nwave * NW <= (items + T - 1) / T * T);
  constexpr bool kWordPerLane = LS != 0 && geo_shape(LS, D).NW == 64;
  if constexpr (kWordPerLane) {
    // every unit is one configuration and lane w always updates word w: the
    // word's coupling words are loaded once per colour
    const int nunits = nres, lane = tid & 63, step = T >> 6;
    for (int c = 0; c < 2; ++c) {
      uint32_t jv[2 * D];
#pragma unroll
      for (int dir = 0; dir < 2 * D; ++dir) jv[dir] = J[(c * 2 * D + dir) * NW + lane];
      for (int u = tid >> 6; u < nunits; u += step) {
        const int slot = slot0 + u;
        const int k = tosl[slot];
        int dE = 0;
        sweep_word_j<D>(g, W + u * W2, jv, c, lane, slot, s, t, thrl[k * 4 + 0], thrl[k * 4 + 1],
                        thrl[k * 4 + 2], dE);
        if (dE) atomicAdd(&El[slot], dE);
      }
      if (c == 0) wave_lds_sync();
    }
  } else if (owned) {
    const int m = NW >= 64 ? NW >> 6 : 1;  // units per configuration (or 1)
    const int nunits = (items + 63) >> 6, lane = tid & 63, step = (T >> 6) * m;
    for (int c = 0; c < 2; ++c) {
      for (int u0 = (tid >> 6) * m; u0 < nunits; u0 += step)
        for (int u = u0; u < u0 + m; ++u) {
          const int it = (u << 6) + lane;
          if (it < items) update(it, c);
        }
      if (c == 0) wave_lds_sync();
    }
  } else {
    for (int it = tid; it < items; it += T) update(it, 0);
    __syncthreads();
    for (int it = tid; it < items; it += T) update(it, 1);
  }
  __syncthreads();
}

// The sweep with the geometry of the shapes the workloads run most folded to
// compile-time constants (3D L = 16, 2D L = 64; for split samples, which run
// one workgroup per CU whatever their registers, also 3D L = 24, 32 and 48),
// else from g.
template <int D, bool kSplitShapes = false>
__device__ __forceinline__ void sweep_resident(const FusedArgs& A, const uint32_t* J, uint32_t* W,
                                               int32_t* El, const int32_t* tosl,
                                               const uint32_t* thrl, int slot0, int nres, int s,
                                               uint32_t t) {
  constexpr int kFixedL = D == 3 ? 16 : 64;
  if (A.g.L == kFixedL) {
    sweep_resident_shape<D, kFixedL>(fixed_shape<D, kFixedL>(A.g), A, J, W, El, tosl, thrl, slot0,
                                     nres, s, t);
    return;
  }
  if constexpr (kSplitShapes && D == 3) {
    if (A.g.L == 32) {
      sweep_resident_shape<3, 32>(fixed_shape<3, 32>(A.g), A, J, W, El, tosl, thrl, slot0, nres,
                                  s, t);
      return;
    }
    if (A.g.L == 48) {
      sweep_resident_shape<3, 48>(fixed_shape<3, 48>(A.g), A, J, W, El, tosl, thrl, slot0, nres,
                                  s, t);
      return;
    }
    if (A.g.L == 24) {
      sweep_resident_shape<3, 24>(fixed_shape<3, 24>(A.g), A, J, W, El, tosl, thrl, slot0, nres,
                                  s, t);
      return;
    }
  }
  sweep_resident_shape<D, 0>(A.g, A, J, W, El, tosl, thrl, slot0, nres, s, t);
}

// ---------------------------------------------------------------------------
// nmcs Monte Carlo steps of sample s with replica sets [c_lo, c_lo + nsets)
// resident in LDS.  With one set only the sweep and the exchange run (the
// Houdayer move and the overlap need both sets).  Only the resident sets'
// state is written back, so the two sets of a sample may run in different
// workgroups at the same time.
// ---------------------------------------------------------------------------
// Adds the round trips a workgroup summed in LDS during the launch to the
// sample's totals (atomically: the sample's two replica sets may have run in
// two workgroups).
__device__ __forceinline__ void flush_trips(const FusedArgs& A, const uint32_t* lds, int s) {
  const uint64_t* bl = reinterpret_cast<const uint64_t*>(lds + A.lay.trip);
  unsigned long long* dst = reinterpret_cast<unsigned long long*>(A.trips) + (size_t)s * 32 * 3;
  for (int i = threadIdx.x; i < 32 * 3; i += blockDim.x)
    if (bl[i]) atomicAdd(dst + i, (unsigned long long)bl[i]);
}

template <int D, bool HOU, bool MEAS, bool WALK, bool MODES>
__device__ __forceinline__ void run_sample(const FusedArgs& A, uint32_t* lds, int s, int c_lo, int nsets) {
  const Geo& g = A.g;
  const int T = blockDim.x, tid = threadIdx.x;
  const int NW = g.NW, NT = g.NT, nslot = g.nslot, W2 = 2 * NW;
  const int slot0 = c_lo * NT, nres = nsets * NT;  // resident slots [slot0, slot0 + nres)
  uint32_t* W = lds + A.lay.W;                     // W[(slot - slot0) * W2 + ...]
  uint32_t* Jl = lds + A.lay.J;
  int32_t* El = reinterpret_cast<int32_t*>(lds + A.lay.E);
  int32_t* sotl = reinterpret_cast<int32_t*>(lds + A.lay.sot);
  int32_t* tosl = reinterpret_cast<int32_t*>(lds + A.lay.tos);
  uint32_t* thrl = lds + A.lay.thr;
  int64_t* mom = reinterpret_cast<int64_t*>(lds + A.lay.mom);
  const size_t lat0 = (size_t)s * nslot + slot0;
  const bool hou = HOU && A.hou && nsets == 2, meas = MEAS && A.meas && nsets == 2;

  // ---- load
  const int items = nres * NW;
  if (g.layout == kLayoutPacked) {
    const uint32_t* src = static_cast<const uint32_t*>(A.spins) + lat0 * W2;
    for (int i = tid; i < nres * W2; i += T) W[i] = src[i];
  } else {
    const int8_t* src = static_cast<const int8_t*>(A.spins) + lat0 * g.N;
#pragma unroll 2
    for (int it = tid; it < items; it += T) {
      const int ls = (int)__umulhi((uint32_t)it, A.magicNW), w = it - ls * NW;
      word_from_int8(g, src + (size_t)ls * g.N, w, W[ls * W2 + w], W[ls * W2 + NW + w]);
    }
  }
  const uint32_t* jws = A.jw + (size_t)s * 2 * 2 * D * NW;
  for (int i = tid; i < 2 * 2 * D * NW; i += T) Jl[i] = jws[i];
  for (int i = tid; i < nslot; i += T) El[i] = A.E[(size_t)s * nslot + i];
  for (int i = tid; i < 2 * NT; i += T) {
    sotl[i] = A.sot[(size_t)s * 2 * NT + i];
    tosl[i] = A.tos[(size_t)s * 2 * NT + i];
  }
  for (int i = tid; i < 4 * NT; i += T) thrl[i] = A.thr[i];
  if (meas)
    for (int i = tid; i < 8 * NT; i += T) mom[i] = A.mom[(size_t)s * NT * 8 + i];
  const bool modes = MODES && meas && A.modes != nullptr;
  const int MH = g.L / 2 + 1;
  int64_t* modl = reinterpret_cast<int64_t*>(lds + A.lay.modes);
  if (modes)
    for (int i = tid; i < NT * MH; i += T) modl[i] = A.modes[(size_t)s * NT * MH + i];
  const bool walk = WALK && A.walk != nullptr;
  int32_t* wkl = reinterpret_cast<int32_t*>(lds + A.lay.walk);
  if (walk) {
    for (int i = tid; i < 2 * nres; i += T) wkl[2 * slot0 + i] = A.walk[2 * lat0 + i];
    for (int i = tid; i < 2 * 32 * 3; i += T) lds[A.lay.trip + i] = 0u;
  }
  if (hou && tid == 0) lds[A.lay.hq] = 0u;
  const uint32_t t0 = A.ctr->t, u0 = A.ctr->u, v0 = A.ctr->v;
  __syncthreads();

  for (int step = 0; step < A.nmcs; ++step) {
    const uint32_t t = t0 + (uint32_t)step, u = u0 + (uint32_t)step;
    exchange_prepare(A, lds, s, u, c_lo, nsets);
    sweep_resident<D>(A, Jl, W, El, tosl, thrl, slot0, nres, s, t);
    if (hou) {
      if (A.hou == 2)
        houdayer_multi_resident<D>(A, lds, s, v0 + (uint32_t)step);
      else
        houdayer_resident<D>(A, lds, s, v0 + (uint32_t)step);
    }
    exchange_resident<WALK>(A, lds, c_lo, nsets, u + 1u, walk);
    if (meas && measures_at(t + 1u, (uint32_t)A.every)) measure_resident<MODES>(A, lds);
  }

  // ---- store the resident sets
  if (g.layout == kLayoutPacked) {
    uint32_t* dst = static_cast<uint32_t*>(A.spins) + lat0 * W2;
    for (int i = tid; i < nres * W2; i += T) dst[i] = W[i];
  } else {
    int8_t* dst = static_cast<int8_t*>(A.spins) + lat0 * g.N;
#pragma unroll 2
    for (int it = tid; it < items; it += T) {
      const int ls = (int)__umulhi((uint32_t)it, A.magicNW), w = it - ls * NW;
      word_to_int8(g, dst + (size_t)ls * g.N, w, W[ls * W2 + w], W[ls * W2 + NW + w]);
    }
  }
  for (int i = tid; i < nres; i += T) A.E[lat0 + i] = El[slot0 + i];
  for (int i = tid; i < nres; i += T) {
    A.sot[(size_t)s * 2 * NT + slot0 + i] = sotl[slot0 + i];
    A.tos[(size_t)s * 2 * NT + slot0 + i] = tosl[slot0 + i];
  }
  if (walk) {
    for (int i = tid; i < 2 * nres; i += T) A.walk[2 * lat0 + i] = wkl[2 * slot0 + i];
    flush_trips(A, lds, s);
  }
  if (modes)
    for (int i = tid; i < NT * MH; i += T) A.modes[(size_t)s * NT * MH + i] = modl[i];
  if (meas)
    for (int i = tid; i < 8 * NT; i += T) A.mom[(size_t)s * NT * 8 + i] = mom[i];
}

// ---------------------------------------------------------------------------
// Samples too large for one workgroup.  The 2 N_T configurations of a sample
// are split into `parts` groups of R slots, one workgroup each, for all steps
// of the launch: a replica exchange only relabels temperatures, so a
// configuration never changes workgroup.  Each step every part publishes the
// energies of its slots (and, when measuring, their configurations) to
// parity-double-buffered global scratch and meets the other parts at a
// per-sample counter barrier; then every part takes the same exchange
// decisions from the same energies and Philox words, so the maps agree
// without further communication, and temperature k is measured by the part
// holding its replica-set-0 configuration, which reads the set-1 partner from
// LDS or from the published configurations (only set-1 slots are published).
// A part overwrites a parity buffer two steps later, after a barrier that
// every reader of it has passed.
// ---------------------------------------------------------------------------

// About 60 s of the 100 MHz constant clock: far beyond any legitimate wait
// (all parts of a sample are taken from the queue together), so reaching it
// means the job's state can no longer be trusted.
constexpr uint64_t kBarrierTicks = 6000000000ull;

// What the parts publish every step (energies and configurations) is written
// and read with agent-scope relaxed accesses, which go past the XCDs' separate
// L2 caches to memory: once a wavefront's stores have completed (vmcnt), an
// agent-scope load on any XCD issued later sees them.  The parts can then meet
// without the release and acquire of ordinary stores, which write back and
// invalidate whole L2 caches at every step, also the coupling words that the
// sweep reads: 3D L = 16, 16 x 2 x 32 over 256 parts, 19.4 -> 15.2 us per measured
// step; with every sample's counter in a cache line of its own 10.3 us.
__device__ __forceinline__ void publish(uint64_t* p, uint64_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish(int32_t* p, int32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T published(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Arrives at a sample's barrier and waits for `target` arrivals in all.
// Returns false if the wait gave up; the job's fault word is then set, and
// every later wait of the job gives up at once.  Every wavefront first waits
// until its own stores have completed, then only thread 0 synchronises with
// the other parts, and the workgroup barrier orders every later load after it.
// FENCED: ordinary stores before it are visible to ordinary loads after it
// (thread 0's release writes back this XCD's L2, its acquire invalidates the
// caches); otherwise only published values are, unless `acquire` lets ordinary
// loads after it see them too.
template <bool FENCED>
__device__ __forceinline__ bool part_barrier(uint32_t* bar, uint32_t target, uint32_t* fault,
                                             int* flag, bool acquire = FENCED) {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0) {
    __hip_atomic_fetch_add(bar, 1u, FENCED ? __ATOMIC_RELEASE : __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    int good = 1;
    const uint64_t t0 = wall_clock64();
    // poll with relaxed loads and acquire once, after the count is reached:
    // an acquire load invalidates caches on every poll, which would also
    // evict the data other workgroups on the same L2 are computing with
    for (uint32_t n = 1;
         __hip_atomic_load(bar, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < target; ++n) {
      if (n % 64u == 0u &&
          (__hip_atomic_load(fault, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u ||
           wall_clock64() - t0 > kBarrierTicks)) {
        __hip_atomic_store(fault, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const uint64_t host = (uint64_t)fault[1] | ((uint64_t)fault[2] << 32);
        if (host)
          __hip_atomic_store(reinterpret_cast<uint32_t*>(host), 1u, __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_SYSTEM);
        good = 0;
        break;
      }
      __builtin_amdgcn_s_sleep(1);
    }
    // the relaxed load read the value of the other parts' increments: this
    // fence makes what they wrote before visible to ordinary loads
    if (acquire) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    *flag = good;
  }
  __syncthreads();
  return *flag != 0;
}

// Overlaps and moment increments of the temperatures whose replica-set-0
// configuration this part holds (its slots below N_T, at temperature tos[r]),
// each against its set-1 partner: from LDS when this part holds the partner
// too, else from the words published this step (`pub`: [nslot][2NW], set-1
// slots).  The increments go to this part's LDS sums, which start each launch
// at zero and are combined across parts at its end (combine_split_moments).
// With the modes kept, the parts publish every slot and temperature k's modes
// are taken by part k mod parts from the published words.
template <bool MODES>
__device__ __forceinline__ void measure_split(const FusedArgs& A, uint32_t* lds, int part, int slot0,
                                              int nres, const uint32_t* W, const uint32_t* pub) {
  const Geo& g = A.g;
  const int NT = g.NT, W2 = 2 * g.NW, tid = threadIdx.x, T = blockDim.x;
  const int32_t* El = reinterpret_cast<const int32_t*>(lds + A.lay.E);
  const int32_t* sotl = reinterpret_cast<const int32_t*>(lds + A.lay.sot);
  const int32_t* tosl = reinterpret_cast<const int32_t*>(lds + A.lay.tos);
  int32_t* qneg = reinterpret_cast<int32_t*>(lds + A.lay.qneg);
  int64_t* mom = reinterpret_cast<int64_t*>(lds + A.lay.mom);
  const int n0 = max(0, min(slot0 + nres, NT) - slot0);  // this part's set-0 slots
  const int wave = tid >> 6, lane = tid & 63, nwave = T >> 6;
  for (int i = tid; i < n0; i += T) qneg[i] = 0;
  __syncthreads();
  // the (pair, chunk of 64 word pairs) space is cut into one contiguous range
  // per wavefront, so that every wavefront has many independent loads in flight
  // whatever the number of pairs; a wavefront adds its lanes' counts of the
  // differing sites once per pair in its range
  const int NW = g.NW, C64 = (NW + 63) >> 6, items = n0 * C64, per = (items + nwave - 1) / nwave;
  const int hi = min(items, (wave + 1) * per);
  for (int it = wave * per; it < hi;) {
    const int i = it / C64, c1 = min(hi - i * C64, C64);
    const int r = slot0 + i, b = NT + sotl[NT + tosl[r]];
    const uint32_t* pa = W + (size_t)i * W2;
    int neg = 0;
    if (b < slot0 + nres) {
      const uint32_t* pb = W + (size_t)(b - slot0) * W2;
      for (int c = it - i * C64; c < c1; ++c) {
        const int w = 2 * (c * 64 + lane);
        if (w < W2) neg += __popc(pa[w] ^ pb[w]) + __popc(pa[w + 1] ^ pb[w + 1]);
      }
    } else {
      const uint64_t* pb = reinterpret_cast<const uint64_t*>(pub + (size_t)b * W2);
#pragma unroll 8
      for (int c = it - i * C64; c < c1; ++c) {
        const int w = c * 64 + lane;
        if (w < NW) {
          const uint64_t x = published(&pb[w]);
          neg += __popc(pa[2 * w] ^ (uint32_t)x) + __popc(pa[2 * w + 1] ^ (uint32_t)(x >> 32));
        }
      }
    }
    neg = wave_total(neg);
    if (lane == 0 && neg) atomicAdd(&qneg[i], neg);
    it = i * C64 + c1;
  }
  __syncthreads();
  for (int i = tid; i < n0; i += T) {
    const int r = slot0 + i, k = tosl[r];
    add_moments(g, mom + (size_t)k * 8, El[r], El[NT + sotl[NT + k]], qneg[i]);
  }
  if (MODES && A.modes) {
    // the owned temperatures' modes, one wavefront each, from the published words
    const int nk = (NT - part + A.parts - 1) / A.parts;
    for (int kl = wave; kl < nk; kl += nwave) {
      const int k = part + kl * A.parts;
      modes_resident(g, A.lay, lds, pub + (size_t)sotl[k] * W2, pub + (size_t)(NT + sotl[NT + k]) * W2,
                     k, wave, lane);
    }
  }
  __syncthreads();
}

// The end of a measuring launch of a split sample: every part writes its
// moment increments to `scr` ([parts][N_T][8] 64-bit words; free once every
// part has passed the last step's barrier), meets the other parts once more,
// and part k mod parts adds the increments of temperature k (the Q^4 sum as a
// 128-bit pair) to the sums in global memory.  False if the wait gave up.
__device__ __forceinline__ bool combine_split_moments(const FusedArgs& A, const int64_t* mom, int s,
                                                      int part, uint64_t* scr, uint32_t* bar,
                                                      uint32_t target, uint32_t* fault, int* flag) {
  const int NT = A.g.NT, tid = threadIdx.x, T = blockDim.x;
  for (int i = tid; i < 8 * NT; i += T) scr[(size_t)part * 8 * NT + i] = (uint64_t)mom[i];
  if (!part_barrier<true>(bar, target, fault, flag)) return false;
  for (int k = part + tid * A.parts; k < NT; k += T * A.parts) {
    uint64_t* dst = reinterpret_cast<uint64_t*>(A.mom) + ((size_t)s * NT + k) * 8;
    uint64_t m[8];
    for (int j = 0; j < 8; ++j) m[j] = dst[j];
    for (int p = 0; p < A.parts; ++p) {
      const uint64_t* q = scr + ((size_t)p * NT + k) * 8;
      for (int j = 0; j < 5; ++j) m[j] += q[j];
      const uint64_t lo = m[5] + q[5];
      m[6] += q[6] + (lo < m[5] ? 1u : 0u);
      m[5] = lo;
      m[7] += q[7];
    }
    for (int j = 0; j < 8; ++j) dst[j] = m[j];
  }
  return true;
}

// nmcs Monte Carlo steps (sweep, exchange, measurement) of part `part` of
// split sample s.
template <int D, bool MEAS, bool WALK, bool MODES>
__device__ __forceinline__ void run_split(const FusedArgs& A, uint32_t* lds, int s, int part,
                                          int* flag) {
  const Geo& g = A.g;
  const int T = blockDim.x, tid = threadIdx.x;
  const int NW = g.NW, NT = g.NT, nslot = g.nslot, W2 = 2 * NW;
  const int slot0 = part * A.R, nres = min(A.R, nslot - slot0);
  uint32_t* W = lds + A.lay.W;
  int32_t* El = reinterpret_cast<int32_t*>(lds + A.lay.E);
  int32_t* sotl = reinterpret_cast<int32_t*>(lds + A.lay.sot);
  int32_t* tosl = reinterpret_cast<int32_t*>(lds + A.lay.tos);
  uint32_t* thrl = lds + A.lay.thr;
  int64_t* mom = reinterpret_cast<int64_t*>(lds + A.lay.mom);
  const size_t lat0 = (size_t)s * nslot + slot0;
  const bool meas = MEAS && A.meas != 0;

  // ---- load this part's slots and the sample's shared state
  const int items = nres * NW;
  if (g.layout == kLayoutPacked) {
    const uint32_t* src = static_cast<const uint32_t*>(A.spins) + lat0 * W2;
    for (int i = tid; i < nres * W2; i += T) W[i] = src[i];
  } else {
    const int8_t* src = static_cast<const int8_t*>(A.spins) + lat0 * g.N;
#pragma unroll 2
    for (int it = tid; it < items; it += T) {
      const int ls = (int)__umulhi((uint32_t)it, A.magicNW), w = it - ls * NW;
      word_from_int8(g, src + (size_t)ls * g.N, w, W[ls * W2 + w], W[ls * W2 + NW + w]);
    }
  }
  const uint32_t* Jsrc = A.jw + (size_t)s * 2 * 2 * D * NW;
  if (A.jlds) {
    uint32_t* Jl = lds + A.lay.J;
    for (int i = tid; i < 2 * 2 * D * NW; i += T) Jl[i] = Jsrc[i];
    Jsrc = Jl;
  }
  for (int i = tid; i < nslot; i += T) El[i] = A.E[(size_t)s * nslot + i];
  for (int i = tid; i < 2 * NT; i += T) {
    sotl[i] = A.sot[(size_t)s * 2 * NT + i];
    tosl[i] = A.tos[(size_t)s * 2 * NT + i];
  }
  for (int i = tid; i < 4 * NT; i += T) thrl[i] = A.thr[i];
  // this launch's moment increments (combined across parts at its end)
  if (meas)
    for (int i = tid; i < 8 * NT; i += T) mom[i] = 0;
  // mode sums of the temperatures this part measures (k = part mod parts)
  const bool modes = MODES && meas && A.modes != nullptr;
  const int MH = g.L / 2 + 1;
  int64_t* modl = reinterpret_cast<int64_t*>(lds + A.lay.modes);
  if (modes)
    for (int k = part; k < NT; k += A.parts)
      for (int i = tid; i < MH; i += T) modl[k * MH + i] = A.modes[((size_t)s * NT + k) * MH + i];
  // part 0 keeps the sample's replica walk
  const bool walk = WALK && A.walk != nullptr && part == 0;
  int32_t* wkl = reinterpret_cast<int32_t*>(lds + A.lay.walk);
  if (walk) {
    for (int i = tid; i < 2 * nslot; i += T) wkl[i] = A.walk[(size_t)s * 2 * nslot + i];
    for (int i = tid; i < 2 * 32 * 3; i += T) lds[A.lay.trip + i] = 0u;
  }
  const uint32_t t0 = A.ctr->t, u0 = A.ctr->u;
  uint32_t* bar = A.bar + (size_t)s * kBarStride;
  uint32_t* fault = A.bar + (size_t)g.S * kBarStride;
  int32_t* Ex = A.Ex + (size_t)s * 2 * nslot;
  uint32_t* snap = A.snap + (size_t)s * 2 * nslot * W2;
  bool good = true;
  __syncthreads();

  for (int step = 0; step < A.nmcs; ++step) {
    const uint32_t t = t0 + (uint32_t)step, u = u0 + (uint32_t)step;
    exchange_prepare(A, lds, s, u, 0, 2);
    sweep_resident<D, true>(A, Jsrc, W, El, tosl, thrl, slot0, nres, s, t);
    // publish, meet, and take the sample-wide steps
    const int par = step & 1;
    const bool mstep = meas && measures_at(t + 1u, (uint32_t)A.every);
    for (int i = tid; i < nres; i += T) publish(&Ex[par * nslot + slot0 + i], El[slot0 + i]);
    if (mstep) {
      // the set-1 slots (every slot when the modes are kept)
      const int first = modes ? 0 : min(nres, max(0, NT - slot0));
      uint64_t* dst = reinterpret_cast<uint64_t*>(snap + ((size_t)par * nslot + slot0) * W2);
      for (int i = first * NW + tid; i < nres * NW; i += T)
        publish(&dst[i], (uint64_t)W[2 * i] | ((uint64_t)W[2 * i + 1] << 32));
    }
    if (!part_barrier<false>(bar, (uint32_t)(A.parts * (step + 1)), fault, flag, mstep && modes)) {
      good = false;
      break;
    }
    for (int i = tid; i < nslot; i += T) El[i] = published(&Ex[par * nslot + i]);
    __syncthreads();
    exchange_resident<WALK>(A, lds, 0, 2, u + 1u, walk);
    if (mstep) measure_split<MODES>(A, lds, part, slot0, nres, W, snap + (size_t)par * nslot * W2);
  }
  if (meas && good)
    combine_split_moments(A, mom, s, part,
                          reinterpret_cast<uint64_t*>(snap + (size_t)(A.nmcs & 1) * nslot * W2), bar,
                          (uint32_t)(A.parts * (A.nmcs + 1)), fault, flag);

  // ---- store this part's slots; part 0 stores the maps, owners the modes
  if (g.layout == kLayoutPacked) {
    uint32_t* dst = static_cast<uint32_t*>(A.spins) + lat0 * W2;
    for (int i = tid; i < nres * W2; i += T) dst[i] = W[i];
  } else {
    int8_t* dst = static_cast<int8_t*>(A.spins) + lat0 * g.N;
#pragma unroll 2
    for (int it = tid; it < items; it += T) {
      const int ls = (int)__umulhi((uint32_t)it, A.magicNW), w = it - ls * NW;
      word_to_int8(g, dst + (size_t)ls * g.N, w, W[ls * W2 + w], W[ls * W2 + NW + w]);
    }
  }
  for (int i = tid; i < nres; i += T) A.E[lat0 + i] = El[slot0 + i];
  if (part == 0)
    for (int i = tid; i < 2 * NT; i += T) {
      A.sot[(size_t)s * 2 * NT + i] = sotl[i];
      A.tos[(size_t)s * 2 * NT + i] = tosl[i];
    }
  if (walk) {
    for (int i = tid; i < 2 * nslot; i += T) A.walk[(size_t)s * 2 * nslot + i] = wkl[i];
    flush_trips(A, lds, s);
  }
  if (modes)
    for (int k = part; k < NT; k += A.parts)
      for (int i = tid; i < MH; i += T) A.modes[((size_t)s * NT + k) * MH + i] = modl[k * MH + i];
}

// ---------------------------------------------------------------------------
// What the last workgroup of a launch leaves behind it: every job's counters
// advanced by its own number of steps, and the queue and the meeting counters
// of split samples at zero for the next launch.  No count of another workgroup
// can arrive after that: each has seen its last queue count returned (it ended
// its loop) and has left every meeting by reading the counter that its own
// arrival is in, before it counts itself done; and it has used the counters that
// it read.  Two kernels around this one, which did the same, cost a call of one
// step (3D L = 8, 8 samples x 16 temperatures, with the read-out of the energies)
// 37.0 us instead of 34.8.
template <bool SPLIT>
__device__ __forceinline__ void batch_finish(const FusedArgs* __restrict__ jobs, int njobs, uint32_t* queue) {
  for (int j = threadIdx.x; j < njobs; j += blockDim.x) {
    const FusedArgs& A = jobs[j];
    DevCounters* c = const_cast<DevCounters*>(A.ctr);
    const uint32_t n = (uint32_t)A.nmcs, t0 = c->t, e = (uint32_t)A.every;
    c->t = t0 + n;
    c->u += n;
    if (A.hou) c->v += n;
    if (A.meas) c->n_meas += e > 1u ? (t0 + n) / e - t0 / e : n;
  }
  if (SPLIT)
    for (int j = 0; j < njobs; ++j) {
      const FusedArgs& A = jobs[j];
      if (A.parts)
        for (int i = threadIdx.x; i < A.g.S; i += blockDim.x) A.bar[(size_t)i * kBarStride] = 0u;
    }
  if (threadIdx.x == 0) queue[0] = queue[kQueueDone] = 0u;
}

// Persistent batch kernel: workgroups take (job, sample, sets) items from a
// shared queue until it is empty.  Each job brings its own geometry,
// tables, state and LDS plan.  F says which kinds of work the launch holds
// (kFeatHou, kFeatMeas, kFeatSplit): code for the others is left out, which
// keeps the register count, and so the number of resident wavefronts, of a
// launch as low as its work allows.
// ---------------------------------------------------------------------------
// Wavefronts per SIMD the register allocation must allow.  The sweep +
// exchange (+ measurement, + replica walk) kernels are held to the 80 VGPRs
// that two 768-thread workgroups per CU need: left alone the scheduler takes
// a few more (for values used once per item, which then go to scratch
// instead, outside the step loop).  Every other variant gets what a
// 1024-thread workgroup needs.
template <int F>
constexpr int kWavesPerSimd = !(F & (kFeatHou | kFeatSplit)) ? 6 : 4;

template <int D, int F>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(kWavesPerSimd<F>)))
k_batch(const FusedArgs* __restrict__ jobs, const BatchItem* __restrict__ items, int nitems,
        uint32_t* queue, int njobs) {
  constexpr bool kHou = (F & kFeatHou) != 0, kMeas = (F & kFeatMeas) != 0;
  constexpr bool kSplit = (F & kFeatSplit) != 0, kWalk = (F & kFeatWalk) != 0;
  constexpr bool kModes = (F & kFeatModes) != 0;
  // 16-byte aligned: the moment words are updated with 64-bit LDS atomics,
  // which need naturally aligned addresses (the plan offsets are 8-byte
  // aligned relative to this base)
  extern __shared__ __align__(16) uint32_t lds[];
  __shared__ int cur, flag;
  for (;;) {
    if (threadIdx.x == 0) cur = (int)atomicAdd(queue, 1u);
    __syncthreads();
    const int i = __builtin_amdgcn_readfirstlane(cur);
    __syncthreads();
    if (i >= nitems) break;
    const BatchItem it = items[i];
    const FusedArgs A = jobs[it.job];
    if (A.nmcs > 0) {
      if (kSplit && it.nsets == 0)
        run_split<D, kMeas, kWalk, kModes>(A, lds, it.sample, it.c_lo, &flag);
      else
        run_sample<D, kHou, kMeas, kWalk, kModes>(A, lds, it.sample, it.c_lo, it.nsets);
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) cur = atomicAdd(queue + kQueueDone, 1u) == gridDim.x - 1u;
  __syncthreads();
  if (__builtin_amdgcn_readfirstlane(cur)) batch_finish<kSplit>(jobs, njobs, queue);
}

// Pointer to one variant of the batch kernel.
using BatchKernel = void (*)(const FusedArgs*, const BatchItem*, int, uint32_t*, int);

// The variant k_batch<D, BASE + feat> for feat in [0, sizeof...(F)).
template <int D, int BASE, int... F>
BatchKernel pick_kernel(int feat, std::integer_sequence<int, F...>, std::integral_constant<int, BASE>) {
  BatchKernel k = nullptr;
  ((k = (feat == F ? &k_batch<D, BASE + F> : k)), ...);
  return k;
}

// Defined in fused_k2a/k2b/k3a/k3b.hip: dimension 2 or 3, feature sets in
// [0, 16) (a) or [16, 32) (b).
BatchKernel batch_kernel_2a(int feat);
BatchKernel batch_kernel_2b(int feat);
BatchKernel batch_kernel_3a(int feat);
BatchKernel batch_kernel_3b(int feat);

}  // namespace ptsg
