// gauss_fused.hip -- whole Monte Carlo steps of Gaussian-coupling jobs in one
// launch (Sec. 2.4 with the Gaussian couplings of Sec. 2.1): Metropolis
// sweep, single-cluster Houdayer move per same-temperature pair, replica
// exchange pass and measurement, n steps per launch.  One workgroup holds
// one disorder sample, all 2 N_T configurations resident in LDS as
// colour-split row words, their 64-bit energies, the maps, the inverse
// temperatures and the moment sums; the coupling groups are read from global
// memory (each workgroup's sample stays in its XCD's L2).  HBM is touched to
// load the state at the start and store it at the end.
//
// Results are bit-identical to the per-step Gaussian kernels (gauss.hip):
// the same site groups and Philox counters, the same acceptance tiers, the
// exchange pass in ascending k with the updated map, the Houdayer seed as the
// m-th q = -1 site in increasing site order and the cluster as its connected
// component (found here by one wavefront per pair).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fused_device.h"
#include "gauss.h"
#include "gauss_kernels.h"

namespace ptsg {

namespace {

// LDS word offsets (64-bit arrays first, so that they stay 8-byte aligned);
// acc < 0: the exchange pass walks serially (ladders above 64 temperatures).
struct GaussLayout {
  int E, beta, mom, cz, sot, tos, hq, W, Qs, sot0, rpt, acc, words;
  int team;  // threads of a team
  int PC;    // wavefronts with a Houdayer scratch area (3D)
};

// Threads of the fused Gaussian workgroup and its LDS plan.  A team of
// threads, one per site group of a colour, sweeps one configuration (in 2D two)
// at a time; a workgroup holds as many teams as its threads allow.  The kernel
// takes four wavefronts per SIMD (its registers), so a CU runs 1024 of its
// threads: one workgroup of 1024 where there are no more samples than CUs or
// two would not fit the LDS, else two of 512.  (One team of 256 to 512 threads
// whatever the sample count, as before: 3D L = 10, 150 samples x 2 x 15, 55 us
// per step against 25 us, the chip holding one wavefront per SIMD.)
int gauss_fused_threads(const Geo& g, int cus, GaussLayout& l);

GaussLayout gauss_layout(const Geo& g, int nwave) {
  GaussLayout l{};
  int o = 0;
  l.E = o;     o += 2 * 2 * g.NT;           // int64 [2 N_T] energies (2^-16 units)
  l.beta = o;  o += 2 * g.NT;               // double [N_T]
  l.mom = o;   o += 2 * 8 * g.NT;           // int64 [N_T][8] moment sums
  l.cz = o;    o += g.NT;                   // float [N_T] the float32 tier's constants
  l.sot = o;   o += 2 * g.NT;               // int32 [2][N_T]
  l.tos = o;   o += 2 * g.NT;               // int32 [2][N_T]
  l.hq = o;    o += 1;                      // the in-register Houdayer move's pair counter
  l.W = o;     o += 2 * g.NT * 2 * g.NW;    // [2 N_T][2 NW] configuration words
  // per wavefront: overlap and cluster words of the word-hop flood fill
  l.PC = rows_houdayer(g) ? 0 : nwave;
  l.Qs = o;    o += l.PC * 4 * g.NW;
  l.words = o;
  // the exchange pass's maps before the pass, Philox words and decisions
  l.acc = -1;
  if (g.NT <= 64) {
    l.sot0 = o;  o += 2 * g.NT;
    l.rpt = o;   o += 2 * g.NT;
    l.acc = o;   o += 2 * (g.NT - 1) * ((g.NT + 31) / 32);
    l.words = o;
  }
  return l;
}

// The LDS of the smallest workgroup (four to eight wavefronts, serial
// exchange): what decides whether a sample's steps run fused.
size_t gauss_least_lds(const Geo& g) {
  const int threads = std::min(512, std::max(256, (gauss_groups(g) + 63) / 64 * 64));
  GaussLayout l = gauss_layout(g, threads / 64);
  return sizeof(uint32_t) * (size_t)(l.acc >= 0 ? l.sot0 : l.words);
}

int gauss_fused_threads(const Geo& g, int cus, GaussLayout& l) {
  const int groups = (gauss_groups(g) + 63) / 64 * 64, configs = g.d == 2 ? g.NT : 2 * g.NT;
  for (int most : {512, 1024}) {
    if (most == 512 && g.S <= cus) continue;
    const int team = std::min(most, groups);
    const int threads = std::max(256, team * std::min(most / team, configs));
    l = gauss_layout(g, threads / 64);
    // fewer scratch areas, then the serial exchange, where the LDS is short
    const size_t limit = kGaussFusedMaxLds / (most == 512 ? 2 : 1);
    while (l.PC > 4 && sizeof(uint32_t) * (size_t)l.words > limit) {
      const int pc = l.PC - 1;
      l = gauss_layout(g, pc);
    }
    if (sizeof(uint32_t) * (size_t)l.words > limit && l.acc >= 0) {
      l.words = l.sot0;
      l.acc = -1;
    }
    l.team = team;
    if (most == 512 && sizeof(uint32_t) * (size_t)l.words > limit) continue;
    return threads;
  }
  return 0;
}

// Wavefront sum of a 64-bit value.
__device__ __forceinline__ int64_t wave_sum64(int64_t v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// Single-cluster Houdayer moves of all N_T pairs, one wavefront per pair at a
// time: overlap words, the seed (the m-th q = -1 site), the flood fill to the
// seed's connected q = -1 component, the energy change of replica a from the
// Gaussian couplings, then the exchange of the two configurations on the
// cluster.  Ends with a workgroup barrier.
template <int D>
__device__ void gauss_houdayer_resident(const Geo& g, uint32_t* W, int64_t* El, const int32_t* sotl,
                                        uint32_t* Qs, int PC, const int4* __restrict__ J0, int s,
                                        uint32_t v) {
  const int NT = g.NT, NW = g.NW, W2 = 2 * NW;
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));  // as in gauss_houdayer_rows
  const int wave = tid >> 6, lane = tid & 63;
  uint32_t* Qw = Qs + (size_t)wave * 2 * W2;
  uint32_t* Cw = Qw + W2;
  const bool in_regs = words_houdayer(g);
  const LaneWord lw = in_regs ? lane_word(g, lane) : LaneWord{};
  for (int k = wave < PC ? wave : NT; k < NT; k += PC) {
    const int a = sotl[k], b = NT + sotl[NT + k];
    uint32_t* Wa = W + (size_t)a * W2;
    uint32_t* Wb = W + (size_t)b * W2;
    if (in_regs) {
      uint32_t c0, c1;
      if (!words_cluster<0>(g, lw, Wa, Wb, s, k, v, c0, c1)) continue;
      if (lw.valid) {
        Cw[lw.w] = c0;
        Cw[NW + lw.w] = c1;
      }
      wave_lds_sync();
    } else if (!lds_cluster<D>(g, Wa, Wb, Qw, Cw, s, k, v, lane)) {
      continue;
    }
    const int64_t delta = wave_sum64(gauss_cluster_delta<D>(g, Cw, Wa, J0, lane, 64));
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
  __syncthreads();
}

// The same for a 2D sample: the cluster is found in registers, one row per
// lane (rows_cluster), pairs from the hottest down; the energy change sums,
// over the cluster's boundary bonds from this row's colour-0 sites, the bond's
// -2n from its coupling group with the sign of replica a across it.  Four
// groups a lane are loaded at once (one at a time waited for the L2 at each;
// eight spill) and added without branches: 2D L = 64, 500 samples x 2 x 24, the
// moves of a step 55 -> 45 us.  Ends with a workgroup barrier, after which the
// pair counter is cleared.
template <int LS>
__device__ void gauss_houdayer_rows(const Geo& gw, uint32_t* W, int64_t* El, const int32_t* sotl,
                                    const int4* __restrict__ J0, int s, uint32_t v, uint32_t* hctr) {
  const Geo g = LS == 64 ? gw : row_geo(gw);
  const int NT = g.NT, NW = gw.NW, NGc = gauss_groups(gw);
  // recomputed at every call: what derives from the lane index (masks,
  // addresses) would otherwise be hoisted out of the step loop and stay live
  // through the sweep
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const bool odd = lane & 1;
  const LaneRow lr = lane_row<LS>(gw, lane);
  // first coupling group of the row (groups of a word: field-major, then q)
  const int g0 = LS == 64 ? lane : lr.w + (lr.sh / g.H) * ((g.H + 3) / 4) * NW;
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
    // the colour-0 sites' bonds: +x0, -x0 in the row, +x1, -x1 to the
    // next/previous row, the order of the coupling groups' directions
    uint32_t nc[4], na[4];
    x0_neighbours(g, c1, odd, nc[0], nc[1]);
    x0_neighbours(g, a1, odd, na[0], na[1]);
    nc[2] = row_next<LS>(lr, c1);
    nc[3] = row_prev<LS>(lr, c1);
    na[2] = row_next<LS>(lr, a1);
    na[3] = row_prev<LS>(lr, a1);
    // (-2n of a bond is at most 2^20 in size, a row has 128: 32 bits hold the
    // sum; a subtracted bond adds its complement, and one from the count)
    int32_t dl = 0;
#pragma unroll
    for (int dir = 0; dir < 4; ++dir) {
      const uint32_t X = c0 ^ nc[dir];             // bonds leaving the cluster
      const uint32_t M = X & ~(a0 ^ na[dir]);      // replica a parallel across them
      dl += __popc(M);
#pragma unroll 1
      for (int q0 = 0; 4 * q0 < g.H; q0 += 4) {    // groups of four sites, four loads in flight
        int4 m[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          m[i] = int4{0, 0, 0, 0};
          if ((X >> (4 * (q0 + i))) & 0xFu) m[i] = J0[(size_t)dir * NGc + g0 + NW * (q0 + i)];
        }
        const uint32_t x4 = X >> (4 * q0), m4 = M >> (4 * q0);
#pragma unroll
        for (int j = 0; j < 16; ++j)
          dl += (lane_of(m[j >> 2], j & 3) & __builtin_amdgcn_sbfe(x4, j, 1)) ^ __builtin_amdgcn_sbfe(m4, j, 1);
      }
    }
    const int64_t delta = wave_sum64((int64_t)dl);
    rows_exchange<LS>(lr, NW, Wa, Wb, ab, c0, c1);
    if (lane == 0) {
      El[a] += delta;
      El[b] -= delta;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) *hctr = 0u;  // the next use is behind the step's barriers
}

// The Metropolis sweep of every configuration, colour 0, then colour 1.  A
// thread takes a group of four same-colour sites (one Philox call, its
// coupling data in registers) and updates it in every configuration of its
// team's share.  The energies come from the colour-1 half alone: a bond has one
// colour-1 end, so E = -(sum of x over the colour-1 sites after their
// updates); El holds zeros before.  Bound by its VALU instructions,
// half of them Philox: 2D L = 64, 500 samples x 2 x 24, sweep + exchange 150 ->
// 99 us per step from the logarithm form of the float32 tier, energies in one
// half instead of a change per flip in both, the L = 64 geometry folded and the
// exchange's decisions taken in parallel (one lane per set walked them before).
// Ends with a workgroup barrier.
template <int D, int LS>
__device__ __forceinline__ void gauss_sweep_resident(const Geo& g, int team_threads, uint32_t* W,
                                                     int64_t* El, const int32_t* tosl, const float* czl,
                                                     const double* bl, const int4* __restrict__ Js,
                                                     int s, uint32_t t) {
  constexpr int U = D == 2 ? 2 : 1;  // configurations per round (2 N_T is even)
  const int NW = g.NW, W2 = 2 * NW, NS = 2 * g.NT, NGc = gauss_groups(g);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), tw = team_threads >> 6;
  const int team = wave / tw, teams = max(1, (int)(blockDim.x >> 6) / tw);
  const int tt = tid - team * team_threads;
  const uint32_t c3 = (kTagMetro << 28) | (uint32_t)s;
  for (int c = 0; c < 2; ++c) {
    const int4* Jc = Js + (size_t)c * (2 * D + 1) * NGc;
    const uint32_t c1 = 2u * t + (uint32_t)c;
    for (int gi0 = 0; gi0 < NGc && team < teams; gi0 += team_threads) {
      // the group's position is recomputed every step: hoisted out of the
      // step loop it would stay live through the Houdayer move, whose
      // in-register cluster then no longer fits the register budget
      const int gi = recomputed(gi0 + tt);
      const bool valid = gi < NGc;
      int4 m[2 * D];
      int4 hs = make_int4(0, 0, 0, 0);
      GroupPos gp{};
      WordNb nb{};
      int p = 0;
      uint32_t c0 = 0;
      if (valid) {
#pragma unroll
        for (int k = 0; k < 2 * D; ++k) m[k] = Jc[(size_t)k * NGc + gi];
        hs = Jc[(size_t)2 * D * NGc + gi];
        gp = group_pos(g, gi);
        nb = word_nb(g, gp.w);
        p = (c + nb.par) & 1;
        c0 = (uint32_t)word_row(g, nb, gp.f) * (uint32_t)g.G + (uint32_t)gp.q;
      }
      const uint32_t vmask = (1u << gp.nv) - 1u;
      // 2D: two configurations per round, two independent chains of loads,
      // Philox rounds and decisions for the scheduler; in 3D two would not fit
      // the register budget of four wavefronts per SIMD
      for (int l = U * team; l < NS; l += U * teams) {
        int e[U];
#pragma unroll
        for (int i = 0; i < U; ++i) e[i] = 0;
        if (valid) {
          Ctr4 r[U];
          int x[U][4], k[U];
          uint32_t F[U];
          bool sure[U];
#pragma unroll
          for (int i = 0; i < U; ++i) {
            uint32_t* Wl = W + (size_t)(l + i) * W2;
            const uint32_t Wc = Wl[c * NW + gp.w];
            uint32_t a[2 * D];
            neighbour_words<D>(g, Wl + (1 - c) * NW, gp.w, nb, p, a);
#pragma unroll
            for (int dir = 0; dir < 2 * D; ++dir) a[dir] ^= Wc;
            r[i] = philox10_u(Ctr4{c0, c1, (uint32_t)(l + i), c3}, g.key0, g.key1);
            k[i] = tosl[l + i];
            gauss_group_fast<D>(a, gp.shift, m, hs, r[i], czl[k[i]], x[i], F[i], sure[i]);
          }
#pragma unroll
          for (int i = 0; i < U; ++i) {
            F[i] = gauss_group_finish(x[i], r[i], czl[k[i]], bl[k[i]], F[i], sure[i], vmask);
            if (F[i]) atomicXor(&W[(size_t)(l + i) * W2 + c * NW + gp.w], F[i] << gp.shift);
            if (c == 1) e[i] = gauss_flip_energy(x[i], F[i]) - (x[i][0] + x[i][1] + x[i][2] + x[i][3]);
          }
        }
        if (c == 1) {
          // every lane of the wavefront is here: DPP sums
          // (|sum| < 64 x 4 x 6 x 2^19 < 2^31), one LDS atomic each
#pragma unroll
          for (int i = 0; i < U; ++i) {
            e[i] = wave_total(e[i]);
            if (lane == 0)
              atomicAdd(reinterpret_cast<unsigned long long*>(&El[l + i]),
                        (unsigned long long)(int64_t)e[i]);
          }
        }
      }
    }
    __syncthreads();
  }
}

// f(l, t, threads) for every lattice l < NS: many at once, each by a group of as many
// of the workgroup's threads as a colour has words, 16 or the next power of two.  (A
// lattice at a time by all threads waits for memory NS times: 3D L = 10, 535 x 2 x
// 48, int8, one step 1553 -> 328 us.  All words flat over the threads: 298, but that
// form's scalars spill into the sweep's loops: 3D L = 8, 69 x 2 x 10, sweep + exchange
// 8.2 -> 8.7 us per step, here 8.0; for the same reason the groups are found at each use.)
template <typename F>
__device__ __forceinline__ void each_lattice(int NW, int NS, F&& f) {
  int sh = 4;
  while ((1 << sh) < NW && (2 << sh) <= (int)blockDim.x) ++sh;
  const int groups = blockDim.x >> sh, group = threadIdx.x >> sh;
  for (int l = group < groups ? group : NS; l < NS; l += groups) f(l, threadIdx.x & ((1 << sh) - 1), 1 << sh);
}

// One workgroup per sample, `n` steps of sweep (+ Houdayer) + exchange
// (+ measurement at the job's interval).  The counters are read at the start;
// the caller advances them by n steps afterwards.
template <int D, bool HOU, bool MEAS>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) k_gfused(Geo g, void* spins, const int4* __restrict__ Jg,
                                                int64_t* __restrict__ E64, int32_t* __restrict__ sot,
                                                int32_t* __restrict__ tos,
                                                const double* __restrict__ beta,
                                                const float* __restrict__ cz, int64_t* __restrict__ mom,
                                                const DevCounters* __restrict__ ctr, int n, int every,
                                                GaussLayout lay) {
  extern __shared__ __align__(16) uint32_t lds[];
  const int T = blockDim.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwave = T >> 6;
  const int NT = g.NT, NW = g.NW, W2 = 2 * NW, NS = 2 * NT, NGc = gauss_groups(g);
  const int s = blockIdx.x;
  int64_t* El = reinterpret_cast<int64_t*>(lds + lay.E);
  double* bl = reinterpret_cast<double*>(lds + lay.beta);
  int64_t* ml = reinterpret_cast<int64_t*>(lds + lay.mom);
  float* czl = reinterpret_cast<float*>(lds + lay.cz);
  int32_t* sotl = reinterpret_cast<int32_t*>(lds + lay.sot);
  int32_t* tosl = reinterpret_cast<int32_t*>(lds + lay.tos);
  uint32_t* W = lds + lay.W;
  const size_t lat0 = (size_t)s * g.nslot;

  // ---- load the sample's state
  each_lattice(NW, NS, [&](int l, int t, int threads) {
    load_lattice(g, spins, lat0 + l, W + (size_t)l * W2, t, threads);
  });
  for (int i = tid; i < NS; i += T) {
    El[i] = E64[lat0 + i];
    sotl[i] = sot[(size_t)s * NS + i];
    tosl[i] = tos[(size_t)s * NS + i];
  }
  for (int i = tid; i < NT; i += T) {
    bl[i] = beta[i];
    czl[i] = cz[i];
  }
  if (MEAS)
    for (int i = tid; i < 8 * NT; i += T) ml[i] = mom[(size_t)s * NT * 8 + i];
  if (tid == 0) lds[lay.hq] = 0u;
  const uint32_t t0 = load_counter(&ctr->t), u0 = load_counter(&ctr->u), v0 = load_counter(&ctr->v);
  __syncthreads();

  const int4* Js = Jg + (size_t)s * 2 * (2 * D + 1) * NGc;
  for (int step = 0; step < n; ++step) {
    const uint32_t t = t0 + (uint32_t)step;
    // what the exchange pass needs from before it; the energies, which the
    // sweep's colour-1 half sums anew
    if (lay.acc >= 0) {
      int32_t* sot0 = reinterpret_cast<int32_t*>(lds + lay.sot0);
      for (int i = tid; i < NS; i += T) sot0[i] = sotl[i];
      for (int i = tid; i < 2 * (NT - 1); i += T) {
        const int c = i / (NT - 1), k = i - c * (NT - 1);
        lds[lay.rpt + c * NT + k] =
            philox10(Ctr4{(uint32_t)k, u0 + (uint32_t)step, (uint32_t)c, (kTagPT << 28) | (uint32_t)s},
                     g.key0, g.key1).x;
      }
    }
    for (int i = tid; i < NS; i += T) El[i] = 0;
    // ---- Metropolis sweep
    if constexpr (D == 2) {
      if (g.L == 64)
        gauss_sweep_resident<D, 64>(fixed_shape<2, 64>(g), lay.team, W, El, tosl, czl, bl, Js, s, t);
      else
        gauss_sweep_resident<D, 0>(g, lay.team, W, El, tosl, czl, bl, Js, s, t);
    } else {
      gauss_sweep_resident<D, 0>(g, lay.team, W, El, tosl, czl, bl, Js, s, t);
    }
    // ---- Houdayer move per pair
    if (HOU) {
      if constexpr (D == 2) {
        if (g.L == 64)
          gauss_houdayer_rows<64>(fixed_shape<2, 64>(g), W, El, sotl, Js, s, v0 + (uint32_t)step,
                                  lds + lay.hq);
        else
          gauss_houdayer_rows<0>(g, W, El, sotl, Js, s, v0 + (uint32_t)step, lds + lay.hq);
      } else {
        gauss_houdayer_resident<D>(g, W, El, sotl, lds + lay.Qs, lay.PC, Js, s, v0 + (uint32_t)step);
      }
    }
    // ---- replica exchange, k ascending with the updated map
    if (lay.acc >= 0) {
      const int32_t* sot0 = reinterpret_cast<const int32_t*>(lds + lay.sot0);
      const uint32_t* rpt = lds + lay.rpt;
      exchange_decide(NT, 0, 2, lds + lay.acc, [&](int c, int k, int j) {
        const int64_t Dl = El[c * NT + sot0[c * NT + k + 1]] - El[c * NT + sot0[c * NT + j]];
        return Dl <= 0 || gauss_accept_d(rpt[c * NT + k], bl[k] - bl[k + 1], Dl);
      });
      __syncthreads();
      exchange_chain<false>(NT, 0, 2, sotl, tosl, sot0, lds + lay.acc, nullptr, nullptr, 0u);
    } else if (lane == 0 && wave < 2) {
      const int c = wave;
      const uint32_t u = u0 + (uint32_t)step;
      int32_t* so = sotl + c * NT;
      int32_t* to = tosl + c * NT;
      const int64_t* Es = El + c * NT;
      for (int k = 0; k + 1 < NT; ++k) {
        const int a = so[k], b = so[k + 1];
        const int64_t Dl = Es[b] - Es[a];
        bool acc = Dl <= 0;
        if (!acc) {
          const Ctr4 r = philox10(Ctr4{(uint32_t)k, u, (uint32_t)c, (kTagPT << 28) | (uint32_t)s},
                                  g.key0, g.key1);
          acc = gauss_accept_d(r.x, bl[k] - bl[k + 1], Dl);
        }
        if (acc) {
          so[k] = b;
          so[k + 1] = a;
          to[b] = k;
          to[a] = k + 1;
        }
      }
    }
    __syncthreads();
    // ---- measurement (Eqs. (3), (4)), one wavefront per temperature
    if (MEAS && measures_at(t + 1u, (uint32_t)every)) {
      for (int k = wave; k < NT; k += nwave) {
        const int a = sotl[k], b = NT + sotl[NT + k];
        const uint32_t* Wa = W + (size_t)a * W2;
        const uint32_t* Wb = W + (size_t)b * W2;
        int neg = 0;
        for (int i = lane; i < W2; i += 64) neg += __popc(Wa[i] ^ Wb[i]);
        neg = wave_total(neg);
        if (lane == 0) {
          const int64_t Q = (int64_t)g.N - 2 * (int64_t)neg;
          const int64_t Ea = El[a], Eb = El[b];
          int64_t* mk = ml + (size_t)k * 8;
          mk[0] += Ea + Eb;
          const uint64_t ua = (uint64_t)(Ea < 0 ? -Ea : Ea), ub = (uint64_t)(Eb < 0 ? -Eb : Eb);
          add128(&mk[1], &mk[7], ua * ua, __umul64hi(ua, ua));
          add128(&mk[1], &mk[7], ub * ub, __umul64hi(ub, ub));
          mk[2] += Q;
          mk[3] += Q < 0 ? -Q : Q;
          const uint64_t q2 = (uint64_t)(Q * Q);
          mk[4] += (int64_t)q2;
          add128(&mk[5], &mk[6], q2 * q2, __umul64hi(q2, q2));
        }
      }
      __syncthreads();
    }
  }

  // ---- store the sample's state
  each_lattice(NW, NS, [&](int l, int t, int threads) {
    store_lattice(g, spins, lat0 + l, W + (size_t)l * W2, t, threads);
  });
  for (int i = tid; i < NS; i += T) {
    E64[lat0 + i] = El[i];
    sot[(size_t)s * NS + i] = sotl[i];
    tos[(size_t)s * NS + i] = tosl[i];
  }
  if (MEAS)
    for (int i = tid; i < 8 * NT; i += T) mom[(size_t)s * NT * 8 + i] = ml[i];
}

template <int D, bool HOU, bool MEAS>
hipError_t launch_gfused(const Geo& g, void* spins, const int4* Jg, int64_t* E64, int32_t* sot,
                         int32_t* tos, const double* beta, const float* cz, int64_t* mom,
                         const DevCounters* ctr, int n, int every, int cus, hipStream_t st) {
  GaussLayout lay;
  const int threads = gauss_fused_threads(g, cus, lay);
  const size_t lds = sizeof(uint32_t) * (size_t)lay.words;
  auto k = k_gfused<D, HOU, MEAS>;
  if (lds > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(k, dim3((unsigned)g.S), dim3(threads), lds, st, g, spins, Jg, E64, sot, tos, beta, cz,
                     mom, ctr, n, every, lay);
  return hipGetLastError();
}

}  // namespace

size_t gauss_fused_lds(const Geo& g, int cus) {
  const size_t least = gauss_least_lds(g);
  if (least > kGaussFusedMaxLds) return least;
  GaussLayout lay;
  gauss_fused_threads(g, cus, lay);
  return sizeof(uint32_t) * (size_t)lay.words;
}

hipError_t launch_gauss_fused(const Geo& g, void* spins, const int4* Jg, int64_t* E64, int32_t* sot,
                              int32_t* tos, const double* beta, const float* cz, int64_t* mom,
                              const DevCounters* ctr, int n, bool hou, bool meas, int every, int cus,
                              hipStream_t st) {
  if (gauss_fused_lds(g, cus) > kGaussFusedMaxLds) return hipErrorInvalidValue;
#define PTSG_GF(DD, HH, MM) \
  return launch_gfused<DD, HH, MM>(g, spins, Jg, E64, sot, tos, beta, cz, mom, ctr, n, every, cus, st)
  if (g.d == 3) {
    if (hou) {
      if (meas) PTSG_GF(3, true, true);
      PTSG_GF(3, true, false);
    }
    if (meas) PTSG_GF(3, false, true);
    PTSG_GF(3, false, false);
  }
  if (hou) {
    if (meas) PTSG_GF(2, true, true);
    PTSG_GF(2, true, false);
  }
  if (meas) PTSG_GF(2, false, true);
  PTSG_GF(2, false, false);
#undef PTSG_GF
}

}  // namespace ptsg
