// exchange_ops.h -- the replica-exchange pass of one sample by a workgroup
// (Sec. 2.2, Eq. (5)), shared by the fused steps and the per-step kernel: all
// candidate decisions in parallel, then the chain of those that apply.
#pragma once
#include "device.h"

namespace ptsg {

// All candidate decisions of one pass for sets [c_lo, c_lo + nsets) as bits:
// decide(c, k, j), j <= k, says whether step k of set c exchanges when the
// configuration carried up from position j meets the one at k + 1.  acc: bit
// j of row (c, k), c-major, (N_T + 31) / 32 words a row.
template <typename F>
__device__ __forceinline__ void exchange_decide(int NT, int c_lo, int nsets, uint32_t* acc, F&& decide) {
  // a half-wavefront per row (ladders of up to 32) or a wavefront: the row's
  // set and step need no division
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwave = blockDim.x >> 6;
  const int rows = nsets * (NT - 1), WB = (NT + 31) >> 5;
  uint32_t* accs = acc + (size_t)c_lo * (NT - 1) * WB;
  if (WB == 1) {
    for (int r0 = 2 * wave; r0 < rows; r0 += 2 * nwave) {
      const int row = r0 + (lane >> 5), j = lane & 31;
      const int cl = row >= NT - 1 ? 1 : 0, k = row - cl * (NT - 1);
      const bool ok = row < rows && j <= k && decide(c_lo + cl, k, j);
      const uint64_t bits = __ballot(ok);
      if (j == 0 && row < rows) accs[row] = lane ? (uint32_t)(bits >> 32) : (uint32_t)bits;
    }
  } else {
    for (int row = wave; row < rows; row += nwave) {
      const int cl = row >= NT - 1 ? 1 : 0, k = row - cl * (NT - 1);
      for (int b = 0; b < WB; b += 2) {
        const int j = 32 * b + lane;
        const uint64_t bits = __ballot(j <= k && decide(c_lo + cl, k, j));
        if (lane == 0) accs[row * WB + b] = (uint32_t)bits;
        if (lane == 32 && b + 1 < WB) accs[row * WB + b + 1] = (uint32_t)(bits >> 32);
      }
    }
  }
}

// Follows the chain of those decisions from the maps before the pass (sot0)
// to the new ones; with WALK and `walk` not null, pass m of the replica walk.
// The caller synchronises before and after.
template <bool WALK>
__device__ __forceinline__ void exchange_chain(int NT, int c_lo, int nsets, int32_t* sotl, int32_t* tosl,
                                               const int32_t* sot0, const uint32_t* acc, int32_t* walk,
                                               uint64_t* trips, uint32_t m) {
  const int tid = threadIdx.x, T = blockDim.x, NB = (NT + 31) & ~31;
  const int wave = tid >> 6, lane = tid & 63, nwave = T >> 6;
  if (NT <= 64) {
    // One wavefront per set; lane k holds decision row k.  From the carried
    // position cur the next rejection is the first step k >= cur whose
    // decision for cur is a rejection, found by one ballot; the configuration
    // carried up from cur stops there and the one at k + 1 is carried on.
    // The walking wavefronts hold up the rest of the workgroup at the next
    // barrier, so they issue ahead of the CU's other wavefronts meanwhile.
    if (wave < nsets) __builtin_amdgcn_s_setprio(2);
    for (int cs = wave; cs < nsets; cs += nwave) {
      const int c = c_lo + cs;
      const int32_t* m0 = sot0 + c * NT;
      int32_t* so = sotl + c * NT;
      int32_t* to = tosl + c * NT;
      const uint32_t* arow = acc + (size_t)c * (NT - 1) * (NB >> 5);
      uint64_t row = 0;
      if (lane < NT - 1) {
        row = arow[lane * (NB >> 5)];
        if (NB > 32) row |= (uint64_t)arow[lane * (NB >> 5) + 1] << 32;
      }
      uint64_t rej = 0;  // steps that rejected
      int cur = 0;
      for (;;) {
        const uint64_t r = __ballot(lane >= cur && lane < NT - 1 && !((row >> cur) & 1u));
        if (r == 0) break;
        const int k = __ffsll((unsigned long long)r) - 1;
        rej |= 1ull << k;
        cur = k + 1;
      }
      // a rejecting step keeps the configuration carried from just after the
      // previous rejection (or from 0); an accepting one takes the one above
      if (lane < NT - 1) {
        int fin;
        if ((rej >> lane) & 1u) {
          const uint64_t below = rej & ((1ull << lane) - 1u);
          fin = m0[below ? 64 - __clzll((long long)below) : 0];
        } else {
          fin = m0[lane + 1];
        }
        so[lane] = fin;
        to[fin] = lane;
      }
      if (lane == 0) {
        const int hot = m0[cur];
        so[NT - 1] = hot;
        to[hot] = NT - 1;
        if (WALK && walk) walk_observe(walk + 2 * c * NT, trips, so[0], hot, m);
      }
    }
    if (wave < nsets) __builtin_amdgcn_s_setprio(0);
  } else if (tid < nsets) {
    const int c = c_lo + tid;
    const int32_t* m0 = sot0 + c * NT;
    int32_t* so = sotl + c * NT;
    int32_t* to = tosl + c * NT;
    const uint32_t* arow = acc + (size_t)c * (NT - 1) * (NB >> 5);
    int cur = 0;
    for (int k = 0; k + 1 < NT; ++k) {
      int fin;
      if ((arow[k * (NB >> 5) + (cur >> 5)] >> (cur & 31)) & 1u) {
        fin = m0[k + 1];
      } else {
        fin = m0[cur];
        cur = k + 1;
      }
      so[k] = fin;
      to[fin] = k;
    }
    so[NT - 1] = m0[cur];
    to[m0[cur]] = NT - 1;
    if (WALK && walk) walk_observe(walk + 2 * c * NT, trips, so[0], m0[cur], m);
  }
}

}  // namespace ptsg
