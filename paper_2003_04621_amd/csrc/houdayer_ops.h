// houdayer_ops.h -- word operations of the Houdayer cluster move (Sec. 2.4,
// Eq. (10)) shared by the per-pair kernel and the fused Monte Carlo step.
// Q = overlap words (bit set <=> q_i = -1), C = cluster words, A = replica a;
// each is 2*NW words, colour c at offset c*NW.
#pragma once
#include "device.h"

namespace ptsg {

// Rank of the seed among a pair's n q = -1 sites (increasing site order).
__device__ __forceinline__ uint32_t seed_rank(const Geo& g, int s, int k, uint32_t v, uint32_t n) {
  const Ctr4 r = philox10(Ctr4{(uint32_t)k, v, 0u, (kTagHou << 28) | (uint32_t)s}, g.key0, g.key1);
  const uint64_t r64 = (uint64_t)r.x | ((uint64_t)r.y << 32);
  return (uint32_t)__umul64hi(r64, (uint64_t)n);
}

// Inclusive prefix sum over the wavefront's lanes (DPP, as wave_total).
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
  v += dpp_zero<kRowShr1>(v);
  v += dpp_zero<kRowShr2>(v);
  v += dpp_zero<kRowShr4>(v);
  v += dpp_zero<kRowShr8>(v);
  v += dpp_zero<kBcast15, 0xA>(v);
  v += dpp_zero<kBcast31, 0xC>(v);
  return v;
}

// Upward fill along the chain F_0, G_0, F_1, G_1, ... of every row field,
// where F_b -> G_b and G_b -> F_(b+1) (no link across a field boundary; nLB
// clears the lowest bit of each field): from seeds SF <= MF, SG <= MG, the
// sites of the masks MF, MG reachable by increasing steps.  F sites that can
// be entered from below form runs of R; adding the entry points Z to R
// carries through each run up to its first gap, so (R + Z) ^ R marks the
// reached bits of the run (an entry point already inside a carry is lost
// from the sum, hence the | Z).
__device__ __forceinline__ void chain_fill_up(uint32_t SF, uint32_t SG, uint32_t MF, uint32_t MG,
                                              uint32_t nLB, uint32_t& UF, uint32_t& UG) {
  const uint32_t Sp = SF | ((SG << 1) & nLB & MF);
  const uint32_t R = (MG << 1) & MF & nLB;
  const uint32_t Z = (Sp << 1) & R;
  const uint32_t V = (R & ((R + Z) ^ R)) | Z;
  UF = Sp | V;
  UG = SG | (UF & MG);
}

// Closure along x0 of the cluster words of one word index in row form: E and
// O hold the even and odd sites of each row field (E_0 O_0 E_1 O_1 ...), ME
// and MO the q sites, rME and rMO their bit reversals.  Every site of q
// linked to the cluster through a run of q sites of its row is added,
// periodic in x0: an upward fill and a bit-reversed (downward) fill cover
// each run from its lowest to its highest seed, and a run through the row's
// end is continued from its other end in one more pass.
__device__ __forceinline__ void row_closure(const Geo& g, uint32_t& E_io, uint32_t& O_io,
                                            uint32_t ME, uint32_t MO, uint32_t rME, uint32_t rMO) {
  const uint32_t nLB = ~g.LB, nLBr = ~__builtin_bitreverse32(g.HB);
  uint32_t SE = E_io, SO = O_io;
  for (;;) {
    uint32_t UE, UO, DO, DE;
    chain_fill_up(SE, SO, ME, MO, nLB, UE, UO);
    chain_fill_up(__builtin_bitreverse32(SO), __builtin_bitreverse32(SE), rMO, rME, nLBr, DO, DE);
    const uint32_t E = UE | __builtin_bitreverse32(DE), O = UO | __builtin_bitreverse32(DO);
    const uint32_t nE = E | (((O & g.HB) >> (g.H - 1)) & ME);  // O_(H-1) -> E_0
    const uint32_t nO = O | (((E & g.LB) << (g.H - 1)) & MO);  // E_0 -> O_(H-1)
    if (nE == E && nO == O) {
      E_io = E;
      O_io = O;
      return;
    }
    SE = nE;
    SO = nO;
  }
}

// One pass of that closure: every run filled upward and downward, but not
// continued through the row's end (a caller that iterates adds the two sites
// linked there, O_(H-1) and E_0, to the next pass's seeds).
__device__ __forceinline__ void row_fill(const Geo& g, uint32_t& E, uint32_t& O, uint32_t ME, uint32_t MO,
                                         uint32_t rME, uint32_t rMO) {
  uint32_t UE, UO, DO, DE;
  chain_fill_up(E, O, ME, MO, ~g.LB, UE, UO);
  chain_fill_up(__builtin_bitreverse32(O), __builtin_bitreverse32(E), rMO, rME,
                ~__builtin_bitreverse32(g.HB), DO, DE);
  E = UE | __builtin_bitreverse32(DE);
  O = UO | __builtin_bitreverse32(DO);
}

// The q site of rank m (counted in increasing x0) of a 64-site row held as
// its even-site word E and odd-site word O (site x0 = 2b + e is bit b of E
// for e = 0, of O for e = 1): sets that bit in SE or SO.  f(b), the number of
// q sites with x0 < 2b, is nondecreasing; a binary search finds the largest
// b with f(b) <= m, whose pair of sites holds the one sought.
__device__ __forceinline__ void rank_in_row64(uint32_t E, uint32_t O, uint32_t m, uint32_t& SE,
                                              uint32_t& SO) {
  int b = 0;
#pragma unroll
  for (int st = 16; st >= 1; st >>= 1) {
    const uint32_t lm = (1u << (b + st)) - 1u;
    if ((uint32_t)(__popc(E & lm) + __popc(O & lm)) <= m) b += st;
  }
  const uint32_t lm = (1u << b) - 1u;
  const bool even = ((E >> b) & 1u) && (uint32_t)(__popc(E & lm) + __popc(O & lm)) == m;
  SE = even ? 1u << b : 0u;
  SO = even ? 0u : 1u << b;
}

// ---------------------------------------------------------------------------
// Clusters in LDS words, in row form: Q (q = -1 sites) and C (cluster) hold
// the even-x0 sites of word w's row fields at [w] and the odd ones at [NW + w].
// ---------------------------------------------------------------------------
// Plants the seed in C (zero before), by one wavefront: the fields of all
// words in turn (site order: field, then word, then x0), the lanes owning
// contiguous words.  Returns the number of q = -1 sites.
__device__ __forceinline__ uint32_t seed_words(const Geo& g, const uint32_t* Q, uint32_t* C, int s, int k,
                                               uint32_t v, int lane) {
  const int NW = g.NW, per = (NW + 63) >> 6;
  const int w0 = min(NW, lane * per), w1 = min(NW, w0 + per);
  uint32_t cnt = 0;
  for (int w = w0; w < w1; ++w) cnt += __popc(Q[w]) + __popc(Q[NW + w]);
  const uint32_t n = (uint32_t)wave_total((int)cnt);
  if (n == 0) return 0;
  uint32_t m = seed_rank(g, s, k, v, n);
  for (int f = 0;; ++f) {
    const int sh = f * g.H;
    uint32_t lc = 0;
    for (int w = w0; w < w1; ++w)
      lc += __popc((Q[w] >> sh) & g.maskH) + __popc((Q[NW + w] >> sh) & g.maskH);
    const uint32_t incl = wave_scan(lc), tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
    if (m >= tot) {
      m -= tot;
      continue;
    }
    if (m >= incl - lc && m < incl) {
      uint32_t r = m - (incl - lc);
      for (int w = w0; w < w1; ++w) {
        const uint32_t e = (Q[w] >> sh) & g.maskH, o = (Q[NW + w] >> sh) & g.maskH;
        const uint32_t cw = __popc(e) + __popc(o);
        if (r < cw) {
          uint32_t se, so;
          rank_in_row64(e, o, r, se, so);
          C[w] = se << sh;
          C[NW + w] = so << sh;
          break;
        }
        r -= cw;
      }
    }
    return n;
  }
}

// Grows both words w of a cluster: neighbours through other words and through
// the row's end, then the runs along x0.  True if anything changed.  Stored
// words are filled along x0, so without new bits there is nothing to do,
// except on the first pass (`first`), which fills the seed's run.
template <int D>
__device__ __forceinline__ bool grow_rows(const Geo& g, uint32_t* C, const uint32_t* Q, int w, bool first) {
  const int NW = g.NW;
  const uint32_t ME = Q[w], MO = Q[NW + w];
  if (!(ME | MO)) return false;
  const WordNb q = word_nb(g, w);
  const uint32_t E0 = C[w], O0 = C[NW + w];
  uint32_t x[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t* Ci = C + i * NW;
    const uint32_t sp = Ci[q.wsp], sm = Ci[q.wsm];
    x[i] = pick(q.crp, rot_fields_down(g, sp), sp) | pick(q.crm, rot_fields_up(g, sm), sm);
    if (D == 3) x[i] |= Ci[q.w1p] | Ci[q.w1m];
  }
  uint32_t E = E0 | (ME & (x[0] | ((O0 & g.HB) >> (g.H - 1))));
  uint32_t O = O0 | (MO & (x[1] | ((E0 & g.LB) << (g.H - 1))));
  if (!(E | O) || (!first && E == E0 && O == O0)) return false;
  row_fill(g, E, O, ME, MO, __builtin_bitreverse32(ME), __builtin_bitreverse32(MO));
  if (E == E0 && O == O0) return false;
  C[w] = E;
  C[NW + w] = O;
  return true;
}

// The cluster of pair k by a whole workgroup (threads t of T): A and Q hold the
// two replicas' colour words on entry, Q the overlap's and C the cluster's colour
// words on return.  False (with Q and C unusable) if there is no q = -1 site.
template <int D>
__device__ __forceinline__ bool team_cluster(const Geo& g, const uint32_t* A, uint32_t* Q, uint32_t* C,
                                             int s, int k, uint32_t v, int t, int T) {
  __shared__ uint32_t n_minus;
  const int NW = g.NW;
  for (int w = t; w < NW; w += T) {
    const uint32_t q0 = A[w] ^ Q[w], q1 = A[NW + w] ^ Q[NW + w];
    const bool par = word_nb(g, w).par;
    Q[w] = par ? q1 : q0;
    Q[NW + w] = par ? q0 : q1;
    C[w] = C[NW + w] = 0u;
  }
  __syncthreads();
  if (t < 64) {
    const uint32_t n = seed_words(g, Q, C, s, k, v, t);
    if (t == 0) n_minus = n;
  }
  __syncthreads();
  if (n_minus == 0) return false;
  // A word read while another thread grows it is seen before or after: the
  // cluster only grows, and a round in which no word changed has read them all
  // as they stay.  One barrier per round: round r raises grew[r mod 3], and
  // the flag of round r - 1, which every thread has read, is cleared for r + 2.
  __shared__ int grew[3];
  if (t < 3) grew[t] = 0;
  if (T >= NW) {
    // one word per thread: its q sites, its cluster bits and where its
    // neighbours lie stay in registers
    const bool mine = t < NW;
    const int w = mine ? t : 0;
    const WordNb nb = word_nb(g, w);
    const uint32_t ME = mine ? Q[w] : 0u, MO = mine ? Q[NW + w] : 0u;
    const uint32_t rME = __builtin_bitreverse32(ME), rMO = __builtin_bitreverse32(MO);
    uint32_t E = mine ? C[w] : 0u, O = mine ? C[NW + w] : 0u;
    const uint32_t *Ce = C, *Co = C + NW;
    if (E | O) {
      row_fill(g, E, O, ME, MO, rME, rMO);
      C[w] = E;
      C[NW + w] = O;
    }
    __syncthreads();
    for (int r = 0;; r = r == 2 ? 0 : r + 1) {
      uint32_t se = Ce[nb.wsp], so = Co[nb.wsp], de = Ce[nb.wsm], od = Co[nb.wsm];
      if (nb.crp) {
        se = rot_fields_down(g, se);
        so = rot_fields_down(g, so);
      }
      if (nb.crm) {
        de = rot_fields_up(g, de);
        od = rot_fields_up(g, od);
      }
      uint32_t xe = se | de | ((O & g.HB) >> (g.H - 1)), xo = so | od | ((E & g.LB) << (g.H - 1));
      if (D == 3) {
        xe |= Ce[nb.w1p] | Ce[nb.w1m];
        xo |= Co[nb.w1p] | Co[nb.w1m];
      }
      const uint32_t nE = E | (ME & xe), nO = O | (MO & xo);
      if (nE != E || nO != O) {
        E = nE;
        O = nO;
        row_fill(g, E, O, ME, MO, rME, rMO);
        C[w] = E;
        C[NW + w] = O;
        grew[r] = 1;
      }
      __syncthreads();
      if (!grew[r]) break;
      if (t == 0) grew[r == 0 ? 2 : r - 1] = 0;
    }
  } else {
    bool first = true;
    __syncthreads();
    for (int r = 0;; r = r == 2 ? 0 : r + 1) {
      bool changed = false;
      for (int w = t; w < NW; w += T) changed |= grow_rows<D>(g, C, Q, w, first);
      first = false;
      if (changed) grew[r] = 1;
      __syncthreads();
      if (!grew[r]) break;
      if (t == 0) grew[r == 0 ? 2 : r - 1] = 0;
    }
  }
  for (int w = t; w < NW; w += T)
    if (word_nb(g, w).par) {
      const uint32_t c = C[w], q = Q[w];
      C[w] = C[NW + w];
      C[NW + w] = c;
      Q[w] = Q[NW + w];
      Q[NW + w] = q;
    }
  __syncthreads();
  return true;
}

// Threads of a team_cluster workgroup: one per word up to 1024.
inline int team_threads(const Geo& g) {
  const int t = (g.NW + 63) / 64 * 64;
  return t < 1024 ? t : 1024;
}

// Energy change of replica a from negating it on the cluster: 2 J_ij s_i s_j
// summed over the bonds leaving the cluster, from the colour-0 word w.
template <int D>
__device__ __forceinline__ int cluster_delta_word(const Geo& g, const uint32_t* C, const uint32_t* A,
                                                  const uint32_t* __restrict__ jw0, int w) {
  const WordNb q = word_nb(g, w);
  const int p = q.par;  // p(0, word)
  uint32_t nc[2 * D], na[2 * D];
  neighbour_words<D>(g, C + g.NW, w, q, p, nc);
  neighbour_words<D>(g, A + g.NW, w, q, p, na);
  const uint32_t C0 = C[w], A0 = A[w];
  int cross = 0, cross_u = 0;
#pragma unroll
  for (int dir = 0; dir < 2 * D; ++dir) {
    const uint32_t X = C0 ^ nc[dir];
    const uint32_t U = A0 ^ na[dir] ^ jw0[(size_t)dir * g.NW + w];
    cross += __popc(X);
    cross_u += __popc(X & U);
  }
  return 2 * (cross - 2 * cross_u);
}

}  // namespace ptsg
