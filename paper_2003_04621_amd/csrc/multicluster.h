// multicluster.h -- the multi-cluster variant of the Houdayer move (Sec. 3 and
// Sec. 5 propose it to remove the load imbalance of single clusters): every
// nearest-neighbour cluster of q = -1 sites of a pair is exchanged,
// independently, with probability 1/2.  A cluster is named by its lowest
// site m (site i = x0 + L x1 + L^2 x2) and is exchanged iff bit m mod 128 of
// the Philox output for counter (m / 128, v, k, 6 << 28 | sample) is set (bit
// j = bit j mod 32 of word j / 32).
//
// Connected components over the runs of q = -1 sites along x0, by a team of
// threads (one wavefront in the fused step, one workgroup in the per-pair
// kernel), with a 16-bit label per run in LDS:
//   1. each row's q = -1 sites form runs along x0 (periodically), found with
//      bit operations on the row's 64-bit mask; a row's runs are numbered in
//      the order of their lowest sites (the run that wraps through x0 = L - 1
//      contains x0 = 0 and comes first).  The label of run r of row R lies at
//      index R S + r, which is also the run's name, so names order runs by their
//      lowest sites and a label is an address.  Every run starts as its own
//      label;
//   2. every overlap segment of two rows adjacent along x1 (or x2) joins two
//      runs.  A run's first segment with the row before it along x1 sets its
//      label to that run; the other segments are edges, listed in LDS;
//   3. rounds until no edge joins two labels: every run takes its label's
//      root; then every edge whose runs have labels lo < hi points hi at lo.
//      Four runs or edges are in flight per thread.  A label only ever points
//      to a lower name of the same component and every round that joins labels
//      leaves fewer roots, whoever wins a concurrent store, so the rounds end,
//      with each run labelled by its component's lowest run;
//   4. the coins of all sites (one Philox call per 128 sites); each root run
//      keeps the coin of its lowest site in its label's top bit, each run takes
//      its root's, and the starts of the exchanged runs added to the row's mask
//      carry through exactly those runs, which makes the exchanged colour words.
// Bound by the instructions of the rounds (3) and their LDS latency at the
// wavefronts per CU that the scratch areas allow (ten at 2D L = 64; six with a
// 32-bit label per site): whole steps at 2D L = 64, 500 samples x 2 x 24, 206 ->
// 127 us against uniting edge by edge with root searches.  3D rows have at most 32
// sites, so their masks are 32-bit and their edges a byte: with 64-bit masks and
// 16-bit edges the scratch was larger than that of site labels at half the sizes
// and many small samples slower than with root searches (us per step, root
// searches / 64-bit / 32-bit): L = 6, 830 x 2 x 16 67.8 / 73.9 / 67.1; L = 10, 500 x
// 2 x 16 77.1 / 85.4 / 77.8; L = 12, 100 x 2 x 20 97.9 / 72.8 / 67.3; L = 16, 300 x
// 2 x 24 456 / 371 / 287; still so L = 4, 1000 x 2 x 16 52.0 / 60.1 / 54.9 (64 x 2 x
// 24 27.4 / 23.6 / 22.5).
#pragma once
#include "device.h"

namespace ptsg {

constexpr uint32_t kTagHouMulti = 6u;

// Sites a team's labels can name (the per-pair kernel's LDS holds them).
constexpr int kMultiMaxSites = 32768;

// A row of L <= 64 sites holds at most L/2 runs.  Places for a row's runs and,
// per direction, its edges (multiples of four), and the labels' row stride S: an
// odd number of words, so that the rows' labels start in different LDS banks
// (L = 4: just its places).
__host__ __device__ constexpr int multi_row_places(int L) { return (L / 2 + 3) & ~3; }
__host__ __device__ constexpr int multi_row_stride(int L) { return multi_row_places(L) + (L > 4 ? 2 : 0); }

// A row's mask and an edge (the two runs' numbers) as held in LDS: a 3D row has
// at most 32 sites (kMultiMaxSites), so 16 runs.
template <int D>
struct MultiRow {
  using Mask = uint64_t;
  using Edge = uint16_t;
  static constexpr int kShift = 8;
};
template <>
struct MultiRow<3> {
  using Mask = uint32_t;
  using Edge = uint8_t;
  static constexpr int kShift = 4;
};

// A label is a run's name, below NR S, with a coin in its top bit; an edge holds
// two numbers of runs, L / 2 at most.
constexpr bool multi_fits() {
  for (int L = 4; L <= 64; L += 2) {
    if (L * multi_row_stride(L) > 0x8000 || L / 2 > 1 << MultiRow<2>::kShift) return false;
    if (L * L * L > kMultiMaxSites) continue;
    if (L * L * multi_row_stride(L) > 0x8000 || L > 32 || L / 2 > 1 << MultiRow<3>::kShift) return false;
  }
  return true;
}
static_assert(multi_fits(), "names, masks and edges of the multi-cluster labels");

// LDS words of one team's scratch for geometry g: overlap and cluster words
// (2 NW each), row masks, coins (one bit per site, 128-bit blocks), labels
// (16-bit), edges and edge counts.
__host__ __device__ constexpr int multi_scratch_words(const Geo& g) {
  const int mask = g.d == 3 ? (int)sizeof(MultiRow<3>::Mask) : (int)sizeof(MultiRow<2>::Mask);
  const int edge = g.d == 3 ? (int)sizeof(MultiRow<3>::Edge) : (int)sizeof(MultiRow<2>::Edge);
  return 4 * g.NW + g.NR * mask / 4 + 4 * ((g.N + 127) / 128) + g.NR * multi_row_stride(g.L) / 2 +
         (g.NR * (g.d - 1) * (multi_row_places(g.L) + 1) * edge + 3) / 4;
}

// Bit b of x moved to bit 2b, for the lower half of a row mask.
__device__ __forceinline__ uint64_t spread_bits(uint64_t v) {
  v = (v | (v << 16)) & 0x0000FFFF0000FFFFull;
  v = (v | (v << 8)) & 0x00FF00FF00FF00FFull;
  v = (v | (v << 4)) & 0x0F0F0F0F0F0F0F0Full;
  v = (v | (v << 2)) & 0x3333333333333333ull;
  v = (v | (v << 1)) & 0x5555555555555555ull;
  return v;
}
__device__ __forceinline__ uint32_t spread_bits(uint32_t v) {
  v = (v | (v << 8)) & 0x00FF00FFu;
  v = (v | (v << 4)) & 0x0F0F0F0Fu;
  v = (v | (v << 2)) & 0x33333333u;
  v = (v | (v << 1)) & 0x55555555u;
  return v;
}

// Bits 2b of x moved to bit b (the inverse of spread_bits).
__device__ __forceinline__ uint32_t compress_even_bits(uint64_t x) {
  x &= 0x5555555555555555ull;
  x = (x | (x >> 1)) & 0x3333333333333333ull;
  x = (x | (x >> 2)) & 0x0F0F0F0F0F0F0F0Full;
  x = (x | (x >> 4)) & 0x00FF00FF00FF00FFull;
  x = (x | (x >> 8)) & 0x0000FFFF0000FFFFull;
  x = (x | (x >> 16)) & 0x00000000FFFFFFFFull;
  return (uint32_t)x;
}
__device__ __forceinline__ uint32_t compress_even_bits(uint32_t x) {
  x &= 0x55555555u;
  x = (x | (x >> 1)) & 0x33333333u;
  x = (x | (x >> 2)) & 0x0F0F0F0Fu;
  x = (x | (x >> 4)) & 0x00FF00FFu;
  x = (x | (x >> 8)) & 0x0000FFFFu;
  return x;
}

__device__ __forceinline__ int mask_count(uint64_t m) { return __popcll(m); }
__device__ __forceinline__ int mask_count(uint32_t m) { return __popc(m); }
// Position of the lowest / highest bit (m != 0).
__device__ __forceinline__ int mask_low(uint64_t m) { return (int)__ffsll((long long)m) - 1; }
__device__ __forceinline__ int mask_low(uint32_t m) { return __ffs((int)m) - 1; }
__device__ __forceinline__ int mask_high(uint64_t m) { return 63 - __clzll((long long)m); }
__device__ __forceinline__ int mask_high(uint32_t m) { return 31 - __clz((int)m); }

// The runs of q = -1 sites of one row (L-bit mask m in x0 order, taken
// periodically).  starts: bit x0 set iff x0 is q = -1 and x0 - 1 is not; n: the
// number of runs; wraps: the last start's run continues at x0 = 0.  A row that
// is q = -1 everywhere has no start and is one run.
template <typename M>
struct RowRuns {
  M m, starts;
  int n;
  bool wraps;
};

template <typename M>
__device__ __forceinline__ RowRuns<M> row_runs(M m, int L, M full) {
  RowRuns<M> r;
  r.m = m;
  r.starts = m & ~(((m << 1) | (m >> (L - 1))) & full);
  r.n = r.starts ? mask_count(r.starts) : (m ? 1 : 0);
  r.wraps = r.starts && (m & 1u) && ((m >> (L - 1)) & 1u);
  return r;
}

// Number (in the order of lowest sites) of the run holding q = -1 site x0.
template <typename M>
__device__ __forceinline__ int run_rank(const RowRuns<M>& r, int x0) {
  const int c = mask_count((M)(r.starts & (((M)2 << x0) - (M)1)));  // the top site: every bit
  if (r.wraps) return c == r.n ? 0 : c;
  return c > 0 ? c - 1 : 0;
}

// The q = -1 sites of row R as an L-bit mask in x0 order.
template <typename M>
__device__ __forceinline__ M row_q_mask(const Geo& g, const uint32_t* Q, int R) {
  int w, f;
  row_word(g, R, w, f);
  const int p0 = row_parity(g, R);  // colour of the even-x0 sites
  const uint32_t e = (Q[p0 * g.NW + w] >> (f * g.H)) & g.maskH;
  const uint32_t o = (Q[(1 - p0) * g.NW + w] >> (f * g.H)) & g.maskH;
  return spread_bits((M)e) | (spread_bits((M)o) << 1);
}

// Rows next to row R in the positive x1 and (3D) x2 directions.
__device__ __forceinline__ void rows_up(const Geo& g, int R, int* up) {
  if (g.d == 3) {
    const int x2 = (int)divL(g, (uint32_t)R), x1 = R - x2 * g.L;
    up[0] = x1 == g.L - 1 ? R - (g.L - 1) : R + 1;
    up[1] = x2 == g.L - 1 ? R - (g.L - 1) * g.L : R + g.L;
  } else {
    up[0] = R == g.L - 1 ? 0 : R + 1;
  }
}

// The exchanged sites of one multi-cluster move of the pair whose overlap
// words are Q (bit set: q = -1) as colour words C (2 NW), by the team's
// threads t < T.  scr: the team's scratch after Q and C (8-byte aligned).
// `sync` orders the team's LDS accesses, `any` does so and tells whether its
// argument is true for some thread of the team.
template <int D, typename Sync, typename Any>
__device__ __forceinline__ void multi_cluster_words(const Geo& g, const uint32_t* Q, uint32_t* C,
                                                    uint32_t* scr, int s, int k, uint32_t v,
                                                    int t, int T, Sync sync, Any any) {
  using Mask = typename MultiRow<D>::Mask;
  using Edge = typename MultiRow<D>::Edge;
  constexpr int kShift = MultiRow<D>::kShift;
  const int L = g.L, NR = g.NR, N = g.N, NW = g.NW;
  const int nblk = (N + 127) / 128, ME = multi_row_places(L), S = multi_row_stride(L);
  Mask* qr = reinterpret_cast<Mask*>(scr);
  uint32_t* coin = scr + NR * (int)(sizeof(Mask) / 4);
  uint16_t* lab = reinterpret_cast<uint16_t*>(coin + 4 * nblk);
  Edge* edge = reinterpret_cast<Edge*>(lab + NR * S);  // edge e of row R, direction j at (j ME + e) NR + R
  Edge* edges = edge + (D - 1) * ME * NR;              // number of them at j NR + R
  const Mask full = L == 8 * (int)sizeof(Mask) ? ~(Mask)0 : (((Mask)1 << L) - (Mask)1);
  // four consecutive labels of a row (two words)
  typedef uint32_t __attribute__((may_alias)) Word;
  auto load4 = [&](int i, uint32_t (&l)[4]) {
    const Word* w = reinterpret_cast<const Word*>(lab + i);
    const uint32_t x = w[0], y = w[1];
    l[0] = x & 0xFFFFu;
    l[1] = x >> 16;
    l[2] = y & 0xFFFFu;
    l[3] = y >> 16;
  };
  auto store4 = [&](int i, const uint32_t (&l)[4]) {
    Word* w = reinterpret_cast<Word*>(lab + i);
    w[0] = l[0] | (l[1] << 16);
    w[1] = l[2] | (l[3] << 16);
  };

  // 1. row masks; every run its own label; coins
  for (int R = t; R < NR; R += T) {
    qr[R] = row_q_mask<Mask>(g, Q, R);
    for (int r = 0; r < ME; r += 4) {  // unused places too
      const uint32_t i = (uint32_t)(R * S + r);
      store4((int)i, {i, i + 1u, i + 2u, i + 3u});
    }
  }
  for (int blk = t; blk < nblk; blk += T) {
    const Ctr4 r = philox10(Ctr4{(uint32_t)blk, v, (uint32_t)k, (kTagHouMulti << 28) | (uint32_t)s},
                            g.key0, g.key1);
    coin[4 * blk + 0] = r.x;
    coin[4 * blk + 1] = r.y;
    coin[4 * blk + 2] = r.z;
    coin[4 * blk + 3] = r.w;
  }
  sync();

  // 2. one edge per segment of overlap along x1 (and x2), except those that set
  // the upper run's label (only row R's thread writes those of the row above);
  // edge = the runs' numbers, the lower row's in the low bits
  for (int R = t; R < NR; R += T) {
    const Mask m = qr[R];
    const RowRuns<Mask> rr = row_runs(m, L, full);
    int up[D - 1];
    rows_up(g, R, up);
#pragma unroll
    for (int j = 0; j < D - 1; ++j) {
      Edge* er = edge + j * ME * NR + R;
      const Mask mu = qr[up[j]];
      const Mask e = m & mu;
      const RowRuns<Mask> ru = row_runs(mu, L, full);
      // first site of each segment (cyclically); a full overlap is one segment
      Mask first = e & ~(((e << 1) | (e >> (L - 1))) & full);
      if (e == full) first = 1;
      uint32_t set = j == 0 && up[j] > R ? 0u : ~0u;  // runs above that have their label
      int n = 0;
      uint32_t ed = 0;
      for (; first; first &= first - (Mask)1) {
        const int x0 = mask_low(first);
        const uint32_t ra = (uint32_t)run_rank(rr, x0), rb = (uint32_t)run_rank(ru, x0);
        if (!((set >> rb) & 1u)) {
          set |= 1u << rb;
          lab[up[j] * S + rb] = (uint16_t)(R * S + ra);
          continue;
        }
        ed = ra | (rb << kShift);
        er[n * NR] = (Edge)ed;
        ++n;
      }
      edges[j * NR + R] = (Edge)n;
      // the last one again up to a multiple of four: no checks when they are read
      for (; n & 3; ++n) er[n * NR] = (Edge)ed;
    }
  }
  sync();

  // 3. take roots and join the labels of every edge, until nothing joins
  for (;;) {
    for (int R = t; R < NR; R += T) {
      const int n = row_runs(qr[R], L, full).n;
      for (int r0 = 0; r0 < n; r0 += 4) {
        uint32_t l[4], p[4];
        load4(R * S + r0, l);
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = lab[l[i]];
        // every thread stores what it has reached, so the distances double
        while (p[0] != l[0] || p[1] != l[1] || p[2] != l[2] || p[3] != l[3]) {
          store4(R * S + r0, p);
#pragma unroll
          for (int i = 0; i < 4; ++i) l[i] = p[i];
#pragma unroll
          for (int i = 0; i < 4; ++i) p[i] = lab[l[i]];
        }
      }
    }
    sync();
    bool joined = false;
    for (int R = t; R < NR; R += T) {
      int up[D - 1];
      rows_up(g, R, up);
#pragma unroll
      for (int j = 0; j < D - 1; ++j) {
        const Edge* er = edge + j * ME * NR + R;
        const int n = edges[j * NR + R];
        const uint16_t *low = lab + R * S, *high = lab + up[j] * S;
        for (int e0 = 0; e0 < n; e0 += 4) {
          uint32_t ed[4], la[4], lb[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) ed[i] = er[(e0 + i) * NR];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            la[i] = low[ed[i] & ((1u << kShift) - 1u)];
            lb[i] = high[ed[i] >> kShift];
          }
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (la[i] != lb[i]) {
              lab[max(la[i], lb[i])] = (uint16_t)min(la[i], lb[i]);
              joined = true;
            }
        }
      }
    }
    if (!any(joined)) break;
  }

  // 4. the roots' coins, then the exchanged sites as colour words
  for (int R = t; R < NR; R += T) {
    const RowRuns<Mask> rr = row_runs(qr[R], L, full);
    Mask rest = rr.starts;
    for (int r = 0; r < rr.n; ++r) {
      const uint32_t name = (uint32_t)(R * S + r);
      int x0 = 0;  // lowest site of run r
      if (rr.starts && !(rr.wraps && r == 0)) {
        x0 = mask_low(rest);
        rest &= rest - (Mask)1;
      }
      if (lab[name] == name) {
        const uint32_t i = (uint32_t)(R * L + x0);
        lab[name] = (uint16_t)(name | (((coin[i >> 5] >> (i & 31)) & 1u) << 15));
      }
    }
  }
  sync();
  for (int w = t; w < NW; w += T) {
    const WordNb q = word_nb(g, w);
    uint32_t out[2] = {0u, 0u};
    for (int f = 0; f < g.P; ++f) {
      const int R = word_row(g, q, f);
      const Mask m = qr[R];
      const RowRuns<Mask> rr = row_runs(m, L, full);
      uint32_t take = 0;  // bit r: run r is exchanged
      for (int r0 = 0; r0 < rr.n; r0 += 4) {
        uint32_t l[4];
        load4(R * S + r0, l);
#pragma unroll
        for (int i = 0; i < 4; ++i) take |= (uint32_t)(lab[l[i] & 0x7FFFu] >> 15) << (r0 + i);
      }
      Mask X = 0;
      if (!rr.starts) {
        X = take ? full : (Mask)0;
      } else {
        Mask St = 0;  // starts of the exchanged runs
        uint32_t bits = take;
        if (rr.wraps) {
          if (take & 1u) St = (Mask)1 | ((Mask)1 << mask_high(rr.starts));
          bits >>= 1;
        }
        for (Mask rest = rr.starts; bits; bits >>= 1, rest &= rest - (Mask)1)
          if (bits & 1u) St |= rest & ((Mask)0 - rest);
        X = m & ~(m + St);
      }
      if (!X) continue;
      const int p0 = row_parity(g, R);  // colour of the even-x0 sites
      out[p0] |= compress_even_bits(X) << (f * g.H);
      out[1 - p0] |= compress_even_bits((Mask)(X >> 1)) << (f * g.H);
    }
    C[w] = out[0];
    C[NW + w] = out[1];
  }
  sync();
}

}  // namespace ptsg
