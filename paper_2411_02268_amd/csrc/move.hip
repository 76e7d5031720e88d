// Local-moving sweeps: LPA iterations (Section 4.3), Louvain/Leiden local moving
// (Sections 4.1-4.2, Fig. 2) and Leiden refinement, with the weighted Misra-Gries
// sketch (Appendix A.1, Algorithm 1) or an exact table (Section 4, Fig. 1).
//
// Per vertex i with current community d = C[i]:
//   pass 1  stream the row (self excluded; refinement: same bound only), key C[j],
//           into a K-slot sketch; rows longer than L positions are cut into chunks
//           of L, each sketched from empty, then merged pairwise left to right,
//           level by level (odd last moves up);
//   pass 2  exact K_{i->c} of every positive slot and K_{i->d} (skipped when the
//           sketch lost no weight: its values are then exact and complete);
//   decide  LPA: largest K_{i->c}, lowest c on ties.  Louvain/Leiden: largest
//           G = W (K_ic - K_id) - K_i (K_i + Sigma_c - Sigma_d) (Eq. 2 times W^2/2),
//           c != d, G > 0, lowest c on ties; applied only in the sweep's direction.
//
// Mapping on CDNA: every chunk is the stream of four lanes with the sketch's slots in
// their VGPRs, 64 chunks per workgroup, the chunks' entries staged in LDS.  A row of at
// most 64 chunks takes 2^b quads of a workgroup (b = 0 for a row of one chunk); its chunk
// sketches are merged in LDS and the same lanes run pass 2 from LDS.  Rows of
// more than 64 chunks write one merged sketch per 64 chunks to scratch, and one
// workgroup per row merges those in LDS.
#include "move.hpp"
#include "primitives.hpp"
#include "quad_sketch.hpp"
#include "sketch.hpp"
#include "wave_sketch.hpp"

namespace mgcd {

// ---- decision ---------------------------------------------------------------------

struct Counters {
  uint32_t moved = 0, prop = 0, cand = 0;
  int32_t g = 0;  // batched: the graph of the rows counted (one row per lane per flush)
  uint64_t sumG = 0;
};

template <int ALGO>
__device__ inline int32_t community_of_self(const SweepArgs &a, int32_t i) {
  return ALGO == ALGO_REFINE ? i : a.C[i];
}

// Evaluate one candidate community c with exact linking weight kc; keep the best.
// Total weight W of vertex i's graph.
__device__ inline uint64_t weight_of(const SweepArgs &a, int32_t i) {
  return a.gid ? (uint64_t)a.Wg[a.gid[i]] : a.W;
}

// Batched runs: a vertex of a graph that no longer moves keeps its community.
__device__ inline bool frozen(const SweepArgs &a, int32_t i) {
  return (a.halt && *a.halt) || (a.gid && !a.active[a.gid[i]]);
}

// Batched runs: no graph moves any more (set after the previous sweep), so this sweep
// does nothing at all and the labels stay in the buffer the last real sweep wrote.
// Wave-uniform (written before the kernel started).
__device__ inline bool level_over(const SweepArgs &a) { return a.live && *a.live == 0; }

// A product of two values that fit 32 signed bits, exact in 64: one multiply-add, where a
// 64-bit product takes several quarter-rate multiplies.  Every factor of the gain fits: W
// and all weights and totals are below 2^31, so are differences of two of them, and
// K_i + Sigma_c - Sigma_d lies within 31 bits of 0 since vertex i's own K_i is part of
// Sigma_d (refinement: Sigma_d = K_i).
__device__ inline int64_t mul32(int64_t x, int64_t y) { return (int64_t)(int32_t)x * (int32_t)y; }

// Evaluate candidate c (present: it exists) with exact linking weight kc and
// community total sc; keep the best.  Branch-free, so gathers feeding sc are issued
// together rather than each inside a branch of its own.
template <int ALGO>
__device__ inline void consider_v(int64_t W, int32_t d, int64_t Ki, int64_t Sd, uint32_t kd, int32_t c,
                                  uint32_t kc, uint32_t sc, bool present, int32_t &best, int64_t &bestG) {
  int64_t G;
  bool ok;
  if (ALGO == ALGO_LPA) {
    G = (int64_t)kc;
    ok = present;
  } else {
    G = mul32(W, (int64_t)kc - (int64_t)kd) - mul32(Ki, Ki + (int64_t)sc - Sd);
    ok = present && c != d && G > 0;
  }
  const bool better = ok && (best < 0 || G > bestG || (G == bestG && c < best));
  best = better ? c : best;
  bestG = better ? G : bestG;
}

template <int ALGO>
__device__ inline void consider(const SweepArgs &a, int64_t W, int32_t d, int64_t Ki, int64_t Sd,
                                uint32_t kd, int32_t c, uint32_t kc, int32_t &best, int64_t &bestG) {
  const uint32_t sc = ALGO == ALGO_LPA ? 0u : a.Sig[c];
  consider_v<ALGO>(W, d, Ki, Sd, kd, c, kc, sc, true, best, bestG);
}

// The best of K candidate slots (EMPTY: no candidate).  LPA scores the linking weights
// alone.  Louvain and Leiden also need each candidate's total Sigma_c, a random read.
// The gain W (k_c - k_d) - K_i (K_i + Sigma_c - Sigma_d) is at most its value at
// Sigma_c = 0, so the heaviest candidate is scored first, and another candidate's total
// is read only when that bound can still beat the best so far (or tie it with a lower
// id); a slot that cannot reads Sigma_d instead (cached; the reads stay branch-free and
// in flight together) and is not scored.  The best gain only grows, so a skipped slot
// could neither win nor tie: the result equals scoring every slot.  Returns the number
// of candidates' totals read.
template <int K, int ALGO>
__device__ MGCD_INLINE int consider_slots(const SweepArgs &a, int64_t W, int32_t d, int64_t Ki, int64_t Sd,
                                     uint32_t kd, const uint32_t (&key)[K], const uint32_t (&ex)[K],
                                     int32_t &best, int64_t &bestG) {
  if constexpr (ALGO == ALGO_LPA) {
#pragma unroll
    for (int p = 0; p < K; ++p)
      consider_v<ALGO>(W, d, Ki, Sd, kd, (int32_t)key[p], ex[p], 0u, key[p] != EMPTY, best, bestG);
    return 0;
  } else {
    const uint32_t ud = (uint32_t)d;
    uint32_t c0 = EMPTY, x0 = 0;  // the heaviest candidate other than d (ties: first slot)
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const bool take = key[p] != EMPTY && key[p] != ud && (c0 == EMPTY || ex[p] > x0);
      c0 = take ? key[p] : c0;
      x0 = take ? ex[p] : x0;
    }
    const uint32_t s0 = a.Sig[c0 != EMPTY ? (int32_t)c0 : d];
    consider_v<ALGO>(W, d, Ki, Sd, kd, (int32_t)c0, x0, s0, c0 != EMPTY, best, bestG);
    const int64_t own = mul32(Ki, Sd - Ki);  // U(c) = W (k_c - k_d) + K_i (Sigma_d - K_i)
    bool live[K];
    uint32_t sc[K];
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const int64_t U = mul32(W, (int64_t)ex[p] - (int64_t)kd) + own;
      const int32_t c = (int32_t)key[p];
      live[p] = key[p] != EMPTY && key[p] != ud && key[p] != c0 && U > 0 &&
                (best < 0 || U > bestG || (U == bestG && c < best));
      sc[p] = a.Sig[live[p] ? c : d];
    }
    int reads = c0 != EMPTY;
#pragma unroll
    for (int p = 0; p < K; ++p) {
      consider_v<ALGO>(W, d, Ki, Sd, kd, (int32_t)key[p], ex[p], sc[p], live[p], best, bestG);
      reads += live[p];
    }
    return reads;
  }
}

template <int ALGO>
__device__ inline void finish(const SweepArgs &a, int32_t i, int32_t d, int32_t best, int64_t bestG,
                              Counters &ct) {
  int32_t target = d;
  if (ALGO == ALGO_LPA) {
    if (best >= 0) target = best;
  } else if (best >= 0) {
    ct.prop += 1;
    ct.sumG += (uint64_t)bestG;
    const int dir = a.gdir ? (int)a.gdir[a.gid[i]] : a.dir;
    bool ok = dir == 0 || (dir < 0 ? best < d : best > d);
    if (ok) target = best;
  }
  a.Cnew[i] = target;
  if (ALGO != ALGO_LPA && a.gain) a.gain[i] = best >= 0 ? bestG : 0;
  ct.moved += target != d;
  if (a.gctr) ct.g = a.gid[i];  // batched: added to the graph's counters when flushed
}

// Batched runs: counts of one graph's rows, kept by a whole wave (wave-uniform) until
// rows of another graph come or the wave ends.  Every atomic on a graph's counters
// queues behind those of the other waves at work on that graph (with one flush per 16
// rows, a sweep over 192 graphs spent more than half its time waiting there).
struct GraphCounts {
  int32_t g;  // -1: none
  uint32_t moved, prop;
  uint64_t sumG;
};

__device__ inline void commit_graph_counts(const SweepArgs &a, const GraphCounts &gc) {  // one lane
  if (gc.g < 0) return;
  unsigned long long *c = a.gctr + 3 * (int64_t)gc.g;
  if (gc.moved) atomicAdd(&c[0], (unsigned long long)gc.moved);
  if (gc.prop) atomicAdd(&c[1], (unsigned long long)gc.prop);
  if (gc.sumG) atomicAdd(&c[2], (unsigned long long)gc.sumG);
}

// Adds the lanes' counts (of at most one row each) to gc, graph by graph; they restart.
__device__ inline void gather_graph_counts(const SweepArgs &a, Counters &ct, GraphCounts &gc) {
  const int lane = lane_id();
  uint64_t todo = __ballot(ct.moved != 0 || ct.prop != 0);  // a gain comes with a proposal
  while (todo) {  // wave-uniform
    const int32_t g = uniform(__shfl(ct.g, __builtin_ctzll(todo)));
    const bool mine = ((todo >> lane) & 1ull) != 0 && ct.g == g;
    if (gc.g != g) {
      if (lane == 0) commit_graph_counts(a, gc);
      gc = GraphCounts{g, 0, 0, 0};
    }
    gc.moved += __popcll(__ballot(mine && ct.moved != 0));
    const uint32_t p = __popcll(__ballot(mine && ct.prop != 0));
    gc.prop += p;
    if (p) gc.sumG += wave_sum((unsigned long long)(mine ? ct.sumG : 0ull));
    todo &= ~__ballot(mine);
  }
  ct = Counters{};
}

// This workgroup's copy of the sweep's counters (the reader adds up the copies).
__device__ inline unsigned long long *sweep_counters(const SweepArgs &a) {
  return a.ctr + (int64_t)spread_copy() * CTR_STRIDE;
}

// One thread's counts of one row, to its graph's counters (batched) or the sweep's.
__device__ inline void commit_counters(const SweepArgs &a, const Counters &ct) {
  unsigned long long *c = a.gctr ? a.gctr + 3 * (int64_t)ct.g : sweep_counters(a);
  if (ct.moved) atomicAdd(&c[0], (unsigned long long)ct.moved);
  if (ct.prop) atomicAdd(&c[1], (unsigned long long)ct.prop);
  if (ct.sumG) atomicAdd(&c[2], (unsigned long long)ct.sumG);
}

// One wave's counts of at most one row per lane.
__device__ inline void flush_wave_counters(const SweepArgs &a, Counters &ct) {
  if (a.gctr) {
    GraphCounts gc{-1, 0, 0, 0};
    gather_graph_counts(a, ct, gc);
    if (lane_id() == 0) commit_graph_counts(a, gc);
    return;
  }
  const uint32_t m = __popcll(__ballot(ct.moved != 0)), p = __popcll(__ballot(ct.prop != 0));
  const uint32_t cands = wave_sum(ct.cand);
  const unsigned long long g = wave_sum((unsigned long long)ct.sumG);
  const int l = lane_id();
  const unsigned long long x = l == 0 ? m : l == 1 ? p : l == 2 ? g : cands;
  if (l < 4 && x) atomicAdd(&sweep_counters(a)[l], x);
}

// Batched runs: the last graphs of a workgroup's waves, together.
__device__ inline void flush_graph_counts(const SweepArgs &a, GraphCounts gc) {
  __shared__ GraphCounts last[BLOCK / WAVE];
  if (lane_id() == 0) last[threadIdx.x / WAVE] = gc;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int q = 1; q < BLOCK / WAVE; ++q) {
      const GraphCounts x = last[q];
      if (x.g < 0) continue;
      if (x.g != gc.g) {
        commit_graph_counts(a, gc);
        gc = x;
      } else {
        gc.moved += x.moved;
        gc.prop += x.prop;
        gc.sumG += x.sumG;
      }
    }
    commit_graph_counts(a, gc);
  }
}

// A workgroup's counts of at most one row per lane.
__device__ inline void flush_counters(const SweepArgs &a, Counters ct) {
  const int w = threadIdx.x / WAVE;
  if (a.gctr) {  // batched (kernel-uniform)
    GraphCounts gc{-1, 0, 0, 0};
    gather_graph_counts(a, ct, gc);
    flush_graph_counts(a, gc);
    return;
  }
  __shared__ unsigned long long red[4][4];
  unsigned long long m = wave_sum((unsigned long long)ct.moved);
  unsigned long long p = wave_sum((unsigned long long)ct.prop);
  unsigned long long g = wave_sum((unsigned long long)ct.sumG);
  unsigned long long c = wave_sum((unsigned long long)ct.cand);
  if (lane_id() == 0) {
    red[0][w] = m;
    red[1][w] = p;
    red[2][w] = g;
    red[3][w] = c;
  }
  __syncthreads();
  if (threadIdx.x < 4) {
    unsigned long long s = red[threadIdx.x][0] + red[threadIdx.x][1] + red[threadIdx.x][2] +
                           red[threadIdx.x][3];
    if (s) atomicAdd(&sweep_counters(a)[threadIdx.x], s);
  }
}

// The device clock at the start of a sweep of one kernel class (SweepArgs::stamp).
__device__ inline void stamp_start(const SweepArgs &a, int64_t first = 0) {
  if (a.stamp && first == 0 && blockIdx.x == 0 && threadIdx.x == 0) *a.stamp = wall_clock64();
}

// Key of entry (i -> j) in the stream of vertex i, or EMPTY when Algorithm 1's
// early exits skip it (self-loop; refinement across bounds).
template <int ALGO>
__device__ inline uint32_t stream_key(const SweepArgs &a, int32_t i, int32_t j, int32_t bi) {
  if (j == i) return EMPTY;
  if (ALGO == ALGO_REFINE) return a.bound[j] == bi ? (uint32_t)j : EMPTY;
  return a.ident ? (uint32_t)j : (uint32_t)a.C[j];
}

// Keys of U neighbours j (any valid ids): their communities C[j], or j itself when C is
// the identity; refinement keys are j when it shares the row's bound b[u], else EMPTY.
// One wave-uniform branch around all U reads keeps them in flight together.
template <int ALGO, int U>
__device__ inline void neighbour_keys(const SweepArgs &a, const int32_t (&j)[U], const int32_t (&b)[U],
                                      uint32_t (&c)[U]) {
  if (ALGO == ALGO_REFINE) {
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = a.bound[j[u]] == b[u] ? (uint32_t)j[u] : EMPTY;
  } else if (a.ident) {
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = (uint32_t)j[u];
  } else {
#pragma unroll
    for (int u = 0; u < U; ++u) c[u] = (uint32_t)a.C[j[u]];
  }
}

// ---- MG: long rows -----------------------------------------------------------------

// Chunk q of a long row: its row, its bounds and whether it is active.
struct LongChunk {
  int32_t m, i;
  int64_t lo, hi;
  bool active;
};

__device__ inline LongChunk long_chunk(const SweepArgs &a, const int32_t *multi,
                                       const int32_t *owner, const int64_t *cstart, int64_t q,
                                       int64_t nchunks, int64_t L) {
  LongChunk c{0, 0, 0, 0, false};
  if (q >= nchunks) return c;
  c.m = owner[q];
  c.i = multi[c.m];
  if (frozen(a, c.i)) return c;
  const int64_t rhi = a.g.off[c.i + 1];
  c.lo = a.g.off[c.i] + (q - cstart[c.m]) * L;
  c.hi = c.lo + L < rhi ? c.lo + L : rhi;
  c.active = true;
  return c;
}

// Choose the best candidate of row i and record the move (one thread).
template <int K, int ALGO>
__device__ inline void decide_long(const SweepArgs &a, int32_t i, int32_t d, const uint32_t (&key)[K],
                                   const uint32_t (&ex)[K], uint32_t kd) {
  Counters ct;
  int32_t best = -1;
  int64_t bestG = 0;
  const int64_t W = ALGO == ALGO_LPA ? 0 : (int64_t)weight_of(a, i);
  const int64_t Ki = ALGO == ALGO_LPA ? 0 : (int64_t)a.K[i];
  const int64_t Sd = ALGO == ALGO_LPA ? 0 : (int64_t)a.Sig[d];
  consider_slots<K, ALGO>(a, W, d, Ki, Sd, kd, key, ex, best, bestG);
  finish<ALGO>(a, i, d, best, bestG, ct);
  commit_counters(a, ct);
}

// cflag[m]: 0 decided here (exact sketch), 1 lossy (candidates in cand), 2 frozen.
template <int K, int ALGO>
__global__ void __launch_bounds__(BLOCK) MGCD_SKETCH_OCCUPANCY(K)
    k_long_merge(SweepArgs a, const int32_t *__restrict__ multi, const int64_t *__restrict__ gstart,
                 int64_t block0, Pair *sk, const uint32_t *__restrict__ skflag, Pair *cand, uint32_t *cflag) {
  if (level_over(a)) return;  // batched: every graph has stopped
  __shared__ Pair lds[BLOCK * K];
  __shared__ int flag_any;
  const int t = threadIdx.x;
  const int32_t m = (int32_t)(block0 + blockIdx.x);
  const int32_t i = multi[m];
  const int64_t cb = gstart[m], nc = gstart[m + 1] - cb;  // group roots of the row
  if (frozen(a, i)) {  // block-uniform
    if (t == 0) {
      a.Cnew[i] = community_of_self<ALGO>(a, i);
      cflag[m] = 2;
    }
    return;
  }
  if (t == 0) flag_any = 0;
  __syncthreads();
  bool f = false;
  for (int64_t q = t; q < nc; q += BLOCK) f |= skflag[cb + q] != 0;
  if (f) flag_any = 1;
  bool lossy = tree_reduce<K>(sk, cb, nc, lds);
  lossy |= flag_any != 0;  // settled by the barriers inside tree_reduce
  if (lossy && second_pass(a, ALGO)) {
    if (t < K) cand[(int64_t)m * K + t] = lds[t];
    if (t == 0) cflag[m] = 1;
    return;
  }
  if (t == 0) {
    cflag[m] = 0;
    uint32_t key[K], ex[K];
#pragma unroll
    for (int p = 0; p < K; ++p) {
      const Pair x = lds[p];
      key[p] = x.val > 0 ? x.key : EMPTY;
      ex[p] = x.val;
    }
    const int32_t d = community_of_self<ALGO>(a, i);
    uint32_t kd = 0;
#pragma unroll
    for (int p = 0; p < K; ++p) kd += key[p] == (uint32_t)d ? ex[p] : 0u;
    decide_long<K, ALGO>(a, i, d, key, ex, kd);
  }
}

// part[q * (K + 1) + p] = weight of chunk q's entries with key cand[p];
// part[q * (K + 1) + K] = weight of those in the row's own community.
template <int K, int ALGO>
__global__ void __launch_bounds__(BLOCK)
    k_long_count(SweepArgs a, const int32_t *__restrict__ multi, const int32_t *__restrict__ owner,
                 const int64_t *__restrict__ cstart, int64_t nchunks, int64_t L, int64_t block0,
                 const Pair *__restrict__ cand, const uint32_t *__restrict__ cflag,
                 const uint32_t *__restrict__ keybuf, uint32_t *part) {
  if (level_over(a)) return;  // batched: every graph has stopped
  const int64_t q = ((block0 + blockIdx.x) * BLOCK + threadIdx.x) / WAVE;  // wave-uniform
  if (q >= nchunks) return;
  const int32_t m = owner[q];
  if (cflag[m] != 1) return;
  const LongChunk c = long_chunk(a, multi, owner, cstart, q, nchunks, L);
  const int32_t d = community_of_self<ALGO>(a, c.i);
  uint32_t key[K], ex[K], kd = 0;
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const Pair x = cand[(int64_t)m * K + p];
    key[p] = x.val > 0 ? x.key : EMPTY;
    ex[p] = 0;
  }
  int64_t e = c.lo + lane_id();
  for (; e + 3 * WAVE < c.hi; e += 4 * WAVE) {
    uint32_t cc[4], w[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) cc[u] = __builtin_nontemporal_load(keybuf + e + u * WAVE);
#pragma unroll
    for (int u = 0; u < 4; ++u) w[u] = __builtin_nontemporal_load(a.g.w + e + u * WAVE);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
#pragma unroll
      for (int p = 0; p < K; ++p) ex[p] += key[p] == cc[u] ? w[u] : 0u;
      kd += cc[u] == (uint32_t)d ? w[u] : 0u;
    }
  }
  for (; e < c.hi; e += WAVE) {
    const uint32_t cc = keybuf[e], w = a.g.w[e];
#pragma unroll
    for (int p = 0; p < K; ++p) ex[p] += key[p] == cc ? w : 0u;
    kd += cc == (uint32_t)d ? w : 0u;
  }
#pragma unroll
  for (int p = 0; p < K; ++p) ex[p] = wave_sum(ex[p]);
  kd = wave_sum(kd);
  const int l = lane_id();
  uint32_t mine = kd;
#pragma unroll
  for (int p = 0; p < K; ++p) mine = l == p ? ex[p] : mine;
  if (l <= K) part[q * (K + 1) + l] = mine;
}

template <int K, int ALGO>
__global__ void __launch_bounds__(BLOCK)
    k_long_decide(SweepArgs a, const int32_t *__restrict__ multi, const int64_t *__restrict__ cstart,
                  int64_t block0, const Pair *__restrict__ cand, const uint32_t *__restrict__ cflag,
                  const uint32_t *__restrict__ part) {
  if (level_over(a)) return;  // batched: every graph has stopped
  __shared__ uint32_t red[K + 1][BLOCK / WAVE];
  const int32_t m = (int32_t)(block0 + blockIdx.x);
  if (cflag[m] != 1) return;  // block-uniform
  const int t = threadIdx.x;
  const int64_t cb = cstart[m], ce = cstart[m + 1];
  uint32_t sum[K + 1];
#pragma unroll
  for (int p = 0; p <= K; ++p) sum[p] = 0;
  for (int64_t q = cb + t; q < ce; q += BLOCK) {
#pragma unroll
    for (int p = 0; p <= K; ++p) sum[p] += part[q * (K + 1) + p];
  }
#pragma unroll
  for (int p = 0; p <= K; ++p) {
    const uint32_t v = wave_sum(sum[p]);
    if (lane_id() == 0) red[p][t / WAVE] = v;
  }
  __syncthreads();
  if (t != 0) return;
  const int32_t i = multi[m];
  uint32_t key[K], ex[K];
#pragma unroll
  for (int p = 0; p < K; ++p) {
    const Pair x = cand[(int64_t)m * K + p];
    key[p] = x.val > 0 ? x.key : EMPTY;
    ex[p] = red[p][0] + red[p][1] + red[p][2] + red[p][3];
  }
  const uint32_t kd = red[K][0] + red[K][1] + red[K][2] + red[K][3];
  decide_long<K, ALGO>(a, i, community_of_self<ALGO>(a, i), key, ex, kd);
}

// ---- MG: 64 chunks per workgroup, four lanes per chunk ---------------------------------

// A workgroup takes 64 chunks, each a quad of lanes (quad_sketch.hpp): an aligned group
// of 64 chunks of a long row (more than 64 chunks), or 64 / P rows of a bucket of P = 2^b
// chunks each (P >= the row's chunk count; b = 0 for rows of one chunk).  The chunks go
// to the quads in order of length, so that a wave's 16 quads end together.
//   stage   windows of CAP entries per chunk: each wave loads those of its 16 chunks with
//           128-bit loads, gathers the keys C[j] (with Algorithm 1's skips) and keeps keys
//           and weights in LDS; the next window's loads are in flight during the fold;
//   fold    every quad runs Algorithm 1 over its chunk from LDS;
//   merge   the fixed tree over the chunk sketches of a row, in LDS, a quad per merge;
//   pass 2  only rows whose sketch lost weight: every lane counts a quarter of its
//           chunk's entries against the row's candidates, from LDS where the chunk had
//           one window, else from the key stream that staging wrote;
//   decide  lane r of the first wave decides row r.
// Rows of more than 64 chunks continue after the sweep kernel:
//   k_long_merge   one workgroup per row: the rest of the fixed merge tree over its
//                  group roots; a row whose sketch lost no weight is decided here;
//   k_long_count   one wave per chunk of a lossy row: pass 2 against the row's
//                  candidates, partial counts per chunk;
//   k_long_decide  one workgroup per lossy row: sum the partial counts, decide.
//
// Why this split.  With one lane per chunk (all slots in its registers) a level-0 sweep of
// R-MAT 2^20 (31.4 M entries, k = 8) took 473 us, waves waiting most of the time: 16 waves
// per CU, rows read twice over (a row's 64-byte pieces came back after its lines had left
// the L2: 1.7 GB for 0.6), and on small levels one wave's serial chain was the launch (80 to
// 170 us for a few hundred rows at k = 16).  A quad per chunk takes 312 us there, 438 us
// against 564 for a Chung-Lu graph of 27 M entries at k = 16, and a Leiden run's sweeps
// on Chung-Lu 2^22 18.5 ms against 38.8.  It is bound by VALU issue (77 % in a first sweep,
// which reads no labels, 108 M wave instructions on R-MAT 2^20) and, in the other sweeps,
// by the label gathers (about 100 us of them there).  Sorting the chunks by length inside
// the workgroup and merging in LDS takes a quarter of the instructions out.  Measured and
// not taken: CAP = 128 with pass 2 from LDS alone (two workgroups per CU: 350 + 63 us, the
// light rows in a second launch), and whole chunks in registers (27 KB of unrolled fold:
// 348 + 75 us, k = 16 spills).
constexpr int WCH = 64;  // chunks per workgroup
constexpr int CAP = 32;  // staged entries per chunk: six workgroups per CU (five at K = 16)

template <int K>
struct RowShare {
  // rows of CAP + 4 words: the 16 quads of a wave read 128 bits each from distinct banks
  __attribute__((aligned(16))) uint32_t key[WCH][CAP + 4];  // by quad: its chunk's staged
  __attribute__((aligned(16))) uint32_t wt[WCH][CAP + 4];   // keys and weights
  uint32_t sk[WCH][K + 1], sv[WCH][K + 1];   // by chunk: candidates and weights; [K]: K_{i->d}
  int64_t lo[WCH], hi[WCH];                  // by quad: its chunk's entries,
  int32_t row[WCH], bnd[WCH], chunk[WCH];    // its row, the row's bound, the chunk
  int32_t nch[WCH], lead[WCH];               // by chunk: chunks of its row here, the row if
                                             // this is its first chunk, else -1; of the row:
  uint32_t own[WCH], ki[WCH], sd[WCH];       // its community, K_i, Sigma of its community,
  uint32_t need[WCH], lossy[WCH];            // needs pass 2, lost weight
  uint32_t any;                              // some row needs pass 2
  uint32_t live;                             // some chunk has entries (of a row that may move)
  int64_t item;                              // persistent: next work item
};

// A window: positions s0 .. s0 + CAP - 1 of this wave's 16 chunks, LPC lanes (four
// entries each) per chunk, CPR chunks per round of loads.
constexpr int LPC = CAP / 4, CPR = WAVE / LPC, ROUNDS = WCH / 4 / CPR;

template <int K>
__device__ MGCD_INLINE void load_window(const SweepArgs &a, const RowShare<K> &S, int64_t s0, v4u (&jj)[ROUNDS],
                                        v4u (&ww)[ROUNDS]) {
  const int lane = lane_id(), c0 = (threadIdx.x / WAVE) * (WCH / 4) + lane / LPC;
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t e = S.lo[c0 + r * CPR] + s0 + 4 * (lane % LPC);
    const bool on = e < S.hi[c0 + r * CPR];
    jj[r] = load4(reinterpret_cast<const uint32_t *>(a.g.idx), e, a.g.nnz, on);
    ww[r] = load4(a.g.w, e, a.g.nnz, on);
  }
}

// The loaded window into LDS: the key C[j] (refinement: j inside the row's bound) and the
// weight, (EMPTY, 0) for skipped entries and past a chunk's end.  keyout: the keys also
// go to the key stream.
template <int K, int ALGO>
__device__ MGCD_INLINE void stage_window(const SweepArgs &a, RowShare<K> &S, int64_t s0, v4u (&jj)[ROUNDS],
                                         const v4u (&ww)[ROUNDS], uint32_t *keyout) {
  const int lane = lane_id(), l = lane % LPC, c0 = (threadIdx.x / WAVE) * (WCH / 4) + lane / LPC;
  // Every gather is issued on every lane with a valid index (0 where there is no entry)
  // and masked with an OR afterwards, so that all of them are in flight together.
  v4u kk[ROUNDS];
  int left[ROUNDS];  // entries of the chunk from this lane's first on, at most 4 matter
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int64_t n = S.hi[c0 + r * CPR] - (S.lo[c0 + r * CPR] + s0 + 4 * l);
    left[r] = n > 4 ? 4 : (int)n;
#pragma unroll
    for (int u = 0; u < 4; ++u) jj[r][u] = u < left[r] ? jj[r][u] : 0u;
  }
  if (ALGO == ALGO_REFINE) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
      for (int u = 0; u < 4; ++u) kk[r][u] = (uint32_t)a.bound[(int32_t)jj[r][u]];
  } else if (!a.ident) {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
      for (int u = 0; u < 4; ++u) kk[r][u] = (uint32_t)a.C[(int32_t)jj[r][u]];
  } else {
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) kk[r] = jj[r];
  }
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r) {
    const int c = c0 + r * CPR;
    const uint32_t i = (uint32_t)S.row[c], b = (uint32_t)S.bnd[c];
    v4u k, w;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const bool skip = u >= left[r] || jj[r][u] == i || (ALGO == ALGO_REFINE && kk[r][u] != b);
      k[u] = (ALGO == ALGO_REFINE ? jj[r][u] : kk[r][u]) | (skip ? EMPTY : 0u);
      w[u] = skip ? 0u : ww[r][u];
    }
    *reinterpret_cast<v4u *>(&S.key[c][4 * l]) = k;
    *reinterpret_cast<v4u *>(&S.wt[c][4 * l]) = w;
    if (keyout && left[r] > 0) {
      typedef uint32_t v4a __attribute__((ext_vector_type(4), aligned(4)));
      uint32_t *o = keyout + S.lo[c] + s0 + 4 * l;
      if (left[r] == 4) {
        *reinterpret_cast<v4a *>(o) = k;
      } else {
#pragma unroll
        for (int u = 0; u < 3; ++u)
          if (u < left[r]) o[u] = k[u];
      }
    }
  }
}

// The longest chunk of this wave's 16 (this lane's quad has len entries).
__device__ inline int64_t wave_max_chunk(int64_t len) {
#pragma unroll
  for (int o = QUAD; o < WAVE; o <<= 1) {
    const int64_t x = __shfl_xor(len, o);
    len = x > len ? x : len;
  }
  return uniform(len);
}

// Work item w: the first bk.ngroups are the groups of long rows, then the buckets' rows
// from b = 6 down to b = 0.  Block-uniform.  ct: the counts of the row decided by this
// thread (first wave).
template <int K, int ALGO, int MODE>
__device__ MGCD_INLINE void row_item(const SweepArgs &a, const Buckets &bk, int64_t L, uint32_t *keybuf,
                                RowShare<K> &S, int64_t w, Counters &ct) {
  constexpr int SL = QuadSketch<K, MODE>::S;
  const int t = threadIdx.x;
  const int c = t / QUAD, ql = t % QUAD;  // this lane's quad and its place there
  const bool group = w < bk.ngroups;
  int logp = 0;
  int64_t wb = w;
  if (group) {
    logp = 6;
  } else {
    wb = w - bk.ngroups;
    logp = 6;
    while (logp > 0 && wb >= bk.item_end[logp]) --logp;
    wb -= bk.item_begin[logp];
  }
  const int P = 1 << logp;
  // the first wave describes the 64 chunks and reads early what the rows' decisions need
  if (t < WCH) {
    int64_t lo = 0, hi = 0, nc = 0;
    int32_t i = 0, d = 0, b = 0;
    uint32_t Ki = 0, Sd = 0;
    bool lead = false;
    if (group) {
      const int32_t m = bk.gowner[w];
      const int64_t base = (w - bk.gstart[m]) * WCH;  // the group's first chunk in the row
      i = bk.multi[m];
      if (!frozen(a, i)) {
        nc = bk.cstart[m + 1] - bk.cstart[m] - base;
        nc = nc < WCH ? nc : WCH;
        const int64_t rhi = a.g.off[i + 1];
        lo = a.g.off[i] + (base + t) * L;
        hi = t < nc ? (lo + L < rhi ? lo + L : rhi) : lo;
        if (ALGO == ALGO_REFINE) b = a.bound[i];
      }
    } else {
      const int q = t & (P - 1);
      const int64_t r = wb * (WCH >> logp) + (t >> logp);
      const bool listed = r < bk.nrows[logp];
      i = listed ? bk.rows[logp][r] : 0;
      if (listed) {
        if (frozen(a, i)) {
          if (q == 0) a.Cnew[i] = community_of_self<ALGO>(a, i);
        } else {
          const int64_t rlo = a.g.off[i], rhi = a.g.off[i + 1];
          nc = (rhi - rlo + L - 1) / L;
          lo = rlo + q * L;
          hi = q < nc ? (lo + L < rhi ? lo + L : rhi) : lo;
          if (ALGO == ALGO_REFINE) b = a.bound[i];
          d = community_of_self<ALGO>(a, i);
          lead = q == 0;
          if (lead && ALGO != ALGO_LPA) {
            Ki = a.K[i];
            Sd = a.Sig[d];
          }
        }
      }
    }
    // longest chunks to the first quads, to within an eighth of 32, 64 or 128 entries
    const int n = hi - lo > 128 ? 128 : (int)(hi - lo);
    const int sh = __ballot(n > 64) ? 4 : __ballot(n > 32) ? 3 : 2;
    const int bin = (n + (1 << sh) - 1) >> sh;
    int slot = 0, base = 0;
#pragma unroll
    for (int v = 8; v >= 0; --v) {
      const uint64_t m = __ballot(bin == v);
      slot = bin == v ? base + (int)__popcll(m & lanemask_lt()) : slot;
      base += (int)__popcll(m);
    }
    S.lo[slot] = lo;
    S.hi[slot] = hi;
    S.row[slot] = i;
    S.bnd[slot] = b;
    S.chunk[slot] = t;
    S.nch[t] = (int32_t)nc;
    S.lead[t] = lead ? i : -1;
    S.ki[t] = Ki;
    S.sd[t] = Sd;
    S.own[t] = (uint32_t)d;
    S.need[t] = 0;
    S.lossy[t] = 0;
    const bool live = __ballot(hi > lo) != 0;
    if (t == 0) {
      S.any = 0;
      S.live = live;
    }
  }
  __syncthreads();
  if (!S.live) return;  // rows that stay where they are: their labels are copied above
  const int64_t clo = S.lo[c], chi = S.hi[c], len = chi - clo;
  const int ch = S.chunk[c];
  const int64_t maxlen = wave_max_chunk(len);
  QuadSketch<K, MODE> s;
  s.reset();
  const bool windows = maxlen > CAP;  // wave-uniform: pass 2 reads the key stream
  uint32_t *const keyout = group || windows ? keybuf : nullptr;
  v4u jj[ROUNDS], ww[ROUNDS];
  load_window(a, S, 0, jj, ww);
  for (int64_t s0 = 0; s0 < maxlen; s0 += CAP) {
    stage_window<K, ALGO>(a, S, s0, jj, ww, keyout);
    wave_sync();
    if (s0 + CAP < maxlen) load_window(a, S, s0 + CAP, jj, ww);  // in flight during the fold
    const int n = (int)(maxlen - s0 < CAP ? maxlen - s0 : CAP);
#pragma unroll 2
    for (int e = 0; e < n; e += 4) {
      const v4u k = *reinterpret_cast<const v4u *>(&S.key[c][e]);
      const v4u x = *reinterpret_cast<const v4u *>(&S.wt[c][e]);
#pragma unroll
      for (int u = 0; u < 4; ++u) s.update(k[u], x[u]);
    }
    wave_sync();
  }
  s.finalize();
  const bool merged = logp > 0;  // block-uniform
  const bool lost = quad_or(s.lost) != 0;
  bool need = lost && second_pass(a, ALGO);
  if (merged) {
    if (lost) S.lossy[ch & ~(P - 1)] = 1;
  } else if (need && ql == 0) {
    S.need[ch] = 1;
  }
  if (merged || !need) {
#pragma unroll
    for (int p = 0; p < SL; ++p) {
      if (p * QUAD + ql < K) {
        S.sk[ch][p * QUAD + ql] = s.key[p];
        S.sv[ch][p * QUAD + ql] = s.val[p];
      }
    }
  }
  if (merged) {
    __syncthreads();
    // level l: node x (a multiple of 2^(l+1) chunks) takes in node x + 2^l if the row has
    // it, a quad per merge: the first two waves for level 0, the first for the others
#pragma unroll 1
    for (int l = 0; l < logp; ++l) {
      if (t < WAVE * (l == 0 ? 2 : 1)) {
        const int x = c << (l + 1);
        if (x < WCH && ((x & (P - 1)) >> l) + 1 < ((S.nch[x] + (1 << l) - 1) >> l)) {
          const int y = x + (1 << l);
          uint32_t bk_[SL], bv_[SL];
#pragma unroll
          for (int p = 0; p < SL; ++p) {
            const bool h = p * QUAD + ql < K;
            s.key[p] = h ? S.sk[x][p * QUAD + ql] : EMPTY;
            s.val[p] = h ? S.sv[x][p * QUAD + ql] : 0u;
            bk_[p] = h ? S.sk[y][p * QUAD + ql] : EMPTY;
            bv_[p] = h ? S.sv[y][p * QUAD + ql] : 0u;
          }
          s.lost = 0;
          s.merge(bk_, bv_);
#pragma unroll
          for (int p = 0; p < SL; ++p) {
            if (p * QUAD + ql < K) {
              S.sk[x][p * QUAD + ql] = s.key[p];
              S.sv[x][p * QUAD + ql] = s.val[p];
            }
          }
          if (s.lost) S.lossy[x & ~(P - 1)] = 1;
        }
        wave_sync();
      }
      if (l == 0) __syncthreads();
    }
    if (group) {
      if (t < K) bk.sk[w * K + t] = Pair{S.sk[0][t], S.sv[0][t]};
      if (t == 0) bk.skflag[w] = S.lossy[0];
      return;
    }
    if (t < WCH && S.lead[t] >= 0 && S.lossy[t] && second_pass(a, ALGO)) {
      S.need[t] = 1;
      S.any = 1;
#pragma unroll
      for (int p = 0; p <= K; ++p) S.sv[t][p] = 0;  // pass 2 counts here
    }
    __syncthreads();
  }
  if (!merged || S.any) {
    const int lc = ch & ~(P - 1);  // the row's first chunk
    if (merged) need = S.need[lc] != 0;
    const int64_t maxlen2 = wave_max_chunk(need ? len : 0);
    if (maxlen2 > 0) {
      uint32_t ck[K], cx[K], kd = 0;
      const uint32_t dk = S.own[lc];
      if (merged) {
#pragma unroll
        for (int p = 0; p < K; ++p) ck[p] = S.sk[lc][p];
      } else {  // the quad's own slots
#pragma unroll
        for (int p = 0; p < K; ++p) {
          const uint32_t x = s.key[p / QUAD];
          ck[p] = p % QUAD == 0 ? quad_bcast<0>(x) : p % QUAD == 1 ? quad_bcast<1>(x)
                  : p % QUAD == 2 ? quad_bcast<2>(x) : quad_bcast<3>(x);
        }
      }
#pragma unroll
      for (int p = 0; p < K; ++p) cx[p] = 0;
      if (windows) __threadfence_block();  // the wave's key stream entries are written
      for (int64_t e = QUAD * ql; e < maxlen2; e += QUAD * QUAD) {
        v4u k, x;
        if (!windows) {
          k = *reinterpret_cast<const v4u *>(&S.key[c][e]);
          x = *reinterpret_cast<const v4u *>(&S.wt[c][e]);
        } else {
          const bool on = need && e < len;
          k = load4(keybuf, clo + e, a.g.nnz, on);
          x = load4(a.g.w, clo + e, a.g.nnz, on);
#pragma unroll
          for (int u = 0; u < 4; ++u) x[u] = on && e + u < len && k[u] != EMPTY ? x[u] : 0u;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
          for (int p = 0; p < K; ++p) cx[p] += ck[p] == k[u] ? x[u] : 0u;
          kd += k[u] == dk ? x[u] : 0u;
        }
      }
      kd = quad_sum(kd);
#pragma unroll
      for (int p = 0; p < K; ++p) cx[p] = quad_sum(cx[p]);
      if (need && merged) {
#pragma unroll
        for (int p = 0; p < K; ++p)
          if (ql == p % QUAD && cx[p]) atomicAdd(&S.sv[lc][p], cx[p]);
        if (ql == 0 && kd) atomicAdd(&S.sv[lc][K], kd);
      } else if (need) {
#pragma unroll
        for (int p = 0; p < K; ++p) {
          if (ql == p % QUAD) {
            S.sk[ch][p] = ck[p];
            S.sv[ch][p] = cx[p];
          }
        }
        if (ql == 0) S.sv[ch][K] = kd;
      }
    }
    __syncthreads();
  }
  if (t < WCH && S.lead[t] >= 0) {
    const int32_t i = S.lead[t], d = (int32_t)S.own[t];
    uint32_t key[K], ex[K];
#pragma unroll
    for (int p = 0; p < K; ++p) {
      key[p] = S.sk[t][p];
      ex[p] = S.sv[t][p];
    }
    uint32_t kd = 0;
    if (S.need[t]) {
      kd = S.sv[t][K];
    } else {
#pragma unroll
      for (int p = 0; p < K; ++p) kd += key[p] == (uint32_t)d ? ex[p] : 0u;
    }
    int32_t best = -1;
    int64_t bestG = 0;
    const int64_t W = ALGO == ALGO_LPA ? 0 : (int64_t)weight_of(a, i);
    ct.cand += consider_slots<K, ALGO>(a, W, d, S.ki[t], S.sd[t], kd, key, ex, best, bestG);
    finish<ALGO>(a, i, d, best, bestG, ct);
  }
}

// ---- MG: light rows, a quad of lanes per row ---------------------------------------------

// Rows of one chunk with at most LIGHT_MAX entries, 16 per wave and nothing shared between
// waves: a lane loads a quarter of its row with 128-bit loads and keeps keys and weights
// in registers; every entry is broadcast to the quad by DPP moves for Algorithm 1 and, if
// the sketch lost weight, again for pass 2, in which each lane counts its own slots; the
// decision, too, is spread over the quad's slots.  No LDS and 47 VGPRs at k = 8: eight
// waves per SIMD.  192 planted graphs (2.5 M rows of about 16 entries) in one batch: 381 us
// per sweep, 728 us with a lane per row, 418 us in the workgroup form above; LPA on one
// planted graph of 10,000 vertices (one wave's latency): 6.5 us per sweep, 15.8 before.
// Bound by VALU issue (72 % on R-MAT 2^20's light rows), then latency.
constexpr int LIGHT_R = LIGHT_MAX / 16;  // 128-bit loads per lane

// The best of a quad's candidates (this lane's slots key, ex): the rule of consider_slots.
// Every lane of the quad returns the best; the result is the number of this lane's
// candidates whose totals were read.
template <int K, int ALGO, int S>
__device__ MGCD_INLINE int consider_quad(const SweepArgs &a, int64_t W, int32_t d, int64_t Ki, int64_t Sd,
                                         uint32_t kd, const uint32_t (&key)[S], const uint32_t (&ex)[S],
                                         int32_t &best, int64_t &bestG) {
  const uint32_t ud = (uint32_t)d;
  int reads = 0;
  if constexpr (ALGO == ALGO_LPA) {
#pragma unroll
    for (int p = 0; p < S; ++p)
      consider_v<ALGO>(W, d, Ki, Sd, kd, (int32_t)key[p], ex[p], 0u, key[p] != EMPTY, best, bestG);
  } else {
    // the heaviest candidate other than d (ties: the lowest slot) is scored first
    uint32_t x0 = 0;
#pragma unroll
    for (int p = 0; p < S; ++p) x0 = key[p] != EMPTY && key[p] != ud ? umax(x0, ex[p]) : x0;
    x0 = quad_max(x0);
    uint32_t f = 255;
#pragma unroll
    for (int p = S - 1; p >= 0; --p)
      f = key[p] != EMPTY && key[p] != ud && ex[p] == x0 ? (uint32_t)(p * QUAD + lane_id() % QUAD) : f;
    const uint32_t f0 = quad_min(f);
    const bool mine = f == f0 && f0 != 255;
    uint32_t c0 = 0;
#pragma unroll
    for (int p = 0; p < S; ++p) c0 = f == (uint32_t)(p * QUAD + lane_id() % QUAD) ? key[p] : c0;
    c0 = quad_or(mine ? c0 : 0u);  // one lane has it
    const bool any = f0 != 255;
    const uint32_t s0 = a.Sig[any ? (int32_t)c0 : d];
    consider_v<ALGO>(W, d, Ki, Sd, kd, (int32_t)c0, x0, s0, any, best, bestG);
    reads = mine;
    const int64_t own = mul32(Ki, Sd - Ki);  // U(c) = W (k_c - k_d) + K_i (Sigma_d - K_i)
    bool live[S];
    uint32_t sc[S];
#pragma unroll
    for (int p = 0; p < S; ++p) {
      const int64_t U = mul32(W, (int64_t)ex[p] - (int64_t)kd) + own;
      const int32_t c = (int32_t)key[p];
      live[p] = key[p] != EMPTY && key[p] != ud && !(any && key[p] == c0) && U > 0 &&
                (best < 0 || U > bestG || (U == bestG && c < best));
      sc[p] = a.Sig[live[p] ? c : d];
    }
#pragma unroll
    for (int p = 0; p < S; ++p) {
      consider_v<ALGO>(W, d, Ki, Sd, kd, (int32_t)key[p], ex[p], sc[p], live[p], best, bestG);
      reads += live[p];
    }
  }
  // the quad's best: larger gain first, then the lower id
#pragma unroll
  for (int o = 0; o < 2; ++o) {
    uint32_t lo = (uint32_t)bestG, hi = (uint32_t)((uint64_t)bestG >> 32), c = (uint32_t)best;
    lo = o ? quad_perm<QP_XOR2>(lo) : quad_perm<QP_XOR1>(lo);
    hi = o ? quad_perm<QP_XOR2>(hi) : quad_perm<QP_XOR1>(hi);
    const int32_t c2 = (int32_t)(o ? quad_perm<QP_XOR2>(c) : quad_perm<QP_XOR1>(c));
    const int64_t g2 = (int64_t)(((uint64_t)hi << 32) | lo);
    const bool take = c2 >= 0 && (best < 0 || g2 > bestG || (g2 == bestG && c2 < best));
    best = take ? c2 : best;
    bestG = take ? g2 : bestG;
  }
  return reads;
}

// Positions 16 r .. n - 1 (n wave-uniform) of the quads' rows, each broadcast in order.
template <int R, int r = 0, typename F>
__device__ MGCD_INLINE void each_entry(int n, const uint32_t (&kk)[R][4], const uint32_t (&ww)[R][4], F &&f) {
  if constexpr (r < R) {
    if (16 * r >= n) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) f(quad_bcast<0>(kk[r][u]), quad_bcast<0>(ww[r][u]));
    if (16 * r + 4 >= n) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) f(quad_bcast<1>(kk[r][u]), quad_bcast<1>(ww[r][u]));
    if (16 * r + 8 >= n) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) f(quad_bcast<2>(kk[r][u]), quad_bcast<2>(ww[r][u]));
    if (16 * r + 12 >= n) return;
#pragma unroll
    for (int u = 0; u < 4; ++u) f(quad_bcast<3>(kk[r][u]), quad_bcast<3>(ww[r][u]));
    each_entry<R, r + 1>(n, kk, ww, f);
  }
}

// Work item w: rows 16 w .. 16 w + 15 of the list, one wave.
template <int K, int ALGO, int MODE>
__device__ MGCD_INLINE void light_item(const SweepArgs &a, const int32_t *rows, int64_t nrows, int64_t w,
                                       Counters &ct) {
  constexpr int R = LIGHT_R, SL = QuadSketch<K, MODE>::S;
  const int lane = lane_id(), ql = lane % QUAD;
  const int64_t r = w * (WAVE / QUAD) + lane / QUAD;
  const bool listed = r < nrows;
  const int32_t i = listed ? rows[r] : 0;
  // the row's bounds are read before it is known whether its graph still moves, the rest
  // after that: a wave of rows that stay where they are copies their labels and is done
  const int64_t rlo = a.g.off[i], rhi = a.g.off[i + 1];
  const int32_t d = community_of_self<ALGO>(a, i);
  const int32_t g = a.gid ? a.gid[i] : 0;
  const bool valid = listed && !(a.halt && *a.halt) && !(a.gid && !a.active[g]);
  if (listed && !valid && ql == 0) a.Cnew[i] = d;
  if (!__ballot(valid)) return;
  const uint32_t Ki = ALGO == ALGO_LPA ? 0u : a.K[i];
  const int32_t b = ALGO == ALGO_REFINE ? a.bound[i] : 0;
  const uint32_t Sd = ALGO == ALGO_LPA ? 0u : a.Sig[d];
  const int64_t W = ALGO == ALGO_LPA ? 0 : a.gid ? (int64_t)a.Wg[g] : (int64_t)a.W;
  const int64_t lo = valid ? rlo : 0, hi = valid ? rhi : 0;
  // this lane's entries lo + 16 x + 4 ql + u
  uint32_t kk[R][4], ww[R][4];
  const int left = (int)(hi - lo) - 4 * ql;
  const int64_t e = lo + 4 * ql;
#pragma unroll
  for (int x = 0; x < R; ++x) {
    const v4u j = load4(reinterpret_cast<const uint32_t *>(a.g.idx), e + 16 * x, a.g.nnz, 16 * x < left);
    const v4u y = load4(a.g.w, e + 16 * x, a.g.nnz, 16 * x < left);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      kk[x][u] = 16 * x + u < left ? j[u] : 0u;  // a valid id: the gathers need no branch
      ww[x][u] = 16 * x + u < left && j[u] != (uint32_t)i ? y[u] : 0u;
    }
  }
  if (ALGO == ALGO_REFINE) {
    uint32_t bb[R][4];
#pragma unroll
    for (int x = 0; x < R; ++x)
#pragma unroll
      for (int u = 0; u < 4; ++u) bb[x][u] = (uint32_t)a.bound[(int32_t)kk[x][u]];
#pragma unroll
    for (int x = 0; x < R; ++x)
#pragma unroll
      for (int u = 0; u < 4; ++u) ww[x][u] = bb[x][u] == (uint32_t)b ? ww[x][u] : 0u;
  } else if (!a.ident) {
#pragma unroll
    for (int x = 0; x < R; ++x)
#pragma unroll
      for (int u = 0; u < 4; ++u) kk[x][u] = (uint32_t)a.C[(int32_t)kk[x][u]];
  }
  // real entries have weights above 0
#pragma unroll
  for (int x = 0; x < R; ++x)
#pragma unroll
    for (int u = 0; u < 4; ++u) kk[x][u] = ww[x][u] ? kk[x][u] : EMPTY;
  const int n = (int)wave_max_chunk(hi - lo);
  QuadSketch<K, MODE> s;
  s.reset();
  each_entry<R>(n, kk, ww, [&](uint32_t c, uint32_t x) MGCD_LAMBDA { s.update(c, x); });
  s.finalize();
  const bool need = quad_or(s.lost) != 0 && second_pass(a, ALGO);
  uint32_t kd = 0;
  if (__ballot(need)) {
    uint32_t cx[SL];
#pragma unroll
    for (int p = 0; p < SL; ++p) cx[p] = 0;
    each_entry<R>(n, kk, ww, [&](uint32_t c, uint32_t x) MGCD_LAMBDA {
#pragma unroll
      for (int p = 0; p < SL; ++p) cx[p] += s.key[p] == c ? x : 0u;
    });
#pragma unroll
    for (int p = 0; p < SL; ++p) s.val[p] = need ? cx[p] : s.val[p];
#pragma unroll
    for (int x = 0; x < R; ++x)
#pragma unroll
      for (int u = 0; u < 4; ++u) kd += kk[x][u] == (uint32_t)d ? ww[x][u] : 0u;
  }
  if (!need) {
    kd = 0;
#pragma unroll
    for (int p = 0; p < SL; ++p) kd += s.key[p] == (uint32_t)d ? s.val[p] : 0u;
  }
  kd = quad_sum(kd);
  if (valid) {
    int32_t best = -1;
    int64_t bestG = 0;
    const int reads = consider_quad<K, ALGO, SL>(a, W, d, Ki, Sd, kd, s.key, s.val, best, bestG);
    ct.cand += reads;
    if (ql == 0) finish<ALGO>(a, i, d, best, bestG, ct);
  }
}

template <int K>
constexpr int row_waves_per_simd() {  // = workgroups per CU: what LDS leaves room for
  return K >= 16 ? 5 : 6;
}
template <int K>
constexpr int light_waves_per_simd() {  // what registers leave room for
  return K >= 16 ? 6 : 8;
}

// The main sweep kernel: a workgroup per work item of the long and ordinary rows, then
// workgroups for the light rows, which fill the chip while the last heavy ones end.
// PERSIST (batched runs; no light rows): as many workgroups as stay resident take work
// items from their counter of the queue (the items of the grid's order whose index is
// c mod QLANES), QGRAB at a time, until none is left.
template <int K, int ALGO, int MODE, bool PERSIST>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(row_waves_per_simd<K>())))
    k_move_rows(SweepArgs a, const Buckets bk, int64_t L, uint32_t *keybuf, int64_t total, const int32_t *light,
                int64_t nlight, int64_t first, unsigned long long *queue) {
  if (level_over(a)) return;  // batched: every graph has stopped
  __shared__ RowShare<K> S;
  Counters ct;
  stamp_start(a, first);
  if constexpr (!PERSIST) {
    const int64_t block = first + blockIdx.x;
    if (block < total) {
      row_item<K, ALGO, MODE>(a, bk, L, keybuf, S, block, ct);
      if (threadIdx.x < WAVE) flush_wave_counters(a, ct);
    } else {
      const int64_t w = (block - total) * (BLOCK / WAVE) + threadIdx.x / WAVE;
      light_item<K, ALGO, MODE>(a, light, nlight, uniform(w), ct);
      flush_counters(a, ct);
    }
  } else {
    GraphCounts gc{-1, 0, 0, 0};
    const int64_t c = blockIdx.x % QLANES;
    unsigned long long *qc = queue + c * QSTRIDE;
    for (;;) {
      __syncthreads();  // the last item's shared state has been read
      if (threadIdx.x == 0) S.item = (int64_t)atomicAdd(qc, (unsigned long long)QGRAB);
      __syncthreads();
      const int64_t j = uniform(S.item);
      if (c + j * QLANES >= total) break;
#pragma unroll 1
      for (int r = 0; r < QGRAB; ++r) {
        const int64_t w = c + (j + r) * QLANES;  // block-uniform
        if (w >= total) break;
        if (r > 0) __syncthreads();
        row_item<K, ALGO, MODE>(a, bk, L, keybuf, S, w, ct);
        if (threadIdx.x < WAVE) gather_graph_counts(a, ct, gc);
      }
    }
    if (threadIdx.x == 0) commit_graph_counts(a, gc);
  }
}

// The light rows of a level that has no others, and of every level of a batch (its own kernel
// has a third more waves per SIMD than k_move_rows).  PERSIST as in k_move_rows, a wave
// taking the items.
template <int K, int ALGO, int MODE, bool PERSIST>
__global__ void __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(light_waves_per_simd<K>())))
    k_move_light(SweepArgs a, const int32_t *__restrict__ rows, int64_t nrows, int64_t first,
                 unsigned long long *queue) {
  if (level_over(a)) return;  // batched: every graph has stopped
  const int64_t wave = uniform(((first + blockIdx.x) * BLOCK + threadIdx.x) / WAVE);
  Counters ct;
  stamp_start(a, first);
  if constexpr (!PERSIST) {
    light_item<K, ALGO, MODE>(a, rows, nrows, wave, ct);
    flush_counters(a, ct);
  } else {
    GraphCounts gc{-1, 0, 0, 0};
    const int64_t total = (nrows + WAVE / QUAD - 1) / (WAVE / QUAD);
    const int64_t c = wave % QLANES;
    unsigned long long *qc = queue + c * QSTRIDE;
    for (;;) {
      unsigned long long j0 = 0;
      if (lane_id() == 0) j0 = atomicAdd(qc, (unsigned long long)1);
      // LGRAB neighbouring items: mostly rows of one graph, whose counts go out together
      const int64_t w0 = (c + uniform((int64_t)__shfl(j0, 0)) * QLANES) * LGRAB;
      if (w0 >= total) break;
#pragma unroll 1
      for (int r = 0; r < LGRAB && w0 + r < total; ++r) {
        light_item<K, ALGO, MODE>(a, rows, nrows, w0 + r, ct);
        gather_graph_counts(a, ct, gc);
      }
    }
    if (lane_id() == 0) commit_graph_counts(a, gc);
  }
}

// ---- MG with K = 32 or 64: one wave per row -------------------------------------------

// The load of wave_chunk for a row of the graph: the entry's key (written to the key
// stream) and weight.
template <int ALGO>
struct RowLoad {
  const SweepArgs &a;
  int32_t i, bi;
  uint32_t *keybuf;
  __device__ inline void operator()(int64_t e, bool in, uint32_t &key, uint32_t &w) const {
    const int32_t j = in ? __builtin_nontemporal_load(a.g.idx + e) : 0;
    w = in ? __builtin_nontemporal_load(a.g.w + e) : 0u;
    key = EMPTY;
    if (in) {
      key = stream_key<ALGO>(a, i, j, bi);
      keybuf[e] = key;
    }
  }
};

// Pass 2 in a wave's map: the candidates' cells, then positions e, e + step, .. below hi of
// the key stream, each item added to its candidate's cell; the result is this lane's part
// of the weight towards d.
template <int K>
__device__ inline void pass2_cells(WaveMap<K> map, const uint32_t (&ck)[WaveSlots<K>::S],
                                   uint32_t (&cell)[WaveSlots<K>::S]) {
  map.clear();
  bool fresh;
#pragma unroll
  for (int u = 0; u < WaveSlots<K>::S; ++u) cell[u] = ck[u] != EMPTY ? map.claim(ck[u], fresh) : 0u;
  wave_sync();
}

template <int K>
__device__ inline uint32_t pass2_items(const SweepArgs &a, WaveMap<K> map, int64_t e, int64_t hi, int step,
                                       const uint32_t *__restrict__ keybuf, uint32_t d) {
  uint32_t kd = 0;
  for (; e < hi; e += step) {
    const uint32_t key = __builtin_nontemporal_load(keybuf + e);
    const uint32_t w = __builtin_nontemporal_load(a.g.w + e);
    kd += key == d ? w : 0u;
    if (key != EMPTY) map.add_present(key, w);
  }
  return kd;
}

// Rows longer than 32 entries when K is 32 or 64 (shorter rows cannot lose weight
// under Algorithm 1 or the textbook rule and take the short rows' kernel).  One wave per
// row.  Pass 1: each chunk's sketch (wave_chunk, keys written to the key stream) goes into
// the fixed merge tree (WaveTree).  Pass 2 (lossy rows only): the key stream again, each
// item added to its candidate's cell.  Decision: every lane scores its candidate, a
// butterfly keeps the best (lowest id on ties), lane 0 records it.
// Bound by the latency of the fold's steps (LDS probes; item by item once a chunk has more
// than K keys).  R-MAT 2^18, K = 64, Leiden's 16 sweeps: 1258 us with an item-by-item fold
// of every entry and of pass 2, 524 us with the map (first sweeps 91 and 50 us).
template <int K, int ALGO, int MODE>
__global__ void __launch_bounds__(BLOCK)
    k_wave_rows(SweepArgs a, const int32_t *__restrict__ rows, int64_t nrows, int64_t L, int depth,
                int64_t block0, uint32_t *keybuf) {
  static_assert(K <= WAVE, "one slot per lane; larger sketches take the split rows");
  if (level_over(a)) return;  // batched: every graph has stopped
  extern __shared__ uint32_t wave_lds[];
  const int lane = lane_id();
  const int64_t r = uniform(((block0 + blockIdx.x) * BLOCK + threadIdx.x) / WAVE);
  Counters ct;
  const bool listed = r < nrows;
  const int32_t i = listed ? uniform(rows[r]) : 0;
  const bool valid = listed && !frozen(a, i);
  if (listed && !valid && lane == 0) a.Cnew[i] = community_of_self<ALGO>(a, i);
  if (valid) {
    const int64_t lo = uniform(a.g.off[i]), hi = uniform(a.g.off[i + 1]);
    const int32_t bi = ALGO == ALGO_REFINE ? uniform(a.bound[i]) : 0;
    const int32_t d = uniform(community_of_self<ALGO>(a, i));
    const RowLoad<ALGO> load{a, i, bi, keybuf};
    const int wave = uniform((int32_t)(threadIdx.x / WAVE));
    WaveTree<K> tree(wave_lds + wave * (WaveMap<K>::WORDS + depth * 2 * WAVE), depth);
    uint32_t ck[1], cv[1];
    bool lossy = false;
    if (hi - lo <= L) {
      lossy = wave_chunk<K, MODE>(tree.map, lo, hi, load, ck, cv);
    } else {
      for (int64_t c0 = lo; c0 < hi; c0 += L) {
        lossy |= wave_chunk<K, MODE>(tree.map, c0, hi - c0 < L ? hi : c0 + L, load, ck, cv);
        tree.push(ck, cv);
      }
      tree.result(ck, cv);
      lossy |= tree.lossy;
    }
    uint32_t kd = 0;
    if (!lossy || !second_pass(a, ALGO)) {
      kd = ck[0] == (uint32_t)d ? cv[0] : 0u;
    } else {
      uint32_t cell[1];
      pass2_cells<K>(tree.map, ck, cell);
      kd = pass2_items<K>(a, tree.map, lo + lane, hi, WAVE, keybuf, (uint32_t)d);
      wave_sync();
      cv[0] = ck[0] != EMPTY ? tree.map.val[cell[0]] : 0u;
    }
    kd = wave_sum(kd);
    int32_t best = -1;
    int64_t bestG = 0;
    if (ck[0] != EMPTY) {
      const int64_t W = ALGO == ALGO_LPA ? 0 : (int64_t)weight_of(a, i);
      const int64_t Ki = ALGO == ALGO_LPA ? 0 : (int64_t)a.K[i];
      const int64_t Sd = ALGO == ALGO_LPA ? 0 : (int64_t)a.Sig[d];
      consider<ALGO>(a, W, d, Ki, Sd, kd, (int32_t)ck[0], cv[0], best, bestG);
    }
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
      const int32_t b2 = __shfl_xor(best, o);
      const int64_t g2 = __shfl_xor(bestG, o);
      if (b2 >= 0 && (best < 0 || g2 > bestG || (g2 == bestG && b2 < best))) {
        best = b2;
        bestG = g2;
      }
    }
    if (lane == 0) finish<ALGO>(a, i, d, best, bestG, ct);
  }
  flush_counters(a, ct);
}

// Rows of more than max(L, WAVE_SPLIT) entries when K is 32 or 64, and every row past the
// short ones when K is 128 or 256 ("split rows"): the same sketch, merge tree and decision
// as k_wave_rows, with the work spread over waves so that a hub row does not hold one wave
// for its whole length.
//   k_wave_chunks: one wave per chunk: its Algorithm 1 sketch (keys written to the key
//                  stream), finalised; the workgroup's chunks (eight neighbouring ones of a
//                  row) are merged into one node (merge_group);
//   k_wave_level:  one launch per tree level l: node x of a row (x a multiple of
//                  2^(l+1)) takes in node x + 2^l if that exists, left operand first,
//                  an odd last node is carried; after ceil(log2(nodes)) levels node 0
//                  is the root, the same tree as WaveTree;
//   k_wave_tree:   the levels at which every row has at most TREE_NODES nodes left, in one
//                  launch: one workgroup per row, a barrier between levels (both over the
//                  rows that may have more than one node; over all 4 M rows of a star at
//                  K = 256, all split, they took 9.2 ms of a sweep);
//   k_wave_count:  pass 2 of lossy rows, one workgroup per node's chunks (K = 128 / 256: one
//                  wave), integer sums added into the row's counts (order-independent);
//   k_wave_decide: one wave per row: scores and the decision, as in k_wave_rows.
// cstart and owner are those of the nodes.
// Bound as k_wave_rows by the latency of the fold.  R-MAT 2^18, K = 64, Leiden's 16 sweeps:
// chunks, levels and counts took 568, 1170 and 328 us; chunks (with their three levels),
// trees and counts now take 496, 120 and 145 us.
template <int K, int ALGO, int MODE>
__global__ void __launch_bounds__(wave_group_block(K))
    k_wave_chunks(SweepArgs a, const int32_t *__restrict__ rows, const int64_t *__restrict__ cstart,
                  const int32_t *__restrict__ owner, int64_t nnodes, int64_t L, uint32_t *keybuf,
                  int64_t block0, Pair *node, uint32_t *nflag, uint32_t *count) {
  if (level_over(a)) return;  // batched: every graph has stopped
  constexpr int S = WaveSlots<K>::S, G = wave_group(K), WAVES = wave_group_waves(K);
  __shared__ uint32_t smap[WAVES][WaveMap<K>::WORDS];
  const int lane = lane_id(), wave = uniform((int32_t)(threadIdx.x / WAVE));
  const int64_t q = G > 1 ? block0 + blockIdx.x : uniform((block0 + blockIdx.x) * WAVES + wave);
  if (q >= nnodes) return;
  const int32_t m = uniform(owner[q]);
  const int32_t i = uniform(rows[m]);
  const int64_t x = q - uniform(cstart[m]);  // node within the row
  if (x == 0) {  // the row's K + 1 pass-2 counts start at zero in every sweep
    uint32_t *cm = count + (int64_t)m * (K + 1);
    for (int p = G > 1 ? (int)threadIdx.x : lane; p <= K; p += G > 1 ? WAVES * WAVE : WAVE) cm[p] = 0u;
  }
  if (frozen(a, i)) return;
  const int64_t rhi = uniform(a.g.off[i + 1]), first = uniform(a.g.off[i]) + x * G * L;
  const int64_t lo = first + (G > 1 ? wave * L : 0);
  const int64_t hi = lo + L < rhi ? lo + L : rhi;
  const int32_t bi = ALGO == ALGO_REFINE ? uniform(a.bound[i]) : 0;
  const WaveMap<K> map(smap[wave]);
  uint32_t ck[S], cv[S];
  bool lossy = false;
  if (G == 1 || lo < hi)
    lossy = wave_chunk<K, MODE>(map, lo, hi, RowLoad<ALGO>{a, i, bi, keybuf}, ck, cv);
  if constexpr (G > 1) {
    __shared__ Pair snode[WAVES][K];
    __shared__ uint32_t sflag[WAVES];
    merge_group<K>(map, snode, sflag, wave, (rhi - first + L - 1) / L, ck, cv, lossy);
    if (wave != 0) return;
  }
#pragma unroll
  for (int r = 0; r < S; ++r)
    if (r * WAVE + lane < K) node[q * K + r * WAVE + lane] = Pair{ck[r], cv[r]};
  if (lane == 0) nflag[q] = lossy ? 1u : 0u;
}

template <int K>
__global__ void __launch_bounds__(BLOCK)
    k_wave_level(SweepArgs a, const int32_t *__restrict__ rows, const int64_t *__restrict__ cstart,
                 const int32_t *__restrict__ owner, int64_t nchunks, int level, int64_t block0, Pair *node,
                 uint32_t *nflag) {
  if (level_over(a)) return;  // batched: every graph has stopped
  __shared__ uint32_t smap[BLOCK / WAVE][WaveMap<K>::WORDS];
  const int64_t q = uniform(((block0 + blockIdx.x) * BLOCK + threadIdx.x) / WAVE);
  if (q >= nchunks) return;
  const int32_t m = uniform(owner[q]);
  const int64_t x = q - cstart[m], half = (int64_t)1 << level;
  if ((x & (2 * half - 1)) != 0) return;  // not a left node of this level
  const int64_t r = q + half;
  if (r >= cstart[m + 1]) return;  // odd last node: carried up
  if (frozen(a, rows[m])) return;
  const bool lossy = merge_nodes<K>(WaveMap<K>(smap[uniform((int32_t)(threadIdx.x / WAVE))]), node, q, r);
  if (lane_id() == 0) nflag[q] = nflag[q] | nflag[r] | (lossy ? 1u : 0u);
}

// Levels from `level` on of every split row, one workgroup each; see k_wave_chunks.
template <int K>
__global__ void __launch_bounds__(TREE_BLOCK)
    k_wave_tree(SweepArgs a, const int32_t *__restrict__ rows, const int64_t *__restrict__ cstart, int level,
                int64_t block0, Pair *node, uint32_t *nflag) {
  if (level_over(a)) return;  // batched: every graph has stopped
  __shared__ uint32_t smap[TREE_BLOCK / WAVE][WaveMap<K>::WORDS];
  const int64_t m = block0 + blockIdx.x;
  if (frozen(a, rows[m])) return;
  const int64_t q0 = cstart[m], n = cstart[m + 1] - q0;
  const int wave = uniform((int32_t)(threadIdx.x / WAVE));
  for (int64_t half = (int64_t)1 << level; half < n; half *= 2) {  // block-uniform
    for (int64_t x = wave * 2 * half; x + half < n; x += TREE_BLOCK / WAVE * 2 * half) {
      const int64_t q = q0 + x, r = q + half;
      const bool lossy = merge_nodes<K>(WaveMap<K>(smap[wave]), node, q, r);
      if (lane_id() == 0) nflag[q] = nflag[q] | nflag[r] | (lossy ? 1u : 0u);
    }
    __syncthreads();
  }
}

// The root of split row m: keys of positive slots, other slots EMPTY.
template <int K, int S = WaveSlots<K>::S>
__device__ inline void wave_root(const Pair *node, const int64_t *cstart, int32_t m, uint32_t (&ck)[S],
                                 uint32_t (&cv)[S]) {
  const int lane = lane_id();
#pragma unroll
  for (int u = 0; u < S; ++u) {
    ck[u] = EMPTY;
    cv[u] = 0;
    if (u * WAVE + lane < K) {
      const Pair p = node[cstart[m] * K + u * WAVE + lane];
      ck[u] = p.val > 0 ? p.key : EMPTY;
      cv[u] = p.val;
    }
  }
}

template <int K, int ALGO>
__global__ void __launch_bounds__(wave_group_block(K))
    k_wave_count(SweepArgs a, const int32_t *__restrict__ rows, const int64_t *__restrict__ cstart,
                 const int32_t *__restrict__ owner, int64_t nnodes, int64_t L, int64_t block0,
                 const uint32_t *__restrict__ keybuf, const Pair *__restrict__ node,
                 const uint32_t *__restrict__ nflag, uint32_t *count) {
  if (level_over(a)) return;  // batched: every graph has stopped
  constexpr int S = WaveSlots<K>::S, G = wave_group(K), WAVES = wave_group_waves(K);
  __shared__ uint32_t smap[G > 1 ? 1 : WAVES][WaveMap<K>::WORDS];
  __shared__ uint32_t skd;
  const int lane = lane_id(), wave = uniform((int32_t)(threadIdx.x / WAVE));
  const int64_t q = G > 1 ? block0 + blockIdx.x : uniform((block0 + blockIdx.x) * WAVES + wave);
  if (q >= nnodes) return;
  const int32_t m = uniform(owner[q]);
  const int32_t i = uniform(rows[m]);
  const int64_t q0 = uniform(cstart[m]);
  if (frozen(a, i) || !uniform(nflag[q0])) return;
  const int64_t rhi = uniform(a.g.off[i + 1]);
  const int64_t lo = uniform(a.g.off[i]) + (q - q0) * G * L;
  const int64_t hi = lo + G * L < rhi ? lo + G * L : rhi;
  const uint32_t d = (uint32_t)uniform(community_of_self<ALGO>(a, i));
  const WaveMap<K> map(smap[G > 1 ? 0 : wave]);  // the workgroup's (or wave's)
  uint32_t ck[S], cv[S], cell[S];
  wave_root<K>(node, cstart, m, ck, cv);
  if (G == 1 || wave == 0) pass2_cells<K>(map, ck, cell);
  if constexpr (G > 1) {
    if (threadIdx.x == 0) skd = 0;
    __syncthreads();
  }
  uint32_t kd;
  if constexpr (G > 1)
    kd = pass2_items<K>(a, map, lo + threadIdx.x, hi, WAVES * WAVE, keybuf, d);
  else
    kd = pass2_items<K>(a, map, lo + lane, hi, WAVE, keybuf, d);
  kd = wave_sum(kd);
  if constexpr (G > 1) {
    if (lane == 0 && kd) atomicAdd(&skd, kd);
    __syncthreads();
    if (wave != 0) return;
    kd = skd;
  } else {
    wave_sync();
  }
  uint32_t *cm = count + (int64_t)m * (K + 1);
#pragma unroll
  for (int u = 0; u < S; ++u) {
    if (ck[u] == EMPTY) continue;
    const uint32_t v = map.val[cell[u]];
    if (v) atomicAdd(&cm[u * WAVE + lane], v);
  }
  if (lane == 0 && kd) atomicAdd(&cm[K], kd);
}

template <int K, int ALGO>
__global__ void __launch_bounds__(BLOCK)
    k_wave_decide(SweepArgs a, const int32_t *__restrict__ rows, const int64_t *__restrict__ cstart,
                  int64_t nrows, int64_t block0, const Pair *__restrict__ node,
                  const uint32_t *__restrict__ nflag, const uint32_t *__restrict__ count) {
  if (level_over(a)) return;  // batched: every graph has stopped
  const int lane = lane_id();
  const int64_t m = uniform(((block0 + blockIdx.x) * BLOCK + threadIdx.x) / WAVE);
  Counters ct;
  if (m < nrows) {
    const int32_t i = uniform(rows[m]);
    if (frozen(a, i)) {
      if (lane == 0) a.Cnew[i] = community_of_self<ALGO>(a, i);
    } else {
      const int32_t d = uniform(community_of_self<ALGO>(a, i));
      constexpr int S = WaveSlots<K>::S;
      uint32_t ck[S], cv[S];
      wave_root<K>(node, cstart, (int32_t)m, ck, cv);
      uint32_t kd;
      if (!nflag[cstart[m]] || !second_pass(a, ALGO)) {
        uint32_t own = 0;
#pragma unroll
        for (int u = 0; u < S; ++u) own += ck[u] == (uint32_t)d ? cv[u] : 0u;
        kd = wave_sum(own);
      } else {
        const uint32_t *cm = count + m * (K + 1);
#pragma unroll
        for (int u = 0; u < S; ++u) cv[u] = u * WAVE + lane < K ? cm[u * WAVE + lane] : 0u;
        kd = cm[K];
      }
      int32_t best = -1;
      int64_t bestG = 0;
      const int64_t W = ALGO == ALGO_LPA ? 0 : (int64_t)weight_of(a, i);
      const int64_t Ki = ALGO == ALGO_LPA ? 0 : (int64_t)a.K[i];
      const int64_t Sd = ALGO == ALGO_LPA ? 0 : (int64_t)a.Sig[d];
#pragma unroll
      for (int u = 0; u < S; ++u)
        if (ck[u] != EMPTY) consider<ALGO>(a, W, d, Ki, Sd, kd, (int32_t)ck[u], cv[u], best, bestG);
#pragma unroll
      for (int o = WAVE / 2; o > 0; o >>= 1) {
        const int32_t b2 = __shfl_xor(best, o);
        const int64_t g2 = __shfl_xor(bestG, o);
        if (b2 >= 0 && (best < 0 || g2 > bestG || (g2 == bestG && b2 < best))) {
          best = b2;
          bestG = g2;
        }
      }
      if (lane == 0) finish<ALGO>(a, i, d, best, bestG, ct);
    }
  }
  flush_counters(a, ct);
}

// ---- exact mode ----------------------------------------------------------------------

// Exact mode, the shortest rows (tier 0, and the rows whose sketch is their exact table):
// G = 1, 2, 4 or 8 lanes per row of at most 4 G entries, each lane with four neighbouring
// entries from one 128-bit load.  Every lane sums the weights of its four keys over the
// whole row (the other lanes' entries come by DPP moves) and scores them; a key that
// occurs twice is scored twice, to the same value.  The group's best is the row's.
// With one lane per row every load of a wave touches a line per lane, 64 a piece, and that
// was the time: a sweep over 0.34 M aggregated rows of up to 16 entries took 70 us and
// takes 43 (Leiden k = 16 on Chung-Lu 2^22), over R-MAT 2^19's rows of up to 32 entries
// 66 and 34 us.  Rows of one to three entries (5 M of k-mer chains: 314 and 309 us) are
// bound by the gathers of C and Sigma, 10 M each from 20 MB tables at the 72 G/s that such
// gathers reach; a row whose neighbours share its community reads no totals.
template <int G>
__device__ inline uint32_t group_perm(uint32_t x, int v) {  // v = 1 .. G - 1: another lane of the group
  const uint32_t y = v & 4 ? quad_perm<QP_HALF_MIRROR>(x) : x;
  return (v & 3) == 1 ? quad_perm<QP_XOR1>(y) : (v & 3) == 2 ? quad_perm<QP_XOR2>(y) : (v & 3) == 3 ? quad_perm<QP_XOR3>(y) : y;
}
// Lanes of a reduction step over the group: v = 1, 2, 4 ... < G.
template <int G>
__device__ inline uint32_t group_sum(uint32_t x) {
#pragma unroll
  for (int v = 1; v < G; v <<= 1) x += group_perm<G>(x, v);
  return x;
}
template <int G>
__device__ inline uint32_t group_or(uint32_t x) {
#pragma unroll
  for (int v = 1; v < G; v <<= 1) x |= group_perm<G>(x, v);
  return x;
}

// Rows w * (WAVE / G) .. of list (count of them), one wave.  SMALL: table keys are slots
// of the small table; a slot's first key (in row order) stands for it.
template <int ALGO, bool SMALL, int G>
__device__ MGCD_INLINE void short_item(const SweepArgs &a, const int32_t *list, int64_t count, int64_t w,
                                       Counters &ct) {
  const int lane = lane_id(), q = lane % G;
  const int64_t r = w * (WAVE / G) + lane / G;
  const bool listed = r < count;
  const int32_t i = listed ? list[r] : 0;
  // as in light_item: a wave of rows that stay where they are ends here
  const int64_t rlo = a.g.off[i], rhi = a.g.off[i + 1];
  const int32_t d = community_of_self<ALGO>(a, i);
  const int32_t gi = a.gid ? a.gid[i] : 0;
  const bool valid = listed && !(a.halt && *a.halt) && !(a.gid && !a.active[gi]);
  if (listed && !valid && q == 0) a.Cnew[i] = d;
  if (!__ballot(valid)) return;
  const uint32_t Ki = ALGO == ALGO_LPA ? 0u : a.K[i];
  const int32_t b = ALGO == ALGO_REFINE ? a.bound[i] : 0;
  const int64_t W = ALGO == ALGO_LPA ? 0 : a.gid ? (int64_t)a.Wg[gi] : (int64_t)a.W;
  const int left = valid ? (int)(rhi - rlo) - 4 * q : 0;
  const v4u j = load4(reinterpret_cast<const uint32_t *>(a.g.idx), rlo + 4 * q, a.g.nnz, left > 0);
  const v4u y = load4(a.g.w, rlo + 4 * q, a.g.nnz, left > 0);
  uint32_t key[4], wt[4], kc[4], sl[4];
  // every gather is issued on every lane with a valid id and masked afterwards
#pragma unroll
  for (int u = 0; u < 4; ++u) key[u] = u < left ? j[u] : 0u;
  if (ALGO == ALGO_REFINE) {
    uint32_t bb[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) bb[u] = (uint32_t)a.bound[(int32_t)key[u]];
#pragma unroll
    for (int u = 0; u < 4; ++u) key[u] |= bb[u] == (uint32_t)b ? 0u : EMPTY;
  } else if (!a.ident) {
#pragma unroll
    for (int u = 0; u < 4; ++u) key[u] = (uint32_t)a.C[(int32_t)key[u]];
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    key[u] |= u < left && j[u] != (uint32_t)i ? 0u : EMPTY;  // self-loops are skipped
    wt[u] = key[u] != EMPTY ? y[u] : 0u;
    sl[u] = SMALL && key[u] != EMPTY ? slot_of(a, key[u]) : key[u];
    kc[u] = 0;
  }
  const uint32_t sd = SMALL ? slot_of(a, (uint32_t)d) : (uint32_t)d;
  uint32_t kd = 0;
#pragma unroll
  for (int u = 0; u < 4; ++u) kd += sl[u] == sd ? wt[u] : 0u;
  kd = group_sum<G>(kd);
  bool stands[4];  // the key may be the row's choice
#pragma unroll
  for (int u = 0; u < 4; ++u) stands[u] = key[u] != EMPTY;
#pragma unroll
  for (int v = 0; v < G; ++v) {
    bool same[4] = {};  // SMALL: the other lane has the slot (this lane, v = 0: at an earlier place)
#pragma unroll
    for (int x = 0; x < 4; ++x) {
      const uint32_t so = group_perm<G>(sl[x], v), wo = group_perm<G>(wt[x], v);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        kc[u] += so == sl[u] ? wo : 0u;
        if (SMALL && (v > 0 || x < u)) same[u] |= so == sl[u];
      }
    }
    if (SMALL) {
      const bool earlier = v == 0 || group_perm<G>((uint32_t)q, v) < (uint32_t)q;
#pragma unroll
      for (int u = 0; u < 4; ++u) stands[u] &= !(same[u] && earlier);
    }
  }
  int32_t best = -1;
  int64_t bestG = 0;
  if constexpr (ALGO == ALGO_LPA) {
#pragma unroll
    for (int u = 0; u < 4; ++u)
      consider_v<ALGO>(W, d, 0, 0, kd, (int32_t)key[u], kc[u], 0u, stands[u], best, bestG);
  } else {
    // a total is read where it can matter; the other lanes read community 0's together
    uint32_t any = 0, sc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      stands[u] = stands[u] && key[u] != (uint32_t)d;
      any |= stands[u];
    }
    any = group_or<G>(any);
    const uint32_t Sd = a.Sig[any ? d : 0];
#pragma unroll
    for (int u = 0; u < 4; ++u) sc[u] = a.Sig[stands[u] ? (int32_t)key[u] : 0];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      consider_v<ALGO>(W, d, Ki, Sd, kd, (int32_t)key[u], kc[u], sc[u], stands[u], best, bestG);
  }
#pragma unroll
  for (int v = 1; v < G; v <<= 1) {
    const uint32_t lo = group_perm<G>((uint32_t)bestG, v), hi = group_perm<G>((uint32_t)((uint64_t)bestG >> 32), v);
    const int32_t c2 = (int32_t)group_perm<G>((uint32_t)best, v);
    const int64_t g2 = (int64_t)(((uint64_t)hi << 32) | lo);
    const bool take = c2 >= 0 && (best < 0 || g2 > bestG || (g2 == bestG && c2 < best));
    best = take ? c2 : best;
    bestG = take ? g2 : bestG;
  }
  if (valid && q == 0) finish<ALGO>(a, i, d, best, bestG, ct);
}

// Many graphs: rows s * 64 .. of list (count of them), one wave, as G items whose counts it
// keeps together; an item whose rows all stay where they are costs no more than the look at
// them, one per lane.
template <int ALGO, bool SMALL, int G>
__device__ MGCD_INLINE void short_rows64(const SweepArgs &a, const int32_t *list, int64_t count, int64_t s,
                                         GraphCounts &gc) {
  const int64_t r = s * WAVE + lane_id();
  const int32_t i = r < count ? list[r] : 0;
  const bool moving = r < count && !frozen(a, i);
  if (r < count && !moving) a.Cnew[i] = community_of_self<ALGO>(a, i);
  const uint64_t todo = __ballot(moving);
#pragma unroll 1
  for (int t = 0; t < G; ++t) {
    if ((todo >> (t * (WAVE / G)) & (~0ull >> (WAVE - WAVE / G))) == 0) continue;
    Counters ct;
    short_item<ALGO, SMALL, G>(a, list, count, s * G + t, ct);
    gather_graph_counts(a, ct, gc);
  }
}

// The short rows, classes of 16..32, 8..15, 4..7 and 1..3 entries one after another in
// the list, each from a wave of its own on (sr.wave).  WIDE (many graphs): the first two
// classes go 64 rows to a wave.
template <int ALGO, bool SMALL, bool WIDE>
__global__ void __launch_bounds__(BLOCK) k_exact_short(SweepArgs a, const int32_t *__restrict__ list, ShortRows sr) {
  if (level_over(a)) return;  // batched: every graph has stopped
  Counters ct;
  GraphCounts gc{-1, 0, 0, 0};
  stamp_start(a);
  const int64_t w = uniform(((int64_t)blockIdx.x * BLOCK + threadIdx.x) / WAVE);
  if (w < sr.wave[1]) {
    if constexpr (WIDE)
      short_rows64<ALGO, SMALL, 8>(a, list, sr.row[1], w, gc);
    else
      short_item<ALGO, SMALL, 8>(a, list, sr.row[1], w, ct);
  } else if (w < sr.wave[2]) {
    if constexpr (WIDE)
      short_rows64<ALGO, SMALL, 4>(a, list + sr.row[1], sr.row[2] - sr.row[1], w - sr.wave[1], gc);
    else
      short_item<ALGO, SMALL, 4>(a, list + sr.row[1], sr.row[2] - sr.row[1], w - sr.wave[1], ct);
  } else if (w < sr.wave[3]) {
    short_item<ALGO, SMALL, 2>(a, list + sr.row[2], sr.row[3] - sr.row[2], w - sr.wave[2], ct);
  } else if (w < sr.wave[4]) {
    short_item<ALGO, SMALL, 1>(a, list + sr.row[3], sr.row[4] - sr.row[3], w - sr.wave[3], ct);
  }
  if constexpr (WIDE) {
    gather_graph_counts(a, ct, gc);
    flush_graph_counts(a, gc);
  } else {
    flush_counters(a, ct);
  }
}

// Tier-0 rows of more than 32 entries (a raised exact_small): one lane per row, which
// re-reads it for every key at its first occurrence.
template <int ALGO>
__global__ void __launch_bounds__(BLOCK)
    k_exact_small(SweepArgs a, const int32_t *__restrict__ list, int64_t count) {
  if (level_over(a)) return;  // batched: every graph has stopped
  Counters ct;
  int64_t t = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  const bool listed = t < count;
  const int32_t i = listed ? list[t] : 0;
  const bool live = listed && !frozen(a, i);
  if (listed && !live) a.Cnew[i] = community_of_self<ALGO>(a, i);
  if (live) {
    const int64_t lo = a.g.off[i], hi = a.g.off[i + 1];
    const int32_t bi = ALGO == ALGO_REFINE ? a.bound[i] : 0;
    const int32_t d = community_of_self<ALGO>(a, i);
    // table key of entry f (EMPTY when Algorithm 1's skips drop it)
    auto tkey = [&](int64_t f) {
      const uint32_t c = stream_key<ALGO>(a, i, a.g.idx[f], bi);
      return c != EMPTY ? slot_of(a, c) : EMPTY;
    };
    const uint32_t sd = slot_of(a, (uint32_t)d);
    uint32_t kd = 0;
    for (int64_t e = lo; e < hi; ++e) kd += tkey(e) == sd ? a.g.w[e] : 0u;
    int32_t best = -1;
    int64_t bestG = 0;
    const int64_t W = ALGO == ALGO_LPA ? 0 : (int64_t)weight_of(a, i);
    const int64_t Ki = ALGO == ALGO_LPA ? 0 : (int64_t)a.K[i];
    const int64_t Sd = ALGO == ALGO_LPA ? 0 : (int64_t)a.Sig[d];
    for (int64_t e = lo; e < hi; ++e) {
      const uint32_t c = stream_key<ALGO>(a, i, a.g.idx[e], bi);
      if (c == EMPTY) continue;
      const uint32_t se = slot_of(a, c);
      bool first = true;
      for (int64_t f = lo; f < e && first; ++f) first = tkey(f) != se;
      if (!first) continue;
      uint32_t kc = 0;
      for (int64_t f = e; f < hi; ++f) kc += tkey(f) == se ? a.g.w[f] : 0u;
      consider<ALGO>(a, W, d, Ki, Sd, kd, (int32_t)c, kc, best, bestG);
    }
    finish<ALGO>(a, i, d, best, bestG, ct);
  }
  flush_counters(a, ct);
}

__device__ inline uint32_t hash_slot(uint32_t c, uint32_t mask) {
  return (c * 0x9E3779B1u) & mask;  // Fibonacci hashing, low bits
}

// The wave's best candidate (larger gain first, then lower id; -1: none) into every lane:
// DPP moves within 16 lanes, then the four rows of 16 by lane reads.
template <int PERM>
__device__ inline void best_step(int32_t &best, int64_t &bestG) {
  const uint32_t lo = quad_perm<PERM>((uint32_t)bestG), hi = quad_perm<PERM>((uint32_t)((uint64_t)bestG >> 32));
  const int32_t c2 = (int32_t)quad_perm<PERM>((uint32_t)best);
  const int64_t g2 = (int64_t)(((uint64_t)hi << 32) | lo);
  const bool take = c2 >= 0 && (best < 0 || g2 > bestG || (g2 == bestG && c2 < best));
  best = take ? c2 : best;
  bestG = take ? g2 : bestG;
}
__device__ inline void wave_best(int32_t &best, int64_t &bestG) {
  best_step<QP_XOR1>(best, bestG);
  best_step<QP_XOR2>(best, bestG);
  best_step<QP_HALF_MIRROR>(best, bestG);
  best_step<QP_MIRROR>(best, bestG);
  int32_t b = -1;
  int64_t g = 0;
#pragma unroll
  for (int r = 0; r < WAVE; r += 16) {
    const int32_t c2 = lane_value(best, r);
    const int64_t g2 = (int64_t)(((uint64_t)lane_value((uint32_t)((uint64_t)bestG >> 32), r) << 32) |
                                 lane_value((uint32_t)bestG, r));
    const bool take = c2 >= 0 && (b < 0 || g2 > g || (g2 == g && c2 < b));
    b = take ? c2 : b;
    g = take ? g2 : g;
  }
  best = b;
  bestG = g;
}

// Add (c, w) of row position f to the LDS table of mask + 1 slots: its slot; fresh: the key
// is new.  The table is at most half full.
template <bool SMALL>
__device__ inline uint32_t table_add(Pair *tab, uint32_t *pos, uint32_t mask, uint32_t c, uint32_t w, uint32_t f,
                                     bool &fresh) {
  uint32_t h = hash_slot(c, mask);
  for (;;) {
    const uint32_t prev = atomicCAS(&tab[h].key, EMPTY, c);
    fresh = prev == EMPTY;
    if (fresh || prev == c) break;
    h = (h + 1) & mask;
  }
  atomicAdd(&tab[h].val, w);
  if (SMALL) atomicMin(&pos[h], f);
  return h;
}

// The sum of key c (0 if it has none).
__device__ inline uint32_t table_sum(const Pair *tab, uint32_t mask, uint32_t c) {
  uint32_t h = hash_slot(c, mask);
  for (;;) {
    const Pair p = tab[h];
    if (p.key == c) return p.val;
    if (p.key == EMPTY) return 0u;
    h = (h + 1) & mask;
  }
}

// Exact mode, tier 1 (rows of up to EXACT_WAVE_MAX entries): one wave per row with an
// LDS open-addressing table of its own, sized to the row (the smallest power of two
// >= 2 * its length), so a block holds four rows instead of one.  The slots that keys
// claim are listed, so that the decision visits keys and not slots.
// Same table keys, sums, first positions (small table) and decision as k_exact_table.
// Bound by the latency of a row's chain of loads, so by the rows in flight: 4.5 KB per wave
// let 32 waves live on a CU (8 KB, for rows of up to 512 entries, 20).  A sweep over R-MAT 2^19's
// rows of 33 to 512 entries took 150 to 176 us here; these of up to 256 take 39 to 47 and
// the others, with tier 2's, are below.
template <int ALGO, bool SMALL = false>
__global__ void __launch_bounds__(BLOCK)
    k_exact_wave(SweepArgs a, const int32_t *__restrict__ list, int64_t count, int64_t block0) {
  if (level_over(a)) return;  // batched: every graph has stopped
  constexpr uint32_t CAPW = 2 * EXACT_WAVE_MAX;
  __shared__ __attribute__((aligned(16))) Pair wtab[BLOCK / WAVE][CAPW];
  __shared__ uint32_t wpos[BLOCK / WAVE][SMALL ? CAPW : 1];
  __shared__ uint16_t wcell[BLOCK / WAVE][EXACT_WAVE_MAX];
  const int lane = lane_id(), w = uniform((int32_t)(threadIdx.x / WAVE));
  const int64_t r = uniform(((block0 + blockIdx.x) * BLOCK + threadIdx.x) / WAVE);
  Counters ct;
  if (r < count) {
    const int32_t i = uniform(list[r]);
    if (frozen(a, i)) {
      if (lane == 0) a.Cnew[i] = community_of_self<ALGO>(a, i);
    } else {
      const int64_t lo = uniform(a.g.off[i]), hi = uniform(a.g.off[i + 1]);
      const int32_t bi = ALGO == ALGO_REFINE ? uniform(a.bound[i]) : 0;
      const int32_t d = uniform(community_of_self<ALGO>(a, i));
      const auto load = [&](int64_t e, uint32_t &key, uint32_t &wt) {
        const bool in = e < hi;
        const int32_t j = in ? __builtin_nontemporal_load(a.g.idx + e) : 0;
        wt = in ? __builtin_nontemporal_load(a.g.w + e) : 0u;
        key = in ? stream_key<ALGO>(a, i, j, bi) : EMPTY;
      };
      uint32_t key, wt;
      load(lo + lane, key, wt);  // on its way while the table is cleared
      uint32_t cap = 64;
      while (cap < CAPW && (int64_t)cap < 2 * (hi - lo)) cap <<= 1;
      const uint32_t mask = cap - 1;
      Pair *tab = wtab[w];
      uint32_t *pos = wpos[w];
      uint16_t *cell = wcell[w];
      for (uint32_t x = 2 * lane; x < cap; x += 2 * WAVE) {
        tab[x] = tab[x + 1] = Pair{EMPTY, 0u};
        if (SMALL) pos[x] = pos[x + 1] = 0xFFFFFFFFu;
      }
      wave_sync();
      int keys = 0;
      for (int64_t e0 = lo; e0 < hi; e0 += WAVE) {  // wave-uniform rounds
        uint32_t nkey = EMPTY, nwt = 0;
        if (e0 + WAVE < hi) load(e0 + WAVE + lane, nkey, nwt);
        uint32_t c = key != EMPTY ? slot_of(a, key) : EMPTY;
        // the lanes holding the first live lane's key add their weights into that lane
        // (one table update instead of one per lane, which serialise on the slot of a
        // community that many neighbours share; the lane is the group's first position)
        const uint64_t lm = __ballot(c != EMPTY);
        if (lm) {
          const int ld = __builtin_ctzll(lm);
          const uint32_t ck = lane_value(c, ld);
          const bool m = c == ck;
          if (__popcll(__ballot(m)) > 1) {
            const uint32_t sum = wave_sum(m ? wt : 0u);
            if (lane == ld)
              wt = sum;
            else if (m)
              c = EMPTY;
          }
        }
        bool fresh = false;
        uint32_t h = 0;
        if (c != EMPTY) h = table_add<SMALL>(tab, pos, mask, c, wt, (uint32_t)(e0 + lane - lo), fresh);
        const uint64_t fm = __ballot(fresh);
        if (fresh) cell[keys + __popcll(fm & lanemask_lt())] = (uint16_t)h;
        keys += __popcll(fm);
        key = nkey;
        wt = nwt;
      }
      wave_sync();
      const uint32_t kd = table_sum(tab, mask, slot_of(a, (uint32_t)d));
      int32_t best = -1;
      int64_t bestG = 0;
      const int64_t W = ALGO == ALGO_LPA ? 0 : (int64_t)weight_of(a, i);
      const int64_t Ki = ALGO == ALGO_LPA ? 0 : (int64_t)a.K[i];
      const int64_t Sd = ALGO == ALGO_LPA ? 0 : (int64_t)a.Sig[d];
      for (int x = lane; x < keys; x += WAVE) {
        Pair p = tab[cell[x]];
        if (SMALL) p.key = stream_key<ALGO>(a, i, a.g.idx[lo + pos[cell[x]]], bi);
        consider<ALGO>(a, W, d, Ki, Sd, kd, (int32_t)p.key, p.val, best, bestG);
      }
      wave_best(best, bestG);
      if (lane == 0) finish<ALGO>(a, i, d, best, bestG, ct);
    }
  }
  flush_counters(a, ct);
}

// Exact mode, tier 2: a workgroup of THREADS per vertex with an open-addressing table
// (linear probing) in LDS, sized to the row, CAP = 8 * THREADS slots at most: a thread has
// four entries of the row, whose loads are all on their way before the table is cleared, and
// the slots that keys claim are listed, so that the decision visits keys and not slots.
// Bound by latency as k_exact_wave: 256 threads with 2048 slots (rows of fewer than 1024
// entries) and 1024 with 8192 fill a CU; 256 threads with 8192 slots were 8 waves on a CU
// and looked at every slot of the largest table for every row: a sweep
// over R-MAT 2^19's rows of 513 to 4096 entries took 136 to 194 us; rows of 257 to 1023 now
// take 52 to 73 us and those of 1024 to 4096 23 to 31.
template <int ALGO, int THREADS, bool SMALL = false>
__global__ void __launch_bounds__(THREADS)
    k_exact_table(SweepArgs a, const int32_t *__restrict__ list, int64_t block0) {
  if (level_over(a)) return;  // batched: every graph has stopped
  constexpr int U = 4;
  constexpr uint32_t CAP = 2 * U * THREADS;
  __shared__ __attribute__((aligned(16))) Pair tab[CAP];
  __shared__ uint32_t pos[SMALL ? CAP : 1];  // small table: first row position per slot
  __shared__ uint16_t cell[CAP / 2];
  __shared__ uint32_t ncell;
  __shared__ int32_t bc[THREADS / WAVE];
  __shared__ int64_t bg[THREADS / WAVE];
  const int t = threadIdx.x;
  const int32_t i = uniform(list[block0 + blockIdx.x]);
  if (frozen(a, i)) {  // block-uniform
    if (t == 0) a.Cnew[i] = community_of_self<ALGO>(a, i);
    return;
  }
  const int64_t lo = uniform(a.g.off[i]), hi = uniform(a.g.off[i + 1]);
  const int32_t bi = ALGO == ALGO_REFINE ? uniform(a.bound[i]) : 0;
  const int32_t d = uniform(community_of_self<ALGO>(a, i));
  // an absent entry reads the row's first and is masked
  uint32_t cs[U], ws[U];
  int32_t js[U], bs[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t e = lo + t + u * THREADS, es = e < hi ? e : lo;
    js[u] = __builtin_nontemporal_load(a.g.idx + es);
    ws[u] = __builtin_nontemporal_load(a.g.w + es);
    bs[u] = bi;
  }
  neighbour_keys<ALGO, U>(a, js, bs, cs);
  uint32_t cap = 2 * THREADS;
  while (cap < CAP && (int64_t)cap < 2 * (hi - lo)) cap <<= 1;
  const uint32_t mask = cap - 1;
  for (uint32_t x = 2 * t; x < cap; x += 2 * THREADS) {
    tab[x] = tab[x + 1] = Pair{EMPTY, 0u};
    if (SMALL) pos[x] = pos[x + 1] = 0xFFFFFFFFu;
  }
  if (t == 0) ncell = 0;
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t f = (uint32_t)(t + u * THREADS);
    if (lo + (int64_t)(f & ~(uint32_t)(WAVE - 1)) >= hi) break;  // wave-uniform: no entry left
    bool fresh = false;
    uint32_t h = 0;
    if (lo + f < hi && js[u] != i && cs[u] != EMPTY)  // self-loops are skipped
      h = table_add<SMALL>(tab, pos, mask, slot_of(a, cs[u]), ws[u], f, fresh);
    const uint64_t fm = __ballot(fresh);
    if (fm == 0) continue;
    uint32_t base = 0;
    if (lane_id() == 0) base = atomicAdd(&ncell, (uint32_t)__popcll(fm));
    base = uniform(base);
    if (fresh) cell[base + __popcll(fm & lanemask_lt())] = (uint16_t)h;
  }
  __syncthreads();
  const uint32_t kd = table_sum(tab, mask, slot_of(a, (uint32_t)d)), keys = ncell;
  int32_t best = -1;
  int64_t bestG = 0;
  const int64_t W = ALGO == ALGO_LPA ? 0 : (int64_t)weight_of(a, i);
  const int64_t Ki = ALGO == ALGO_LPA ? 0 : (int64_t)a.K[i];
  const int64_t Sd = ALGO == ALGO_LPA ? 0 : (int64_t)a.Sig[d];
  for (uint32_t x = t; x < keys; x += THREADS) {
    Pair p = tab[cell[x]];
    // a small table's slot stands for its first key: the key of its earliest row entry
    if (SMALL) p.key = stream_key<ALGO>(a, i, a.g.idx[lo + pos[cell[x]]], bi);
    consider<ALGO>(a, W, d, Ki, Sd, kd, (int32_t)p.key, p.val, best, bestG);
  }
  // block arg-max: larger gain first, then lower community id
  wave_best(best, bestG);
  if (lane_id() == 0) {
    bc[t / WAVE] = best;
    bg[t / WAVE] = bestG;
  }
  __syncthreads();
  if (t == 0) {
    for (int q = 1; q < THREADS / WAVE; ++q) {
      bool take = bc[q] >= 0 && (best < 0 || bg[q] > bestG || (bg[q] == bestG && bc[q] < best));
      best = take ? bc[q] : best;
      bestG = take ? bg[q] : bestG;
    }
    Counters ct;
    finish<ALGO>(a, i, d, best, bestG, ct);
    commit_counters(a, ct);
  }
}

// Exact mode, rows of more than exact_t2 entries: a global open-addressing table per
// row (hbase), filled by one workgroup per segment of GSEG entries (global atomics,
// so the segments of one row insert concurrently); then K_{i->d} by a probe, one
// workgroup per TSEG table slots scores them and clears them for the next sweep (the
// tables are cleared once when the schedule is built), and one thread per row
// combines the segments' best (the rule is associative) and decides.  Same keys,
// sums, positions and decision as k_exact_table.
template <int ALGO, bool SMALL>
__global__ void __launch_bounds__(BLOCK)
    k_gtab_insert(SweepArgs a, const int32_t *__restrict__ list, const int64_t *__restrict__ hbase,
                  const int64_t *__restrict__ sstart, const int32_t *__restrict__ sowner, int64_t block0,
                  Pair *htab, uint32_t *hpos) {
  if (level_over(a)) return;  // batched: every graph has stopped
  // Each round's U * BLOCK entries are first combined in an LDS table (at most U * BLOCK
  // keys in 2 * U * BLOCK slots), then every distinct key goes to the global table
  // once: the entries of a hub row concentrate on a few communities, whose slots
  // would otherwise serialise the global atomics of all the row's workgroups.
  constexpr int U = 4;  // entries per thread and round, loads and gathers issued together
  constexpr uint32_t LCAP = 2 * U * BLOCK;
  __shared__ uint32_t lk[LCAP], lv[LCAP];
  __shared__ uint32_t lp[SMALL ? LCAP : 1];
  const int t = threadIdx.x;
  const int64_t sg = block0 + blockIdx.x;
  const int32_t r = sowner[sg];
  const int32_t i = list[r];
  if (frozen(a, i)) return;  // block-uniform
  const int64_t rlo = a.g.off[i], rhi = a.g.off[i + 1];
  const int64_t lo = rlo + (sg - sstart[r]) * GSEG;
  const int64_t hi = lo + GSEG < rhi ? lo + GSEG : rhi;
  Pair *tab = htab + hbase[r];
  uint32_t *pos = hpos + hbase[r];
  const uint32_t mask = (uint32_t)(hbase[r + 1] - hbase[r]) - 1;
  const int32_t bi = ALGO == ALGO_REFINE ? a.bound[i] : 0;
  for (int64_t b0 = lo; b0 < hi; b0 += U * BLOCK) {  // block-uniform rounds
    for (uint32_t x = t; x < LCAP; x += BLOCK) {
      lk[x] = EMPTY;
      lv[x] = 0u;
      if (SMALL) lp[x] = 0xFFFFFFFFu;
    }
    __syncthreads();
    uint32_t cs[U], ws[U];
    int32_t js[U], bs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t e = b0 + t + (int64_t)u * BLOCK;
      const bool v = e < hi;
      const int64_t es = v ? e : lo;
      js[u] = a.g.idx[es];
      bs[u] = bi;
      ws[u] = a.g.w[es];
    }
    neighbour_keys<ALGO, U>(a, js, bs, cs);
#pragma unroll
    for (int u = 0; u < U; ++u)  // self-loops are skipped
      cs[u] |= ((b0 + t + (int64_t)u * BLOCK) < hi && js[u] != i) ? 0u : EMPTY;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (cs[u] == EMPTY) continue;
      const uint32_t c = slot_of(a, cs[u]);
      uint32_t h = hash_slot(c, LCAP - 1);
      while (true) {
        const uint32_t prev = atomicCAS(&lk[h], EMPTY, c);
        if (prev == EMPTY || prev == c) break;
        h = (h + 1) & (LCAP - 1);
      }
      atomicAdd(&lv[h], ws[u]);
      if (SMALL) atomicMin(&lp[h], (uint32_t)(b0 + t + (int64_t)u * BLOCK - rlo));
    }
    __syncthreads();
    // key and sum go in by one 64-bit swap when the slot is free, by an add when it holds
    // the key; four swaps of a thread are under way together (a first sweep over R-MAT
    // 2^19's rows of more than 4096 entries: 108 us; with a swap of the key and an add one
    // after another 150 to 179)
    for (uint32_t x0 = t; x0 < LCAP; x0 += U * BLOCK) {
      uint32_t c[U], h[U];
      unsigned long long old[U];
      const auto swap = [&](uint32_t slot, uint32_t key, uint32_t sum) {
        return atomicCAS(reinterpret_cast<unsigned long long *>(tab + slot), (unsigned long long)EMPTY,
                         ((unsigned long long)sum << 32) | key);
      };
#pragma unroll
      for (int u = 0; u < U; ++u) {
        c[u] = lk[x0 + u * BLOCK];
        h[u] = hash_slot(c[u], mask);
        if (c[u] != EMPTY) old[u] = swap(h[u], c[u], lv[x0 + u * BLOCK]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (c[u] == EMPTY) continue;
        while ((uint32_t)old[u] != EMPTY && (uint32_t)old[u] != c[u]) {
          h[u] = (h[u] + 1) & mask;
          old[u] = swap(h[u], c[u], lv[x0 + u * BLOCK]);
        }
        if ((uint32_t)old[u] == c[u]) atomicAdd(&tab[h[u]].val, lv[x0 + u * BLOCK]);
        if (SMALL) atomicMin(&pos[h[u]], lp[x0 + u * BLOCK]);
      }
    }
    __syncthreads();  // the flush has read the table before the next round clears it
  }
}

// K_{i->d} of every global-table row, by probing its table for d's key (before any
// workgroup of k_gtab_scan clears a segment of the table).
template <int ALGO>
__global__ void __launch_bounds__(BLOCK)
    k_gtab_kd(SweepArgs a, const int32_t *__restrict__ list, int64_t count, const int64_t *__restrict__ hbase,
              const Pair *__restrict__ htab, uint32_t *kdout) {
  if (level_over(a)) return;  // batched: every graph has stopped
  const int64_t r = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (r >= count) return;
  const int32_t i = list[r];
  if (frozen(a, i)) return;
  const Pair *tab = htab + hbase[r];
  const uint32_t mask = (uint32_t)(hbase[r + 1] - hbase[r]) - 1;
  const uint32_t sd = slot_of(a, (uint32_t)community_of_self<ALGO>(a, i));
  uint32_t h = hash_slot(sd, mask), kd = 0;
  while (true) {  // the table is at most half full, so an EMPTY slot ends the probe
    const Pair p = tab[h];
    if (p.key == sd) {
      kd = p.val;
      break;
    }
    if (p.key == EMPTY) break;
    h = (h + 1) & mask;
  }
  kdout[r] = kd;
}

// One workgroup per TSEG slots of a row's table: the best candidate among them
// (larger gain, then lower id) into part[], then the slots are cleared for the next
// sweep.
template <int ALGO, bool SMALL>
__global__ void __launch_bounds__(BLOCK)
    k_gtab_scan(SweepArgs a, const int32_t *__restrict__ list, const int64_t *__restrict__ hbase,
                const int64_t *__restrict__ tstart, const int32_t *__restrict__ towner, int64_t block0,
                Pair *htab, uint32_t *hpos, const uint32_t *__restrict__ kdin, int32_t *pbest, int64_t *pgain) {
  if (level_over(a)) return;  // batched: every graph has stopped
  __shared__ int32_t bc[BLOCK / WAVE];
  __shared__ int64_t bg[BLOCK / WAVE];
  const int t = threadIdx.x;
  const int64_t sg = block0 + blockIdx.x;
  const int32_t r = towner[sg];
  const int32_t i = list[r];
  if (frozen(a, i)) return;  // block-uniform; the table was not filled
  const int64_t lo = a.g.off[i];
  const int64_t x0 = hbase[r] + (sg - tstart[r]) * TSEG;
  const int64_t x1 = x0 + TSEG < hbase[r + 1] ? x0 + TSEG : hbase[r + 1];
  const int32_t bi = ALGO == ALGO_REFINE ? a.bound[i] : 0;
  const int32_t d = community_of_self<ALGO>(a, i);
  const uint32_t kd = kdin[r];
  int32_t best = -1;
  int64_t bestG = 0;
  const int64_t W = ALGO == ALGO_LPA ? 0 : (int64_t)weight_of(a, i);
  const int64_t Ki = ALGO == ALGO_LPA ? 0 : (int64_t)a.K[i];
  const int64_t Sd = ALGO == ALGO_LPA ? 0 : (int64_t)a.Sig[d];
  for (int64_t x = x0 + t; x < x1; x += BLOCK) {
    Pair p = htab[x];
    const bool present = p.key != EMPTY;
    if (SMALL && present) p.key = stream_key<ALGO>(a, i, a.g.idx[lo + hpos[x]], bi);
    const uint32_t sc = ALGO == ALGO_LPA ? 0u : a.Sig[present ? (int32_t)p.key : d];
    consider_v<ALGO>(W, d, Ki, Sd, kd, (int32_t)p.key, p.val, sc, present, best, bestG);
  }
#pragma unroll
  for (int o = WAVE / 2; o > 0; o >>= 1) {
    const int32_t ob = __shfl_xor(best, o);
    const int64_t og = __shfl_xor(bestG, o);
    const bool take = ob >= 0 && (best < 0 || og > bestG || (og == bestG && ob < best));
    best = take ? ob : best;
    bestG = take ? og : bestG;
  }
  if (lane_id() == 0) {
    bc[t / WAVE] = best;
    bg[t / WAVE] = bestG;
  }
  __syncthreads();  // every slot of the segment has been read: clear them
  for (int64_t x = x0 + t; x < x1; x += BLOCK) {
    htab[x] = Pair{EMPTY, 0u};
    if (SMALL) hpos[x] = 0xFFFFFFFFu;
  }
  if (t == 0) {
    for (int q = 1; q < BLOCK / WAVE; ++q) {
      const bool take = bc[q] >= 0 && (best < 0 || bg[q] > bestG || (bg[q] == bestG && bc[q] < best));
      best = take ? bc[q] : best;
      bestG = take ? bg[q] : bestG;
    }
    pbest[sg] = best;
    pgain[sg] = bestG;
  }
}

// One thread per global-table row: the best over its segments, then the decision.
template <int ALGO>
__global__ void __launch_bounds__(BLOCK)
    k_gtab_finish(SweepArgs a, const int32_t *__restrict__ list, int64_t count,
                  const int64_t *__restrict__ tstart, const int32_t *__restrict__ pbest,
                  const int64_t *__restrict__ pgain) {
  if (level_over(a)) return;  // batched: every graph has stopped
  const int64_t r = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  Counters ct;
  if (r < count) {
    const int32_t i = list[r];
    const int32_t d = community_of_self<ALGO>(a, i);
    if (frozen(a, i)) {
      a.Cnew[i] = d;
    } else {
      int32_t best = -1;
      int64_t bestG = 0;
      for (int64_t q = tstart[r]; q < tstart[r + 1]; ++q) {
        const bool take = pbest[q] >= 0 && (best < 0 || pgain[q] > bestG || (pgain[q] == bestG && pbest[q] < best));
        best = take ? pbest[q] : best;
        bestG = take ? pgain[q] : bestG;
      }
      finish<ALGO>(a, i, d, best, bestG, ct);
    }
  }
  flush_counters(a, ct);
}

__global__ void k_gtab_clear(Pair *htab, uint32_t *hpos, int64_t n, int64_t block0) {
  const int64_t x = (block0 + blockIdx.x) * BLOCK + threadIdx.x;
  if (x < n) {
    htab[x] = Pair{EMPTY, 0u};
    hpos[x] = 0xFFFFFFFFu;
  }
}

// ---- schedule ------------------------------------------------------------------------

// Category of every vertex for this level's schedule, and per-category counts
// (wave ballots, then one atomic per category and workgroup).
//   MG:    0 = row fits one chunk (sort key: heavy first), 1 + b = a long row of at
//          most 2^b <= 64 chunks (b = 1..6), 7 = longer rows;
//   MG with K = 32 / 64: 0 = at most exact_t0 entries, 1 = one wave per row, 2 = split
//          rows (more than max(L, WAVE_SPLIT) entries);
//          (4 counts those of the split rows that may have more than one node: the first
//          ones, heavy rows being first)
//   exact: tiers 0..3 by degree; 4 counts the tier-2 rows for the smaller workgroup.
//   every mode: rows without entries (category 8) are sorted last and listed in no
//          kernel's work: their label can never change, so no sweep writes it, and
//          callers keep both label buffers equal for them.
//   MG:    10 = light rows: category 0 with at most LIGHT_MAX entries (they follow the
//          other single-chunk rows in the heavy-first order).
//   every mode: 11..15 count the rows of category 0 or 9 that take the short rows' kernel
//          by class: 1..3, 4..7, 8..15, 16..32 entries, and longer ones.
constexpr int NCAT = 16;
constexpr int CAT_BLOCK = 4;  // exact: tier-2 rows of fewer than EXACT_BLOCK_MAX entries
constexpr int CAT_TREE = 4;   // K >= 32: split rows of SchedParams::tree_class and up
constexpr int CAT_EMPTY = 8;
constexpr int CAT_LIGHT = 10;
constexpr int CAT_CLASS = 11;
constexpr int CAT_SHORT = 9;  // MG: rows whose sketch cannot lose weight (short rows' kernel)

// The class of rows of deg entries that lists are ordered by: the bits of deg, 32 with 16..31
// (the longest of their class of short rows).
__host__ __device__ inline int row_class(int64_t deg) {
  int b = 0;
  while (b < 63 && (deg >> b) != 0) ++b;
  return deg == 32 ? 5 : b;
}

__global__ void __launch_bounds__(BLOCK)
    k_schedule_keys(const int64_t *off, int32_t n, SchedParams sp, uint64_t *key, uint32_t *val,
                    unsigned long long *cnt) {
  const int mode = sp.mode;
  const int64_t L = sp.L;
  __shared__ unsigned long long bc[NCAT];
  if (threadIdx.x < NCAT) bc[threadIdx.x] = 0;
  __syncthreads();
  int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  int cat = -1, cls = -1;
  int64_t dmax = 0;
  if (i < n) {
    int64_t deg = off[i + 1] - off[i];
    dmax = deg;
    const int b = row_class(deg);
    uint64_t k;
    bool shortrow = false;
    if (deg == 0) {
      cat = CAT_EMPTY;
      k = 255;  // after every other key of every mode
    } else if (mode == MODE_EXACT) {
      const int64_t t1 = sp.exact_t1 < EXACT_WAVE_MAX ? sp.exact_t1 : EXACT_WAVE_MAX;
      cat = deg <= sp.exact_t0 ? 0 : deg <= t1 ? 1 : deg <= sp.exact_t2 ? 2 : 3;
      // heavy rows first in each tier
      k = cat == 0 ? (uint64_t)(64 - b) : (uint64_t)(128 + (cat - 1) * 32 + (b < 31 ? 31 - b : 0));
      shortrow = cat == 0;
      if (cat == 2 && deg < EXACT_BLOCK_MAX) cls = CAT_BLOCK;
    } else if (sp.wave) {  // K >= 32: short rows exact, split rows, the rest one wave each
      // (K = 128 / 256: every other row is a split row, one wave per chunk)
      cat = deg <= sp.exact_t0 ? 0 : (sp.k > WAVE || (deg > L && deg > WAVE_SPLIT)) ? 2 : 1;
      k = (uint64_t)(cat * 64 + 64 - b);  // heavy rows first in each tier
      shortrow = cat == 0;
      if (cat == 2 && b >= sp.tree_class) cls = CAT_TREE;
    } else if (deg <= sp.mg_short) {  // after the single-chunk rows, heavy rows first
      cat = CAT_SHORT;
      shortrow = true;
      k = (uint64_t)(128 + 64 - b);  // b <= 5: below 200
    } else if (deg <= L) {
      cat = deg <= LIGHT_MAX ? CAT_LIGHT : 0;
      k = (uint64_t)(64 - b) + (deg <= LIGHT_MAX ? 64 : 0);  // heavy rows first, then light ones
    } else {
      int64_t nc = (deg + L - 1) / L;
      int lp = 0;
      while ((1ll << lp) < nc) ++lp;
      cat = lp <= sp.row_lanes_log2 ? lp : 7;
      k = 200ull + (uint64_t)cat;
    }
    key[i] = k;
    val[i] = (uint32_t)i;
    if (shortrow) cls = CAT_CLASS + (b <= 2 ? 0 : b <= 5 ? b - 2 : 4);
  }
#pragma unroll
  for (int q = 0; q < NCAT; ++q) {
    uint64_t m = __ballot(cat == q || cls == q);
    if (lane_id() == 0 && m) atomicAdd(&bc[q], (unsigned long long)__popcll(m));
  }
  __syncthreads();
  cnt += spread_copy() * (NCAT + 1);
  if (threadIdx.x < NCAT && bc[threadIdx.x]) atomicAdd(&cnt[threadIdx.x], bc[threadIdx.x]);
  // block maximum, then one atomic per block, skipped when it cannot raise the value
  __shared__ unsigned long long bmax[BLOCK / WAVE];
#pragma unroll
  for (int o = WAVE / 2; o > 0; o >>= 1) {
    const int64_t x = __shfl_xor(dmax, o);
    dmax = x > dmax ? x : dmax;
  }
  if (lane_id() == 0) bmax[threadIdx.x / WAVE] = (unsigned long long)dmax;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned long long mx = bmax[0];
    for (int q = 1; q < BLOCK / WAVE; ++q) mx = bmax[q] > mx ? bmax[q] : mx;
    if (mx > 0 && mx > __hip_atomic_load(&cnt[NCAT], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&cnt[NCAT], mx);
  }  // longest row
}

__global__ void k_chunk_counts(const int64_t *off, const int32_t *multi, int64_t nmulti, int64_t L,
                               int64_t *nch) {
  int64_t m = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (m >= nmulti) return;
  int32_t i = multi[m];
  nch[m] = (off[i + 1] - off[i] + L - 1) / L;
}

__global__ void k_group_counts(const int64_t *cstart, int64_t nmulti, int64_t *ng) {
  int64_t m = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (m >= nmulti) return;
  ng[m] = (cstart[m + 1] - cstart[m] + WAVE - 1) / WAVE;
}

__global__ void k_chunk_owner(const int64_t *cstart, int64_t block0, int32_t *owner) {
  const int64_t m = block0 + blockIdx.x;
  for (int64_t q = cstart[m] + threadIdx.x; q < cstart[m + 1]; q += BLOCK) owner[q] = (int32_t)m;
}

static void chunk_owners(const int64_t *cstart, int64_t nmulti, int32_t *owner, hipStream_t st) {
  launch_slices(nmulti, BLOCK, [&](int64_t first, unsigned blocks) {
    k_chunk_owner<<<blocks, BLOCK, 0, st>>>(cstart, first, owner);
    MGCD_LAUNCHED();
  });
}

__global__ void k_table_segs(const int64_t *hbase, int64_t count, int64_t *nt) {
  const int64_t r = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (r < count) nt[r] = (hbase[r + 1] - hbase[r] + TSEG - 1) / TSEG;
}

__global__ void k_hash_caps(const int64_t *off, const int32_t *list, int64_t count, int64_t *cap) {
  int64_t m = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (m >= count) return;
  int32_t i = list[m];
  int64_t need = 2 * (off[i + 1] - off[i]);
  int64_t c = 1;
  while (c < need) c <<= 1;
  cap[m] = c;
}

__global__ void k_u32_from_u64(const uint32_t *v, int32_t *out, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) out[i] = (int32_t)v[i];
}

static unsigned grid_for(int64_t n) { return (unsigned)ceil_div(n > 0 ? n : 1, BLOCK); }

size_t schedule_ws_bytes(int32_t n, int64_t nnz, int mode, int k, int64_t L) {
  size_t b = 0;
  b += (size_t)n * (8 + 4) * 2 + 4096;         // sort keys/values, two buffers
  b += radix_sort_ws_bytes(n) + 4096;
  b += (size_t)n * 4 + 1024;                   // ordered list
  if (mode == MODE_EXACT) {
    // rows on global tables: at most min(n, nnz) (each has an entry)
    const int64_t c3 = n < nnz ? n : nnz;
    // per row: table capacity and base, insert-segment count and start, scan-segment
    // count and start (8 B each), K_{i->d} (4 B); three scans
    b += (size_t)(c3 + 2) * (6 * 8 + 4) + 3 * scan_ws_bytes(c3 + 1) + 8192;
    b += (size_t)(4 * nnz + 64) * (sizeof(Pair) + 4) + 2048;  // tables (cap <= 4*deg), positions
    // insert segments (owner) and scan segments (owner, best, gain)
    const int64_t ns = nnz / GSEG + c3 + 2, nt = (4 * nnz + 64) / TSEG + c3 + 2;
    b += (size_t)ns * 4 + (size_t)nt * (4 + 4 + 8) + 4096;
  } else {
    // a long row has more than one chunk, so more than L entries: at most nnz / L
    // long rows, at most 2 nnz / L + 1 of their chunks, and groups of 64 chunks at
    // most chunks / 64 + long rows
    const int64_t Lc = L > 0 ? L : 1;
    const int64_t nl = nnz / Lc + 1, cl = 2 * (nnz / Lc) + 2, gl = cl / 64 + nl + 1;
    b += (size_t)nnz * 4 + 1024;                                     // key stream
    b += (size_t)(nl + 1) * 8 * 2 + scan_ws_bytes(nl) + 2048;        // chunk counts, cstart
    b += (size_t)cl * (4 + (size_t)(k + 1) * 4) + 4096;              // owner, pass-2 counts
    b += (size_t)(nl + 1) * 8 * 2 + scan_ws_bytes(nl) + 2048;        // group counts, gstart
    b += (size_t)gl * (4 + (size_t)k * sizeof(Pair) + 4) + 4096;     // gowner, roots, flags
    b += (size_t)nl * ((size_t)k * sizeof(Pair) + 4) + 2048;         // candidates, flags
    if (k > 16)  // split rows of the 32/64-slot sketch: chunk nodes, flags, pass-2 counts
      b += (size_t)cl * ((size_t)k * sizeof(Pair) + 4) + (size_t)nl * (k + 1) * 4 + 4096;
    if (k > WAVE) {  // 128/256 slots: every row of more than 32 (or, unconditional, 0)
      // entries is split: at most min(n, nnz) rows and nnz / L + that many chunks
      const int64_t rs = (n < nnz ? (int64_t)n : nnz) + 1, cs = nnz / Lc + rs + 1;
      b += (size_t)(rs + 1) * 8 * 2 + scan_ws_bytes(rs) + (size_t)cs * 4 + 4096;  // counts, cstart, owner
      b += (size_t)cs * ((size_t)k * sizeof(Pair) + 4) + (size_t)rs * (k + 1) * 4 + 4096;
    }
  }
  return b + 64 * 1024;
}

static void build_lists(const Graph &g, const SchedParams &sp_in, Schedule &s, Arena &a, hipStream_t st) {
  SchedParams sp = sp_in;
  if (sp.short_auto && g.nnz > sp.mg_short * (int64_t)g.n) sp.mg_short = 0;
  const int mode = sp.mode, k = sp.k;
  const int64_t L = sp.L;
  const int32_t n = g.n;
  if (sp.wave) sp.tree_class = row_class(wave_group(k) * L + 1);
  s = Schedule{};
  if (n == 0) return;
  unsigned long long *cnt = a.take<unsigned long long>(SPREAD * (NCAT + 1));
  uint64_t *k0 = a.take<uint64_t>(n);
  uint32_t *v0 = a.take<uint32_t>(n);
  uint64_t *k1 = a.take<uint64_t>(n);
  uint32_t *v1 = a.take<uint32_t>(n);
  int32_t *order = a.take<int32_t>(n);
  launch_zero_u64(cnt, SPREAD * (NCAT + 1), st);
  k_schedule_keys<<<grid_for(n), BLOCK, 0, st>>>(g.off, n, sp, k0, v0, cnt);
  MGCD_LAUNCHED();
  bool flip = radix_sort_pairs(k0, v0, k1, v1, n, 8, a, st);
  k_u32_from_u64<<<grid_for(n), BLOCK, 0, st>>>(flip ? v1 : v0, order, n);
  MGCD_LAUNCHED();
  unsigned long long h[NCAT + 1];
  read_spread(cnt, NCAT, h, st);
  s.maxdeg = (int64_t)h[NCAT];
  {  // the short rows' classes, heavy first: longer ones, then 8, 4, 2 and 1 lanes per row
    ShortRows &sr = s.shorts;
    s.ntail = (int64_t)h[CAT_CLASS + 4];
    for (int q = 0; q < 4; ++q) {
      const int64_t rows = (int64_t)h[CAT_CLASS + 3 - q];
      sr.row[q + 1] = sr.row[q] + rows;
      sr.wave[q + 1] = sr.wave[q] + ceil_div(rows * (8 >> q), WAVE);
    }
  }
  if (sp.wave) {
    s.tier[0] = order;
    s.ntier[0] = (int64_t)h[0];
    s.tier[1] = order + h[0];
    s.ntier[1] = (int64_t)h[1];
    s.keybuf = a.take<uint32_t>(g.nnz);
    s.multi = order + h[0] + h[1];
    s.nmulti = (int64_t)h[2];
    if (s.nmulti > 0) {
      int64_t *nch = a.take<int64_t>(s.nmulti);
      s.cstart = a.take<int64_t>(s.nmulti + 1);
      k_chunk_counts<<<grid_for(s.nmulti), BLOCK, 0, st>>>(g.off, s.multi, s.nmulti, wave_group(k) * L, nch);
      MGCD_LAUNCHED();
      scan_i64(nch, s.cstart, s.nmulti, s.cstart + s.nmulti, a, st);
      s.ntree = (int64_t)h[CAT_TREE];
      HostRead rd(st);
      rd.add(&s.nchunks, s.cstart + s.nmulti, sizeof(int64_t));
      rd.add(&s.tree_nodes, s.cstart + s.ntree, sizeof(int64_t));
      rd.wait();
      s.owner = a.take<int32_t>(s.nchunks);
      chunk_owners(s.cstart, s.nmulti, s.owner, st);
      s.wnode = a.take<Pair>(s.nchunks * k);
      s.wflag = a.take<uint32_t>(s.nchunks);
      s.wcount = a.take<uint32_t>(s.nmulti * (k + 1));
    }
    return;
  }
  if (mode == MODE_EXACT) {
    int64_t pos = 0;
    for (int q = 0; q < 4; ++q) {
      s.tier[q] = order + pos;
      s.ntier[q] = (int64_t)h[q];
      pos += (int64_t)h[q];
    }
    s.nblock = (int64_t)h[CAT_BLOCK];
    if (s.ntier[3] > 0) {
      int64_t c3 = s.ntier[3];
      s.hbase = a.take<int64_t>(c3 + 1);
      int64_t *caps = a.take<int64_t>(c3);
      k_hash_caps<<<grid_for(c3), BLOCK, 0, st>>>(g.off, s.tier[3], c3, caps);
      MGCD_LAUNCHED();
      scan_i64(caps, s.hbase, c3, s.hbase + c3, a, st);
      int64_t *nseg = a.take<int64_t>(c3);
      s.sstart = a.take<int64_t>(c3 + 1);
      k_chunk_counts<<<grid_for(c3), BLOCK, 0, st>>>(g.off, s.tier[3], c3, GSEG, nseg);
      MGCD_LAUNCHED();
      scan_i64(nseg, s.sstart, c3, s.sstart + c3, a, st);
      int64_t *ntab = a.take<int64_t>(c3);
      s.tstart = a.take<int64_t>(c3 + 1);
      k_table_segs<<<grid_for(c3), BLOCK, 0, st>>>(s.hbase, c3, ntab);
      MGCD_LAUNCHED();
      scan_i64(ntab, s.tstart, c3, s.tstart + c3, a, st);
      int64_t tot = 0;  // table slots, insert and scan segments in one host round trip
      HostRead rd(st);
      rd.add(&tot, s.hbase + c3, sizeof(int64_t));
      rd.add(&s.nseg, s.sstart + c3, sizeof(int64_t));
      rd.add(&s.ntseg, s.tstart + c3, sizeof(int64_t));
      rd.wait();
      s.sowner = a.take<int32_t>(s.nseg);
      chunk_owners(s.sstart, c3, s.sowner, st);
      s.towner = a.take<int32_t>(s.ntseg);
      chunk_owners(s.tstart, c3, s.towner, st);
      s.gkd = a.take<uint32_t>(c3);
      s.pbest = a.take<int32_t>(s.ntseg);
      s.pgain = a.take<int64_t>(s.ntseg);
      s.htab = a.take<Pair>(tot);
      s.hpos = a.take<uint32_t>(tot);
      launch_slices(ceil_div(tot, BLOCK), BLOCK, [&](int64_t first, unsigned blocks) {
        k_gtab_clear<<<blocks, BLOCK, 0, st>>>(s.htab, s.hpos, tot, first);
        MGCD_LAUNCHED();
      });
    }
    return;
  }
  s.keybuf = a.take<uint32_t>(g.nnz);
  int64_t pos = 0;
  s.single = order;
  s.nsingle = (int64_t)h[0];
  s.light = order + s.nsingle;
  s.nlight = (int64_t)h[CAT_LIGHT];
  pos = s.nsingle + s.nlight;
  s.tier[0] = order + pos;  // short rows
  s.ntier[0] = (int64_t)h[CAT_SHORT];
  pos += s.ntier[0];
  for (int b = 1; b <= 6; ++b) {
    s.packed[b] = order + pos;
    s.npacked[b] = (int64_t)h[b];
    pos += (int64_t)h[b];
  }
  s.multi = order + pos;
  s.nmulti = (int64_t)h[7];
  if (s.nmulti > 0) {
    int64_t *nch = a.take<int64_t>(s.nmulti);
    s.cstart = a.take<int64_t>(s.nmulti + 1);
    k_chunk_counts<<<grid_for(s.nmulti), BLOCK, 0, st>>>(g.off, s.multi, s.nmulti, L, nch);
    MGCD_LAUNCHED();
    scan_i64(nch, s.cstart, s.nmulti, s.cstart + s.nmulti, a, st);
    int64_t *ng = a.take<int64_t>(s.nmulti);
    s.gstart = a.take<int64_t>(s.nmulti + 1);
    k_group_counts<<<grid_for(s.nmulti), BLOCK, 0, st>>>(s.cstart, s.nmulti, ng);
    MGCD_LAUNCHED();
    scan_i64(ng, s.gstart, s.nmulti, s.gstart + s.nmulti, a, st);
    // chunk and group totals in one host round trip
    HostRead rd(st);
    rd.add(&s.nchunks, s.cstart + s.nmulti, sizeof(int64_t));
    rd.add(&s.ngroups, s.gstart + s.nmulti, sizeof(int64_t));
    rd.wait();
    s.owner = a.take<int32_t>(s.nchunks);
    chunk_owners(s.cstart, s.nmulti, s.owner, st);
    s.gowner = a.take<int32_t>(s.ngroups);
    chunk_owners(s.gstart, s.nmulti, s.gowner, st);
    s.sk = a.take<Pair>(s.ngroups * k);
    s.skflag = a.take<uint32_t>(s.ngroups);
    s.part = a.take<uint32_t>(s.nchunks * (k + 1));
    s.cand = a.take<Pair>(s.nmulti * k);
    s.cflag = a.take<uint32_t>(s.nmulti);
  }
  {  // bucket table of k_move_rows, heaviest bucket first in the grid
    Buckets bk{};
    int64_t w = 0;
    for (int b = 6; b >= 0; --b) {
      const int64_t rows = b == 0 ? s.nsingle : s.npacked[b];
      bk.rows[b] = b == 0 ? s.single : s.packed[b];
      bk.nrows[b] = rows;
      bk.item_begin[b] = w;
      w += ceil_div(rows << b, WCH);
      bk.item_end[b] = w;
    }
    s.row_items = w;
    bk.ngroups = s.ngroups;
    bk.multi = s.multi;
    bk.gowner = s.gowner;
    bk.gstart = s.gstart;
    bk.cstart = s.cstart;
    bk.sk = s.sk;
    bk.skflag = s.skflag;
    s.buckets = bk;  // a kernel argument: no upload, no host round trip
  }
}

static void set_classes(Schedule &s, const SchedParams &sp);

void build_schedule(const Graph &g, const SchedParams &sp, Schedule &s, Arena &a, hipStream_t st) {
  build_lists(g, sp, s, a, st);
  set_classes(s, sp);
}

// ---- launch -------------------------------------------------------------------------

// Event i of a sweep bounds the kernel classes i - 1 and i: recorded (4 us of the stream's
// time each) only where one of them has kernels.
static inline void mark(const Schedule &s, hipEvent_t *ev, int i, hipStream_t st) {
  if (ev && (s.classes & (1u << i | (i > 0 ? 1u << (i - 1) : 0u)) & 7u)) MGCD_HIP(hipEventRecord(ev[i], st));
}

// The kernel classes that a sweep on this schedule has (bits, as launched below); `clock`:
// one class, whose first kernel writes SweepArgs::stamp.
static void set_classes(Schedule &s, const SchedParams &sp) {
  const bool shorts = s.ntail > 0 || s.shorts.wave[4] > 0;
  bool c[3];
  if (sp.wave) {
    c[0] = shorts;
    c[1] = s.ntier[1] > 0;
    c[2] = s.nmulti > 0;
  } else if (sp.mode == MODE_EXACT) {
    c[0] = shorts;
    c[1] = s.ntier[1] > 0 || s.ntier[2] > 0;
    c[2] = s.ntier[3] > 0;
  } else {
    c[0] = s.ngroups + s.row_items > 0 || s.nlight > 0;
    c[1] = s.nmulti > 0;
    c[2] = shorts;
  }
  s.classes = (c[0] ? 1u : 0u) | (c[1] ? 2u : 0u) | (c[2] ? 4u : 0u);
  const bool mg = !sp.wave && sp.mode != MODE_EXACT;
  s.clock = (s.classes == 1u && (mg || s.ntail == 0)) || (mg && s.classes == 4u);
}

// Compute units of the current device.
static int64_t compute_units() {
  int dev = 0, cus = 0;
  MGCD_HIP(hipGetDevice(&dev));
  MGCD_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  return cus > 0 ? cus : 1;
}

// One launch of the main sweep kernel over `items` work items; persistent (a.queue): as
// many workgroups as stay resident at once, each pulling work until the queue is empty.
template <int K, int ALGO, int MODE>
static void launch_rows(const SweepArgs &a, const Schedule &s, int64_t L, hipStream_t st) {
  const int64_t items = s.ngroups + s.row_items, lblocks = ceil_div(s.nlight, BLOCK / QUAD);
  const bool own = a.queue || items == 0;  // the light rows in a launch of their own
  if (items > 0) {
    if (a.queue) {
      const int64_t grid = std::min<int64_t>(items, compute_units() * row_waves_per_simd<K>());
      k_move_rows<K, ALGO, MODE, true><<<(unsigned)grid, BLOCK, 0, st>>>(a, s.buckets, L, s.keybuf, items, nullptr, 0,
                                                                        0, a.queue);
      MGCD_LAUNCHED();
    } else {
      launch_slices(items + lblocks, BLOCK, [&](int64_t first, unsigned blocks) {
        k_move_rows<K, ALGO, MODE, false><<<blocks, BLOCK, 0, st>>>(a, s.buckets, L, s.keybuf, items, s.light,
                                                                    s.nlight, first, nullptr);
        MGCD_LAUNCHED();
      });
    }
  }
  if (own && lblocks > 0) {
    if (a.queue) {
      const int64_t grid = std::min<int64_t>(lblocks, compute_units() * light_waves_per_simd<K>());
      k_move_light<K, ALGO, MODE, true><<<(unsigned)grid, BLOCK, 0, st>>>(a, s.light, s.nlight, 0,
                                                                         a.queue + QLANES * QSTRIDE);
      MGCD_LAUNCHED();
    } else {
      launch_slices(lblocks, BLOCK, [&](int64_t first, unsigned blocks) {
        k_move_light<K, ALGO, MODE, false><<<blocks, BLOCK, 0, st>>>(a, s.light, s.nlight, first, nullptr);
        MGCD_LAUNCHED();
      });
    }
  }
}

// Many graphs: from so many waves on the short rows of 8 and more entries go 64 to a wave,
// which then adds to a graph's counters once for 64 rows and passes over the rows of a graph
// that has stopped at one look.  63 graphs of equal rows, the first sweep with its set-up and
// a sweep in which all but one graph stand: 2.56 M rows of 23 entries 759 and 37 us, with 8
// rows to a wave 1317 and 99; of 11 entries 550 and 37, with 16 rows to a wave 874 and 63.
// At 160,000 rows (2500 waves) 194 us against 217, at 80,000 187 against 179, at 20,000 179
// against 156: a wave's items then take their turns on an idle chip.
constexpr int64_t SHORT_WIDE = 2048;

// Tier 0: the list's longer rows (a raised exact_small), then the short rows.
template <int ALGO, bool SMALL = false>
static void launch_short(const SweepArgs &a, const Schedule &s, hipStream_t st) {
  if (s.ntail > 0) {
    k_exact_small<ALGO><<<grid_for(s.ntail), BLOCK, 0, st>>>(a, s.tier[0], s.ntail);
    MGCD_LAUNCHED();
  }
  const auto launch = [&](auto kernel, const ShortRows &sr) {
    kernel<<<(unsigned)ceil_div(sr.wave[4], BLOCK / WAVE), BLOCK, 0, st>>>(a, s.tier[0] + s.ntail, sr);
    MGCD_LAUNCHED();
  };
  ShortRows wide = s.shorts;  // 64 rows per wave in the first two classes
  for (int q = 0; q < 4; ++q)
    wide.wave[q + 1] = wide.wave[q] + (q < 2 ? ceil_div(wide.row[q + 1] - wide.row[q], WAVE)
                                             : s.shorts.wave[q + 1] - s.shorts.wave[q]);
  if (a.gctr && wide.wave[2] >= SHORT_WIDE)
    launch(k_exact_short<ALGO, SMALL, true>, wide);
  else if (s.shorts.wave[4] > 0)
    launch(k_exact_short<ALGO, SMALL, false>, s.shorts);
}

template <int K, int ALGO, int MODE>
static void sweep_mg(const SweepArgs &a, const Schedule &s, int64_t L, hipStream_t st, hipEvent_t *ev) {
  mark(s, ev, 0, st);
  launch_rows<K, ALGO, MODE>(a, s, L, st);
  mark(s, ev, 1, st);
  // long rows: rest of the merge tree, pass 2, decision
  if (s.nmulti > 0) {
    launch_slices(s.nmulti, BLOCK, [&](int64_t first, unsigned blocks) {
      k_long_merge<K, ALGO><<<blocks, BLOCK, 0, st>>>(a, s.multi, s.gstart, first, s.sk, s.skflag, s.cand, s.cflag);
      MGCD_LAUNCHED();
    });
    launch_slices(ceil_div(s.nchunks, BLOCK / WAVE), BLOCK, [&](int64_t first, unsigned blocks) {
      k_long_count<K, ALGO><<<blocks, BLOCK, 0, st>>>(a, s.multi, s.owner, s.cstart, s.nchunks, L, first, s.cand,
                                                      s.cflag, s.keybuf, s.part);
      MGCD_LAUNCHED();
    });
    launch_slices(s.nmulti, BLOCK, [&](int64_t first, unsigned blocks) {
      k_long_decide<K, ALGO><<<blocks, BLOCK, 0, st>>>(a, s.multi, s.cstart, first, s.cand, s.cflag, s.part);
      MGCD_LAUNCHED();
    });
  }
  mark(s, ev, 2, st);
  launch_short<ALGO>(a, s, st);  // rows whose sketch is their exact table
  mark(s, ev, 3, st);
}

template <int ALGO, bool SMALL = false>
static void sweep_exact(const SweepArgs &a, const Schedule &s, hipStream_t st, hipEvent_t *ev) {
  mark(s, ev, 0, st);
  launch_short<ALGO, SMALL>(a, s, st);
  mark(s, ev, 1, st);
  if (s.ntier[1] > 0) {
    launch_slices(ceil_div(s.ntier[1], BLOCK / WAVE), BLOCK, [&](int64_t first, unsigned blocks) {
      k_exact_wave<ALGO, SMALL><<<blocks, BLOCK, 0, st>>>(a, s.tier[1], s.ntier[1], first);
      MGCD_LAUNCHED();
    });
  }
  if (s.ntier[2] > 0) {
    const int64_t big = s.ntier[2] - s.nblock;
    launch_slices(big, EXACT_T2_MAX / 4, [&](int64_t first, unsigned blocks) {
      k_exact_table<ALGO, EXACT_T2_MAX / 4, SMALL><<<blocks, EXACT_T2_MAX / 4, 0, st>>>(a, s.tier[2], first);
      MGCD_LAUNCHED();
    });
    launch_slices(s.nblock, EXACT_BLOCK_MAX / 4, [&](int64_t first, unsigned blocks) {
      k_exact_table<ALGO, EXACT_BLOCK_MAX / 4, SMALL><<<blocks, EXACT_BLOCK_MAX / 4, 0, st>>>(a, s.tier[2] + big,
                                                                                            first);
      MGCD_LAUNCHED();
    });
  }
  mark(s, ev, 2, st);
  if (s.ntier[3] > 0) {
    launch_slices(s.nseg, BLOCK, [&](int64_t first, unsigned blocks) {
      k_gtab_insert<ALGO, SMALL><<<blocks, BLOCK, 0, st>>>(a, s.tier[3], s.hbase, s.sstart, s.sowner, first, s.htab,
                                                           s.hpos);
      MGCD_LAUNCHED();
    });
    k_gtab_kd<ALGO><<<grid_for(s.ntier[3]), BLOCK, 0, st>>>(a, s.tier[3], s.ntier[3], s.hbase, s.htab, s.gkd);
    MGCD_LAUNCHED();
    launch_slices(s.ntseg, BLOCK, [&](int64_t first, unsigned blocks) {
      k_gtab_scan<ALGO, SMALL><<<blocks, BLOCK, 0, st>>>(a, s.tier[3], s.hbase, s.tstart, s.towner, first, s.htab,
                                                         s.hpos, s.gkd, s.pbest, s.pgain);
      MGCD_LAUNCHED();
    });
    k_gtab_finish<ALGO><<<grid_for(s.ntier[3]), BLOCK, 0, st>>>(a, s.tier[3], s.ntier[3], s.tstart, s.pbest,
                                                                s.pgain);
    MGCD_LAUNCHED();
  }
  mark(s, ev, 3, st);
}

template <int K, int ALGO, int MODE>
static void sweep_wave(const SweepArgs &a, const Schedule &s, int64_t L, hipStream_t st, hipEvent_t *ev) {
  mark(s, ev, 0, st);
  launch_short<ALGO>(a, s, st);  // rows that cannot lose weight
  mark(s, ev, 1, st);
  if constexpr (K <= WAVE) {  // K = 128 / 256: every row the sketch takes is a split row
    if (s.ntier[1] > 0) {
      const int depth = wave_tree_depth(WAVE_SPLIT, L);  // longer rows are one chunk or split
      launch_slices(ceil_div(s.ntier[1], BLOCK / WAVE), BLOCK, [&](int64_t first, unsigned blocks) {
        k_wave_rows<K, ALGO, MODE><<<blocks, BLOCK, BLOCK / WAVE * wave_tree_lds<K>(depth), st>>>(
            a, s.tier[1], s.ntier[1], L, depth, first, s.keybuf);
        MGCD_LAUNCHED();
      });
    }
  }
  mark(s, ev, 2, st);
  if (s.nmulti > 0) {  // split rows
    const int64_t groups = wave_group_blocks(K, s.nchunks);
    launch_slices(groups, wave_group_block(K), [&](int64_t first, unsigned blocks) {
      k_wave_chunks<K, ALGO, MODE><<<blocks, wave_group_block(K), 0, st>>>(
          a, s.multi, s.cstart, s.owner, s.nchunks, L, s.keybuf, first, s.wnode, s.wflag, s.wcount);
      MGCD_LAUNCHED();
    });
    const int64_t G = wave_group(K), maxch = (s.maxdeg + G * L - 1) / (G * L);
    int l = 0;
    for (; (maxch >> l) > TREE_NODES; ++l) {
      launch_slices(ceil_div(s.tree_nodes, BLOCK / WAVE), BLOCK, [&](int64_t first, unsigned blocks) {
        k_wave_level<K><<<blocks, BLOCK, 0, st>>>(a, s.multi, s.cstart, s.owner, s.tree_nodes, l, first, s.wnode,
                                                  s.wflag);
        MGCD_LAUNCHED();
      });
    }
    if (((int64_t)1 << l) < maxch) {
      launch_slices(s.ntree, TREE_BLOCK, [&](int64_t first, unsigned blocks) {
        k_wave_tree<K><<<blocks, TREE_BLOCK, 0, st>>>(a, s.multi, s.cstart, l, first, s.wnode, s.wflag);
        MGCD_LAUNCHED();
      });
    }
    if (second_pass(a, ALGO)) {
      launch_slices(groups, wave_group_block(K), [&](int64_t first, unsigned blocks) {
        k_wave_count<K, ALGO><<<blocks, wave_group_block(K), 0, st>>>(
            a, s.multi, s.cstart, s.owner, s.nchunks, L, first, s.keybuf, s.wnode, s.wflag, s.wcount);
        MGCD_LAUNCHED();
      });
    }
    launch_slices(ceil_div(s.nmulti, BLOCK / WAVE), BLOCK, [&](int64_t first, unsigned blocks) {
      k_wave_decide<K, ALGO><<<blocks, BLOCK, 0, st>>>(a, s.multi, s.cstart, s.nmulti, first, s.wnode, s.wflag,
                                                       s.wcount);
      MGCD_LAUNCHED();
    });
  }
  mark(s, ev, 3, st);
}

template <int ALGO, int MODE>
static void sweep_k(const SweepArgs &a, const Schedule &s, int k, int64_t L, hipStream_t st,
                    hipEvent_t *ev) {
  switch (k) {
    case 32: sweep_wave<32, ALGO, MODE>(a, s, L, st, ev); break;
    case 64: sweep_wave<64, ALGO, MODE>(a, s, L, st, ev); break;
    case 128: sweep_wave<128, ALGO, MODE>(a, s, L, st, ev); break;
    case 256: sweep_wave<256, ALGO, MODE>(a, s, L, st, ev); break;
    case 1: sweep_mg<1, ALGO, MODE>(a, s, L, st, ev); break;
    case 2: sweep_mg<2, ALGO, MODE>(a, s, L, st, ev); break;
    case 4: sweep_mg<4, ALGO, MODE>(a, s, L, st, ev); break;
    case 8: sweep_mg<8, ALGO, MODE>(a, s, L, st, ev); break;
    case 16: sweep_mg<16, ALGO, MODE>(a, s, L, st, ev); break;
    default: throw Error(-6, "k must be 1, 2, 4, 8, 16, 32, 64, 128 or 256");
  }
}

template <int ALGO>
static void sweep_algo(const SweepArgs &a, const Schedule &s, int mode, int k, int64_t L,
                       hipStream_t st, hipEvent_t *ev) {
  switch (mode) {
    case MODE_EXACT: sweep_exact<ALGO>(a, s, st, ev); break;
    case MODE_SMALL: {  // the exact kernels keyed by small-table slots (k of them)
      SweepArgs b = a;
      b.small_slots = k;
      sweep_exact<ALGO, true>(b, s, st, ev);
      break;
    }
    case MODE_ALG1: sweep_k<ALGO, MODE_ALG1>(a, s, k, L, st, ev); break;
    case MODE_UNCOND: sweep_k<ALGO, MODE_UNCOND>(a, s, k, L, st, ev); break;
    case MODE_STD: sweep_k<ALGO, MODE_STD>(a, s, k, L, st, ev); break;
    default: throw Error(-6, "unknown sketch mode");
  }
}

void launch_sweep(const SweepArgs &a, const Schedule &s, int algo, int mode, int k, int64_t L,
                  hipStream_t st, hipEvent_t *ev) {
  switch (algo) {
    case ALGO_LPA: sweep_algo<ALGO_LPA>(a, s, mode, k, L, st, ev); break;
    case ALGO_MOVE: sweep_algo<ALGO_MOVE>(a, s, mode, k, L, st, ev); break;
    case ALGO_REFINE: sweep_algo<ALGO_REFINE>(a, s, mode, k, L, st, ev); break;
    default: throw Error(-1, "unknown sweep");
  }
}

// ---- bookkeeping kernels ---------------------------------------------------------------

// Run by one whole wave: each lane takes its copy of the sweep's counters.
__device__ inline void level_converge(int algo, const LevelRule &r) {
  // Read and clear in one atomic step: a plain load of these addresses may overtake the
  // store of 0 that follows it.
  static_assert(SPREAD == WAVE, "one copy of the counters per lane");
  unsigned long long *ctr = r.ctr + lane_id() * CTR_STRIDE;
  const unsigned long long moved = wave_sum(atomicExch(&ctr[0], 0ull)), prop = wave_sum(atomicExch(&ctr[1], 0ull)),
                           sumG = wave_sum(atomicExch(&ctr[2], 0ull)), cands = wave_sum(atomicExch(&ctr[3], 0ull));
  if (lane_id() != 0) return;
  LevelState *ls = r.ls;
  if (ls->halt) return;
  ls->cands += cands;
  ls->sweeps += 1;
  ls->edges += (unsigned long long)r.nnz;
  ls->moved_last = moved;
  if (r.stamp) {
    const uint64_t now = wall_clock64(), then = *r.stamp;
    ls->ticks += now > then ? now - then : 0;
  }
  const bool stop = algo == ALGO_LPA ? (double)moved <= r.tol * (double)r.n
                                     : prop == 0 || 2.0 * (double)sumG <= r.tol * r.WW;
  if (stop) ls->halt = 1;
}

__global__ void k_apply_moves(const int32_t *Cold, const int32_t *Cnew, const uint32_t *K, uint32_t *Sig,
                              int32_t n, LevelRule rule) {
  int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (rule.live && *rule.live == 0) return;  // batched: the sweep did nothing
  if (rule.ls && i < WAVE) level_converge(ALGO_MOVE, rule);  // the sweep's counters are final
  if (i >= n) return;
  int32_t d = Cold[i], c = Cnew[i];
  if (c == d) return;
  uint32_t k = K[i];
  atomicSub(&Sig[d], k);
  atomicAdd(&Sig[c], k);
}

void launch_apply_moves(const int32_t *Cold, const int32_t *Cnew, const uint32_t *K, uint32_t *Sig,
                        int32_t n, hipStream_t st, const LevelRule *rule) {
  const LevelRule r = rule ? *rule : LevelRule{};
  if (n <= 0 && !rule) return;
  k_apply_moves<<<n > 0 ? grid_for(n) : 1, BLOCK, 0, st>>>(Cold, Cnew, K, Sig, n, r);
  MGCD_LAUNCHED();
}

__global__ void k_zero_totals(uint32_t *Sig, int32_t n) {
  int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) Sig[i] = 0;
}

__global__ void k_totals(const int32_t *C, const uint32_t *K, uint32_t *Sig, int32_t n) {
  int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) atomicAdd(&Sig[C[i]], K[i]);
}

void launch_community_totals(const int32_t *C, const uint32_t *K, uint32_t *Sig, int32_t n,
                             hipStream_t st) {
  if (n <= 0) return;
  k_zero_totals<<<grid_for(n), BLOCK, 0, st>>>(Sig, n);
  MGCD_LAUNCHED();
  k_totals<<<grid_for(n), BLOCK, 0, st>>>(C, K, Sig, n);
  MGCD_LAUNCHED();
}

__global__ void k_count_proposals(const int32_t *prop, int32_t *nprop, int32_t *from, int32_t n) {
  int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i >= n) return;
  int32_t t = prop[i];
  if (t != (int32_t)i) {
    atomicAdd(&nprop[t], 1);
    from[t] = (int32_t)i;  // read only where exactly one vertex proposed t
  }
}

__global__ void k_accept(const int32_t *prop, const int32_t *nprop, const int32_t *from, int32_t *R,
                         int32_t n) {
  int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i >= n) return;
  int32_t t = prop[i];
  bool ok = t != (int32_t)i &&
            (nprop[i] == 0 || (nprop[i] == 1 && from[i] == t && t < (int32_t)i));
  R[i] = ok ? t : (int32_t)i;
}

void launch_refine_accept(const int32_t *prop, int32_t *nprop, int32_t *from, int32_t *R, int32_t n,
                          hipStream_t st) {
  if (n <= 0) return;
  launch_fill_i32(nprop, 0, n, st);
  k_count_proposals<<<grid_for(n), BLOCK, 0, st>>>(prop, nprop, from, n);
  MGCD_LAUNCHED();
  k_accept<<<grid_for(n), BLOCK, 0, st>>>(prop, nprop, from, R, n);
  MGCD_LAUNCHED();
}

__global__ void k_fill_i32(int32_t *p, int32_t v, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) p[i] = v;
}
__global__ void k_iota(int32_t *p, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) p[i] = (int32_t)i;
}
__global__ void k_level_converge(int algo, LevelRule r) { level_converge(algo, r); }

void launch_level_converge(int algo, const LevelRule &r, hipStream_t st) {
  k_level_converge<<<1, WAVE, 0, st>>>(algo, r);
  MGCD_LAUNCHED();
}

// A level's start: its state and the sweep counters (may be null) cleared.
__global__ void k_level_start(LevelState *ls, unsigned long long *ctr) {
  if (threadIdx.x == 0) *ls = LevelState{0, 0, 0, 0, 0, 0};
  if (ctr)
    for (int64_t i = threadIdx.x; i < CTR_WORDS; i += BLOCK) ctr[i] = 0;
}

void launch_level_start(LevelState *ls, unsigned long long *ctr, hipStream_t st) {
  k_level_start<<<1, BLOCK, 0, st>>>(ls, ctr);
  MGCD_LAUNCHED();
}

__global__ void k_zero_u64(unsigned long long *p, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * BLOCK + threadIdx.x;
  if (i < n) p[i] = 0;
}

void launch_fill_i32(int32_t *p, int32_t v, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  k_fill_i32<<<grid_for(n), BLOCK, 0, st>>>(p, v, n);
  MGCD_LAUNCHED();
}
void launch_iota(int32_t *p, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  k_iota<<<grid_for(n), BLOCK, 0, st>>>(p, n);
  MGCD_LAUNCHED();
}
void launch_zero_u64(unsigned long long *p, int64_t n, hipStream_t st) {
  if (n <= 0) return;
  k_zero_u64<<<grid_for(n), BLOCK, 0, st>>>(p, n);
  MGCD_LAUNCHED();
}

}  // namespace mgcd
