// The weighted Misra-Gries sketch spread over a wavefront, for K = 32, 64, 128 or 256
// slots (Appendix A.1, Algorithm 1, and its variants): slot p lives in lane p mod 64,
// register p / 64.  Stream items arrive wave-uniform (the same (c, w) in every lane);
// matching a key is one compare per slot register plus a ballot, and the free slot
// that takes a new key is the first free one (slot placement does not change the
// sketch's positive entries).
#pragma once
#include "common.hpp"

namespace mgcd {

__device__ inline int first_lane(uint64_t m) { return __builtin_ctzll(m); }

template <typename T>
__device__ inline T lane_value(T v, int lane) {  // v of `lane` (wave-uniform lane)
  return (T)__builtin_amdgcn_readlane((int)v, lane);
}

// Slots per lane of a K-slot wave sketch: one for K <= 64, K / 64 for 128 and 256
// (slot p = s * 64 + lane lives in lane `lane`, register s).
template <int K>
struct WaveSlots {
  static_assert(K == 32 || K == 64 || K == 128 || K == 256, "wave sketch sizes");
  static constexpr int S = K <= WAVE ? 1 : K / WAVE;
  // lanes whose slot s exists (all lanes unless K < 64)
  static constexpr uint64_t VALID = K >= WAVE ? ~0ull : ((1ull << K) - 1);
};

template <int K, int MODE>
struct WaveSketch {
  static constexpr int S = WaveSlots<K>::S;
  static constexpr uint64_t VALID = WaveSlots<K>::VALID;
  uint32_t key[S], val[S];  // this lane's slots (lanes >= K stay empty)
  bool lossy;               // wave-uniform

  __device__ inline void reset() {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      key[s] = EMPTY;
      val[s] = 0;
    }
    lossy = false;
  }

  // The first free slot (value 0; register-major, then lowest lane) takes (c, w);
  // returns false (wave-uniform) when every slot is in use.
  __device__ inline bool insert(uint32_t c, uint32_t w) {
    const int lane = lane_id();
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const uint64_t fr = __ballot(val[s] == 0) & VALID;
      if (fr) {
        if (lane == first_lane(fr)) {
          key[s] = c;
          val[s] = w;
        }
        return true;
      }
    }
    return false;
  }

  // Add w to the slot whose key is c (present: value positive, or any value for
  // Algorithm 1, whose stale keys revive); false (wave-uniform) when c has none.
  __device__ inline bool add(uint32_t c, uint32_t w, bool positive_only) {
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const bool m = key[s] == c && (!positive_only || val[s] > 0);
      if (__ballot(m) & VALID) {
        if (m) val[s] += w;
        return true;
      }
    }
    return false;
  }

  // Add (c, w) (wave-uniform, c != EMPTY); true (wave-uniform) if the slots lost weight.
  __device__ inline bool update(uint32_t c, uint32_t w) {
    const int lane = lane_id();
    if constexpr (MODE == MODE_ALG1) {
      // accumulate into the slot holding c (a stale key revives); else the first free
      // slot; else subtract w from every slot (clamped at 0) and drop the item
      if (add(c, w, false)) return false;
      if (insert(c, w)) return false;
      lossy = true;
#pragma unroll
      for (int s = 0; s < S; ++s) val[s] = val[s] > w ? val[s] - w : 0u;
      return true;
    } else if constexpr (MODE == MODE_UNCOND) {
      // present = positive; on a miss subtract w from every slot, then insert
      if (add(c, w, true)) return false;
      bool any = false;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        any |= (__ballot(val[s] > 0) & VALID) != 0;
        val[s] = val[s] > w ? val[s] - w : 0u;
      }
      const bool put = insert(c, w);
      lossy |= any || !put;
      return true;
    } else {  // MODE_STD: textbook weighted MG
      if (add(c, w, true)) return false;
      if (insert(c, w)) return false;
      lossy = true;
      uint32_t d = ~0u;
#pragma unroll
      for (int s = 0; s < S; ++s) {
        const uint32_t x = lane < K ? val[s] : ~0u;
        d = x < d ? x : d;
      }
#pragma unroll
      for (int o = WAVE / 2; o > 0; o >>= 1) {
        const uint32_t x = __shfl_xor(d, o);
        d = x < d ? x : d;
      }
      d = d < w ? d : w;
      if (lane < K) {
#pragma unroll
        for (int s = 0; s < S; ++s) val[s] -= d;
      }
      const uint32_t rest = w - d;
      if (rest > 0) insert(c, rest);
      return true;
    }
  }

  __device__ inline int free_slots() const {
    int n = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) n += __popcll(__ballot(val[s] == 0) & VALID);
    return n;
  }

  // Keep only the candidates (positive slots); other keys become EMPTY.
  __device__ inline void finalize() {
#pragma unroll
    for (int s = 0; s < S; ++s) key[s] = val[s] > 0 ? key[s] : EMPTY;
  }
};

// A map of 32-bit keys to summed weights in one wave's LDS, one item per lane at a time:
// open addressing over H cells, a key's cell claimed by compare-and-swap.  While no more
// than K different keys have come the sketch of a stream is this map whatever the order of
// its items (Algorithm 1 and the textbook rule only take weight away at the (K + 1)-th),
// so 64 items go in with one probe loop instead of 64 wave-uniform updates of about ten
// instructions each.  A batch adds at most 64 keys to at most K, a merge K keys to K: at
// most half of the H cells are ever in use, every probe loop ends, and the longest of a
// wave's 64 probe chains stays short (with 2 K cells a merge of full sketches filled the
// table, and k_wave_chunks of R-MAT 2^18's first sweeps took 215 us; with 4 K it is 93).
template <int K>
struct WaveMap {
  static constexpr int S = WaveSlots<K>::S;
  static constexpr int BITS = K <= 64 ? 8 : K == 128 ? 9 : 10;
  static constexpr int H = 1 << BITS;      // >= 2 (K + 64) and >= 4 K
  static constexpr int CELLS = H / WAVE;   // cells per lane
  static constexpr int WORDS = 2 * H;      // LDS words of one wave
  uint32_t *key, *val;  // LDS, H each

  __device__ inline explicit WaveMap(uint32_t *lds) : key(lds), val(lds + H) {}

  __device__ inline void clear() {
#pragma unroll
    for (int c = 0; c < CELLS; ++c) {
      key[c * WAVE + lane_id()] = EMPTY;
      val[c * WAVE + lane_id()] = 0;
    }
    wave_sync();
  }

  // The cells tried for c: from h in steps of `step` (odd, so that it visits every cell).
  struct Probe {
    uint32_t h, step;
    __device__ inline explicit Probe(uint32_t c) {
      const uint32_t x = c * 0x9E3779B1u;
      h = x >> (32 - BITS);
      step = (x >> 7) | 1u;
    }
    __device__ inline void next() { h = (h + step) & (H - 1); }
  };

  // The cell of c (c != EMPTY), claimed if c has none yet; fresh: this lane claimed it.
  __device__ inline uint32_t claim(uint32_t c, bool &fresh) {
    Probe p(c);
    for (;;) {
      const uint32_t old = atomicCAS(&key[p.h], EMPTY, c);
      fresh = old == EMPTY;
      if (fresh || old == c) return p.h;
      p.next();
    }
  }

  // Add the items (c != EMPTY) of lanes t and up to a map of `used` keys, up to the lane
  // returned (64: all of them): the items of the lanes before it bring at most K keys in
  // all.  When it returns less than 64, `used` no longer holds and the map is only good
  // for take().
  __device__ inline int add(uint32_t c, uint32_t w, int t, int &used) {
    const bool in = c != EMPTY && lane_id() >= t;
    bool fresh = false, miss = false;
    uint32_t h = 0;
    if (in) h = claim(c, fresh);
    int upto = WAVE;
    const int free = K - used;
    used += __popcll(__ballot(fresh));
    if (used > K) {  // up to the lane whose item may be the first without a slot
      if (in) miss = val[h] == 0;
      wave_sync();
      const uint64_t m = __ballot(miss);
      const uint64_t over = __ballot(miss && __popcll(m & lanemask_lt()) == free);
      upto = over ? first_lane(over) : WAVE - 1;
    }
    if (in && lane_id() < upto) atomicAdd(&val[h], w);
    return upto;
  }

  // The positive slots of a sketch in place of what the map held: their cells and number.
  __device__ inline int load(const uint32_t (&ck)[S], const uint32_t (&cv)[S], uint32_t (&cell)[S]) {
    int n = 0;
    bool fresh;
    clear();
#pragma unroll
    for (int s = 0; s < S; ++s) {
      cell[s] = 0;
      if (cv[s] > 0) {
        cell[s] = claim(ck[s], fresh);
        val[cell[s]] = cv[s];
      }
      n += __popcll(__ballot(cv[s] > 0));
    }
    wave_sync();
    return n;
  }

  // Add w to the cell of c if c (!= EMPTY) has one; the map holds fewer than H keys.
  __device__ inline void add_present(uint32_t c, uint32_t w) {
    Probe p(c);
    for (;;) {
      const uint32_t k = key[p.h];
      if (k == c) atomicAdd(&val[p.h], w);
      if (k == c || k == EMPTY) return;
      p.next();
    }
  }

  // The positive entries among the wave's N per lane (at most K) as slots; other slots are
  // EMPTY with value 0.  The map's contents are gone afterwards.
  template <int N>
  __device__ inline void pack(const uint32_t (&xk)[N], const uint32_t (&xv)[N], uint32_t (&ck)[S],
                              uint32_t (&cv)[S]) {
    const int lane = lane_id();
    wave_sync();  // every lane has read the map
    int n = 0;
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const uint64_t m = __ballot(xv[c] > 0);
      const int r = n + __popcll(m & lanemask_lt());
      if (xv[c] > 0) {
        key[r] = xk[c];
        val[r] = xv[c];
      }
      n += __popcll(m);
    }
    wave_sync();
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const bool in = s * WAVE + lane < n;
      ck[s] = in ? key[s * WAVE + lane] : EMPTY;
      cv[s] = in ? val[s * WAVE + lane] : 0u;
    }
    wave_sync();
  }

  __device__ inline void take(uint32_t (&ck)[S], uint32_t (&cv)[S]) {
    uint32_t xk[CELLS], xv[CELLS];
    wave_sync();
#pragma unroll
    for (int c = 0; c < CELLS; ++c) {
      xk[c] = key[c * WAVE + lane_id()];
      xv[c] = val[c * WAVE + lane_id()];
    }
    pack(xk, xv, ck, cv);
  }

  // Merge sketch (bk, bv) into (ak, av) (mergeable summaries, Agarwal et al. 2012): add
  // the values of equal keys; if more than K keys are positive, subtract the (K+1)-th
  // largest value from all and keep the positive ones.  Returns true (wave-uniform)
  // when the threshold step removed weight.
  // A key's partner is found in the map: matching slot by slot took two loops of up to K
  // rounds, 2.5 us a merge at K = 64, and that was most of a level of the merge tree.
  __device__ inline bool merge(uint32_t (&ak)[S], uint32_t (&av)[S], const uint32_t (&bk)[S],
                               const uint32_t (&bv)[S]) {
    uint32_t cell[S], xk[2 * S], xv[2 * S];  // a's slots and those of b that a has not
    int cnt = load(ak, av, cell);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      bool fresh = false;
      if (bv[s] > 0) {
        const uint32_t h = claim(bk[s], fresh);
        if (!fresh) val[h] += bv[s];  // a sketch's keys differ: no other lane has this cell
      }
      xk[S + s] = bk[s];
      xv[S + s] = fresh ? bv[s] : 0u;
      cnt += __popcll(__ballot(fresh));
    }
    wave_sync();
#pragma unroll
    for (int s = 0; s < S; ++s) {
      xk[s] = ak[s];
      xv[s] = av[s] > 0 ? val[cell[s]] : 0u;
    }
    const bool lossy = cnt > K;
    if (lossy) {
      // t = the largest value with at least K+1 values >= it (the (K+1)-th largest)
      const auto at_least = [&](uint32_t v) {
        int ge = 0;
#pragma unroll
        for (int c = 0; c < 2 * S; ++c) ge += __popcll(__ballot(xv[c] >= v));
        return ge;
      };
      uint32_t t = 0;
      for (int bit = at_least(1u << 16) ? 31 : at_least(1u << 8) ? 15 : 7; bit >= 0; --bit) {
        const uint32_t cand = t | (1u << bit);
        if (at_least(cand) >= K + 1) t = cand;
      }
#pragma unroll
      for (int c = 0; c < 2 * S; ++c) xv[c] = xv[c] > t ? xv[c] - t : 0u;
    }
    pack(xk, xv, ak, av);
    return lossy;
  }
};

// The sketch of one chunk, positions lo .. hi - 1 of a stream, as slots (positive ones
// first or not, others EMPTY); load(e, in, key, w) gives position e (EMPTY, 0 unless `in`).
// Returns true (wave-uniform) if it lost weight.
// Batches of 64 items go into the map while at most K keys are in use.  From the first item
// that may be the (K + 1)-th key on they are folded one by one, until a step that takes
// weight leaves REFILL slots free, which is worth another turn with the map (a map's turn
// costs about as much as a dozen items).  Leiden on R-MAT 2^18 at K = 64 and 32: 2.93 and
// 3.07 ms with 16, 2.91 and 2.88 with 8, 3.18 and 3.55 with 32, 3.06 and 3.11 without ever
// going back; at K = 64 on a Chung-Lu graph of 1 M vertices 9.98, 9.91, 10.57 and 10.53.
// The unconditional rule takes weight at every miss and is folded one by one throughout.
template <int K, int MODE, typename Load>
__device__ inline bool wave_chunk(WaveMap<K> map, int64_t lo, int64_t hi, const Load &load,
                                  uint32_t (&ck)[WaveSlots<K>::S], uint32_t (&cv)[WaveSlots<K>::S]) {
  constexpr int REFILL = 16;
  WaveSketch<K, MODE> s;
  s.reset();
  bool fold = MODE == MODE_UNCOND;  // the sketch is in s, else in the map
  int used = 0;
  if (!fold) map.clear();
  uint32_t key, w;
  load(lo + lane_id(), lo + lane_id() < hi, key, w);
  for (int64_t e0 = lo; e0 < hi; e0 += WAVE) {
    uint32_t nkey = EMPTY, nw = 0;  // the next batch is on its way while this one is folded
    if (e0 + WAVE < hi) load(e0 + WAVE + lane_id(), e0 + WAVE + lane_id() < hi, nkey, nw);
    const int nb = hi - e0 < WAVE ? (int)(hi - e0) : WAVE;
    bool refill = MODE != MODE_UNCOND && fold && s.free_slots() >= REFILL;
    for (int t = 0; t < nb;) {
      if (refill) {
        uint32_t cell[WaveSlots<K>::S];
        used = map.load(s.key, s.val, cell);
        fold = false;
        refill = false;
      }
      if (!fold) {
        t = map.add(key, w, t, used);
        if (t >= nb) break;
        map.take(s.key, s.val);
        fold = true;
      }
      while (t < nb && !refill) {
        const uint32_t c = lane_value(key, t);
        if (c != EMPTY && s.update(c, lane_value(w, t)) && MODE != MODE_UNCOND)
          refill = nb - t > REFILL && s.free_slots() >= REFILL;
        ++t;
      }
    }
    key = nkey;
    w = nw;
  }
  if (!fold) {
    map.take(ck, cv);
    return s.lossy;
  }
  s.finalize();
#pragma unroll
  for (int q = 0; q < WaveSlots<K>::S; ++q) {
    ck[q] = s.key[q];
    cv[q] = s.val[q];
  }
  return s.lossy;
}

// The fixed merge tree over a stream's chunk sketches, kept as a binary counter:
// level l of `stack` (LDS, `depth` levels of 2 x 64 words) holds the merged sketch of
// the last complete aligned run of 2^l chunks.  push() merges a finished chunk
// sketch in (left operand = the older run); result() merges the pending runs from
// the right, which is the order of the level-by-level tree with an odd last node
// carried up.  A stream of fewer than 2^depth chunks fits.
// One wave's LDS is its map and its stack.
inline int wave_tree_depth(int64_t max_len, int64_t L) {  // streams of max_len positions, or one chunk
  const int64_t chunks = L >= max_len ? 1 : ceil_div(max_len, L);
  int d = 1;
  while (chunks >> d) ++d;
  return d;
}
template <int K>
constexpr size_t wave_tree_lds(int depth) {
  return (size_t)(WaveMap<K>::WORDS + depth * 2 * WAVE) * sizeof(uint32_t);
}

template <int K>
struct WaveTree {
  WaveMap<K> map;
  uint32_t *stack;
  int depth;
  uint32_t mask = 0;  // occupied levels (wave-uniform)
  bool lossy = false;

  __device__ inline WaveTree(uint32_t *lds, int d) : map(lds), stack(lds + WaveMap<K>::WORDS), depth(d) {}

  __device__ inline void put(int l, const uint32_t (&k)[1], const uint32_t (&v)[1]) {
    stack[(2 * l) * WAVE + lane_id()] = k[0];
    stack[(2 * l + 1) * WAVE + lane_id()] = v[0];
  }
  __device__ inline void get(int l, uint32_t (&k)[1], uint32_t (&v)[1]) const {
    k[0] = stack[(2 * l) * WAVE + lane_id()];
    v[0] = stack[(2 * l + 1) * WAVE + lane_id()];
  }

  __device__ inline void push(uint32_t (&k)[1], uint32_t (&v)[1]) {
    int l = 0;
    while ((mask >> l) & 1u) {
      uint32_t lk[1], lv[1];
      get(l, lk, lv);
      lossy |= map.merge(lk, lv, k, v);
      k[0] = lk[0];
      v[0] = lv[0];
      mask &= ~(1u << l);
      ++l;
    }
    put(l, k, v);
    mask |= 1u << l;
  }

  // The root (empty if no chunk was pushed).
  __device__ inline void result(uint32_t (&k)[1], uint32_t (&v)[1]) {
    k[0] = EMPTY;
    v[0] = 0;
    bool have = false;
    for (int l = 0; l < depth; ++l) {
      if (!((mask >> l) & 1u)) continue;
      uint32_t lk[1], lv[1];
      get(l, lk, lv);
      if (have) lossy |= map.merge(lk, lv, k, v);
      k[0] = lk[0];
      v[0] = lv[0];
      have = true;
    }
    k[0] = v[0] > 0 ? k[0] : EMPTY;
  }
};

// Chunks of a split stream that share a workgroup, a chunk per wave, and become one node of
// the stream's merge tree: the first three levels need no launch and no trip to memory.
// With K = 128 and 256 every stream past the short ones is split and most are one chunk,
// so there a node is a chunk and a workgroup has four.
constexpr int wave_group(int k) { return k <= WAVE ? 8 : 1; }
constexpr int wave_group_waves(int k) { return k <= WAVE ? 8 : BLOCK / WAVE; }
constexpr int wave_group_block(int k) { return wave_group_waves(k) * WAVE; }
inline int64_t wave_group_blocks(int k, int64_t nodes) {
  return wave_group(k) > 1 ? nodes : ceil_div(nodes, wave_group_waves(k));
}

// The levels of the fixed merge tree within a workgroup's `n` chunk sketches (K <= 64, wave
// w holds chunk w in ck, cv); the root is wave 0's.  Every wave of the workgroup calls it.
template <int K>
__device__ inline void merge_group(WaveMap<K> map, Pair (*snode)[K], uint32_t *sflag, int wave, int64_t n,
                                   uint32_t (&ck)[1], uint32_t (&cv)[1], bool &lossy) {
  const int lane = lane_id();
#pragma unroll 1
  for (int half = 1; half < wave_group(K); half *= 2) {
    const int place = wave & (2 * half - 1);
    if (place == half) {
      if (lane < K) snode[wave][lane] = Pair{ck[0], cv[0]};
      if (lane == 0) sflag[wave] = lossy ? 1u : 0u;
    }
    __syncthreads();
    if (place == 0 && wave + half < n) {
      const Pair b = lane < K ? snode[wave + half][lane] : Pair{EMPTY, 0};
      const uint32_t bk[1] = {b.key}, bv[1] = {b.val};
      const bool taken = map.merge(ck, cv, bk, bv);
      lossy |= taken || uniform(sflag[wave + half]) != 0;
    }
  }
}

// Nodes q and r (K pairs each) of a merge tree become node q; returns true (wave-uniform)
// if that lost weight.
template <int K>
__device__ inline bool merge_nodes(WaveMap<K> map, Pair *node, int64_t q, int64_t r) {
  constexpr int S = WaveSlots<K>::S;
  const int lane = lane_id();
  uint32_t ak[S], av[S], bk[S], bv[S];
#pragma unroll
  for (int u = 0; u < S; ++u) {
    const int p = u * WAVE + lane;
    const Pair none{EMPTY, 0};
    const Pair pa = p < K ? node[q * K + p] : none, pb = p < K ? node[r * K + p] : none;
    ak[u] = pa.key;
    av[u] = pa.val;
    bk[u] = pb.key;
    bv[u] = pb.val;
  }
  const bool lossy = map.merge(ak, av, bk, bv);
#pragma unroll
  for (int u = 0; u < S; ++u)
    if (u * WAVE + lane < K) node[q * K + u * WAVE + lane] = Pair{ak[u], av[u]};
  return lossy;
}

}  // namespace mgcd
