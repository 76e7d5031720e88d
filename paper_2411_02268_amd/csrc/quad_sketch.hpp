// A K-slot (K <= 16) weighted Misra-Gries sketch spread over a quad of lanes: slot
// 4p + q lives in register p of the quad's lane q, so one stream's chain of updates is
// about a third as long as with all slots in one lane, and a wave holds 16 streams,
// whose entries fit in LDS whole.  The lanes of a quad see the same items and take the
// same branches; they agree through DPP quad permutes (no LDS).  The sketch depends on the
// stream only, not on which free slot a new key takes (a slot of value 0 is free; reviving
// a stale key equals inserting it afresh).
#pragma once
#include "common.hpp"

namespace mgcd {

constexpr int QUAD = 4;

template <int CTRL>
__device__ inline uint32_t quad_perm(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, true);
}
// lanes [1,0,3,2], [2,3,0,1], [3,2,1,0], [1,2,3,0]; and lane 7 - x of each eight
constexpr int QP_XOR1 = 0xB1, QP_XOR2 = 0x4E, QP_XOR3 = 0x1B, QP_ROT1 = 0x39, QP_HALF_MIRROR = 0x141, QP_MIRROR = 0x140;

// The value of the quad's lane J.
template <int J>
__device__ inline uint32_t quad_bcast(uint32_t x) {
  return quad_perm<J * 0x55>(x);
}
__device__ inline uint32_t quad_or(uint32_t x) {
  x |= quad_perm<QP_XOR1>(x);
  return x | quad_perm<QP_XOR2>(x);
}
__device__ inline uint32_t quad_sum(uint32_t x) {
  x += quad_perm<QP_XOR1>(x);
  return x + quad_perm<QP_XOR2>(x);
}
__device__ inline uint32_t umin(uint32_t a, uint32_t b) { return a < b ? a : b; }
__device__ inline uint32_t umax(uint32_t a, uint32_t b) { return a > b ? a : b; }
__device__ inline uint32_t sub_sat(uint32_t a, uint32_t b) { return a > b ? a - b : 0u; }
__device__ inline uint32_t quad_min(uint32_t x) {
  x = umin(x, quad_perm<QP_XOR1>(x));
  return umin(x, quad_perm<QP_XOR2>(x));
}
__device__ inline uint32_t quad_max(uint32_t x) {
  x = umax(x, quad_perm<QP_XOR1>(x));
  return umax(x, quad_perm<QP_XOR2>(x));
}

template <int K, int MODE>
struct QuadSketch {
  static constexpr int S = K >= QUAD ? K / QUAD : 1;  // slots per lane
  uint32_t key[S];
  uint32_t val[S];
  uint32_t lost;  // nonzero in some lane of the quad: counted weight was removed

  // K < 4: only the first K lanes of the quad hold a slot
  __device__ static bool slot_here() { return K >= QUAD || (lane_id() & (QUAD - 1)) < K; }

  __device__ inline void reset() {
#pragma unroll
    for (int p = 0; p < S; ++p) {
      key[p] = EMPTY;
      val[p] = 0;
    }
    lost = 0;
  }

  // The quad's lowest-numbered free slot (p * QUAD + lane), or NONE.
  static constexpr uint32_t NONE = 255;
  __device__ inline uint32_t free_slot() const {
    const uint32_t q = lane_id() & (QUAD - 1);
    uint32_t f = NONE;
#pragma unroll
    for (int p = S - 1; p >= 0; --p) f = val[p] == 0 ? (uint32_t)(p * QUAD) + q : f;
    if (K < QUAD) f = slot_here() ? f : NONE;
    return quad_min(f);
  }
  __device__ inline void put(uint32_t f, uint32_t c, uint32_t w) {
    const uint32_t q = lane_id() & (QUAD - 1);
#pragma unroll
    for (int p = 0; p < S; ++p) {
      const bool t = f == (uint32_t)(p * QUAD) + q;
      key[p] = t ? c : key[p];
      val[p] = t ? w : val[p];
    }
  }

  // Add (c, w).  A skipped entry is passed as (EMPTY, 0): it leaves every value, every
  // positive slot's key and `lost` as they are.
  __device__ MGCD_INLINE void update(uint32_t c, uint32_t w) {
    uint32_t hit = 0;  // the weight taken up by a slot holding c (w > 0 for a real entry)
#pragma unroll
    for (int p = 0; p < S; ++p) {
      const bool m = key[p] == c && (MODE == MODE_ALG1 || val[p] > 0);
      const uint32_t x = m ? w : 0u;
      val[p] += x;
      hit |= x;
    }
    if (quad_or(hit) != 0) return;
    if constexpr (MODE == MODE_ALG1) {
      // into a free slot, else subtract w from every slot and drop the item
      const uint32_t f = free_slot();
      put(f, c, w);
      const uint32_t x = f == NONE ? w : 0u;
#pragma unroll
      for (int p = 0; p < S; ++p) val[p] = sub_sat(val[p], x);
      lost |= x;
    } else if constexpr (MODE == MODE_UNCOND) {
      // subtract w from every slot first, then into a free slot if there is one
      uint32_t any = 0;
#pragma unroll
      for (int p = 0; p < S; ++p) {
        any |= val[p];
        val[p] = sub_sat(val[p], w);
      }
      const uint32_t f = free_slot();
      put(f, c, w);
      lost |= (any != 0 || f == NONE) ? w : 0u;
    } else {  // MODE_STD: textbook weighted MG
      const uint32_t f = free_slot();
      if (f != NONE) {
        put(f, c, w);
      } else {
        uint32_t d = w;
#pragma unroll
        for (int p = 0; p < S; ++p) d = slot_here() ? umin(val[p], d) : d;
        d = quad_min(d);
#pragma unroll
        for (int p = 0; p < S; ++p) val[p] = slot_here() ? val[p] - d : 0u;
        if (w - d > 0) put(free_slot(), c, w - d);
        lost |= w;
      }
    }
  }

  // Keep only the candidates (positive slots); other keys become EMPTY.
  __device__ inline void finalize() {
#pragma unroll
    for (int p = 0; p < S; ++p) key[p] = val[p] > 0 ? key[p] : EMPTY;
  }

  // Merge the finalised sketch (bk, bv) of another quad (slot 4p + q in this lane's
  // bk[p]) into this finalised one, with the rule of merge_sketch: add equal keys; if
  // more than K values are positive subtract the (K+1)-th largest; keep the positive
  // ones.  Every lane of the quad calls it.
  __device__ MGCD_INLINE void merge(uint32_t (&bk)[S], uint32_t (&bv)[S]) {
    // a's slots visit the quad's lanes in turn and take up the equal keys of b there
    // (an EMPTY key meets EMPTY keys of value 0 only)
#pragma unroll
    for (int r = 0; r < QUAD; ++r) {
#pragma unroll
      for (int x = 0; x < S; ++x) {
#pragma unroll
        for (int y = 0; y < S; ++y) {
          const bool m = key[x] == bk[y];
          val[x] += m ? bv[y] : 0u;
          bv[y] = m ? 0u : bv[y];
        }
      }
#pragma unroll
      for (int x = 0; x < S; ++x) {
        key[x] = quad_perm<QP_ROT1>(key[x]);
        val[x] = quad_perm<QP_ROT1>(val[x]);
      }
    }
    uint32_t cnt = 0;
#pragma unroll
    for (int x = 0; x < S; ++x) cnt += (val[x] > 0) + (bv[x] > 0);
    cnt = quad_sum(cnt);
    if (cnt > (uint32_t)K) {
      lost = 1;
      // t = the largest value with at least K+1 values >= it (the (K+1)-th largest)
      uint32_t ge[2 * S], o[2 * S];
#pragma unroll
      for (int x = 0; x < S; ++x) {
        o[x] = val[x];
        o[S + x] = bv[x];
        ge[x] = 0;
        ge[S + x] = 0;
      }
#pragma unroll
      for (int r = 0; r < QUAD; ++r) {
#pragma unroll
        for (int x = 0; x < S; ++x) {
#pragma unroll
          for (int y = 0; y < 2 * S; ++y) {
            ge[x] += o[y] >= val[x];
            ge[S + x] += o[y] >= bv[x];
          }
        }
#pragma unroll
        for (int y = 0; y < 2 * S; ++y) o[y] = quad_perm<QP_ROT1>(o[y]);
      }
      uint32_t t = 0;
#pragma unroll
      for (int x = 0; x < S; ++x) {
        t = ge[x] >= K + 1 ? umax(t, val[x]) : t;
        t = ge[S + x] >= K + 1 ? umax(t, bv[x]) : t;
      }
      t = quad_max(t);
#pragma unroll
      for (int x = 0; x < S; ++x) {
        val[x] = sub_sat(val[x], t);
        bv[x] = sub_sat(bv[x], t);
      }
    }
    // b's survivors visit the lanes until each has found a free slot of a (at most K
    // values are positive in all, and a quad has K slots)
#pragma unroll
    for (int r = 0; r < QUAD; ++r) {
#pragma unroll
      for (int y = 0; y < S; ++y) {
#pragma unroll
        for (int x = 0; x < S; ++x) {
          const bool e = bv[y] > 0 && val[x] == 0 && slot_here();
          key[x] = e ? bk[y] : key[x];
          val[x] = e ? bv[y] : val[x];
          bv[y] = e ? 0u : bv[y];
        }
      }
      if (r + 1 < QUAD) {
#pragma unroll
        for (int y = 0; y < S; ++y) {
          bk[y] = quad_perm<QP_ROT1>(bk[y]);
          bv[y] = quad_perm<QP_ROT1>(bv[y]);
        }
      }
    }
    finalize();
  }
};

}  // namespace mgcd
