// Exclusive scan (tile reduce -> recursive scan of tile sums -> tile scan) and a
// stable least-significant-digit radix sort with 8-bit digits.  Both are plain
// data-parallel primitives used by bucketing, renumbering and aggregation.
#include "primitives.hpp"

namespace mgcd {

constexpr int SCAN_ITEMS = 8;
constexpr int SCAN_TILE = BLOCK * SCAN_ITEMS;  // 2048 items per workgroup
// Scans of at most so many tiles are one launch: the last of eight workgroups reads the
// seven tiles before its own in 14 loads per thread, all on their way at once.  32-bit
// counts of 2, 4 and 8 tiles take 5.5, 5.9 and 7.0 us, in three launches 11.2 to 11.4 (one
// tile 4.7).  With a limit of 16, scans of 9 and 16 tiles take 8.0 and 9.7 us instead of 11.4,
// but those of 2 to 8 tiles 0.7 more, for the loads of the largest; most scans are small.
constexpr int SCAN_ALONE = 8;

template <typename Tin>
__global__ void __launch_bounds__(BLOCK) k_tile_sums(const Tin *in, int64_t n, int64_t *sums) {
  __shared__ int64_t lds[4];
  int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
  int64_t acc = 0;
#pragma unroll
  for (int r = 0; r < SCAN_ITEMS; ++r) {
    int64_t i = base + (int64_t)r * BLOCK + threadIdx.x;
    if (i < n) acc += (int64_t)in[i];
  }
  acc = block_sum(acc, lds);
  if (threadIdx.x == 0) sums[blockIdx.x] = acc;
}

// Wave w of the tile scans its SCAN_ITEMS * WAVE consecutive items 64 at a time (one
// coalesced load and store per round, a carry across rounds); the waves' totals give
// their offsets within the tile, tile_off the tile's; without tile_off a workgroup adds up
// the tiles before its own by itself (in and out apart).
template <typename Tin>
__global__ void __launch_bounds__(BLOCK)
    k_tile_scan(const Tin *in, int64_t *out, int64_t n, const int64_t *tile_off, int64_t *total) {
  __shared__ int64_t wtot[BLOCK / WAVE], wbefore[BLOCK / WAVE];
  const int w = threadIdx.x / WAVE, lane = lane_id();
  if (!tile_off) {
    const int64_t before = (int64_t)blockIdx.x * SCAN_TILE;
    int64_t acc = 0;
    if constexpr (sizeof(Tin) == 4) {  // whole tiles: 128-bit loads, all on their way at once
      if (before > 0) {  // block-uniform
#pragma unroll
        for (int r = 0; r < (SCAN_ALONE - 1) * SCAN_ITEMS / 4; ++r) {
          const int64_t i = ((int64_t)r * BLOCK + threadIdx.x) * 4;
          const v4u x = load4(reinterpret_cast<const uint32_t *>(in), i, n, i < before);
          acc += (int64_t)x.x + x.y + x.z + x.w;
        }
      }
    } else {
#pragma unroll 8
      for (int64_t i = threadIdx.x; i < before; i += BLOCK) acc += (int64_t)in[i];
    }
    acc = wave_sum(acc);
    if (lane == 0) wbefore[w] = acc;
  }
  const int64_t wbase = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)w * (SCAN_ITEMS * WAVE) + lane;
  int64_t ex[SCAN_ITEMS];
  int64_t carry = 0;
#pragma unroll
  for (int r = 0; r < SCAN_ITEMS; ++r) {
    const int64_t i = wbase + (int64_t)r * WAVE;
    const int64_t x = i < n ? (int64_t)in[i] : 0;
    const int64_t incl = wave_inclusive_scan(x);
    ex[r] = carry + incl - x;
    carry += __shfl(incl, WAVE - 1);
  }
  if (lane == 0) wtot[w] = carry;
  __syncthreads();
  int64_t off = 0;
  if (tile_off) {
    off = tile_off[blockIdx.x];
  } else {
    for (int q = 0; q < BLOCK / WAVE; ++q) off += wbefore[q];
  }
  for (int q = 0; q < w; ++q) off += wtot[q];
#pragma unroll
  for (int r = 0; r < SCAN_ITEMS; ++r) {
    const int64_t i = wbase + (int64_t)r * WAVE;
    if (i < n) out[i] = off + ex[r];
  }
  if (total && blockIdx.x == gridDim.x - 1 && w == BLOCK / WAVE - 1 && lane == 0) *total = off + carry;
}

template <typename Tin>
static void scan_impl(const Tin *in, int64_t *out, int64_t n, int64_t *total, Arena &a,
                      hipStream_t s) {
  if (n <= 0) {
    if (total) MGCD_HIP(hipMemsetAsync(total, 0, sizeof(int64_t), s));
    return;
  }
  int64_t tiles = ceil_div(n, SCAN_TILE);
  if (tiles == 1 || (tiles <= SCAN_ALONE && static_cast<const void *>(in) != static_cast<const void *>(out))) {
    k_tile_scan<Tin><<<(unsigned)tiles, BLOCK, 0, s>>>(in, out, n, nullptr, total);
    MGCD_LAUNCHED();
    return;
  }
  size_t m = a.mark();
  int64_t *sums = a.take<int64_t>(tiles);
  k_tile_sums<Tin><<<(unsigned)tiles, BLOCK, 0, s>>>(in, n, sums);
  MGCD_LAUNCHED();
  scan_impl<int64_t>(sums, sums, tiles, nullptr, a, s);
  k_tile_scan<Tin><<<(unsigned)tiles, BLOCK, 0, s>>>(in, out, n, sums, total);
  MGCD_LAUNCHED();
  a.release(m);
}

void scan_u32_i64(const uint32_t *in, int64_t *out, int64_t n, int64_t *total, Arena &a,
                  hipStream_t s) {
  scan_impl<uint32_t>(in, out, n, total, a, s);
}
void scan_i64(const int64_t *in, int64_t *out, int64_t n, int64_t *total, Arena &a,
              hipStream_t s) {
  scan_impl<int64_t>(in, out, n, total, a, s);
}

size_t scan_ws_bytes(int64_t n) {
  size_t b = 0;
  int64_t t = ceil_div(n > 0 ? n : 1, SCAN_TILE);
  while (t > 1) {
    b += (size_t)t * sizeof(int64_t) + 256;
    t = ceil_div(t, SCAN_TILE);
  }
  return b + 256;
}

// ------------------------------------------------------------------------------------
// radix sort
// ------------------------------------------------------------------------------------
constexpr int RS_ITEMS = 16;
constexpr int RS_TILE = BLOCK * RS_ITEMS;  // 4096 items per workgroup
constexpr int RS_BINS = 256;

// hist[d * tiles + t] = items of tile t whose digit is d (digit-major, so one
// exclusive scan yields every (digit, tile) output offset in stable order).
__global__ void __launch_bounds__(BLOCK)
    k_rs_hist(const uint64_t *keys, int64_t n, int shift, uint32_t *hist, int64_t tiles) {
  __shared__ uint32_t h[RS_BINS];
  h[threadIdx.x] = 0;
  __syncthreads();
  int64_t base = (int64_t)blockIdx.x * RS_TILE;
#pragma unroll 4
  for (int r = 0; r < RS_ITEMS; ++r) {
    int64_t i = base + (int64_t)r * BLOCK + threadIdx.x;
    if (i < n) atomicAdd(&h[(uint32_t)(keys[i] >> shift) & 255u], 1u);
  }
  __syncthreads();
  hist[(int64_t)threadIdx.x * tiles + blockIdx.x] = h[threadIdx.x];
}

// Wave w takes items base + 1024 w .. of the tile in order, 64 per round: an item's rank
// among the wave's items of its digit is the wave's count so far (its own LDS row, no
// barrier between rounds) plus its rank among the round's lanes (ballots).  The waves'
// counts, scanned once per tile, and the tile's digit offsets then give every position.
// All loads of the tile are in flight together.  On one tile (the smallest sorts) it takes
// 8 us against 15 for 16 rounds between barriers.
// ORDER: the tile is put in order in LDS (keys, then values through the same words) and
// stored from there, so that a wave's stores are runs of the same digit: bound by the
// scattered stores, 12 bytes per item to a line each, otherwise.  15.5 M pairs by digits
// in no order: 218 to 316 us without, 90 to 104 with (3.9 TB/s).
template <bool ORDER>
__global__ void __launch_bounds__(BLOCK)
    k_rs_scatter(const uint64_t *kin, const uint32_t *vin, uint64_t *kout, uint32_t *vout,
                 int64_t n, int shift, const int64_t *offs, int64_t tiles) {
  constexpr int WAVES = BLOCK / WAVE;
  __shared__ uint32_t cnt[WAVES][RS_BINS];
  __shared__ int64_t off_lds[RS_BINS];
  __shared__ uint64_t sorted[ORDER ? RS_TILE : 1];
  __shared__ uint32_t wsum[WAVES];
  const int t = threadIdx.x, w = t / WAVE;
  static_assert(BLOCK == RS_BINS, "thread t owns digit t");
  off_lds[t] = offs[(int64_t)t * tiles + blockIdx.x];
#pragma unroll
  for (int q = 0; q < WAVES; ++q) cnt[q][t] = 0;
  const int64_t first = (int64_t)blockIdx.x * RS_TILE + (int64_t)w * (RS_TILE / WAVES) + lane_id();
  uint64_t key[RS_ITEMS];
  uint32_t val[RS_ITEMS], rank[RS_ITEMS];
#pragma unroll
  for (int r = 0; r < RS_ITEMS; ++r) {
    const int64_t i = first + (int64_t)r * WAVE;
    key[r] = i < n ? kin[i] : 0;
    val[r] = i < n ? vin[i] : 0;
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < RS_ITEMS; ++r) {
    const bool valid = first + (int64_t)r * WAVE < n;
    const uint32_t d = (uint32_t)(key[r] >> shift) & (RS_BINS - 1);
    uint64_t peers = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const bool bit = (d >> b) & 1u;
      const uint64_t m = __ballot(bit);
      peers &= bit ? m : ~m;
    }
    const uint32_t before = cnt[w][d];
    rank[r] = (uint32_t)__popcll(peers & lanemask_lt());
    wave_sync();
    if (valid && rank[r] == 0) cnt[w][d] = before + (uint32_t)__popcll(peers);
    wave_sync();
    rank[r] += before;
  }
  __syncthreads();
  uint32_t sum = 0;
#pragma unroll
  for (int q = 0; q < WAVES; ++q) {
    const uint32_t c = cnt[q][t];
    cnt[q][t] = sum;
    sum += c;
  }
  __syncthreads();
  if constexpr (!ORDER) {
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
      if (first + (int64_t)r * WAVE < n) {
        const uint32_t d = (uint32_t)(key[r] >> shift) & (RS_BINS - 1);
        const int64_t pos = off_lds[d] + cnt[w][d] + rank[r];
        kout[pos] = key[r];
        vout[pos] = val[r];
      }
    }
  } else {
    // digit t's first place in the tile, added to the waves' counts and taken off its
    // offset, which then turns a place into a position
    const uint32_t incl = wave_inclusive_scan(sum);
    if (lane_id() == WAVE - 1) wsum[w] = incl;
    __syncthreads();
    uint32_t place = incl - sum;
    for (int q = 0; q < w; ++q) place += wsum[q];
#pragma unroll
    for (int q = 0; q < WAVES; ++q) cnt[q][t] += place;
    off_lds[t] -= place;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * RS_TILE;
    const int count = n - base < RS_TILE ? (int)(n - base) : RS_TILE;
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
      const uint32_t d = (uint32_t)(key[r] >> shift) & (RS_BINS - 1);
      rank[r] += cnt[w][d];
      if (first + (int64_t)r * WAVE < n) sorted[rank[r]] = key[r];
    }
    __syncthreads();
    int64_t pos[RS_ITEMS];
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
      const int x = r * BLOCK + t;
      if (x < count) {
        const uint64_t k = sorted[x];
        pos[r] = off_lds[(uint32_t)(k >> shift) & (RS_BINS - 1)] + x;
        kout[pos[r]] = k;
      }
    }
    __syncthreads();
    uint32_t *sv = reinterpret_cast<uint32_t *>(sorted);
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r)
      if (first + (int64_t)r * WAVE < n) sv[rank[r]] = val[r];
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RS_ITEMS; ++r) {
      const int x = r * BLOCK + t;
      if (x < count) vout[pos[r]] = sv[x];
    }
  }
}

// Sorts of at least so many tiles put them in order before the stores: at 64 tiles that is
// 11 to 12 us against 9 to 13, at 256 tiles 13 to 15 against 17 to 22 (two more barriers
// and trips through LDS, which do not pay while the tiles do not fill the chip).
constexpr int64_t RS_ORDER_TILES = 128;

bool radix_sort_pairs(uint64_t *k0, uint32_t *v0, uint64_t *k1, uint32_t *v1, int64_t n,
                      int bits, Arena &a, hipStream_t s, int from) {
  if (n <= 1 || bits <= from) return false;
  int64_t tiles = ceil_div(n, RS_TILE);
  size_t m = a.mark();
  uint32_t *hist = a.take<uint32_t>(tiles * RS_BINS);
  int64_t *offs = a.take<int64_t>(tiles * RS_BINS);
  bool flip = false;
  for (int shift = from; shift < bits; shift += 8) {
    const uint64_t *ki = flip ? k1 : k0;
    const uint32_t *vi = flip ? v1 : v0;
    uint64_t *ko = flip ? k0 : k1;
    uint32_t *vo = flip ? v0 : v1;
    k_rs_hist<<<(unsigned)tiles, BLOCK, 0, s>>>(ki, n, shift, hist, tiles);
    MGCD_LAUNCHED();
    scan_u32_i64(hist, offs, tiles * RS_BINS, nullptr, a, s);
    if (tiles >= RS_ORDER_TILES)
      k_rs_scatter<true><<<(unsigned)tiles, BLOCK, 0, s>>>(ki, vi, ko, vo, n, shift, offs, tiles);
    else
      k_rs_scatter<false><<<(unsigned)tiles, BLOCK, 0, s>>>(ki, vi, ko, vo, n, shift, offs, tiles);
    MGCD_LAUNCHED();
    flip = !flip;
  }
  a.release(m);
  return flip;
}

size_t radix_sort_ws_bytes(int64_t n) {
  int64_t tiles = ceil_div(n > 0 ? n : 1, RS_TILE);
  return (size_t)tiles * RS_BINS * (sizeof(uint32_t) + sizeof(int64_t)) + 1024 +
         scan_ws_bytes(tiles * RS_BINS);
}

}  // namespace mgcd
