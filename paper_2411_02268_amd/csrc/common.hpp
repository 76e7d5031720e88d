// Shared device and host helpers of the MI355X (gfx950) community-detection library.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <cstring>
#include <stdexcept>
#include <string>
#include <vector>

#include "launch.hpp"

namespace mgcd {

constexpr uint32_t EMPTY = 0xFFFFFFFFu;  // key of a fresh sketch slot; never a community id
constexpr int WAVE = 64;                 // CDNA wavefront width
constexpr int BLOCK = 256;               // four waves per workgroup

enum Algo : int { ALGO_LPA = 0, ALGO_MOVE = 1, ALGO_REFINE = 2 };
enum Mode : int { MODE_EXACT = 0, MODE_ALG1 = 1, MODE_UNCOND = 2, MODE_STD = 3, MODE_SMALL = 5 };

// A CSR graph in device memory (Section 3): rows are the out-entries of a vertex.
struct Graph {
  int32_t n;
  int64_t nnz;
  const int64_t *off;
  const int32_t *idx;
  const uint32_t *w;
};

struct Pair {
  uint32_t key;
  uint32_t val;
};

// ---- errors (host) -------------------------------------------------------------
struct Error : std::runtime_error {
  int code;
  Error(int c, const std::string &m) : std::runtime_error(m), code(c) {}
};

#define MGCD_HIP(x)                                                                     \
  do {                                                                                  \
    hipError_t e_ = (x);                                                                \
    if (e_ != hipSuccess)                                                               \
      throw ::mgcd::Error(-5, std::string(#x) + ": " + hipGetErrorString(e_));          \
  } while (0)

// Set while this thread records work into a HIP graph: the runtime refuses
// hipGetLastError then, and launch errors surface when the capture ends instead.
inline thread_local bool in_capture = false;

#define MGCD_LAUNCHED()                                      \
  do {                                                       \
    if (!::mgcd::in_capture) MGCD_HIP(hipGetLastError());    \
  } while (0)

// Kernels that hold a K-slot sketch per lane in registers: at K = 16 two waves per
// SIMD leave room for the sketch and its merge partner without spilling.
#define MGCD_SKETCH_OCCUPANCY(K) __attribute__((amdgpu_waves_per_eu(1, (K) >= 16 ? 2 : 8)))

// Inlined always: as a call, arrays held in registers would go to scratch memory.
#define MGCD_INLINE __attribute__((always_inline)) inline
#define MGCD_LAMBDA __attribute__((always_inline))

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Sets the calling thread's message returned by mgcd_last_error().
void set_last_error(const std::string &msg);

inline int bits_for(uint64_t maxval) {  // bits needed to hold values <= maxval
  int b = 0;
  while (b < 64 && (maxval >> b) != 0) ++b;
  return b;
}

// ---- bump allocator over the caller's workspace (host) ---------------------------
struct Arena {
  char *base = nullptr;
  size_t cap = 0, used = 0, peak = 0;
  bool dry = false;  // sizing pass: count bytes only
  template <typename T>
  T *take(int64_t count) {
    size_t bytes = (size_t)(count > 0 ? count : 1) * sizeof(T);
    size_t start = (used + 255) & ~(size_t)255;
    size_t end = start + bytes;
    if (end > peak) peak = end;
    if (!dry && end > cap)
      throw Error(-4, "workspace too small: need more than " + std::to_string(end) + " bytes");
    used = end;
    return dry ? nullptr : reinterpret_cast<T *>(base + start);
  }
  size_t mark() const { return used; }
  void release(size_t m) { used = m; }
};

// ---- small reads from the device (host) ---------------------------------------------
// Results that the host waits for land in pinned memory first: a copy into pageable
// memory is staged by the runtime and its round trip takes 22 us, into pinned memory 14.
// A read leases a pinned block for its own duration from a pool of at most POOL_BLOCKS
// (any thread, stream and device; a block beyond the pool is freed at once).
constexpr size_t PINNED_BYTES = 16 * 1024;
void *pinned_lease();            // null when none can be had: the read is pageable then
void pinned_return(void *block);
inline thread_local bool no_pinned = false;  // this thread's calls may not allocate

struct HostRead {
  explicit HostRead(hipStream_t s) : st(s) {}
  HostRead(const HostRead &) = delete;
  HostRead &operator=(const HostRead &) = delete;
  ~HostRead() {
    if (!block) return;
    if (count) (void)hipStreamSynchronize(st);  // an error on the way: nothing may still write to it
    pinned_return(block);
  }
  void add(void *dst, const void *src, size_t bytes) {
    if (!block && !tried && !no_pinned) {
      block = static_cast<char *>(pinned_lease());
      tried = true;
    }
    if (!block || count == MAX || used + bytes > PINNED_BYTES) {
      MGCD_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDeviceToHost, st));
      return;
    }
    piece[count++] = Piece{dst, used, bytes};
    MGCD_HIP(hipMemcpyAsync(block + used, src, bytes, hipMemcpyDeviceToHost, st));
    used += (bytes + 15) & ~(size_t)15;
  }
  void wait() {
    MGCD_HIP(hipStreamSynchronize(st));
    for (int q = 0; q < count; ++q) std::memcpy(piece[q].dst, block + piece[q].at, piece[q].bytes);
    count = 0;
    used = 0;
  }

 private:
  static constexpr int MAX = 4;
  struct Piece {
    void *dst;
    size_t at, bytes;
  };
  hipStream_t st;
  char *block = nullptr;
  bool tried = false;
  size_t used = 0;
  int count = 0;
  Piece piece[MAX];
};

// Copies device memory to the host and waits for the stream.
inline void read_back(void *dst, const void *src, size_t bytes, hipStream_t st) {
  HostRead r(st);
  r.add(dst, src, bytes);
  r.wait();
}

// ---- device time of a stretch of stream work (host) --------------------------------
struct Timer {
  hipEvent_t a = nullptr, b = nullptr;
  hipStream_t st;
  explicit Timer(hipStream_t s) : st(s) {
    MGCD_HIP(hipEventCreate(&a));
    MGCD_HIP(hipEventCreate(&b));
  }
  ~Timer() {
    if (a) (void)hipEventDestroy(a);
    if (b) (void)hipEventDestroy(b);
  }
  void start() { MGCD_HIP(hipEventRecord(a, st)); }
  float stop() {  // synchronises
    MGCD_HIP(hipEventRecord(b, st));
    MGCD_HIP(hipEventSynchronize(b));
    float ms = 0;
    MGCD_HIP(hipEventElapsedTime(&ms, a, b));
    return ms;
  }
};

// ---- device time by phase (host): one event per boundary, read once at the end -----------
struct PhaseClock {
  explicit PhaseClock(hipStream_t s) : st(s) { mark(-1); }
  ~PhaseClock() {
    for (hipEvent_t e : ev) (void)hipEventDestroy(e);
  }
  // The stream's work since the last mark belongs to phase p (< 0: to none).
  void mark(int p) {
    hipEvent_t e = nullptr;
    MGCD_HIP(hipEventCreate(&e));
    ev.push_back(e);
    phase.push_back(p);
    MGCD_HIP(hipEventRecord(e, st));
  }
  // Milliseconds of phases 0 .. n - 1 into ms; returns the time from first to last mark.
  float read(float *ms, int n) {
    MGCD_HIP(hipEventSynchronize(ev.back()));
    float total = 0;
    for (int q = 0; q < n; ++q) ms[q] = 0;
    for (size_t x = 1; x < ev.size(); ++x) {
      float t = 0;
      MGCD_HIP(hipEventElapsedTime(&t, ev[x - 1], ev[x]));
      if (phase[x] >= 0 && phase[x] < n) ms[phase[x]] += t;
      total += t;
    }
    return total;
  }

 private:
  hipStream_t st;
  std::vector<hipEvent_t> ev;
  std::vector<int> phase;
};

// ---- wave helpers (device) -------------------------------------------------------
__device__ inline int lane_id() { return (int)(threadIdx.x & (WAVE - 1)); }

// Orders a wave's LDS accesses before this point with those after it.
__device__ inline void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

typedef uint32_t v4u __attribute__((ext_vector_type(4)));

// Entries e .. e + 3 of p (nnz entries; 0 past the end); nothing when off.
__device__ inline v4u load4(const uint32_t *p, int64_t e, int64_t nnz, bool on) {
  typedef uint32_t v4a __attribute__((ext_vector_type(4), aligned(4)));
  v4u x = {0u, 0u, 0u, 0u};
  if (on) {
    if (e + 4 <= nnz) {
      x = *reinterpret_cast<const v4a *>(p + e);
    } else {
      x.x = p[e];
      x.y = e + 1 < nnz ? p[e + 1] : 0u;
      x.z = e + 2 < nnz ? p[e + 2] : 0u;
    }
  }
  return x;
}

// A value that is the same in every lane, moved to a scalar register so that the
// compiler treats what depends on it as wave-uniform (scalar branches and loops).
__device__ inline int32_t uniform(int32_t v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline uint32_t uniform(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)v);
}
__device__ inline int64_t uniform(int64_t v) {
  const uint64_t u = (uint64_t)v;
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)u);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)(u >> 32));
  return (int64_t)(((uint64_t)hi << 32) | lo);
}

__device__ inline uint64_t lanemask_lt() {
  int l = lane_id();
  return l == 0 ? 0ull : ((~0ull) >> (64 - l));
}

template <typename T>
__device__ inline T wave_sum(T v) {
#pragma unroll
  for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

template <typename T>
__device__ inline T wave_inclusive_scan(T v) {
  int l = lane_id();
#pragma unroll
  for (int o = 1; o < WAVE; o <<= 1) {
    T u = __shfl_up(v, o);
    if (l >= o) v += u;
  }
  return v;
}

// Totals that every block adds to one device counter go to one of SPREAD copies (by
// block index), so the atomics of blocks that finish together do not serialise on a
// single address; the reader adds up (or takes the maximum of) the copies.
constexpr int SPREAD = 64;
__device__ inline int spread_copy() { return (int)(blockIdx.x & (SPREAD - 1)); }

// Host: fold SPREAD copies of (nsum counters, then one maximum), each copy nsum + 1
// values, into out[0 .. nsum] (sums, then the maximum).  Synchronises st.
inline void read_spread(const unsigned long long *dev, int nsum, unsigned long long *out,
                        hipStream_t st) {
  std::vector<unsigned long long> h((size_t)SPREAD * (nsum + 1));
  read_back(h.data(), dev, h.size() * sizeof(unsigned long long), st);
  for (int q = 0; q <= nsum; ++q) out[q] = 0;
  for (int c = 0; c < SPREAD; ++c) {
    const unsigned long long *x = h.data() + (size_t)c * (nsum + 1);
    for (int q = 0; q < nsum; ++q) out[q] += x[q];
    out[nsum] = x[nsum] > out[nsum] ? x[nsum] : out[nsum];
  }
}

// Sum over a 256-thread block; every thread gets the total.
template <typename T>
__device__ inline T block_sum(T v, T *lds4) {
  v = wave_sum(v);
  int w = threadIdx.x / WAVE;
  __syncthreads();
  if (lane_id() == 0) lds4[w] = v;
  __syncthreads();
  T t = lds4[0] + lds4[1] + lds4[2] + lds4[3];
  __syncthreads();
  return t;
}

}  // namespace mgcd
