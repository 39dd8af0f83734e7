// Shared host/device helpers of the LOR assembly library (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <string>
#include <type_traits>

#include "../../include/lor.h"

namespace lor {

// ----------------------------------------------------------------- errors

// Thread-local message of the last failing call (lor_last_error).
void set_error(const char* fmt, ...);
void clear_error();

struct Status {
  int code = LOR_OK;
  bool ok() const { return code == LOR_OK; }
};

#define LOR_FAIL(CODE, ...)        \
  do {                             \
    ::lor::set_error(__VA_ARGS__); \
    return (CODE);                 \
  } while (0)

#define LOR_HIP(CALL)                                                                  \
  do {                                                                                 \
    hipError_t e_ = (CALL);                                                            \
    if (e_ != hipSuccess) {                                                            \
      ::lor::set_error("%s failed: %s (%s:%d)", #CALL, hipGetErrorString(e_), __FILE__, \
                       __LINE__);                                                      \
      return LOR_EDEVICE;                                                              \
    }                                                                                  \
  } while (0)

// Launch-error check right after a <<<>>> launch.
#define LOR_LAUNCHED(NAME)                                                             \
  do {                                                                                 \
    hipError_t e_ = hipGetLastError();                                                 \
    if (e_ != hipSuccess) {                                                            \
      ::lor::set_error("launch of %s failed: %s", NAME, hipGetErrorString(e_));         \
      return LOR_EDEVICE;                                                              \
    }                                                                                  \
  } while (0)

inline hipStream_t as_stream(void* s) { return reinterpret_cast<hipStream_t>(s); }

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

// ------------------------------------------------------ reference element

// Local dof counts per element.
inline int nloc_h1(int p) { return (p + 1) * (p + 1) * (p + 1); }
inline int nloc_nd(int p) { return 3 * p * (p + 1) * (p + 1); }
inline int nloc_rt(int p) { return 3 * p * p * (p + 1); }

// Per-element table entry: bits 0..6 = position of the entry inside its CSR
// row, bit 7 = this element is the first (lowest colour) contributor.
constexpr uint8_t kFirstBit = 0x80u;
constexpr uint8_t kRankMask = 0x7fu;

// Workgroup barrier for LDS traffic only.  __syncthreads() is also a
// workgroup-scope memory fence, which makes every wave wait for all of its
// outstanding global loads and stores first; the assembly kernels keep global
// prefetches and stores in flight across phases, so they synchronise LDS with
// this barrier instead (wait for the wave's LDS operations, then s_barrier).
__device__ __forceinline__ void lds_barrier() {
  __asm__ volatile("" ::: "memory");
  // s_waitcnt lgkmcnt(0) with vmcnt and expcnt left at their maxima
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_s_barrier();
  __asm__ volatile("" ::: "memory");
}

// Box lattices (H1 meshes whose vertex at lattice point (X, Y, Z) has id
// X + LX (Y + LY Z)): the row of a point holds its in-box 3 x 3 x 3
// neighbours in (dz, dy, dx) order.  box_count: neighbours of a point along
// one axis of L >= 2 points; box_prefix: their sum over the points before X
// (X in [0, L]); box_row_start: the CSR row start of point (X, Y, Z).
__host__ __device__ __forceinline__ int box_count(int64_t X, int64_t L) { return 1 + (X > 0) + (X < L - 1); }
__host__ __device__ __forceinline__ int64_t box_prefix(int64_t X, int64_t L) {
  return X == 0 ? 0 : 3 * X - 1 - (X == L ? 1 : 0);
}
__host__ __device__ __forceinline__ int64_t box_row_start(int64_t X, int64_t Y, int64_t Z, int64_t LX, int64_t LY,
                                                          int64_t LZ) {
  const int64_t SX = 3 * LX - 2, SY = 3 * LY - 2;
  const int64_t cz = box_count(Z, LZ), cyz = box_count(Y, LY) * cz;
  return box_prefix(Z, LZ) * SY * SX + cz * box_prefix(Y, LY) * SX + cyz * box_prefix(X, LX);
}

// Segment length of a marching kernel: `layers` steps per tile, split into
// segments of equal length, each of which takes `extra` steps more when there
// are several (the layer below it, integrated again for its carry, and its
// start).  The waves run in rounds over the chip's `slots` resident waves, so
// a launch takes about ceil(waves / slots) x (length + extra) steps; the length
// with the fewest (*steps) is taken, so that neither the last round nor, on a small
// mesh, the chip is left mostly idle.  `tiles`: waves per segment (all batch
// entries).  Short segments are what a small mesh needs: H1 p = 2 on 4^3
// elements (4 tiles) takes 48 us as segments of 8 layers and 12.5 us of 1 layer (most
// of it the launch), p = 5 on 13 x 9 x 11 47.7 us of 8 and 25.0 us of 4.
inline int64_t march_segment(int64_t layers, int64_t tiles, int64_t slots, int64_t extra, int64_t* steps = nullptr) {
  constexpr int64_t kMaxSegments = 65535;  // second grid dimension
  int64_t seglen = layers, best = -1;
  // Only the shortest length of each number of segments: about 2 sqrt(layers) of
  // them (each value call searches, on the host: 480 us a call on 60,000 layers over
  // all lengths, 16 so).
  for (int64_t len = ceil_div(layers, kMaxSegments);;) {
    const int64_t ns = ceil_div(layers, len);
    const int64_t cost = ceil_div(tiles * ns, slots) * (len + (ns > 1 ? extra : 0));
    if (best < 0 || cost < best) {
      best = cost;
      seglen = len;
    }
    if (ns <= 1) break;
    len = ceil_div(layers, ns - 1);
  }
  if (steps) *steps = best;
  return seglen;
}

// Whether a mesh without an owner-computes schedule is assembled row by row:
// up to `per_color` cells (all batch entries) per colour, and rows that fit 64 KB
// of LDS (256 lanes, `lanes` per row; max_row_nnz 0: unknown).  The batch counts,
// since it shares the launches per colour: by the mesh alone batches would be
// slower (24,300 cells, p = 3, batch 8: H(curl) 219 -> 369 us in FP64, 159 -> 362 in
// FP32; H1, batch 32: 224 -> 380).  So a batch can take another kernel than one of
// its entries alone; LOR_COLORED gives both the same.
inline bool rows_pay(const lor_sched* s, int64_t cells, int64_t per_color, int lanes) {
  const int row = (s->max_row_nnz > 0 ? s->max_row_nnz : LOR_MAX_ROW_NNZ) | 1;
  return cells <= per_color * s->ncolors && 256 / lanes * row * 8 <= 64 * 1024;
}

template <typename T>
inline T* dev_at(const lor_sched* s, size_t off) {
  return reinterpret_cast<T*>(static_cast<char*>(s->dev) + off);
}

}  // namespace lor
