// dispatch.h -- compile-time instantiation of the vector kernels.
//
// (kind, vector class) selects the element type / metric and the lane
// layout of row gathers:
//   class A: rows of <= 8 chunks of 16 B   -> 8 lanes per row, 1 chunk per lane
//   class B: rows of <= 32 chunks          -> 8 lanes per row, <= 4 chunks per lane
//   class C: rows of <= 64 chunks          -> 16 lanes per row, <= 4 chunks per lane
//   class D: rows of <= 128 chunks         -> 32 lanes per row, <= 4 chunks per lane
//   class E: rows of <= 256 chunks         -> 64 lanes per row, <= 4 chunks per lane
// Four chunks a lane keep the query in 16 registers: with 16 lanes and 16
// chunks for every row above class B a search held 296 registers, one wave per
// SIMD (2,000 searches of 100K x 960 fp32 2.09 ms; now 1.55).  Few searches
// gain as well below class E: one, and 1,000, of 50K x 300 0.91 -> 0.49 and 1.23
// -> 0.71 ms, of 50K x 512 1.04 -> 0.52 and 1.35 -> 1.06.
#pragma once
#include "index.h"
#include "vec.h"

#define GR_DISPATCH_KV(kind, vc, ...)                                                       \
  do {                                                                                      \
    const int k__ = (kind), v__ = (vc);                                                     \
    if (k__ == ::gr::kU8L2 && v__ == ::gr::kVcA) {                                          \
      constexpr int KIND = ::gr::kU8L2, LPV = 8, CPL = 1; __VA_ARGS__;                      \
    } else if (k__ == ::gr::kU8L2 && v__ == ::gr::kVcB) {                                   \
      constexpr int KIND = ::gr::kU8L2, LPV = 8, CPL = 4; __VA_ARGS__;                      \
    } else if (k__ == ::gr::kU8L2 && v__ == ::gr::kVcC) {                                   \
      constexpr int KIND = ::gr::kU8L2, LPV = 16, CPL = 4; __VA_ARGS__;                     \
    } else if (k__ == ::gr::kU8L2 && v__ == ::gr::kVcD) {                                   \
      constexpr int KIND = ::gr::kU8L2, LPV = 32, CPL = 4; __VA_ARGS__;                     \
    } else if (k__ == ::gr::kU8L2 && v__ == ::gr::kVcE) {                                   \
      constexpr int KIND = ::gr::kU8L2, LPV = 64, CPL = 4; __VA_ARGS__;                     \
    } else if (k__ == ::gr::kF32L2 && v__ == ::gr::kVcA) {                                  \
      constexpr int KIND = ::gr::kF32L2, LPV = 8, CPL = 1; __VA_ARGS__;                     \
    } else if (k__ == ::gr::kF32L2 && v__ == ::gr::kVcB) {                                  \
      constexpr int KIND = ::gr::kF32L2, LPV = 8, CPL = 4; __VA_ARGS__;                     \
    } else if (k__ == ::gr::kF32L2 && v__ == ::gr::kVcC) {                                  \
      constexpr int KIND = ::gr::kF32L2, LPV = 16, CPL = 4; __VA_ARGS__;                    \
    } else if (k__ == ::gr::kF32L2 && v__ == ::gr::kVcD) {                                  \
      constexpr int KIND = ::gr::kF32L2, LPV = 32, CPL = 4; __VA_ARGS__;                    \
    } else if (k__ == ::gr::kF32L2 && v__ == ::gr::kVcE) {                                  \
      constexpr int KIND = ::gr::kF32L2, LPV = 64, CPL = 4; __VA_ARGS__;                    \
    } else if (k__ == ::gr::kF32IP && v__ == ::gr::kVcA) {                                  \
      constexpr int KIND = ::gr::kF32IP, LPV = 8, CPL = 1; __VA_ARGS__;                     \
    } else if (k__ == ::gr::kF32IP && v__ == ::gr::kVcB) {                                  \
      constexpr int KIND = ::gr::kF32IP, LPV = 8, CPL = 4; __VA_ARGS__;                     \
    } else if (k__ == ::gr::kF32IP && v__ == ::gr::kVcC) {                                  \
      constexpr int KIND = ::gr::kF32IP, LPV = 16, CPL = 4; __VA_ARGS__;                    \
    } else if (k__ == ::gr::kF32IP && v__ == ::gr::kVcD) {                                  \
      constexpr int KIND = ::gr::kF32IP, LPV = 32, CPL = 4; __VA_ARGS__;                    \
    } else if (k__ == ::gr::kF32IP && v__ == ::gr::kVcE) {                                  \
      constexpr int KIND = ::gr::kF32IP, LPV = 64, CPL = 4; __VA_ARGS__;                    \
    } else {                                                                                \
      return hipErrorInvalidValue;                                                          \
    }                                                                                       \
  } while (0)

// Class E rows for launches that leave a SIMD to every wave: 16 lanes per row,
// <= 16 chunks per lane.
#define GR_DISPATCH_ALONE(kind, ...)                                                        \
  do {                                                                                      \
    const int k__ = (kind);                                                                 \
    if (k__ == ::gr::kU8L2) {                                                               \
      constexpr int KIND = ::gr::kU8L2, LPV = 16, CPL = 16; __VA_ARGS__;                    \
    } else if (k__ == ::gr::kF32L2) {                                                       \
      constexpr int KIND = ::gr::kF32L2, LPV = 16, CPL = 16; __VA_ARGS__;                   \
    } else {                                                                                \
      constexpr int KIND = ::gr::kF32IP, LPV = 16, CPL = 16; __VA_ARGS__;                   \
    }                                                                                       \
  } while (0)

// Register rows (64 keys each) needed to hold `n` keys: 1, 2 or 4.
#define GR_DISPATCH_N(n, ...)                                                               \
  do {                                                                                      \
    const uint32_t n__ = (n);                                                               \
    if (n__ <= 64) {                                                                        \
      constexpr int NR = 1; __VA_ARGS__;                                                    \
    } else if (n__ <= 128) {                                                                \
      constexpr int NR = 2; __VA_ARGS__;                                                    \
    } else if (n__ <= 256) {                                                                \
      constexpr int NR = 4; __VA_ARGS__;                                                    \
    } else {                                                                                \
      return hipErrorInvalidValue;                                                          \
    }                                                                                       \
  } while (0)

namespace gr {
// Workgroups of 64 lanes of `kern` (no dynamic LDS) that are resident on
// the current device at once, or 0 if the runtime cannot say.  A persistent
// loop over a queue split over exactly this many workgroups leaves no
// workgroup to start after the first ones finish.
static inline uint32_t resident_blocks(const void *kern) {
  int dev = 0, ncu = 0, per = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, 64, 0) != hipSuccess) return 0;
  return per > 0 && ncu > 0 ? (uint32_t)per * (uint32_t)ncu : 0u;
}
static inline uint32_t clamp_resident(uint32_t grid, uint32_t res) { return res && res < grid ? res : grid; }
}  // namespace gr
