// Output tiles written in a caller's index order (internal; OutMap in
// internal.h): the kernel stages a sub-tile in LDS and writes it to C in
// 16-byte runs of consecutive positions.  It takes the place of a permute of
// the whole output (one more read and write of C): 2^21 x 2^7 outputs over
// K = 64 in BF16 850 -> 527 us, 2^22 x 2^4 over K = 32 in complex64 550 -> 357
// us.  (Nontemporal stores measured 2 % slower: a line's runs come from one
// workgroup but not from one instruction.)
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "internal.h"

namespace tnrcs {

struct NoOut {};  // kernels that write their natural layout [rows, columns]
template <typename OM>
constexpr bool has_out = std::is_same<OM, OutMap>::value;

// LDS entry of the row bits r (0, 1, 3, 4) of accumulator register r: rows
// 8 (r >> 2) + (r & 3) of a 32x32 block; the same in every lane.
__device__ __forceinline__ int out_reg(const OutMap& o, int r) {
  return (r & 1 ? o.srow[0] : 0) ^ (r & 2 ? o.srow[1] : 0) ^ (r & 4 ? o.srow[3] : 0) ^ (r & 8 ? o.srow[4] : 0);
}

// LDS entry of this lane's column (bits 0 .. 4) and of row bit 2.
__device__ __forceinline__ int out_lane(const OutMap& o, int c, int kh) {
  int s = kh ? o.srow[2] : 0;
#pragma unroll
  for (int b = 0; b < 5; ++b) s ^= c >> b & 1 ? o.scol[b] : 0;
  return s;
}

// Position offset in C of the 16-byte groups tid + 256 i of a sub-tile: the
// thread's part, and (uniform) the part of i.
template <typename E>
__device__ __forceinline__ uint64_t out_thread(const OutMap& o, int tid) {
  constexpr int LV = sizeof(E) == 8 ? 1 : 2;
  uint64_t p = 0;
#pragma unroll
  for (int b = 0; b < 8; ++b)
    if (LV + b < o.bits) p |= (uint64_t)(tid >> b & 1) << o.cpos[LV + b];
  return p;
}

// Writes the staged sub-tile to C + base.  Every thread of the 256 calls it,
// after a barrier that follows the staging.
// MB: the most bits that the sub-tile has.
template <typename E, int MB>
__device__ __forceinline__ void out_write(const OutMap& o, E* C, const E* Cs, uint64_t base, uint64_t thread_off,
                                          int tid) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  constexpr int LV = sizeof(E) == 8 ? 1 : 2;
  const int groups = 1 << (o.bits - LV);
  const uint32_t st = out_swizzle((uint32_t)tid << LV, LV);
  if (tid >= groups) return;
#pragma unroll
  for (int i = 0; i < 1 << (MB - LV - 8); ++i) {
    if (i * 256 >= groups) break;
    uint64_t off = base;
#pragma unroll
    for (int b = 0; b < MB - LV - 8; ++b)
      if (i >> b & 1) off += (uint64_t)1 << o.cpos[LV + 8 + b];
    const u32x4 v = *reinterpret_cast<const u32x4*>(Cs + (st ^ out_swizzle((uint32_t)i << (8 + LV), LV)));
    *reinterpret_cast<u32x4*>(C + (off + thread_off)) = v;
  }
}

}  // namespace tnrcs
