// Address-ordered gathers of a 128-row x 16-k (or 32-k) chunk of an
// operand stored in an arbitrary bit layout (internal): shared by the skewed
// matrix-core kernels and the complex GEMMs that read their large operand in
// place.
#pragma once

#include <hip/hip_runtime.h>

#include "internal.h"

namespace tnrcs {

constexpr int kSkewMaxV = 12;  // index bits of one chunk: 7 row bits + up to 5 k bits

// Address order of one chunk: chunk element e (0 .. 2^v) has its bit i at
// A position pos[i], and is row bit mb[i] (or -1) / k bit kb[i] (or -1) of
// the chunk; the bits are sorted by A position.  Row m, k of the chunk sits
// in LDS at k * (row stride) + (m ^ h), h = XOR of hk[i] over the set k bits
// i and of hm[j] over the set row bits 5 + j: a swizzle that keeps the 32
// rows a matrix-core operand reads at one k in 32 distinct banks, and gives
// the 32 entries that one half-wave stores (consecutive in address order)
// distinct banks too.  All-zero hk and hm: no swizzle.
struct SkewMap {
  int32_t v;
  int8_t pos[kSkewMaxV];
  int8_t mb[kSkewMaxV];
  int8_t kb[kSkewMaxV];
  int8_t hk[5];
  int8_t hm[2];
};

// The slab bits of a K split: bit i of the slab's number at position pos[i]
// of A (the uppermost k bits; n of them).
struct SlabMap {
  int32_t n = 0;
  int8_t pos[6] = {0, 0, 0, 0, 0, 0};
};

__device__ __forceinline__ uint64_t slab_offset(const SlabMap& s, int64_t z) {
  uint64_t o = 0;
#pragma unroll
  for (int i = 0; i < 6; ++i)
    if (i < s.n) o |= (uint64_t)((z >> i) & 1) << s.pos[i];
  return o;
}

// splits (a power of two up to 64) slabs of idx's sum, each a whole number of
// 2^stage_bits terms
inline bool slab_map(const IndexOp& idx, int splits, int stage_bits, SlabMap* s) {
  *s = SlabMap{};
  while ((1 << s->n) < splits) ++s->n;
  if (splits < 1 || (1 << s->n) != splits || s->n > 6 || idx.nK - s->n < stage_bits) return false;
  for (int i = 0; i < s->n; ++i) s->pos[i] = (int8_t)run_pos(idx.aK, idx.nK - s->n + i);
  return true;
}

__device__ __forceinline__ int skew_h(const SkewMap& mp, int m, int k) {
  int h = 0;
#pragma unroll
  for (int i = 0; i < 5; ++i)
    if ((k >> i) & 1) h ^= mp.hk[i];
#pragma unroll
  for (int j = 0; j < 2; ++j)
    if ((m >> (5 + j)) & 1) h ^= mp.hm[j];
  return h;
}

// Chunk element e -> its offset from the chunk's first entry, its row m and
// its k within the chunk.  Unrolled over the largest map, so that the map's
// fields are read at fixed offsets of the kernel argument (scalar loads): the
// GEMMs that read A in place evaluate it in every workgroup, one per tile.
__device__ __forceinline__ void skew_split(const SkewMap& mp, int e, uint64_t& off, int& m, int& k) {
  off = 0;
  m = 0;
  k = 0;
#pragma unroll
  for (int i = 0; i < kSkewMaxV; ++i) {
    if (i < mp.v) {
      const int b = (e >> i) & 1;
      off |= (uint64_t)b << mp.pos[i];
      if (mp.mb[i] >= 0) m |= b << mp.mb[i];
      if (mp.kb[i] >= 0) k |= b << mp.kb[i];
    }
  }
}

// 16-bit storage, 16-byte loads: the four entries of a load differ in the
// chunk's two lowest address bits.  The planar LDS rows hold k contiguously,
// so a thread keeps all four entries of k bits 0 and 1 of its rows and stores
// them together: the k bits that the load does not cover are the ones that
// tell the thread's loads apart.  How they sit: kQuadKK: the load covers k0,
// k1; kQuadKR: k0, then a row bit; kQuadRK: a row bit, then k0; kQuadRR: two
// row bits.  kQuadNone: entries stored one by one.
enum QuadMode : int { kQuadNone = -1, kQuadKK = 0, kQuadKR = 1, kQuadRK = 2, kQuadRR = 3 };

// Host: the mode of a chunk map (entries sorted by position), whose entries
// are reordered so that the last ones tell a thread's 2^lj loads apart: k1
// (kQuadKR, kQuadRK), or k0 and, with lj = 2, k1 (kQuadRR; then k0 before k1).
// -1: the two lowest positions are not in the chunk, or hold k bits other
// than these.
int quad_mode(SkewMap* mp, int lj);

// Four 16-bit pairs (re, im) as two words of re and two of im.
__device__ __forceinline__ void quad_split(uint32_t w0, uint32_t w1, uint32_t w2, uint32_t w3, uint2& re, uint2& im) {
  re = make_uint2(__builtin_amdgcn_perm(w1, w0, 0x05040100u), __builtin_amdgcn_perm(w3, w2, 0x05040100u));
  im = make_uint2(__builtin_amdgcn_perm(w1, w0, 0x07060302u), __builtin_amdgcn_perm(w3, w2, 0x07060302u));
}

// Host: the chunk map of rows 0..127 (op.aM bits 0..6) and k bits
// 0..kcb-1 (op.aK), with the bank swizzle for stores that cover chunk bits
// lv .. lv+4.  False when a bit has no position.
bool skew_map(const IndexOp& op, int kcb, int lv, SkewMap* mp);

}  // namespace tnrcs
