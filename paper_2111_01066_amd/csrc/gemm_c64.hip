// Complex GEMM on FP32 matrix cores for complex64 storage (the matrix product
// of Supplement Eq. (matmul)).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "elem.h"
#include "gather.h"
#include "kernels.h"
#include "outmap.h"

namespace tnrcs {

typedef float floatx16 __attribute__((ext_vector_type(16)));

// ------------------------------------------------------------------- GEMM --
// C[M][N] = sum_k A[M][K] B[N][K], complex64 in and out, FP32 accumulation on
// v_mfma_f32_32x32x2_f32.  4M form: Cr += ArBr + (-Ai)Bi, Ci += ArBi + AiBr
// (four real products).  3M form: T1 = ArBr, T2 = AiBi,
// T3 = (Ar+Ai)(Br+Bi); Cr = T1 - T2, Ci = T3 - T1 - T2 (three products).
// Workgroup tile 64x64, four waves of 32x32, K staged through LDS in steps of
// 16 as (re, im) pairs; the next stage is loaded into registers while the
// current one is multiplied.  With few workgroups per CU a stage's load
// latency bounds it, with many the FP32 products: with planes in LDS and each
// stage loaded where it was used, 3 x 1984 x 1088 x 1200 took 465 us (now 403),
// 192 x 320 x 2048 in 4 slabs 52 (37), 64 x 64 x 1024 80 (64).  Four waves per
// SIMD: five spill and are no faster.

constexpr int GBM = 64, GBN = 64, GBK = 16;

// blockIdx.z selects a batch entry or a split-K slab through the strides sA,
// sB, sC; each sums k_len terms of rows that are K long.
template <int FORM>
__global__ __launch_bounds__(256, 4) void k_cgemm(const float2* __restrict__ A, const float2* __restrict__ B,
                                              float2* __restrict__ C, int64_t N, int64_t K, int64_t k_len,
                                              int64_t sA, int64_t sB, int64_t sC, int chunk) {
  constexpr int LD = GBM;
  // entry (k, row) of A and B at k * LD + (row ^ swz(k)): the four k quarters
  // of a row that neighbouring threads store go to different banks
  __shared__ __attribute__((aligned(16))) float2 As[GBK * LD], Bs[GBK * LD];
  auto swz = [](int k) { return (k & 12) << 1; };
  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int64_t bm = (int64_t)blockIdx.x * GBM, bn = (int64_t)blockIdx.y * GBN;
  const int64_t z = blockIdx.z;
  A += z * sA;
  B += z * sB;
  C += z * sC;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;
  floatx16 c0 = {}, c1 = {}, c2 = {};
  const int lrow = tid >> 2, lk = (tid & 3) * 4;
  const float2* Ap = A + (bm + lrow) * K + lk;
  const float2* Bp = B + (bn + lrow) * K + lk;
  const int slot0 = lk * LD + (lrow ^ swz(lk));  // entries (lk + q, lrow) at slot0 + q * LD
  float4 ra[2], rb[2];
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    ra[q] = *reinterpret_cast<const float4*>(Ap + 2 * q);
    rb[q] = *reinterpret_cast<const float4*>(Bp + 2 * q);
  }
  const int j = lane & 31, kh = lane >> 5;
  // adds (ADD false: stores) the running FP32 sums to C and restarts them
  auto flush = [&](auto add) {
    constexpr bool ADD = decltype(add)::value;
    // the row stride is made opaque here so that the compiler does not keep
    // the 16 output addresses live across the K loop
    int64_t ld = N;
    asm volatile("" : "+s"(ld));
    float2* Cw = C + (bm + wm + 4 * kh) * ld + bn + wn + j;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      float2 v;
      if (FORM == TN_GEMM_3M) {
        v.x = c0[r] - c1[r];
        v.y = c2[r] - c0[r] - c1[r];
      } else {
        v.x = c0[r];
        v.y = c1[r];
      }
      float2* p = Cw + (8 * (r >> 2) + (r & 3)) * ld;
      if constexpr (ADD) {
        const float2 o = *p;
        v.x += o.x;
        v.y += o.y;
      }
      *p = v;
    }
    c0 = floatx16{};
    c1 = floatx16{};
    c2 = floatx16{};
  };
  // this lane's operands: rows wm + j and wn + j at k = 4 q + kh and 4 q + 2 + kh
  const float2 *Al[4], *Bl[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    Al[q] = As + (4 * q + kh) * LD + ((wm + j) ^ (8 * q));
    Bl[q] = Bs + (4 * q + kh) * LD + ((wn + j) ^ (8 * q));
  }
  bool first = true;
  int it = 0;
  for (int64_t k0 = 0; k0 < k_len; k0 += GBK, ++it) {
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      As[slot0 + 2 * q * LD] = make_float2(ra[q].x, ra[q].y);
      As[slot0 + (2 * q + 1) * LD] = make_float2(ra[q].z, ra[q].w);
      Bs[slot0 + 2 * q * LD] = make_float2(rb[q].x, rb[q].y);
      Bs[slot0 + (2 * q + 1) * LD] = make_float2(rb[q].z, rb[q].w);
    }
    if (chunk > 0 && it > 0 && it % chunk == 0) {
      if (first)
        flush(std::false_type{});
      else
        flush(std::true_type{});
      first = false;
    }
    __syncthreads();
    if (k0 + GBK < k_len) {
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        ra[q] = *reinterpret_cast<const float4*>(Ap + k0 + GBK + 2 * q);
        rb[q] = *reinterpret_cast<const float4*>(Bp + k0 + GBK + 2 * q);
      }
    }
#pragma unroll
    for (int kk = 0; kk < GBK; kk += 2) {
      const float2 a = Al[kk >> 2][(kk & 2) * LD], b = Bl[kk >> 2][(kk & 2) * LD];
      const float ar = a.x, ai = a.y, br = b.x, bi = b.y;
      if (FORM == TN_GEMM_3M) {
        c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, br, c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, bi, c1, 0, 0, 0);
        c2 = __builtin_amdgcn_mfma_f32_32x32x2f32(ar + ai, br + bi, c2, 0, 0, 0);
      } else {
        c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, br, c0, 0, 0, 0);
        c0 = __builtin_amdgcn_mfma_f32_32x32x2f32(-ai, bi, c0, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, bi, c1, 0, 0, 0);
        c1 = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, br, c1, 0, 0, 0);
      }
    }
  }
  if (first)
    flush(std::false_type{});
  else
    flush(std::true_type{});
}

// A read in place (GA = 1): the large operand's rows and contracted bits
// sit anywhere in its stored layout (row bit i at the position of aM bit i,
// k bit i at that of aK bit i, the k bits above 3 in increasing positions),
// so no permute runs before the product.  Each 128 x 16 chunk is gathered in
// A's address order (the chunk map) in 16-byte loads of two entries: A's
// lowest index bit is the lowest row or k bit, so it belongs to the chunk.
// The chunk's K offset moves by a carrying add restricted to the K bits
// (valid because they are in increasing positions).
struct GatherA {
  SkewMap mp;
  Runs aM;
  uint64_t maskK = 0, incK = 0;
  SlabMap slab{};
};

// 128x128 workgroup tile, four waves of 64x64 (2x2 blocks of 32x32 MFMA
// tiles, 64 rows and columns apart), K staged through LDS 16 at a time; the
// next K tile is loaded into registers while the current one is multiplied.
// The 3M operand sums re+im are formed in registers after the LDS reads, which
// keeps the kernel within 256 registers per lane (two waves per SIMD).
// A vector instruction does not overlap an FP32 product of the same SIMD: one
// between two products costs 12 cycles, each further one 4 (a product takes
// 64).  So LDS holds (re, im) pairs at strides that fit the read
// instruction's two offsets: no address arithmetic in the K loop, and half
// the LDS instructions of separate planes (8192 x 8192 x 2048 in 3M 178 -> 186
// complex TFLOP/s, 2^18 x 128 x 256 161 -> 167; the rank-26 x rank-26 pair
// 3.28 -> 3.16 ms, with A read in place).
// z selects a batch entry or a split-K slab through the strides sA, sB, sC
// (GA: slabs only, A's through g.slab).
template <int FORM, int GA, typename OM>
__global__ __launch_bounds__(256, 2) void k_cgemm128(const float2* __restrict__ A, const float2* __restrict__ B,
                                                 float2* __restrict__ C, int64_t N, int64_t K, int64_t k_len,
                                                 int64_t sA, int64_t sB, int64_t sC, int64_t Mt, int64_t Nt,
                                                 int chunk, const GatherA g, const OM om) {
  constexpr int P = (FORM == TN_GEMM_3M) ? 3 : 2;
  constexpr int BM = 128, BN = 128, BK = 16, LD = 128;
  constexpr int LPT = 4;  // gathered A: 16-byte loads per thread per chunk
  // entry (k, row) of A and B at k * LD + (row ^ swz(k)): the two k halves of
  // a row that neighbouring threads store go to different banks
  __shared__ __attribute__((aligned(16))) float2 AB[2][BK * LD];
  float2* As = AB[0];
  float2* Bs = AB[1];
  auto swz = [](int k) { return (k & 8) << 1; };
  // gathered A: its stores' lanes may differ in any k bits, so bits 0 (which a
  // lane's reads do not change) and 1 move rows too; the planner gives the
  // lanes' k bits the numbers 3, 0 and 1 first (swizzle_order).  With bit 3
  // alone, A's with several k bits in their lowest positions were up to 14 %
  // slower (2^14 x 2^9 over 2^11, k at positions 1 to 5: 896 us, 797 now)
  auto swz_a = [&](int k) { return swz(k) ^ (GA != 0 ? (k & 1) << 3 ^ (k & 2) << 1 : 0); };
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int64_t tm, tn, z;
  xcd_tile(blockIdx.x, Mt, Nt, gridDim.x, tm, tn, z);
  const int64_t bm = tm * BM, bn = tn * BN;
  A += z * sA;
  B += z * sB;
  C += z * sC;
  const int wm = (wave & 1) * 32, wn = (wave >> 1) * 32;  // and 64 further on
  floatx16 acc[P][2][2];
#pragma unroll
  for (int p = 0; p < P; ++p)
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[p][i][j] = floatx16{};
  const int lrow = tid >> 1, lk = (tid & 1) * 8;
  const int slot0 = lk * LD + (lrow ^ swz(lk));  // entries (lk + q, lrow) at slot0 + q * LD
  const float2* Ap = A + (bm + lrow) * K + lk;
  int64_t brow_b = bn + lrow;
  if constexpr (has_out<OM>) brow_b = (int64_t)dep((uint64_t)brow_b, om.nmap);
  const float2* Bp = B + brow_b * K + lk;
  float4 ra[4], rb[4];
  // gathered A: a thread's entries are (j * 256 + tid) * 2 and the next one.
  // Offsets and LDS entries are sums (XORs) over the bits of that number, so
  // only tid's part is held per lane; j's and the odd entry's are uniform
  uint32_t eoff = 0, eidx = 0, uidx[GA ? LPT : 1], uodd = 0;
  uint64_t uoff[GA ? LPT : 1];
  uint64_t abase = 0, kofs = 0;
  float4 rg[GA ? LPT : 1];
  if constexpr (GA != 0) {
    auto entry = [&](int e, uint64_t& off) {
      int m, k;
      skew_split(g.mp, e, off, m, k);
      return (uint32_t)(k * LD + (m ^ swz_a(k)));
    };
    uint64_t off;
    uodd = entry(1, off);
    eidx = entry(tid * 2, off);
    eoff = (uint32_t)off;
#pragma unroll
    for (int j = 0; j < LPT; ++j) uidx[j] = entry(j * 512, uoff[j]);
    abase = dep_u<12>((uint64_t)bm, g.aM);
    kofs = slab_offset(g.slab, z);
  }
  auto load_a = [&]() {
    if constexpr (GA != 0) {
      const float2* base = A + (abase + kofs);
#pragma unroll
      for (int j = 0; j < LPT; ++j) rg[j] = *reinterpret_cast<const float4*>(base + uoff[j] + eoff);
    }
  };
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if constexpr (GA == 0) ra[j] = *reinterpret_cast<const float4*>(Ap + 2 * j);
    rb[j] = *reinterpret_cast<const float4*>(Bp + 2 * j);
  }
  load_a();
  const int c = lane & 31, kh = lane >> 5;
  // Adds (ADD false: stores) the running FP32 sums to C and restarts them.
  // Called every `chunk` K stages, where the staged operands have just been
  // written to LDS and the prefetch registers are free, so one FP32
  // accumulation chain covers at most chunk * BK terms.
  auto flush = [&](auto add) {
    constexpr bool ADD = decltype(add)::value;
    // the row stride is made opaque here so that the compiler does not keep
    // the 64 output addresses live across the K loop
    int64_t ld = N;
    asm volatile("" : "+s"(ld));
    float2* Cw = C + (bm + wm + 4 * kh) * ld + bn + wn + c;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float2 v;
          if (FORM == TN_GEMM_3M) {
            v.x = acc[0][i][j][r] - acc[1][i][j][r];
            v.y = acc[P - 1][i][j][r] - acc[0][i][j][r] - acc[1][i][j][r];
          } else {
            v.x = acc[0][i][j][r];
            v.y = acc[1][i][j][r];
          }
          float2* p = Cw + (64 * i + 8 * (r >> 2) + (r & 3)) * ld + 64 * j;
          if constexpr (ADD) {
            const float2 o = *p;
            v.x += o.x;
            v.y += o.y;
          }
          *p = v;
        }
#pragma unroll
        for (int q = 0; q < P; ++q) acc[q][i][j] = floatx16{};
        __builtin_amdgcn_sched_barrier(0);  // one 32x32 block's loads in flight at a time
      }
  };
  // this lane's operands: rows wm + c and wm + 64 + c at k = kk + kh
  const float2* a_at[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) a_at[q] = As + kh * LD + ((wm + c) ^ swz_a((q & 2) << 2 | (q & 1) << 1 | kh));
  const float2* b_lo = Bs + kh * LD + wn + c;
  const float2* b_hi = Bs + kh * LD + ((wn + c) ^ 16);
  bool first = true;
  int it = 0;
  for (int64_t k0 = 0; k0 < k_len; k0 += BK, ++it) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if constexpr (GA == 0) {
        As[slot0 + 2 * j * LD] = make_float2(ra[j].x, ra[j].y);
        As[slot0 + (2 * j + 1) * LD] = make_float2(ra[j].z, ra[j].w);
      }
      Bs[slot0 + 2 * j * LD] = make_float2(rb[j].x, rb[j].y);
      Bs[slot0 + (2 * j + 1) * LD] = make_float2(rb[j].z, rb[j].w);
    }
    if constexpr (GA != 0) {
      uint32_t e = eidx;
      asm volatile("" : "+v"(e));  // the XORs stay here: no registers for them across the K loop
#pragma unroll
      for (int j = 0; j < LPT; ++j) {
        As[e ^ uidx[j]] = make_float2(rg[j].x, rg[j].y);
        As[e ^ uidx[j] ^ uodd] = make_float2(rg[j].z, rg[j].w);
      }
    }
    if (chunk > 0 && it > 0 && it % chunk == 0) {
      if (first)
        flush(std::false_type{});
      else
        flush(std::true_type{});
      first = false;
    }
    __syncthreads();
    if (k0 + BK < k_len) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if constexpr (GA == 0) ra[j] = *reinterpret_cast<const float4*>(Ap + k0 + BK + 2 * j);
        rb[j] = *reinterpret_cast<const float4*>(Bp + k0 + BK + 2 * j);
      }
      if constexpr (GA != 0) {
        kofs = ((kofs | ~g.maskK) + g.incK) & g.maskK;
        load_a();
      }
    }
#pragma unroll
    for (int kk = 0; kk < BK; kk += 2) {
      float a[P][2], b[P][2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const float2 x = a_at[(kk >> 2 & 2) | (kk >> 1 & 1)][kk * LD + 64 * i], y = (kk < 8 ? b_lo : b_hi)[kk * LD + 64 * i];
        a[0][i] = x.x;
        a[1][i] = x.y;
        b[0][i] = y.x;
        b[1][i] = y.y;
      }
      if (P == 3)  // 3M operand sums, formed in FP32 from the staged re/im
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          a[P - 1][i] = a[0][i] + a[1][i];
          b[P - 1][i] = b[0][i] + b[1][i];
        }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          if (FORM == TN_GEMM_3M) {
            acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0][i], b[0][j], acc[0][i][j], 0, 0, 0);
            acc[1][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[1][i], b[1][j], acc[1][i][j], 0, 0, 0);
            acc[P - 1][i][j] =
                __builtin_amdgcn_mfma_f32_32x32x2f32(a[P - 1][i], b[P - 1][j], acc[P - 1][i][j], 0, 0, 0);
          } else {
            acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0][i], b[0][j], acc[0][i][j], 0, 0, 0);
            acc[0][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(-a[1][i], b[1][j], acc[0][i][j], 0, 0, 0);
            acc[1][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[0][i], b[1][j], acc[1][i][j], 0, 0, 0);
            acc[1][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[1][i], b[0][j], acc[1][i][j], 0, 0, 0);
          }
        }
    }
  }
  if constexpr (has_out<OM>) {
    // (sums of at most one chunk: nothing has been stored yet.)  Blocks (i, j)
    // of all four waves: one sub-tile in C's order at a time
    float2* Cs = AB[0];
    const int at = out_lane(om, c, kh) ^ (wave & 1 ? om.srow[5] : 0) ^ (wave >> 1 ? om.scol[5] : 0);
    const uint64_t tile = dep_u<12>((uint64_t)bm, om.cM) | dep_u<12>((uint64_t)bn, om.cN);
    const uint64_t toff = out_thread<float2>(om, tid);
    const uint64_t oi = dep_u<12>(64, om.cM), oj = dep_u<12>(64, om.cN);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float2 v;
          if (FORM == TN_GEMM_3M) {
            v.x = acc[0][i][j][r] - acc[1][i][j][r];
            v.y = acc[P - 1][i][j][r] - acc[0][i][j][r] - acc[1][i][j][r];
          } else {
            v.x = acc[0][i][j][r];
            v.y = acc[1][i][j][r];
          }
          Cs[at ^ out_reg(om, r)] = v;
        }
        __syncthreads();
        out_write<float2, 12>(om, C, Cs, tile | (i ? oi : 0) | (j ? oj : 0), toff, tid);
      }
    return;
  }
  if (first)
    flush(std::false_type{});
  else
    flush(std::true_type{});
}

// C[i] = sum over slabs s (in order) of W[s][i], summed in FP64 and rounded
// once.
__global__ __launch_bounds__(256) void k_splitk_sum(const float2* __restrict__ W, float2* __restrict__ C, int64_t n,
                                                   int slabs) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    double r = 0.0, im = 0.0;
    for (int sl = 0; sl < slabs; ++sl) {
      const float2 v = W[(int64_t)sl * n + i];
      r += (double)v.x;
      im += (double)v.y;
    }
    C[i] = make_float2((float)r, (float)im);
  }
}

bool gemm_shape_ok(int64_t M, int64_t N, int64_t K) {
  return M > 0 && N > 0 && K > 0 && M % GBM == 0 && N % GBN == 0 && K % GBK == 0;
}

hipError_t launch_gemm_c64(const float2* A, const float2* B, float2* C, int64_t M, int64_t N, int64_t K,
                           int64_t batch, int form, hipStream_t s, float2* work, int splits, int tile) {
  if (!gemm_shape_ok(M, N, K) || batch < 0) return hipErrorInvalidValue;
  if (batch == 0) return hipSuccess;
  if (splits < 1) splits = 1;
  const bool fits128 = (M % 128 == 0) && (N % 128 == 0);
  if (tile == 128 && !fits128) return hipErrorInvalidValue;
  const bool big = fits128 && tile != 64;
  const int chunk = kAccChain / 16;  // K stages of the 128x128 kernel per FP32 chain
  if (splits > 1) {
    if (batch != 1 || !work || K % (16 * splits) != 0 || splits > 65535) return hipErrorInvalidValue;
    const int64_t kl = K / splits;
    const int64_t n = M * N;
    if (!big) {  // 64x64 tiles, one slab per blockIdx.z
      if (N / GBN > 65535) return hipErrorInvalidValue;
      dim3 grid((unsigned)(M / GBM), (unsigned)(N / GBN), (unsigned)splits);
      if (form == TN_GEMM_3M)
        hipLaunchKernelGGL(k_cgemm<TN_GEMM_3M>, grid, dim3(256), 0, s, A, B, work, N, K, kl, kl, kl, n,
                           kAccChain / GBK);
      else
        hipLaunchKernelGGL(k_cgemm<TN_GEMM_4M>, grid, dim3(256), 0, s, A, B, work, N, K, kl, kl, kl, n,
                           kAccChain / GBK);
      hipLaunchKernelGGL(k_splitk_sum, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 8192)), dim3(256), 0, s,
                         work, C, n, splits);
      return hipGetLastError();
    }
    const int64_t Mt = M / 128, Nt = N / 128;
    dim3 grid((unsigned)(Mt * Nt * splits));
    if (form == TN_GEMM_3M)
      hipLaunchKernelGGL((k_cgemm128<TN_GEMM_3M, 0, NoOut>), grid, dim3(256), 0, s, A, B, work, N, K, kl, kl, kl, M * N, Mt, Nt,
                         chunk, GatherA{}, NoOut{});
    else
      hipLaunchKernelGGL((k_cgemm128<TN_GEMM_4M, 0, NoOut>), grid, dim3(256), 0, s, A, B, work, N, K, kl, kl, kl, M * N, Mt, Nt,
                         chunk, GatherA{}, NoOut{});
    hipLaunchKernelGGL(k_splitk_sum, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 8192)), dim3(256), 0, s,
                       work, C, n, splits);
    return hipGetLastError();
  }
  if (batch > 65535) return hipErrorInvalidValue;
  // short contractions are store-bound: the 64x64 kernel keeps more
  // workgroups in flight
  if (big && (K > 64 || tile == 128)) {
    const int64_t Mt = M / 128, Nt = N / 128;
    dim3 grid((unsigned)(Mt * Nt * batch));
    if (form == TN_GEMM_3M)
      hipLaunchKernelGGL((k_cgemm128<TN_GEMM_3M, 0, NoOut>), grid, dim3(256), 0, s, A, B, C, N, K, K, M * K, N * K, M * N, Mt, Nt,
                         chunk, GatherA{}, NoOut{});
    else
      hipLaunchKernelGGL((k_cgemm128<TN_GEMM_4M, 0, NoOut>), grid, dim3(256), 0, s, A, B, C, N, K, K, M * K, N * K, M * N, Mt, Nt,
                         chunk, GatherA{}, NoOut{});
    return hipGetLastError();
  }
  if (N / GBN > 65535) return hipErrorInvalidValue;
  dim3 grid((unsigned)(M / GBM), (unsigned)(N / GBN), (unsigned)batch);
  if (form == TN_GEMM_3M)
    hipLaunchKernelGGL(k_cgemm<TN_GEMM_3M>, grid, dim3(256), 0, s, A, B, C, N, K, K, M * K, N * K, M * N,
                       kAccChain / GBK);
  else
    hipLaunchKernelGGL(k_cgemm<TN_GEMM_4M>, grid, dim3(256), 0, s, A, B, C, N, K, K, M * K, N * K, M * N,
                       kAccChain / GBK);
  return hipGetLastError();
}

static uint64_t dep_host(uint64_t x, const Runs& r) {
  uint64_t o = 0;
  for (int i = 0; i < r.n; ++i) o |= ((x >> r.src[i]) & ((1ull << r.len[i]) - 1ull)) << r.dst[i];
  return o;
}

hipError_t launch_gemm_c64_ga(const float2* A, const float2* B, float2* C, const IndexOp& idx, int form,
                              hipStream_t s, float2* work, int splits, const OutMap* out) {
  if (!gemm_gather_ok(idx) || (splits > 1 && (!work || out))) return hipErrorInvalidValue;
  const int64_t M = (int64_t)1 << idx.nM, N = (int64_t)1 << idx.nN, K = (int64_t)1 << idx.nK;
  GatherA g{};
  skew_map(idx, 4, 0, &g.mp);
  g.aM = idx.aM;
  g.maskK = dep_host((uint64_t)(K - 1) & ~(uint64_t)15, idx.aK);
  g.incK = K > 16 ? dep_host(16, idx.aK) : 0;
  if (!slab_map(idx, splits, 4, &g.slab)) return hipErrorInvalidValue;
  if (g.mp.pos[0] != 0) return hipErrorInvalidValue;  // A's lowest bit must belong to the chunk
  const int chunk = kAccChain / 16;
  const int64_t Mt = M / 128, Nt = N / 128;
  const dim3 grid((unsigned)(Mt * Nt * splits));
  if (splits > 1) {
    const int64_t kl = K / splits, n = M * N;
    if (form == TN_GEMM_3M)
      hipLaunchKernelGGL((k_cgemm128<TN_GEMM_3M, 1, NoOut>), grid, dim3(256), 0, s, A, B, work, N, K, kl, 0, kl, n, Mt,
                         Nt, chunk, g, NoOut{});
    else
      hipLaunchKernelGGL((k_cgemm128<TN_GEMM_4M, 1, NoOut>), grid, dim3(256), 0, s, A, B, work, N, K, kl, 0, kl, n, Mt,
                         Nt, chunk, g, NoOut{});
    hipLaunchKernelGGL(k_splitk_sum, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 8192)), dim3(256), 0, s, work,
                       C, n, splits);
  } else if (out && form == TN_GEMM_3M)
    hipLaunchKernelGGL((k_cgemm128<TN_GEMM_3M, 1, OutMap>), grid, dim3(256), 0, s, A, B, C, N, K, K, 0, 0, 0, Mt, Nt,
                       chunk, g, *out);
  else if (out)
    hipLaunchKernelGGL((k_cgemm128<TN_GEMM_4M, 1, OutMap>), grid, dim3(256), 0, s, A, B, C, N, K, K, 0, 0, 0, Mt, Nt,
                       chunk, g, *out);
  else if (form == TN_GEMM_3M)
    hipLaunchKernelGGL((k_cgemm128<TN_GEMM_3M, 1, NoOut>), grid, dim3(256), 0, s, A, B, C, N, K, K, 0, 0, 0, Mt, Nt,
                       chunk, g, NoOut{});
  else
    hipLaunchKernelGGL((k_cgemm128<TN_GEMM_4M, 1, NoOut>), grid, dim3(256), 0, s, A, B, C, N, K, K, 0, 0, 0, Mt, Nt,
                       chunk, g, NoOut{});
  return hipGetLastError();
}

}  // namespace tnrcs
