// Small networks (gfx950): a slice whose tensors all fit one workgroup's LDS
// is contracted by one workgroup in one launch, all slices of a call side by
// side, instead of a bind, one launch per step and an accumulation per slice.
//
// What bounds such a network is latency: a launch in a captured chain costs
// 4-8 us however little it does.  Here the leaves of the slice (the sub-block
// that its sliced wires select) and the steps' offset tables are read once
// into LDS, every step runs from LDS with one barrier after it, and the
// slices' results are added to the amplitudes in slice order in FP64 by a
// second kernel (by the same one for a single slice), so that the sum is the
// same for any split of a range.  A 12-qubit, 16-slice network of three steps
// took 398 us slice by slice and takes 20 us.
//
// Arithmetic per step as in the gathered kernel: FP32 sums, scaled by the
// step's output scale and rounded to the storage type; several lanes share an
// output while the outputs are fewer than the threads, and a thread takes a
// block of outputs when they are more.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "elem.h"
#include "kernels.h"

namespace tnrcs {

namespace {

// root factor of a slice: 2^e_root, the unsliced leaves' rounding factor and
// the sliced leaves' for this slice
__device__ __forceinline__ double2 root_factor(const AccumDesc& d, double2 kap, bool sliced) {
  double kr = d.kappa0_re * d.root_scale, ki = d.kappa0_im * d.root_scale;
  if (sliced) {
    const double t = kr * kap.x - ki * kap.y;
    ki = kr * kap.y + ki * kap.x;
    kr = t;
  }
  return make_double2(kr, ki);
}

// A slice's share of an amplitude.  Spelled out: the single-slice kernel and
// the sum over slices must round alike.
__device__ __forceinline__ double2 slice_share(float2 v, double2 f) {
  const double x = v.x, y = v.y;
  return make_double2(__builtin_fma(x, f.x, -(y * f.y)), __builtin_fma(x, f.y, y * f.x));
}

constexpr int kSmallThreads = 256;

// One step's outputs in TM x TN blocks per thread (rows m and columns n at
// stride 2^nM / TM and 2^nN / TN, so that neighbouring lanes stay neighbours):
// TM + TN LDS operand reads and two table reads serve TM x TN multiply-adds.
// With one output per thread and 1024 threads the LDS reads bound wide steps
// (2^18.6 multiply-adds 98 us, 22 us in blocks, launch
// aside).
template <int TM, int TN, typename E>
__device__ __forceinline__ float small_blocks(const SmallOp& op, E* T, const uint16_t* tm, const uint16_t* tn,
                                              const uint16_t* ka, const uint16_t* kb, float sc) {
  constexpr int LM = TM == 4 ? 2 : TM == 2 ? 1 : 0, LN = TN == 4 ? 2 : TN == 2 ? 1 : 0;
  const int bM = op.nM - LM, bN = op.nN - LN, K = 1 << op.nK;
  float mx = 0.f;
  for (int i = threadIdx.x; i < 1 << (bM + bN); i += kSmallThreads) {
    const int m = i >> bN, n = i & ((1 << bN) - 1);
    const E *A[TM], *B[TN];
#pragma unroll
    for (int u = 0; u < TM; ++u) A[u] = T + op.a + tm[m + (u << bM)];
#pragma unroll
    for (int v = 0; v < TN; ++v) B[v] = T + op.b + tn[n + (v << bN)];
    float re[TM][TN], im[TM][TN];
#pragma unroll
    for (int u = 0; u < TM; ++u)
#pragma unroll
      for (int v = 0; v < TN; ++v) re[u][v] = im[u][v] = 0.f;
#pragma unroll 2
    for (int k = 0; k < K; ++k) {
      const int ak = ka[k], bk = kb[k];
      float2 x[TM], y[TN];
#pragma unroll
      for (int u = 0; u < TM; ++u) x[u] = to_f2(A[u][ak]);
#pragma unroll
      for (int v = 0; v < TN; ++v) y[v] = to_f2(B[v][bk]);
#pragma unroll
      for (int u = 0; u < TM; ++u)
#pragma unroll
        for (int v = 0; v < TN; ++v) {
          re[u][v] = fmaf(x[u].x, y[v].x, re[u][v]);
          re[u][v] = fmaf(-x[u].y, y[v].y, re[u][v]);
          im[u][v] = fmaf(x[u].x, y[v].y, im[u][v]);
          im[u][v] = fmaf(x[u].y, y[v].x, im[u][v]);
        }
    }
#pragma unroll
    for (int u = 0; u < TM; ++u)
#pragma unroll
      for (int v = 0; v < TN; ++v) {
        mx = mag_max(mx, re[u][v], im[u][v]);
        T[op.c + ((m + (u << bM)) << op.nN) + n + (v << bN)] = from_f2<E>(re[u][v] * sc, im[u][v] * sc);
      }
  }
  return mx;
}

// A lane's sum of up to 2^10 terms, four at a time, in a tree of degree four
// (a chain of 2^9 terms would round 2^10 times in a row; this as often as a
// split sum of a few terms per thread and a tree over the threads).
struct SumTree {
  float2 s[5] = {};
  // adds the g-th (from 1) group of four
  __device__ __forceinline__ void add(float re, float im, int g) {
    s[0].x += re;
    s[0].y += im;
#pragma unroll
    for (int l = 1; l < 5; ++l) {
      if (g & ((1 << 2 * l) - 1)) break;
      s[l].x += s[l - 1].x;
      s[l].y += s[l - 1].y;
      s[l - 1] = make_float2(0.f, 0.f);
    }
  }
  __device__ __forceinline__ void total(float& re, float& im) const {
    re = ((s[0].x + s[1].x) + (s[2].x + s[3].x)) + s[4].x;
    im = ((s[0].y + s[1].y) + (s[2].y + s[3].y)) + s[4].y;
  }
};

struct SmallShape {
  int32_t n_ops, n_leaves, n_tabs, root, root_tab, n_open, n_slots, pad_elems;
};

template <typename E>
__global__ __launch_bounds__(kSmallThreads) void k_small(const E* __restrict__ leaf_data, const SmallArgs g, const SmallShape h,
                                               const AccumDesc d, const double2* __restrict__ kappa, Ctrl* ctrl,
                                               const float* __restrict__ out_scales, float over, float under,
                                               int64_t s_begin, int64_t count, double* __restrict__ amp) {
  extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
  E* T = reinterpret_cast<E*>(lds);                               // tensors
  uint16_t* tabs = reinterpret_cast<uint16_t*>(T + h.pad_elems);  // offset tables
  SmallOp* ops = reinterpret_cast<SmallOp*>(tabs + h.n_tabs);
  unsigned* slot_max = reinterpret_cast<unsigned*>(ops + h.n_ops);
  __shared__ double2 kap;
  constexpr int nt = kSmallThreads, nw = nt / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  for (int i = tid; i < h.n_tabs / 8; i += nt)
    reinterpret_cast<uint4*>(tabs)[i] = reinterpret_cast<const uint4*>(g.tabs)[i];
  for (int i = tid; i < h.n_ops * (int)(sizeof(SmallOp) / 4); i += nt)
    reinterpret_cast<int*>(ops)[i] = reinterpret_cast<const int*>(g.ops)[i];
  const int n_amp = 1 << h.n_open;
  bool bad = false;
  unsigned flags = 0;
  for (int64_t sl = blockIdx.x; sl < count; sl += gridDim.x) {
    const int64_t s = s_begin + sl;
    for (int i = tid; i < h.n_slots; i += nt) slot_max[i] = 0u;
    if (kappa && tid == 0) {  // in leaf order, as the bind kernel does
      double kr = 1.0, ki = 0.0;
      for (int i = 0; i < h.n_leaves; ++i) {
        const SmallLeaf& l = g.leaves[i];
        if (l.kappa_off < 0) continue;
        int64_t b = 0;
        for (int j = 0; j < l.n_sl; ++j) b |= ((s >> l.sbit[j]) & 1ll) << (l.n_sl - 1 - j);
        const double2 f = kappa[l.kappa_off + b];
        const double t = kr * f.x - ki * f.y;
        ki = kr * f.y + ki * f.x;
        kr = t;
      }
      kap = make_double2(kr, ki);
    }
    for (int i = wave; i < h.n_leaves; i += nw) {
      const SmallLeaf& l = g.leaves[i];
      int64_t off = l.src;
      for (int j = 0; j < l.n_sl; ++j) off += ((s >> l.sbit[j]) & 1ll) << l.pos[j];
      for (int e = lane; e < l.n; e += 64) T[l.dst + e] = leaf_data[off + e];
    }
    __syncthreads();
    for (int o = 0; o < h.n_ops; ++o) {
      const SmallOp op = ops[o];
      const int lc = op.nM + op.nN, K = 1 << op.nK;
      const uint16_t* tm = tabs + op.tab;
      const uint16_t* tn = tm + (1 << op.nM);
      const uint16_t* ka = tn + (1 << op.nN);
      const uint16_t* kb = ka + K;
      const float sc = op.slot >= 0 ? out_scales[op.slot] : 1.f;
      float mx = 0.f;
      if (lc >= 12 && op.nM >= 2 && op.nN >= 2) {
        mx = small_blocks<4, 4, E>(op, T, tm, tn, ka, kb, sc);
      } else if (lc >= 11 && op.nM >= 2 && op.nN >= 1) {
        mx = small_blocks<4, 2, E>(op, T, tm, tn, ka, kb, sc);
      } else if (lc >= 10 && op.nM >= 1 && op.nN >= 1) {
        mx = small_blocks<2, 2, E>(op, T, tm, tn, ka, kb, sc);
      } else {
        // 2^L lanes share an output, lane t taking the terms t, t + 2^L, ... (a
        // sum of two terms rounds less in one chain than as the sum of two lanes)
        const int L = op.nK > 1 ? max(0, min(min(6, op.nK), 8 - lc)) : 0;
        const int t = tid & ((1 << L) - 1);
        for (int i = tid; i < 1 << (lc + L); i += kSmallThreads) {
          const int c = i >> L;
          const E* A = T + op.a + tm[c >> op.nN];
          const E* B = T + op.b + tn[c & ((1 << op.nN) - 1)];
          float re = 0.f, im = 0.f;
          auto madd = [&](int k, float& pr, float& pi) {
            const float2 x = to_f2(A[ka[k]]), y = to_f2(B[kb[k]]);
            pr = fmaf(x.x, y.x, pr);
            pr = fmaf(-x.y, y.y, pr);
            pi = fmaf(x.x, y.y, pi);
            pi = fmaf(x.y, y.x, pi);
          };
          if (K >> L < 4) {
            for (int k = t; k < K; k += 1 << L) madd(k, re, im);
          } else {
            SumTree sum;
            for (int k = t, g = 1; k < K; k += 4 << L, ++g) {
              float pr = 0.f, pi = 0.f;
#pragma unroll
              for (int q = 0; q < 4; ++q) madd(k + (q << L), pr, pi);
              sum.add(pr, pi, g);
            }
            sum.total(re, im);
          }
          for (int q = 1 << L >> 1; q > 0; q >>= 1) {
            re += __shfl_xor(re, q);
            im += __shfl_xor(im, q);
          }
          mx = mag_max(mx, re, im);
          if (t == 0) T[op.c + c] = from_f2<E>(re * sc, im * sc);
        }
      }
      if (op.slot >= 0) {
        for (int q = 32; q > 0; q >>= 1) mx = fmaxf(mx, __shfl_xor(mx, q));
        if (lane == 0) atomicMax(&slot_max[op.slot], __float_as_uint(mx));
      }
      __syncthreads();
    }
    const double2 f = root_factor(d, kap, kappa != nullptr);
    for (int y = tid; y < n_amp; y += nt) {
      const float2 v = to_f2(T[h.root + tabs[h.root_tab + y]]);
      bad |= !(isfinite(v.x) && isfinite(v.y));
      if (count == 1) {
        const double2 w = slice_share(v, f);
        amp[2 * y] += w.x;
        amp[2 * y + 1] += w.y;
      } else {
        g.roots[sl * n_amp + y] = v;
      }
    }
    if (count > 1 && tid == 0) g.factors[sl] = f;
    for (int i = tid; i < h.n_slots; i += nt) {
      const float m = __uint_as_float(slot_max[i]) * out_scales[i];
      if (!(m < over)) flags |= TN_FLAG_OVERFLOW;
      if (m < under) flags |= TN_FLAG_UNDERFLOW;
    }
    __syncthreads();  // the next slice's leaves overwrite the tensors
  }
  if (bad) flags |= TN_FLAG_NONFINITE;
  if (flags) atomicOr(&ctrl->flags, flags);
}

// amp += the slices' results in slice order, in FP64.  A block owns up to 256
// amplitudes; the slices' values pass through LDS in chunks, so that the chain
// of additions waits on LDS and not on memory.
constexpr int kSmallChunk = 2048;  // values per chunk

__global__ __launch_bounds__(256) void k_small_sum(const float2* __restrict__ roots,
                                                   const double2* __restrict__ factors, int n_open, int64_t count,
                                                   double* __restrict__ amp) {
  __shared__ float2 v[kSmallChunk];
  __shared__ double2 f[kSmallChunk];
  const int ln = n_open < 8 ? n_open : 8, ny = 1 << ln;  // amplitudes of this block
  const int per = kSmallChunk >> ln;                     // slices per chunk
  const int64_t n_amp = (int64_t)1 << n_open, y0 = (int64_t)blockIdx.x << ln;
  const int tid = threadIdx.x;
  double re = 0.0, im = 0.0;
  if (tid < ny) {
    re = amp[2 * (y0 + tid)];
    im = amp[2 * (y0 + tid) + 1];
  }
  for (int64_t s0 = 0; s0 < count; s0 += per) {
    const int ns = (int)(count - s0 < per ? count - s0 : per);
    for (int i = tid; i < ns << ln; i += 256) v[i] = roots[(s0 + (i >> ln)) * n_amp + y0 + (i & (ny - 1))];
    for (int i = tid; i < ns; i += 256) f[i] = factors[s0 + i];
    __syncthreads();
    if (tid < ny)
      for (int i = 0; i < ns; ++i) {
        const double2 w = slice_share(v[(i << ln) + tid], f[i]);
        re += w.x;
        im += w.y;
      }
    __syncthreads();
  }
  if (tid < ny) {
    amp[2 * (y0 + tid)] = re;
    amp[2 * (y0 + tid) + 1] = im;
  }
}

int32_t pad_elems(const SmallNet& net, int eb) { return (net.elems * eb + 15) / 16 * 16 / eb; }

size_t small_lds(const SmallNet& net, int eb, int n_slots) {
  return (size_t)pad_elems(net, eb) * eb + net.tabs.size() * 2 + net.ops.size() * sizeof(SmallOp) +
         (size_t)n_slots * 4;
}

template <typename E>
hipError_t launch_t(const void* leaf_data, const SmallNet& net, const SmallArgs& a, const AccumDesc& d,
                    const double2* kappa, Ctrl* ctrl, const float* out_scales, int n_slots, int64_t s_begin,
                    int64_t count, double* amp, float over, float under, hipStream_t s) {
  SmallShape h{};
  h.n_ops = (int32_t)net.ops.size();
  h.n_leaves = (int32_t)net.leaves.size();
  h.n_tabs = (int32_t)net.tabs.size();
  h.root = net.root;
  h.root_tab = net.root_tab;
  h.n_open = d.n_open;
  h.n_slots = n_slots;
  h.pad_elems = pad_elems(net, (int)sizeof(E));
  const dim3 grid((unsigned)std::min<int64_t>(count, 2048));
  hipLaunchKernelGGL(k_small<E>, grid, dim3(kSmallThreads), small_lds(net, (int)sizeof(E), n_slots), s, (const E*)leaf_data, a, h,
                     d, kappa, ctrl, out_scales, over, under, s_begin, count, amp);
  if (count > 1) {
    const dim3 g2((unsigned)std::max<int64_t>(1, (int64_t)1 << std::max(0, d.n_open - 8)));
    hipLaunchKernelGGL(k_small_sum, g2, dim3(256), 0, s, a.roots, a.factors, d.n_open, count, amp);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_small(int dtype, const void* leaf_data, const SmallNet& net, const SmallArgs& a, const AccumDesc& d,
                        const double2* kappa, Ctrl* ctrl, const float* out_scales, int n_slots, int64_t s_begin,
                        int64_t count, double* amp, hipStream_t s) {
  if (!net.ok || count < 1 || (count > 1 && (!a.roots || !a.factors))) return hipErrorInvalidValue;
  if (dtype == TN_DTYPE_F16S)
    return launch_t<cf16>(leaf_data, net, a, d, kappa, ctrl, out_scales, n_slots, s_begin, count, amp, 65504.f, 0.25f,
                          s);
  if (dtype == TN_DTYPE_BF16S)
    return launch_t<cbf16>(leaf_data, net, a, d, kappa, ctrl, out_scales, n_slots, s_begin, count, amp, 3.0e38f,
                           0.25f, s);
  return launch_t<float2>(leaf_data, net, a, d, nullptr, ctrl, out_scales, 0, s_begin, count, amp, 3.0e38f, 0.f, s);
}

hipError_t prepare_small(int dtype, const SmallNet& net, int n_slots) {
  const int bytes = (int)small_lds(net, elem_bytes_of(dtype), n_slots);
  if (bytes <= 64 * 1024) return hipSuccess;
  // raised for the device, never lowered: plans on other threads share it
  const void* k = dtype == TN_DTYPE_F16S    ? (const void*)k_small<cf16>
                  : dtype == TN_DTYPE_BF16S ? (const void*)k_small<cbf16>
                                            : (const void*)k_small<float2>;
  return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, kSmallLdsBytes);
}

}  // namespace tnrcs
