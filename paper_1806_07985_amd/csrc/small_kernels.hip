// Bandwidth- and latency-bound kernels of the NNCP iteration:
//  * multi-TTV (Section IV-A, Figure 2b): R independent matrix-vector products
//    over the contiguous blocks of a tree-node temporary, FP64 accumulation;
//  * the NLS-Update of one factor (Section II-B): HALS column sweep or the
//    multiplicative rule, one lane group per row, FP64 arithmetic;
//  * Gram matrix, column norms (lambda), the Hadamard product S of the other
//    modes' Grams, and the relative error from ||X||^2 - 2<X,M> + ||M||^2
//    (Section IV-B, appendix algorithm), all accumulated in FP64 with a
//    deterministic two-stage reduction;
//  * ||X||^2 and FP32 -> BF16/FP16 quantisation of the stored tensor.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "nncp_internal.hpp"

// (hipcc has no builtin for v_writelane_b32; the label names the intrinsic)
extern __device__ int writelane_i32(int v, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

namespace nncpk {
namespace {

constexpr int NT = 256;

template <typename T>
__device__ __forceinline__ double to_f64(T v);
template <>
__device__ __forceinline__ double to_f64<float>(float v) { return (double)v; }
template <>
__device__ __forceinline__ double to_f64<__bf16>(__bf16 v) { return (double)(float)v; }
template <>
__device__ __forceinline__ double to_f64<_Float16>(_Float16 v) { return (double)(float)v; }

// Element i of a buffer that holds doubles (f64 != 0) or floats.
__device__ __forceinline__ double ldv(const void* p, int64_t i, int f64) {
  return f64 ? as_global((const double*)p)[i] : (double)as_global((const float*)p)[i];
}
__device__ __forceinline__ void stv(void* p, int64_t i, int f64, double v) {
  if (f64) as_global((double*)p)[i] = v;
  else as_global((float*)p)[i] = (float)v;
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  __syncthreads();
  if (l == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) t += sh[i];
  return t;  // valid in thread 0
}

// --------------------------------------------------------------------------
// ||X||^2 in FP64
// --------------------------------------------------------------------------
// A group sums a contiguous run of the tensor; a thread reads 16-byte vectors (4
// FP32 or 8 16-bit values), eight of them, 4 KB apart, issued before any is used;
// the vector type is aligned to the element only, so any element-aligned base
// works. Up to four groups per CU hide one another's waits. 45.4 M values: FP32
// 65.9 -> 26.6 us (6.8 TB/s), BF16 55.4 -> 14.3 (6.3 TB/s); 268 M: 212 -> 152 and
// 124 -> 77 (one group per CU, sums added by the last of them to arrive). The
// n % VEC tail is read by block 0. Squares are exact in FP64 (a 24-bit significand
// squared fits 53 bits) and summed in FP64; the block sums are added in a fixed
// order by a second kernel of one block, so the result does not depend on
// scheduling (a sum by the last block to arrive needs a device-scope release per
// block, which writes the XCD's L2 back: 0.1 us each, one after the other).
template <typename T>
__global__ __launch_bounds__(NT) void norm_sq_kernel(const T* X, int64_t n, double* partial) {
  constexpr int VEC = 16 / sizeof(T);
  constexpr int U = 8;
  typedef T vT __attribute__((ext_vector_type(VEC), aligned(sizeof(T))));
  __shared__ double sh[NT / 64];
  const vT* V = (const vT*)X;
  const int64_t nv = n / VEC;
  // the group's run, a multiple of U * NT vectors
  const int64_t per = (nv + (int64_t)gridDim.x * U * NT - 1) / ((int64_t)gridDim.x * U * NT) * U * NT;
  const int64_t v0 = (int64_t)blockIdx.x * per;
  const int64_t v1 = v0 + per < nv ? v0 + per : nv;
  // four independent FP64 sums (vector lane e adds into e % 4), added in a fixed
  // order at the end, so the FMA chains do not serialise the stream
  double s4[4] = {0.0, 0.0, 0.0, 0.0};
  int64_t i = v0 + threadIdx.x;
  for (; i + (U - 1) * NT < v1; i += U * NT) {
    vT v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(V + i + u * NT);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < VEC; ++e) {
        const double x = to_f64<T>(v[u][e]);
        s4[e % 4] = __builtin_fma(x, x, s4[e % 4]);
      }
  }
  double s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
  for (; i < v1; i += NT) {
    const vT v = __builtin_nontemporal_load(V + i);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
      const double x = to_f64<T>(v[e]);
      s = __builtin_fma(x, x, s);
    }
  }
  if (blockIdx.x == 0)
    for (int64_t e = nv * VEC + threadIdx.x; e < n; e += NT) {
      const double x = to_f64<T>(X[e]);
      s = __builtin_fma(x, x, s);
    }
  double t = block_sum(s, sh);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}
__global__ __launch_bounds__(NT) void norm_sq_sum_kernel(const double* partial, int nb, double* out) {
  __shared__ double sh[NT / 64];
  double u = 0.0;
  for (int b = threadIdx.x; b < nb; b += NT) u += partial[b];
  u = block_sum(u, sh);
  if (threadIdx.x == 0) out[0] = u;
}

// --------------------------------------------------------------------------
// FP32 -> BF16 / FP16 (round to nearest even)
// --------------------------------------------------------------------------
// Eight values per thread and round (two 16-byte loads, one 16-byte store, aligned
// to the element only); the n % 8 tail by block 0. Bound by HBM: 45.4 M values 49
// -> 44 us (6.2 TB/s), 268 M 383 -> 299, against one value per thread (6 bytes each; 40 us at the rate of a
// large copy).
template <typename T>
__global__ __launch_bounds__(NT) void quantize_kernel(const float* src, T* dst, int64_t n) {
  typedef float f4e __attribute__((ext_vector_type(4), aligned(4)));
  typedef T t8 __attribute__((ext_vector_type(8), aligned(2)));
  const int64_t nv = n / 8, stride = (int64_t)gridDim.x * NT;
  for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < nv; i += stride) {
    const f4e a = __builtin_nontemporal_load((const f4e*)src + 2 * i);
    const f4e b = __builtin_nontemporal_load((const f4e*)src + 2 * i + 1);
    t8 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] = (T)a[e];
      o[e + 4] = (T)b[e];
    }
    *((t8*)dst + i) = o;
  }
  if (blockIdx.x == 0)
    for (int64_t i = nv * 8 + threadIdx.x; i < n; i += NT) dst[i] = (T)src[i];
}

__global__ void fill_u32_kernel(unsigned* p, int64_t n, unsigned v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
__global__ void fill_f64_kernel(double* p, int64_t n, double v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
__global__ void copy_f64_kernel(double* d, const double* s, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) d[i] = s[i];
}
__global__ void widen_f32_kernel(double* d, const float* s, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) d[i] = (double)s[i];
}
__global__ void unit_lambda_kernel(double* lam, int64_t n) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) lam[i] = lam[i] > 0.0 ? 1.0 : 0.0;
}

// --------------------------------------------------------------------------
// Multi-TTV, trailing modes: out(i, r) = sum_j T(i, j, r) K(j, r).
// Block: 64 rows i x 4 interleaved phases of j; K(:, r) formed in LDS chunks.
// --------------------------------------------------------------------------
constexpr int TRAIL_KCH = 1024;

// A node with few rows and a long J is split over nz runs of J (FP64 partials,
// added in order by the split-K sum kernel): one group per 64 rows and column
// leaves the chip idle then (64 rows, J = 262144 / 64, R = 32: 32 groups, 105 us).
template <typename TN>
__device__ __forceinline__ void mttv_trail_body(const MttvArgs& a, int bxz, int r) {
  __shared__ double kv[TRAIL_KCH];
  __shared__ double red[4][64];
  const int ti = threadIdx.x & 63, ph = threadIdx.x >> 6;
  const int bx = a.nz > 1 ? bxz / a.nz : bxz, z = a.nz > 1 ? bxz - bx * a.nz : 0;
  const int64_t jb = a.nz > 1 ? (int64_t)z * a.jz : 0;
  const int64_t je = a.nz > 1 && jb + a.jz < a.J ? jb + a.jz : a.J;
  const int64_t i = (int64_t)bx * 64 + ti;
  const double scale = krp_colscale(a.krp, r);
  const TN* Tr = as_global((const TN*)a.T) + (int64_t)r * a.Ia * a.J;
  double acc = 0.0;
  for (int64_t j0 = jb; j0 < je; j0 += TRAIL_KCH) {
    const int cnt = (int)((je - j0) < TRAIL_KCH ? (je - j0) : TRAIL_KCH);
    __syncthreads();
    // the Khatri-Rao column chunk: every factor load is issued (from a valid
    // address) before any product is formed
    for (int e = threadIdx.x; e < cnt; e += NT) {
      uint32_t rem = (uint32_t)(j0 + e);
      float fv[kMaxModes];
#pragma unroll
      for (int m = 0; m < kMaxModes; ++m) {
        const int mm = m < a.krp.nm ? m : 0;
        const uint32_t d = (uint32_t)a.krp.dim[mm];
        const uint32_t q = rem / d;
        const uint32_t dig = m < a.krp.nm ? rem - q * d : 0u;
        if (m < a.krp.nm) rem = q;
        fv[m] = as_global(a.krp.f[mm])[(int64_t)dig + (int64_t)a.krp.dim[mm] * r];
      }
      double p = scale;
#pragma unroll
      for (int m = 0; m < kMaxModes; ++m)
        if (m < a.krp.nm) p *= (double)fv[m];
      kv[e] = p;
    }
    __syncthreads();
    // sixteen rows j of this phase in flight per step (each thread still adds
    // its rows j = ph, ph + 4, ... in increasing order); rows past the chunk
    // (or past I_a) read a valid element and are weighted by zero
    const int64_t ic = i < a.Ia ? i : 0;
    const TN* base = Tr + ic + a.Ia * j0;
    for (int e = ph; e < cnt; e += 64) {
      TN t[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int ej = e + 4 * u;
        t[u] = base[a.Ia * (int64_t)(ej < cnt ? ej : e)];
      }
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const int ej = e + 4 * u;
        if (ej < cnt) acc += (double)t[u] * kv[ej];
      }
    }
  }
  red[ph][ti] = acc;
  __syncthreads();
  if (ph == 0 && i < a.Ia) {
    double s = red[0][ti] + red[1][ti] + red[2][ti] + red[3][ti];
    if (a.nz > 1) as_global(a.part)[((int64_t)z * a.R + r) * a.Ia + i] = s;
    else stv(a.out, i + a.Ia * r, a.out_f64, s);
  }
}
template <typename TN>
__global__ __launch_bounds__(NT) void mttv_trail_kernel(MttvArgs a) {
  mttv_trail_body<TN>(a, blockIdx.x, blockIdx.y);
}

// --------------------------------------------------------------------------
// Multi-TTV, leading modes: out(j, r) = sum_i T(i, j, r) K(i, r), i over the
// leading mode(s) of the node (K = their Khatri-Rao product, the first
// fastest; one mode: K = H), one lane group of GS lanes per output
// (contiguous dot product, shuffle reduction).
// --------------------------------------------------------------------------
template <int GS, typename TN>
__device__ __forceinline__ void mttv_lead_body(const MttvArgs& a, int bx) {
  constexpr int OPB = NT / GS;
  const int g = threadIdx.x / GS, p = threadIdx.x % GS;
  const int64_t o = (int64_t)bx * OPB + g;  // output index j + J*r
  const int64_t total = a.J * a.R;
  double acc = 0.0;
  int r = 0;
  if (o < total) {
    r = (int)(o / a.J);
    const int64_t j = o - (int64_t)r * a.J;
    const TN* Tc = as_global((const TN*)a.T) + a.Ia * (j + a.J * (int64_t)r);
    if (a.krp.nm == 1) {
      // eight products of the lane in flight, added in increasing i
      const float* Hc = as_global(a.krp.f[0]) + a.Ia * (int64_t)r;
      int64_t i = p;
      for (; i + 7 * GS < a.Ia; i += 8 * GS) {
        TN t[8];
        float h[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          t[u] = Tc[i + u * GS];
          h[u] = Hc[i + u * GS];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += (double)t[u] * (double)h[u];
      }
      for (; i < a.Ia; i += GS) acc += (double)Tc[i] * (double)Hc[i];
    } else {
      const bool narrow = a.Ia <= (int64_t)UINT32_MAX;  // 32-bit index arithmetic suffices
      for (int64_t i = p; i < a.Ia; i += GS) {
        double k = 1.0;
        if (narrow) {
          uint32_t rem = (uint32_t)i;
          for (int m = 0; m < a.krp.nm; ++m) {
            const uint32_t d = (uint32_t)a.krp.dim[m];
            const uint32_t q = rem / d;
            k *= (double)as_global(a.krp.f[m])[(int64_t)(rem - q * d) + (int64_t)d * r];
            rem = q;
          }
        } else {
          int64_t rem = i;
          for (int m = 0; m < a.krp.nm; ++m) {
            const int64_t d = a.krp.dim[m];
            const int64_t q = rem / d;
            k *= (double)as_global(a.krp.f[m])[(rem - q * d) + d * r];
            rem = q;
          }
        }
        acc += (double)Tc[i] * k;
      }
    }
  }
#pragma unroll
  for (int off = GS / 2; off > 0; off >>= 1) acc += __shfl_xor(acc, off, GS);
  if (p == 0 && o < total) stv(a.out, o, a.out_f64, acc * krp_colscale(a.krp, r));
}
template <int GS, typename TN>
__global__ __launch_bounds__(NT) void mttv_lead_kernel(MttvArgs a) {
  mttv_lead_body<GS, TN>(a, blockIdx.x);
}

// --------------------------------------------------------------------------
// NLS update (Section II-B), one wave per row. Lane p holds columns
// k = p + 64*v (v < VPL) of the warm start w, the MTTKRP row m and the running
// product g = w S. HALS visits r = 0..R-1 in order (Gauss-Seidel): every lane
// forms its candidate change, the owner's one is broadcast with readlane, and
// every lane updates g += d S(r, :). S and 1/S(r,r) live in LDS; all FP64.
// --------------------------------------------------------------------------
__device__ __forceinline__ double readlane_f64(double v, int lane) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)u, lane);
  const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(u >> 32), lane);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

template <int VPL>
__device__ __forceinline__ void update_body(const UpdateArgs& a, int bx) {
  extern __shared__ double Sl[];  // R*R, then R inverse diagonals
  const int R = a.R;
  double* invd = Sl + R * R;
  const int p = threadIdx.x & 63;
  const int64_t row = (int64_t)bx * (NT / 64) + (threadIdx.x >> 6);
  const bool live = row < a.I;  // wave-uniform
  // this row's loads are issued before S is staged, so their latency overlaps it
  double w[VPL], m[VPL], g[VPL];
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    const int k = p + 64 * v;
    w[v] = 0.0;
    m[v] = 0.0;
    g[v] = 0.0;
    if (live && k < R) {
      const double ls = a.lam_self[k];
      const double f = ls > 0.0 ? a.lam_model[k] / ls : 0.0;
      w[v] = (double)a.W[row + a.I * k] * f;
      m[v] = ldv(a.M, row + a.I * k, a.m_f64);
    }
  }
  for (int e = threadIdx.x; e < R * R; e += NT) Sl[e] = a.S[e];
  for (int k = threadIdx.x; k < R; k += NT) {
    const double d = a.S[k * R + k];
    invd[k] = d > 0.0 ? 1.0 / d : 0.0;
  }
  __syncthreads();
  if (!live) return;  // whole wave leaves together

  // g = w S with the starting w
  auto wS = [&]() {
#pragma unroll
    for (int q = 0; q < VPL; ++q) g[q] = 0.0;
    for (int r = 0; r < R; ++r) {
      const int v = r >> 6;
      double wv = w[0];
#pragma unroll
      for (int q = 1; q < VPL; ++q)
        if (v == q) wv = w[q];
      const double wr = readlane_f64(wv, r & 63);
#pragma unroll
      for (int q = 0; q < VPL; ++q) {
        const int k = p + 64 * q;
        if (k < R) g[q] += wr * Sl[r * R + k];
      }
    }
  };
  wS();
  const int sweeps = a.sweeps > 1 ? a.sweeps : 1;
  const double tol = a.tol;
  // the row's largest |w| (all lanes), for the relative change of a sweep
  auto wave_absmax = [&]() {
    double m = 0.0;
#pragma unroll
    for (int q = 0; q < VPL; ++q) m = fmax(m, fabs(w[q]));
    for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o, 64));
    return m;
  };
  if (a.update == NNCP_HALS) {
    // g stays equal to w S across sweeps: every column change is added to it
    for (int sw = 0; sw < sweeps; ++sw) {
      double dmax = 0.0;  // the sweep's largest |change| (uniform: every change is broadcast)
      for (int r = 0; r < R; ++r) {
        const int v = r >> 6;
        double wv = w[0], mv = m[0], gv = g[0];
  #pragma unroll
        for (int q = 1; q < VPL; ++q)
          if (v == q) {
            wv = w[q];
            mv = m[q];
            gv = g[q];
          }
        // column r: W(:,r) <- max(0, W(:,r) + (M(:,r) - (W S)(:,r)) / S(r,r)); a zero
        // diagonal (all-zero column elsewhere) sets the column to zero
        const double id = invd[r];
        double wn = id > 0.0 ? wv + (mv - gv) * id : 0.0;
        wn = wn > 0.0 ? wn : 0.0;
        const double d = readlane_f64(wn - wv, r & 63);
        dmax = fmax(dmax, fabs(d));
        if (p == (r & 63)) {
  #pragma unroll
          for (int q = 0; q < VPL; ++q)
            if (v == q) w[q] += d;
        }
  #pragma unroll
        for (int q = 0; q < VPL; ++q) {
          const int k = p + 64 * q;
          if (k < R) g[q] += d * Sl[r * R + k];
        }
      }
      if (tol > 0.0 && dmax <= tol * wave_absmax()) break;  // uniform
    }
  } else {
    for (int sw = 0; sw < sweeps; ++sw) {
      if (sw > 0) wS();
      double dloc = 0.0;
#pragma unroll
      for (int v = 0; v < VPL; ++v) {
        const double den = g[v] > 1e-16 ? g[v] : 1e-16;
        const double wn = w[v] * m[v] / den;
        dloc = fmax(dloc, fabs(wn - w[v]));
        w[v] = wn;
      }
      if (tol > 0.0) {
        for (int o = 32; o > 0; o >>= 1) dloc = fmax(dloc, __shfl_xor(dloc, o, 64));
        if (dloc <= tol * wave_absmax()) break;  // uniform
      }
    }
  }
#pragma unroll
  for (int v = 0; v < VPL; ++v) {
    const int k = p + 64 * v;
    if (k < R) {
      a.W[row + a.I * k] = (float)w[v];
      if (a.W64) a.W64[row + a.I * k] = w[v];
    }
  }
}
template <int VPL>
__global__ __launch_bounds__(NT) void update_kernel(UpdateArgs a) {
  update_body<VPL>(a, blockIdx.x);
}

// One row's update with lane k's column of S in registers (R <= RB <= 64): w =
// W(row, k) scaled to the model, m = M(row, k), srow[r] = S(r, k) (zero for r >= R
// or k >= R), invd = 1 / S(k, k) (zero unless positive). The column sweeps are
// unrolled over RB, so every broadcast uses a constant lane and the Gauss-Seidel
// chain touches no memory. Returns the new w.
// The row's latency is the chain of R column steps, so the chain is kept short:
// lanes hold the residual y = m - (w S) instead of m and w S, and column r's change
// is max(y / S(r,r), -w), which is W(:,r) <- max(0, W(:,r) + (M(:,r) - (W S)(:,r)) /
// S(r,r)) written as a difference: two operations, a broadcast and one update of y
// per step (1344 rows, R = 50: 11.6 -> 9.7 us; 50 sweeps of them 200 -> 103).
// With tol > 0 the sweeps stop early, once a sweep changes no entry of the row
// by more than tol times the row's largest entry (the row is one NNLS
// subproblem of the block; the rows are independent).
__device__ __forceinline__ double wave_max_f64(double v) {
  for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
  return v;
}
template <int RB>
__device__ __forceinline__ double update_row_reg(double w, const double m, const double (&srow)[RB],
                                                 const double invd, const int k, const int R, const int update,
                                                 const int sweeps, const double tol) {
  auto wS = [&]() {  // w S, two sums
    double g0 = 0.0, g1 = 0.0;
#pragma unroll
    for (int r = 0; r < RB; r += 2) {
      g0 += readlane_f64(w, r) * srow[r];
      g1 += readlane_f64(w, r + 1) * srow[r + 1];
    }
    return g0 + g1;
  };
  if (update == NNCP_HALS) {
    double y = m - wS();
    // a zero diagonal (all-zero column elsewhere) sets the column to zero: its
    // candidate change is -inf, so the maximum is -w
    const double bias = invd > 0.0 ? 0.0 : -__builtin_huge_val();
    // A sweep. Column r's change goes from lane r to all lanes; lane r's own w is
    // read in its own step only, so the changes are collected in lane r of `dl` and
    // added to w at the end. Steps at or past R change nothing (their w, y and S are
    // zero), so the rank is looked at once per eight columns: a branch per column
    // costs as much as the step.
    auto sweep = [&]() {
      int lo = 0, hi = 0;
#pragma unroll
      for (int r0 = 0; r0 < RB; r0 += 8) {
        if (r0 < R) {  // uniform
#pragma unroll
          for (int r = r0; r < r0 + 8; ++r) {
            const uint64_t u = __builtin_bit_cast(uint64_t, fmax(__builtin_fma(y, invd, bias), -w));
            const int dlo = __builtin_amdgcn_readlane((int)(uint32_t)u, r);
            const int dhi = __builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), r);
            const double dlt = __builtin_bit_cast(double, ((uint64_t)(uint32_t)dhi << 32) | (uint32_t)dlo);
            y = __builtin_fma(-dlt, srow[r], y);
            lo = writelane_i32(dlo, r, lo);
            hi = writelane_i32(dhi, r, hi);
          }
        }
      }
      const double dl = __builtin_bit_cast(double, ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
      w += dl;
      return dl;
    };
    // y stays m - w S across sweeps: every column change is taken off it
    if (tol > 0.0) {
      for (int sw = 0; sw < sweeps; ++sw) {
        const double dl = sweep();
        if (wave_max_f64(fabs(dl)) <= tol * wave_max_f64(fabs(w))) break;  // uniform
      }
    } else {
      for (int sw = 0; sw < sweeps; ++sw) sweep();
    }
  } else {
    for (int sw = 0; sw < sweeps; ++sw) {
      const double g = wS();
      const double den = g > 1e-16 ? g : 1e-16;
      const double wn = w * m / den;
      const double d = fabs(wn - w);
      w = wn;
      if (tol > 0.0 && wave_max_f64(d) <= tol * wave_max_f64(fabs(w))) break;  // uniform
    }
  }
  return w;
}

// Lane k's column of S (zero outside R x R) and 1 / S(k, k), loaded unconditionally.
template <int RB>
__device__ __forceinline__ void load_s_column(const UpdateArgs& a, int k, double (&srow)[RB], double& invd) {
  const int R = a.R;
  const bool col = k < R;
  const int kc = col ? k : 0;
#pragma unroll
  for (int r = 0; r < RB; ++r) srow[r] = a.S[(int64_t)(r < R ? r : 0) * R + kc];  // S symmetric
  const double dg = a.S[(int64_t)kc * R + kc];
  invd = (col && dg > 0.0) ? 1.0 / dg : 0.0;
#pragma unroll
  for (int r = 0; r < RB; ++r)
    if (!(col && r < R)) srow[r] = 0.0;
}

// The update for R <= RB <= 64: one wave per row.
template <int RB>
__device__ __forceinline__ void update_reg_body(const UpdateArgs& a, int bx) {
  const int R = a.R;
  const int k = threadIdx.x & 63;
  const int64_t row = (int64_t)bx * (NT / 64) + (threadIdx.x >> 6);
  if (row >= a.I) return;  // wave-uniform; no barrier in this kernel
  const bool col = k < R;
  const int kc = col ? k : 0;  // every load is unconditional (from a valid index), masked after
  const double ls = a.lam_self[kc], lm = a.lam_model[kc];
  const double w0 = (double)a.W[row + a.I * kc];
  const double m0 = ldv(a.M, row + a.I * kc, a.m_f64);
  double srow[RB], invd;
  load_s_column<RB>(a, k, srow, invd);
  const double f = ls > 0.0 ? lm / ls : 0.0;
  const double w = update_row_reg<RB>(col ? w0 * f : 0.0, col ? m0 : 0.0, srow, invd, k, R, a.update,
                                      a.sweeps > 1 ? a.sweeps : 1, a.tol);
  if (col) {
    a.W[row + a.I * k] = (float)w;
    if (a.W64) a.W64[row + a.I * k] = w;
  }
}
// The update for R <= RB <= 32 and many rows: one lane per row. The lane holds the
// whole row of W in registers and forms (W S)(:,r) afresh for every column from S
// in LDS (read by broadcast, two entries per load), so a wave updates 64 rows with
// R multiply-adds per column instead of one row with a broadcast chain per column,
// and its loads of M and W are 64 consecutive rows of a column. 30012 rows, R = 10:
// one wave per row 23.7 us (each wave reads a line per column for one row), so 6.
template <int RB>
__device__ __forceinline__ void update_lane_body(const UpdateArgs& a, int bx) {
  __shared__ double Sl[RB * RB], inv[RB], low[RB], fs[RB];  // low: 0, or -inf where a column is set to zero
  const int R = a.R;
  const int64_t row = (int64_t)bx * NT + threadIdx.x;
  const bool live = row < a.I;
  const int64_t rc = live ? row : a.I - 1;
  double w[RB], m[RB];
#pragma unroll
  for (int k = 0; k < RB; ++k) {
    const int kc = k < R ? k : 0;
    w[k] = (double)a.W[rc + a.I * kc];
  }
  // (one branch for all of M's loads: a branch around each would wait for each)
  if (a.m_f64) {
    const double* Mp = as_global((const double*)a.M) + rc;
#pragma unroll
    for (int k = 0; k < RB; ++k) m[k] = Mp[a.I * (k < R ? k : 0)];
  } else {
    const float* Mp = as_global((const float*)a.M) + rc;
    float mf[RB];
#pragma unroll
    for (int k = 0; k < RB; ++k) mf[k] = Mp[a.I * (k < R ? k : 0)];
#pragma unroll
    for (int k = 0; k < RB; ++k) m[k] = (double)mf[k];
  }
  for (int e = threadIdx.x; e < RB * RB; e += NT) {
    const int r = e / RB, k = e % RB;
    Sl[e] = r < R && k < R ? a.S[r * R + k] : 0.0;
  }
  if (threadIdx.x < RB) {
    const int k = threadIdx.x < R ? threadIdx.x : 0;
    const double d = a.S[k * R + k];
    inv[threadIdx.x] = d > 0.0 ? 1.0 / d : 0.0;
    low[threadIdx.x] = d > 0.0 ? 0.0 : -__builtin_huge_val();
    const double ls = a.lam_self[k], lm = a.lam_model[k];
    fs[threadIdx.x] = threadIdx.x < R && ls > 0.0 ? lm / ls : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < RB; ++k) w[k] *= fs[k];
  // `z` is zero, but not to the compiler: S stays in LDS instead of being hoisted
  // out of the sweeps into registers that there are not
  int z = 0;
  auto dot = [&](int r) {  // (w S)(r), four sums
    double g[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < RB; ++k) g[k & 3] = __builtin_fma(w[k], Sl[z + r * RB + k], g[k & 3]);
    __builtin_amdgcn_sched_barrier(0);
    return (g[0] + g[1]) + (g[2] + g[3]);
  };
  const int sweeps = a.sweeps > 1 ? a.sweeps : 1;
  bool go = live;  // this row still sweeps
  for (int sw = 0; sw < sweeps; ++sw) {
    double dmax = 0.0, wmax = 0.0;
    asm volatile("v_mov_b32 %0, 0" : "=v"(z));
    if (a.update == NNCP_HALS) {
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        if (r < R) {  // uniform
          const double y = m[r] - dot(r);
          const double d = fmax(__builtin_fma(y, inv[r], low[r]), -w[r]);
          w[r] = go ? w[r] + d : w[r];
          dmax = fmax(dmax, fabs(d));
        }
      }
    } else {
      double wn[RB];
#pragma unroll
      for (int r = 0; r < RB; ++r) {
        wn[r] = 0.0;
        if (r < R) {
          const double g = dot(r), den = g > 1e-16 ? g : 1e-16;
          wn[r] = w[r] * m[r] / den;
          dmax = fmax(dmax, fabs(wn[r] - w[r]));
        }
      }
#pragma unroll
      for (int r = 0; r < RB; ++r) w[r] = go ? wn[r] : w[r];
    }
    if (a.tol > 0.0) {
#pragma unroll
      for (int r = 0; r < RB; ++r) wmax = fmax(wmax, fabs(w[r]));
      go = go && !(dmax <= a.tol * wmax);
      if (!__any(go)) break;
    }
  }
  if (live) {
#pragma unroll
    for (int k = 0; k < RB; ++k)
      if (k < R) {
        a.W[row + a.I * k] = (float)w[k];
        if (a.W64) a.W64[row + a.I * k] = w[k];
      }
  }
}
template <int RB>
__global__ __launch_bounds__(NT) void update_lane_kernel(UpdateArgs a) {
  update_lane_body<RB>(a, blockIdx.x);
}

template <int RB>
__global__ __launch_bounds__(NT) void update_reg_kernel(UpdateArgs a) {
  update_reg_body<RB>(a, blockIdx.x);
}

constexpr int kUpdLane = 100;  // update variants of one lane per row: 100 + registers

// Rows of W staged in LDS at a time (FP64): about 32 KB.
__host__ __device__ inline int fin_sub_rows(int R) {
  int r = 4096 / (R > 0 ? R : 1);
  return r < 1 ? 1 : (r > 256 ? 256 : r);
}

// Stage 1: W^T W (and <M, W> when the fit is due) over this block's row chunk,
// written to partial[chunk] (R*R + 1 doubles).
__device__ void gram_chunk(const FinalizeArgs& a, double* fl, double* sh, int bx) {
  const int R = a.R, RR = R * R;
  const int sub = fin_sub_rows(R);
  const int64_t r0 = (int64_t)bx * a.rows_per_chunk;
  int64_t r1 = r0 + a.rows_per_chunk;
  if (r1 > a.I) r1 = a.I;
  double* part = a.partial + (size_t)bx * (RR + 1);
  // Each thread owns entries e = tid, tid + NT, ...; the running sums live in
  // this block's partial slot (only this thread touches them).
  double bsum = 0.0;
  bool first = true;
  for (int64_t s0 = r0; s0 < r1 || first; s0 += sub) {
    const int cnt = (int)((r1 - s0) < sub ? (r1 - s0) : sub);
    __syncthreads();
    for (int e = threadIdx.x; e < cnt * R; e += NT) {
      const int k = e / cnt, rw = e - k * cnt;
      const double wv = (double)a.W[s0 + rw + a.I * k];
      fl[rw * R + k] = wv;
      if (a.do_fit && a.M) bsum += wv * ldv(a.M, s0 + rw + a.I * k, a.m_f64);
    }
    __syncthreads();
    // four entries per thread at a time (independent FMA chains), rows unrolled
    for (int eg = threadIdx.x; eg < RR; eg += 4 * NT) {
      int ex[4], ey[4];
      double sacc[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = eg + q * NT < RR ? eg + q * NT : eg;
        ex[q] = e / R;
        ey[q] = e - ex[q] * R;
        sacc[q] = 0.0;
      }
#pragma unroll 4
      for (int rw = 0; rw < cnt; ++rw) {
        const double* row = fl + rw * R;
#pragma unroll
        for (int q = 0; q < 4; ++q) sacc[q] += row[ex[q]] * row[ey[q]];
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int e = eg + q * NT;
        if (e < RR) part[e] = first ? sacc[q] : part[e] + sacc[q];
      }
    }
    first = false;
  }
  double bt = block_sum(bsum, sh);
  if (threadIdx.x == 0) part[RR] = bt;
}

// Stage 2 (one block): reduce the chunk partials in chunk order, then lambda =
// sqrt(diag G_hat), the normalised Gram, the model weights, S for the next mode
// and, after the last mode, the fit.
__device__ void finalize_tail(const FinalizeArgs& a, double* fl, double* sh) {
  const int R = a.R, RR = R * R;
  double* Gh = fl;  // R*R + 1 scratch
  for (int e = threadIdx.x; e < RR + 1; e += NT) {
    double s = 0.0;
    for (int c = 0; c < a.nchunks; ++c) s += a.partial[(size_t)c * (RR + 1) + e];
    Gh[e] = s;
  }
  __syncthreads();
  if (a.gram_raw)
    for (int e = threadIdx.x; e < RR; e += NT) a.gram_raw[e] = Gh[e];
  double* lamm = a.lam + (int64_t)a.mode * R;
  for (int k = threadIdx.x; k < R; k += NT) {
    const double l = sqrt(Gh[k * R + k]);
    lamm[k] = l;
    if (a.set_model) a.lam_model[k] = l;
  }
  double* Gm = a.G + (int64_t)a.mode * RR;
  for (int e = threadIdx.x; e < RR; e += NT) {
    const int x = e / R, y = e - x * R;
    const double lx = sqrt(Gh[x * R + x]), ly = sqrt(Gh[y * R + y]);
    Gm[e] = (lx > 0.0 && ly > 0.0) ? Gh[e] / (lx * ly) : 0.0;
  }
  __syncthreads();
  if (a.do_fit) {
    // gamma = 1^T (S^(mode) * G_hat) 1, S^(mode) the Hadamard of the other Grams
    const double* Sm = a.S + (int64_t)a.mode * RR;
    double gp = 0.0;
    for (int e = threadIdx.x; e < RR; e += NT) gp += Sm[e] * Gh[e];
    double gamma = block_sum(gp, sh);
    if (threadIdx.x == 0) {
      const double alpha = a.alpha[0];
      const double beta = Gh[RR];
      double num = alpha - 2.0 * beta + gamma;
      num = num > 0.0 ? num : 0.0;
      const double eps = alpha > 0.0 ? sqrt(num / alpha) : 0.0;
      const int it = *a.iter_counter;
      if (it < a.fit_capacity) a.fit_out[it] = 1.0 - eps;
      *a.iter_counter = it + 1;
    }
    __syncthreads();
  }
  if (a.next_mode >= 0) {
    // this block wrote G[mode] above; the other modes' Grams are from earlier kernels
    double* Sn = a.S + (int64_t)a.next_mode * RR;
    for (int e = threadIdx.x; e < RR; e += NT) {
      double s = 1.0;
      for (int k = 0; k < a.N; ++k)
        if (k != a.next_mode) s *= a.G[(int64_t)k * RR + e];
      Sn[e] = s;
    }
  }
}

// Ranks up to this use the 1024-thread Gram kernels below.
constexpr int kSmallMaxR = 64;

// One block does both stages (a single row chunk).
__device__ __forceinline__ void finalize_fused_body(const FinalizeArgs& a) {
  extern __shared__ double fl[];
  __shared__ double sh[NT / 64];
  gram_chunk(a, fl, sh, 0);
  __syncthreads();
  finalize_tail(a, fl, sh);
}
__device__ __forceinline__ void gram_chunks_body(const FinalizeArgs& a, int bx) {
  extern __shared__ double fl[];
  __shared__ double sh[NT / 64];
  gram_chunk(a, fl, sh, bx);
}
__device__ __forceinline__ void finalize_tail_body(const FinalizeArgs& a) {
  extern __shared__ double fl[];
  __shared__ double sh[NT / 64];
  finalize_tail(a, fl, sh);
}
__global__ __launch_bounds__(NT) void finalize_fused_kernel(FinalizeArgs a) { finalize_fused_body(a); }
__global__ __launch_bounds__(NT) void gram_chunks_kernel(FinalizeArgs a) { gram_chunks_body(a, blockIdx.x); }
__global__ __launch_bounds__(NT) void finalize_tail_kernel(FinalizeArgs a) { finalize_tail_body(a); }

// ---------------------------------------------------------------------------
// Gram, lambda, next S and the fit for R <= 64 with 1024-thread work-groups. W^T W
// runs on the FP64 matrix instruction (16x16x4): a wave takes one pair of 16-column
// blocks of the upper triangle and every ns-th group of 16 rows, both operands
// straight from global memory (a lane's four rows of one column are one 16-byte
// load and feed four products; the order of the rows in a sum is free), and the
// waves of a pair add up through LDS in a fixed order. These kernels are bound by
// latency: staging the rows through LDS and 4x4 register blocks took five barriers
// and a long chain of LDS reads (1344 x 50 in four groups: 26.5 us, one group of
// 128 x 32: 10.4 us; now, in seven groups, 12.5 and 7.2). Entry e of an R x R matrix belongs
// to thread e mod 1024, slot e / 1024 (at most four slots).
constexpr int NTF = 1024;
typedef double d4 __attribute__((ext_vector_type(4)));

__host__ __device__ inline int fin_nb(int R) { return (R + 15) >> 4; }
__host__ __device__ inline int fin_pairs(int R) { return fin_nb(R) * (fin_nb(R) + 1) / 2; }
__host__ __device__ inline int fin_ns(int R) { return 16 / fin_pairs(R); }
// dynamic LDS doubles: one 16 x 16 block per wave (<= 32 KB)
__host__ __device__ inline int fin_work_doubles(int R) { return fin_ns(R) * fin_pairs(R) * 256; }
// R x R entries per thread: 1, 2 or 4
__host__ __device__ inline int fin_ep(int R) { return R * R <= NTF ? 1 : (R * R <= 2 * NTF ? 2 : 4); }

__device__ __forceinline__ int tri_index(int bx, int by, int nb) { return bx * nb - bx * (bx - 1) / 2 + (by - bx); }

// Rows row .. row + 3 of column col in FP64, zero for rows at or past r1 and for
// columns at or past R. `whole`: the four rows exist (a 16-byte load, aligned to
// the element); else element loads from clamped rows.
__device__ __forceinline__ d4 fin_rows4(const FinalizeArgs& a, int64_t row, int64_t r1, int col, bool whole) {
  typedef float f4e __attribute__((ext_vector_type(4), aligned(4)));
  const float* W = as_global(a.W) + a.I * (int64_t)(col < a.R ? col : 0);
  f4e v;
  if (whole) {
    v = *(const f4e*)(W + row);
  } else {
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = W[row + u < a.I ? row + u : a.I - 1];
  }
  d4 x;
#pragma unroll
  for (int u = 0; u < 4; ++u) x[u] = col < a.R && row + u < r1 ? (double)v[u] : 0.0;
  return x;
}

// W^T W over rows [r0, r1) into g[q] (entry tid + NTF*q; raw, unnormalised) and
// beta = sum of M o W over those rows (thread 0, when the fit is due). Block-wide;
// work: fin_work_doubles.
template <int EP>
__device__ __forceinline__ void gram1k_rows(const FinalizeArgs& a, int64_t r0, int64_t r1, double* work, double* sh,
                                            double (&g)[EP], double& beta) {
  const int R = a.R, RR = R * R, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lq = lane >> 4;
  const int nb = fin_nb(R), np = fin_pairs(R), ns = fin_ns(R);
  const int p = wave % np, q0 = wave / np;
  const bool active = q0 < ns;
  int bi = 0, bj = p;  // the pair's blocks, bi <= bj (row-major over the triangle)
  while (bj >= nb - bi) {
    bj -= nb - bi;
    ++bi;
  }
  bj += bi;
  d4 acc = {0.0, 0.0, 0.0, 0.0};
  if (active) {
    for (int64_t t = r0 + 16 * q0; t < r1; t += 32 * ns) {  // two row groups in flight
      const int64_t t2 = t + 16 * ns;
      const bool w1 = t + 16 <= a.I, w2 = t2 + 16 <= a.I;  // uniform
      const int64_t ra = t + 4 * lq, rb = t2 + 4 * lq;
      const d4 x0 = fin_rows4(a, ra, r1, 16 * bi + li, w1);
      const d4 x1 = fin_rows4(a, rb, r1, 16 * bi + li, w2);
      d4 y0 = x0, y1 = x1;
      if (bj != bi) {
        y0 = fin_rows4(a, ra, r1, 16 * bj + li, w1);
        y1 = fin_rows4(a, rb, r1, 16 * bj + li, w2);
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x0[u], y0[u], acc, 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x1[u], y1[u], acc, 0, 0, 0);
    }
  }
  beta = 0.0;
  if (a.do_fit && a.M) {
    // element e = tid + NTF * q is row r0 + e mod cnt of column e / cnt; (k, rw) step
    // with e, and four elements' loads are in flight
    const unsigned cnt = (unsigned)(r1 - r0), dk = NTF / cnt, drw = NTF - dk * cnt;  // (an extent is below 2^31)
    const int64_t n = (int64_t)cnt * R;
    unsigned k = tid / cnt, rw = tid - k * cnt;
    double bsum = 0.0;
    for (int64_t e = tid; e < n; e += 4 * NTF) {
      float w[4];
      double m[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const bool in = e + u * NTF < n;
        const int64_t idx = in ? r0 + rw + a.I * (int64_t)k : r0;
        w[u] = as_global(a.W)[idx];
        m[u] = in ? ldv(a.M, idx, a.m_f64) : 0.0;
        k += dk;
        rw += drw;
        if (rw >= cnt) {
          rw -= cnt;
          ++k;
        }
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
        if (e + u * NTF < n) bsum += (double)w[u] * m[u];
    }
    beta = block_sum(bsum, sh);
  }
  // acc[v]: row 4v + lq, column li of the block; splits summed in order
  if (active) {
#pragma unroll
    for (int v = 0; v < 4; ++v) work[(q0 * np + p) * 256 + (4 * v + lq) * 16 + li] = acc[v];
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < EP; ++q) {
    const int e = tid + NTF * q;
    const int ec = e < RR ? e : 0;
    const int x = ec / R, y = ec - (ec / R) * R;
    const int X = x >> 4, Y = y >> 4;
    const int b = X <= Y ? tri_index(X, Y, nb) : tri_index(Y, X, nb);
    const int at = X <= Y ? (x & 15) * 16 + (y & 15) : (y & 15) * 16 + (x & 15);
    double s = 0.0;
    for (int c = 0; c < ns; ++c) s += work[(c * np + b) * 256 + at];
    g[q] = s;
  }
}

// What the tail needs from global memory, requested up front: the product P of
// the Grams of the modes other than `mode` and `next_mode` (for S of the next
// mode), S of this mode (for gamma), alpha and the iteration counter.
template <int EP>
struct FinPre {
  double P[EP], Sm[EP];
  double alpha;
  int it;
};
template <int EP>
__device__ __forceinline__ void fin_preload(const FinalizeArgs& a, FinPre<EP>& p) {
  const int RR = a.R * a.R, tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < EP; ++q) p.P[q] = 1.0;
  double t[kMaxModes - 2][EP];
#pragma unroll
  for (int j = 0; j < kMaxModes - 2; ++j)
#pragma unroll
    for (int q = 0; q < EP; ++q) t[j][q] = 1.0;
  if (a.next_mode >= 0) {
    const int lo = a.mode < a.next_mode ? a.mode : a.next_mode;
    const int hi = a.mode < a.next_mode ? a.next_mode : a.mode;
#pragma unroll
    for (int j = 0; j < kMaxModes - 2; ++j) {
      int k = j;
      if (k >= lo) ++k;
      if (k >= hi) ++k;
      if (k < a.N) {  // uniform
#pragma unroll
        for (int q = 0; q < EP; ++q) {
          const int e = tid + NTF * q;
          t[j][q] = a.G[(int64_t)k * RR + (e < RR ? e : 0)];
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < EP; ++q) p.Sm[q] = 0.0;
  p.alpha = 0.0;
  p.it = 0;
  if (a.do_fit) {  // S, alpha and the counter are only there when the fit is due
#pragma unroll
    for (int q = 0; q < EP; ++q) {
      const int e = tid + NTF * q;
      p.Sm[q] = a.S[(int64_t)a.mode * RR + (e < RR ? e : 0)];
    }
    p.alpha = a.alpha[0];
    p.it = *a.iter_counter;
  }
#pragma unroll
  for (int j = 0; j < kMaxModes - 2; ++j)
#pragma unroll
    for (int q = 0; q < EP; ++q) p.P[q] *= t[j][q];
}

// lambda, normalised Gram, S of the next mode, the raw Gram if asked, and the fit.
template <int EP>
__device__ __forceinline__ void fin1k_tail(const FinalizeArgs& a, const double (&g)[EP], double beta, const FinPre<EP>& p,
                           double* sh) {
  __shared__ double dg[kSmallMaxR], il[kSmallMaxR];
  const int R = a.R, RR = R * R, tid = threadIdx.x;
  int xs[EP], ys[EP];
#pragma unroll
  for (int q = 0; q < EP; ++q) {
    const int e = tid + NTF * q;
    const int ec = e < RR ? e : 0;
    xs[q] = ec / R;
    ys[q] = ec - xs[q] * R;
    if (e < RR && xs[q] == ys[q]) dg[xs[q]] = g[q];
  }
  __syncthreads();
  double* lamm = a.lam + (int64_t)a.mode * R;
  if (tid < R) {
    const double l = sqrt(dg[tid]);
    lamm[tid] = l;
    if (a.set_model) a.lam_model[tid] = l;
    il[tid] = l > 0.0 ? 1.0 / l : 0.0;
  }
  __syncthreads();
  double* Gm = a.G + (int64_t)a.mode * RR;
  double* Sn = a.next_mode >= 0 ? a.S + (int64_t)a.next_mode * RR : nullptr;
  double gp = 0.0;
#pragma unroll
  for (int q = 0; q < EP; ++q) {
    const int e = tid + NTF * q;
    if (e < RR) {
      const double gn = g[q] * il[xs[q]] * il[ys[q]];
      Gm[e] = gn;
      if (Sn) Sn[e] = p.P[q] * gn;
      if (a.gram_raw) a.gram_raw[e] = g[q];
      gp += p.Sm[q] * g[q];
    }
  }
  if (a.do_fit) {
    // gamma = 1^T (S^(mode) * G_hat) 1 with G_hat the Gram of the unnormalised factor
    const double gamma = block_sum(gp, sh);
    if (tid == 0) {
      double num = p.alpha - 2.0 * beta + gamma;
      num = num > 0.0 ? num : 0.0;
      const double eps = p.alpha > 0.0 ? sqrt(num / p.alpha) : 0.0;
      if (p.it < a.fit_capacity) a.fit_out[p.it] = 1.0 - eps;
      *a.iter_counter = p.it + 1;
    }
  }
}

// One row chunk: everything in one group.
template <int EP>
__device__ __forceinline__ void fin1k_body(const FinalizeArgs& a) {
  extern __shared__ double lds[];
  __shared__ double sh[NTF / 64];
  FinPre<EP> p;
  fin_preload(a, p);
  double g[EP], beta;
  gram1k_rows<EP>(a, 0, a.I, lds, sh, g, beta);
  fin1k_tail<EP>(a, g, beta, p, sh);
}
// Several row chunks: chunk bx's Gram and beta into partial[bx] ...
template <int EP>
__device__ __forceinline__ void gram1k_chunk_body(const FinalizeArgs& a, int bx) {
  extern __shared__ double lds[];
  __shared__ double sh[NTF / 64];
  const int RR = a.R * a.R;
  const int64_t r0 = (int64_t)bx * a.rows_per_chunk;
  const int64_t r1 = r0 + a.rows_per_chunk < a.I ? r0 + a.rows_per_chunk : a.I;
  double g[EP], beta;
  gram1k_rows<EP>(a, r0, r1, lds, sh, g, beta);
  double* out = a.partial + (size_t)bx * (RR + 1);
#pragma unroll
  for (int q = 0; q < EP; ++q) {
    const int e = threadIdx.x + NTF * q;
    if (e < RR) out[e] = g[q];
  }
  if (threadIdx.x == 0) out[RR] = beta;
}
// ... then one group sums the partials in chunk order and finishes.
template <int EP>
__device__ __forceinline__ void tail1k_body(const FinalizeArgs& a) {
  __shared__ double sh[NTF / 64];
  const int RR = a.R * a.R, tid = threadIdx.x;
  FinPre<EP> p;
  fin_preload(a, p);
  double g[EP];
#pragma unroll
  for (int q = 0; q < EP; ++q) g[q] = 0.0;
  double beta = 0.0;
  constexpr int CB = EP == 1 ? 16 : (EP == 2 ? 8 : 4);  // chunks whose loads fly together
  for (int c0 = 0; c0 < a.nchunks; c0 += CB) {
    double t[CB][EP], tb[CB];
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      const int c = c0 + u < a.nchunks ? c0 + u : 0;
      const double* pc = a.partial + (size_t)c * (RR + 1);
#pragma unroll
      for (int q = 0; q < EP; ++q) {
        const int e = tid + NTF * q;
        t[u][q] = pc[e < RR ? e : 0];
      }
      tb[u] = pc[RR];
    }
#pragma unroll
    for (int u = 0; u < CB; ++u) {
      if (c0 + u < a.nchunks) {
#pragma unroll
        for (int q = 0; q < EP; ++q) g[q] += t[u][q];
        beta += tb[u];
      }
    }
  }
  fin1k_tail<EP>(a, g, beta, p, sh);
}

template <int EP>
__global__ __launch_bounds__(NTF) void fin1k_kernel(FinalizeArgs a) { fin1k_body<EP>(a); }
template <int EP>
__global__ __launch_bounds__(NTF) void gram1k_chunk_kernel(FinalizeArgs a) { gram1k_chunk_body<EP>(a, blockIdx.x); }
template <int EP>
__global__ __launch_bounds__(NTF) void tail1k_kernel(FinalizeArgs a) { tail1k_body<EP>(a); }

__device__ __forceinline__ void fin_op(const KOp& op, int bx) {
  FinalizeArgs a = op.u.fin;
  globalize(a);
  switch (op.kind) {
    case K_FIN1K:
      if (op.variant == 1) fin1k_body<1>(a);
      else if (op.variant == 2) fin1k_body<2>(a);
      else fin1k_body<4>(a);
      break;
    case K_GRAM1K:
      if (op.variant == 1) gram1k_chunk_body<1>(a, bx);
      else if (op.variant == 2) gram1k_chunk_body<2>(a, bx);
      else gram1k_chunk_body<4>(a, bx);
      break;
    case K_TAIL1K:
      if (op.variant == 1) tail1k_body<1>(a);
      else if (op.variant == 2) tail1k_body<2>(a);
      else tail1k_body<4>(a);
      break;
    default: break;
  }
}
// Persistent batched form of the 1024-thread finalize kernels.
__global__ __launch_bounds__(NTF) void fin_batch_kernel(const BItem* __restrict__ items, const int* __restrict__ grp,
                                                        const KOp* __restrict__ ops) {
  const int off = grp[0], n = grp[1];
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const BItem it = items[off + i];
    fin_op(ops[it.op], it.bx);
    __syncthreads();
  }
}

// Split-K sum of partial-MTTKRP partials: T(m, col0 + r) = sum over splits (in
// split order) of part[(sp*RP + r)*Mpad + m], one thread per output (coalesced along
// m), sixteen splits' loads in flight: a short output of a long K is a chain of loads
// (12000001x4x4, R = 5: 10417 splits of 80 outputs, 1.23 -> 0.66 ms against four in flight, which took
// 0.88 while the tensor was streamed past the cache that holds the partials).
template <typename TO>
__device__ __forceinline__ void pm_reduce_body(const ReduceArgs& ra, int bx) {
  const int64_t e = (int64_t)bx * NT + threadIdx.x;
  const int64_t total = ra.Mtot * ra.R;
  if (e >= total) return;
  const int r = (int)(e / ra.Mtot);
  const int64_t m = e - (int64_t)r * ra.Mtot;
  const double* p = ra.part + (size_t)r * ra.Mpad + m;
  const size_t st = (size_t)ra.RP * ra.Mpad;
  double s = 0.0;
  int sp = 0;
  for (; sp + 16 <= ra.nsplit; sp += 16) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = p[(sp + u) * st];
#pragma unroll
    for (int u = 0; u < 16; ++u) s += v[u];
  }
  for (; sp + 4 <= ra.nsplit; sp += 4) {
    const double v0 = p[(sp + 0) * st], v1 = p[(sp + 1) * st], v2 = p[(sp + 2) * st], v3 = p[(sp + 3) * st];
    s += v0;
    s += v1;
    s += v2;
    s += v3;
  }
  for (; sp < ra.nsplit; ++sp) s += p[sp * st];
  ((TO*)ra.T)[m + ra.Mtot * (int64_t)(ra.col0 + r)] = (TO)s;
}
template <typename TO>
__global__ __launch_bounds__(NT) void pm_reduce_kernel(ReduceArgs ra) {
  pm_reduce_body<TO>(ra, blockIdx.x);
}

// Persistent batched forms of the small kernels of the iteration: one kernel
// per kind (and per register variant of the update), so that each runs at its
// own occupancy rather than at that of the most register-hungry one.
template <int KIND, int VAR, typename A>
__device__ __forceinline__ void small_op(const A& a, int variant, int bx, int by) {
  if constexpr (KIND == K_PM_REDUCE) {
    if (variant) pm_reduce_body<double>(a, bx);
    else pm_reduce_body<float>(a, bx);
  } else if constexpr (KIND == K_MTTV_TRAIL) {
    if (variant) mttv_trail_body<double>(a, bx, by);
    else mttv_trail_body<float>(a, bx, by);
  } else if constexpr (KIND == K_MTTV_LEAD) {
    switch (variant) {
      case 41: mttv_lead_body<4, double>(a, bx); break;
      case 40: mttv_lead_body<4, float>(a, bx); break;
      case 81: mttv_lead_body<8, double>(a, bx); break;
      case 80: mttv_lead_body<8, float>(a, bx); break;
      case 161: mttv_lead_body<16, double>(a, bx); break;
      case 160: mttv_lead_body<16, float>(a, bx); break;
      case 321: mttv_lead_body<32, double>(a, bx); break;
      case 320: mttv_lead_body<32, float>(a, bx); break;
      case 641: mttv_lead_body<64, double>(a, bx); break;
      default: mttv_lead_body<64, float>(a, bx); break;
    }
  } else if constexpr (KIND == K_UPDATE) {
    if constexpr (VAR >= kUpdLane) update_lane_body<VAR - kUpdLane>(a, bx);
    else update_reg_body<VAR>(a, bx);
  }
}

// A small op's arguments: a copy with its pointers marked global, or, for a
// multi-TTV, the record itself (its arrays are indexed by the mode, and a copy of
// them would live in scratch memory; its body marks the pointers).
template <int KIND>
__device__ __forceinline__ decltype(auto) small_args(const KOp& op) {
  if constexpr (KIND == K_PM_REDUCE) {
    ReduceArgs a = op.u.red;
    globalize(a);
    return a;
  } else if constexpr (KIND == K_UPDATE) {
    UpdateArgs a = op.u.up;
    globalize(a);
    return a;
  } else {
    return (op.u.mt);
  }
}
template <int KIND, int VAR>
__global__ __launch_bounds__(NT) void small_items_kernel(const BItem* __restrict__ items, const int* __restrict__ grp,
                                                         const KOp* __restrict__ ops) {
  const int off = grp[0], n = grp[1];
  for (int i = blockIdx.x; i < n; i += gridDim.x) {
    const BItem it = items[off + i];
    const KOp& op = ops[it.op];
    decltype(auto) a = small_args<KIND>(op);
    const unsigned b0 = (unsigned)it.bx * op.coarse, b1 = min(b0 + op.coarse, op.gx);
    for (unsigned b = b0; b < b1; ++b) {
      small_op<KIND, VAR>(a, op.variant, (int)b, it.by);
      __syncthreads();  // LDS is reused by the next work-group's share
    }
  }
}

__global__ void init_model_kernel(const double* lam_in, const double* lam, double* lam_model,
                                  const double* G, double* S, int N, int R) {
  for (int k = threadIdx.x; k < R; k += blockDim.x) {
    double l = lam_in ? lam_in[k] : 1.0;
    for (int n = 0; n < N; ++n) l *= lam[(int64_t)n * R + k];
    lam_model[k] = l;
  }
  const int RR = R * R;
  for (int e = threadIdx.x; e < RR; e += blockDim.x) {
    double s = 1.0;
    for (int n = 1; n < N; ++n) s *= G[(int64_t)n * RR + e];
    S[e] = s;
  }
}

__global__ void normalize_out_kernel(float* W, int64_t I, int R, const double* lam) {
  const int64_t n = I * R;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
       e += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(e / I);
    const double l = lam[k];
    W[e] = l > 0.0 ? (float)((double)W[e] / l) : 0.f;
  }
}

inline unsigned grid_for(int64_t n, int threads, unsigned cap = 65535u * 32u) {
  int64_t g = (n + threads - 1) / threads;
  if (g < 1) g = 1;
  if (g > (int64_t)cap) g = cap;
  return (unsigned)g;
}

}  // namespace

int norm_sq_blocks(int64_t n) {
  // 32 values per thread at least, at most four groups per CU of this chip. A
  // fixed count keeps the summation order, and so the result, the same on every
  // device.
  int64_t b = (n + NT * 32 - 1) / (NT * 32);
  if (b < 1) b = 1;
  if (b > kNormSqMaxBlocks) b = kNormSqMaxBlocks;
  return (int)b;
}

hipError_t norm_sq_launch(const void* X, int dtype, int64_t n, double* out, double* partial,
                          int nblocks, hipStream_t st) {
  dim3 g(nblocks), b(NT);
  switch (dtype) {
    case NNCP_F32: hipLaunchKernelGGL(norm_sq_kernel<float>, g, b, 0, st, (const float*)X, n, partial); break;
    case NNCP_BF16: hipLaunchKernelGGL(norm_sq_kernel<__bf16>, g, b, 0, st, (const __bf16*)X, n, partial); break;
    case NNCP_F16: hipLaunchKernelGGL(norm_sq_kernel<_Float16>, g, b, 0, st, (const _Float16*)X, n, partial); break;
    default: return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(norm_sq_sum_kernel, dim3(1), b, 0, st, partial, nblocks, out);
  return hipGetLastError();
}

hipError_t quantize_launch(const float* src, void* dst, int dtype, int64_t n, hipStream_t st) {
  dim3 g(grid_for(n, NT * 8, 8192)), b(NT);
  if (dtype == NNCP_BF16) hipLaunchKernelGGL(quantize_kernel<__bf16>, g, b, 0, st, src, (__bf16*)dst, n);
  else if (dtype == NNCP_F16) hipLaunchKernelGGL(quantize_kernel<_Float16>, g, b, 0, st, src, (_Float16*)dst, n);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t fill_u32_launch(unsigned* p, int64_t n, unsigned v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(n, NT)), dim3(NT), 0, st, p, n, v);
  return hipGetLastError();
}
hipError_t fill_f64_launch(double* p, int64_t n, double v, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(fill_f64_kernel, dim3(grid_for(n, NT)), dim3(NT), 0, st, p, n, v);
  return hipGetLastError();
}
hipError_t widen_f32_launch(double* d, const float* s, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(widen_f32_kernel, dim3(grid_for(n, NT)), dim3(NT), 0, st, d, s, n);
  return hipGetLastError();
}
hipError_t copy_f64_launch(double* d, const double* s, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(copy_f64_kernel, dim3(grid_for(n, NT)), dim3(NT), 0, st, d, s, n);
  return hipGetLastError();
}
hipError_t unit_lambda_launch(double* lam, int64_t n, hipStream_t st) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(unit_lambda_kernel, dim3(grid_for(n, NT)), dim3(NT), 0, st, lam, n);
  return hipGetLastError();
}

static hipError_t record_or_launch(const Sink& sk, int kind, int variant, unsigned gx, unsigned gy, size_t lds,
                                   const void* kernel, const void* arg_struct, size_t arg_bytes, int threads = NT) {
  if (sk.rec) {
    KOp op{};
    op.kind = kind;
    op.variant = variant;
    op.gx = gx;
    op.gy = gy;
    op.lds = (unsigned)lds;
    std::memcpy(&op.u, arg_struct, arg_bytes);
    return sink_record(sk, op);
  }
  void* args[] = {const_cast<void*>(arg_struct)};
  return hipLaunchKernel(kernel, dim3(gx, gy), dim3(threads), args, lds, sk.st);
}

// Runs of J for a trailing multi-TTV: at least 128 j each, and no more groups than
// two per CU; none below 384 j. (Splitting costs one more launch, about 3 us; a
// group takes about 30 ns per j: 437 j, 16 groups, 14.5 us in one run,
// 7.8 + 3.8 in three.)
int mttv_trail_split(int64_t Ia, int64_t J, int R) {
  if (J < 384) return 1;
  const int64_t groups = (Ia + 63) / 64 * R;
  int64_t nz = 512 / groups;
  if (nz > J / 128) nz = J / 128;
  return nz < 2 ? 1 : (int)nz;
}

hipError_t mttv_trail_launch(const MttvArgs& a0, const Sink& sk) {
  MttvArgs a = a0;
  if (a.Ia <= 0 || a.R <= 0) return hipSuccess;
  a.nz = a.part ? mttv_trail_split(a.Ia, a.J, a.R) : 1;
  a.jz = (a.J + a.nz - 1) / a.nz;
  const void* k = a.t_f64 ? (const void*)mttv_trail_kernel<double> : (const void*)mttv_trail_kernel<float>;
  hipError_t e = record_or_launch(sk, K_MTTV_TRAIL, a.t_f64 ? 1 : 0, (unsigned)((a.Ia + 63) / 64 * a.nz),
                                  (unsigned)a.R, 0, k, &a, sizeof(a));
  if (e != hipSuccess || a.nz == 1) return e;
  ReduceArgs r{};
  r.part = a.part;
  r.T = a.out;
  r.t_f64 = a.out_f64;
  r.Mtot = r.Mpad = a.Ia;
  r.RP = r.R = a.R;
  r.nsplit = a.nz;
  return pm_reduce_launch(r, sk);
}

hipError_t mttv_lead_launch(const MttvArgs& a, const Sink& sk) {
  const int64_t outputs = a.J * a.R;
  if (outputs <= 0) return hipSuccess;
  // lanes per output: about 8 elements of the contracted range per lane (at
  // least 4 lanes, at most a wave), so that short ranges still give each
  // work-group many outputs and each lane several independent loads
  int gs = 4;
  while (gs < 64 && gs * 8 < a.Ia) gs <<= 1;
  const unsigned blocks = (unsigned)((outputs * gs + NT - 1) / NT);
  const void* k = nullptr;
#define NNCP_LEAD(GSV) \
  k = a.t_f64 ? (const void*)mttv_lead_kernel<GSV, double> : (const void*)mttv_lead_kernel<GSV, float>;
  switch (gs) {
    case 4: NNCP_LEAD(4) break;
    case 8: NNCP_LEAD(8) break;
    case 16: NNCP_LEAD(16) break;
    case 32: NNCP_LEAD(32) break;
    default: NNCP_LEAD(64) break;
  }
#undef NNCP_LEAD
  return record_or_launch(sk, K_MTTV_LEAD, gs * 10 + (a.t_f64 ? 1 : 0), blocks, 1, 0, k, &a, sizeof(a));
}

// Rows from which the update takes one lane per row (R <= 32; above, a row does not
// fit a lane's registers). Below, a wave per row has the shorter chain. Lanes' time
// hardly grows with the rows; per sweep it is R * rb products (rb register columns). A
// wave's grows with them; per sweep it is a step per column (HALS, in eights), or the
// products of W S at 0.6 of a step each (MU), and seven steps' worth of reductions if
// the sweeps may stop early. With many sweeps the line is where those meet, with one
// where loads and stores do. us, wave / lane per row: HALS R = 16, one sweep: 4096
// rows 8 / 9, 32768 29 / 9; 50 sweeps: 4096 50 / 161, 16384 174 / 163, 32768 337 / 166; R = 5,
// 50 sweeps: 8192 50 / 62, 12288 72 / 62, to a tolerance 8192 103 / 66; R = 32, one: 8192 18 / 19,
// 50: 8192 176 / 567, 32768 652 / 573; MU R = 32, one: 12288 21 / 19, ten: 8192 28 / 118, 65536
// 156 / 122.
int64_t update_lane_rows(int R, int update, int sweeps, double tol) {
  const int rb = R <= 16 ? 16 : 32;
  const bool mu = update == NNCP_MU;
  const double steps = (mu ? 0.6 * rb : (double)((R + 7) / 8 * 8)) + (tol > 0.0 ? 7.0 : 0.0);
  const double one = std::max(256.0 * rb, mu ? 375.0 * R : 0.0);
  const double many = std::max(one, 920.0 * R * rb / steps);
  return (int64_t)(many - (many - one) * 2.0 / (std::max(sweeps, 1) + 1.0));
}

hipError_t update_launch(const UpdateArgs& a, const Sink& sk) {
  if (a.I <= 0) return hipSuccess;
  const int rpb = NT / 64;
  const unsigned g = (unsigned)((a.I + rpb - 1) / rpb);
  if (a.R <= 64) {
    const int rb = a.R <= 16 ? 16 : (a.R <= 32 ? 32 : 64);
    if (a.R <= 32 && a.I >= update_lane_rows(a.R, a.update, a.sweeps, a.tol)) {
      const void* k = rb == 16 ? (const void*)update_lane_kernel<16> : (const void*)update_lane_kernel<32>;
      return record_or_launch(sk, K_UPDATE, kUpdLane + rb, (unsigned)((a.I + NT - 1) / NT), 1, 0, k, &a, sizeof(a));
    }
    const void* k = rb == 16 ? (const void*)update_reg_kernel<16>
                             : (rb == 32 ? (const void*)update_reg_kernel<32> : (const void*)update_reg_kernel<64>);
    return record_or_launch(sk, K_UPDATE, rb, g, 1, 0, k, &a, sizeof(a));
  }
  const size_t lds = ((size_t)a.R * a.R + a.R) * sizeof(double);
  const int vpl = a.R <= 64 ? 1 : 2;
  const void* k = vpl == 1 ? (const void*)update_kernel<1> : (const void*)update_kernel<2>;
  return record_or_launch(sk, K_UPDATE, vpl, g, 1, lds, k, &a, sizeof(a));
}

hipError_t pm_reduce_launch(const ReduceArgs& r, const Sink& sk) {
  const int64_t total = r.Mtot * r.R;
  if (total <= 0) return hipSuccess;
  const void* k = r.t_f64 ? (const void*)pm_reduce_kernel<double> : (const void*)pm_reduce_kernel<float>;
  return record_or_launch(sk, K_PM_REDUCE, r.t_f64 ? 1 : 0, (unsigned)((total + NT - 1) / NT), 1, 0, k, &r,
                          sizeof(r));
}

hipError_t mttv_trail_launch(const MttvArgs& a, hipStream_t st) {
  Sink sk;
  sk.st = st;
  return mttv_trail_launch(a, sk);
}
hipError_t mttv_lead_launch(const MttvArgs& a, hipStream_t st) {
  Sink sk;
  sk.st = st;
  return mttv_lead_launch(a, sk);
}
hipError_t update_launch(const UpdateArgs& a, hipStream_t st) {
  Sink sk;
  sk.st = st;
  return update_launch(a, sk);
}

hipError_t sink_record(const Sink& s, const KOp& op) {
  if (!s.rec) return hipErrorInvalidValue;
  try {
    KOp o = op;
    o.stage = 64 * s.mode + 4 * s.step + kslot(op.kind);
    static_cast<std::vector<KOp>*>(s.rec)->push_back(o);
  } catch (...) {
    return hipErrorOutOfMemory;
  }
  return hipSuccess;
}

const void* small_batch_kernel_ptr(int kind, int variant) {
  switch (kind) {
    case K_PM_REDUCE: return (const void*)small_items_kernel<K_PM_REDUCE, 0>;
    case K_MTTV_TRAIL: return (const void*)small_items_kernel<K_MTTV_TRAIL, 0>;
    case K_MTTV_LEAD: return (const void*)small_items_kernel<K_MTTV_LEAD, 0>;
    case K_UPDATE:
      switch (variant) {
        case 16: return (const void*)small_items_kernel<K_UPDATE, 16>;
        case 32: return (const void*)small_items_kernel<K_UPDATE, 32>;
        case 64: return (const void*)small_items_kernel<K_UPDATE, 64>;
        case kUpdLane + 16: return (const void*)small_items_kernel<K_UPDATE, kUpdLane + 16>;
        case kUpdLane + 32: return (const void*)small_items_kernel<K_UPDATE, kUpdLane + 32>;
        default: return nullptr;
      }
    default: return nullptr;
  }
}
const void* fin_batch_kernel_ptr() { return (const void*)fin_batch_kernel; }
// The most dynamic LDS a 1024-thread Gram/finalize op of rank <= 64 uses.
size_t fin_batch_max_lds() {
  size_t m = 0;
  for (int R = 1; R <= kSmallMaxR; ++R) {
    const size_t b = (size_t)fin_work_doubles(R) * sizeof(double);
    if (b > m) m = b;
  }
  return m;
}

// Row chunks for the Gram. R <= 64: a chunk's waves take about six groups of 16
// rows each (fin_ns waves per column-block pair; twelve at R > 48, whose partials
// are the largest to add up: 1344 x 50 in 14 chunks 8.6 + 14.4 us, in 7 12.5 + 8.4),
// one group without a second launch up to twice that. Past 32 chunks the walk of a
// chunk (about 1.5 us per two row groups of a wave) is set against the sum over the
// chunks, and the least total lies near a multiple of sqrt(I), at most one chunk per
// CU (us with 32 / 64 / 128 / 256 chunks: 100000 x 10 19 / 19 / 26 / 42, x 50 148 /
// 103 / 102 / 147; 1000000 x 10 103 / 62 / 48 / 54, x 50 1459 / 763 / 436 / 314).
// R > 64: chunks of about 2^19 products, at most 64.
int finalize_chunks(int64_t I, int R, int* rows_per_chunk) {
  int64_t chunks;
  if (R <= kSmallMaxR) {
    const int64_t rows = 16 * (R > 48 ? 12 : 6) * fin_ns(R);
    chunks = I <= 2 * rows ? 1 : (I + rows - 1) / rows;
    if (chunks > 32) {
      const int64_t c = (int64_t)((R <= 16 ? 0.15 : 0.28) * std::sqrt((double)I));
      chunks = std::min(chunks, std::max<int64_t>(32, std::min<int64_t>(256, c)));
    }
  } else {
    chunks = (I * R * R + (1ll << 19) - 1) >> 19;
    if (chunks > 64) chunks = 64;
  }
  if (chunks > I) chunks = I;
  if (chunks < 1) chunks = 1;
  int64_t rpc = (I + chunks - 1) / chunks;
  if (rpc < 1) rpc = 1;
  chunks = (I + rpc - 1) / rpc;
  *rows_per_chunk = (int)rpc;
  return (int)chunks;
}

hipError_t finalize_launch(const FinalizeArgs& a, const Sink& sk) {
  const size_t RR = (size_t)a.R * a.R;
  if (a.R <= kSmallMaxR) {
    const int ep = fin_ep(a.R);
    const size_t lds = (size_t)fin_work_doubles(a.R) * sizeof(double);
    if (a.nchunks <= 1) {
      const void* k = ep == 1 ? (const void*)fin1k_kernel<1>
                              : (ep == 2 ? (const void*)fin1k_kernel<2> : (const void*)fin1k_kernel<4>);
      return record_or_launch(sk, K_FIN1K, ep, 1, 1, lds, k, &a, sizeof(a), NTF);
    }
    const void* kc = ep == 1 ? (const void*)gram1k_chunk_kernel<1>
                             : (ep == 2 ? (const void*)gram1k_chunk_kernel<2> : (const void*)gram1k_chunk_kernel<4>);
    hipError_t e = record_or_launch(sk, K_GRAM1K, ep, (unsigned)a.nchunks, 1, lds, kc, &a, sizeof(a), NTF);
    if (e != hipSuccess) return e;
    const void* kt = ep == 1 ? (const void*)tail1k_kernel<1>
                             : (ep == 2 ? (const void*)tail1k_kernel<2> : (const void*)tail1k_kernel<4>);
    return record_or_launch(sk, K_TAIL1K, ep, 1, 1, 0, kt, &a, sizeof(a), NTF);
  }
  size_t lds = (size_t)fin_sub_rows(a.R) * a.R * sizeof(double);
  const size_t need = (RR + 1) * sizeof(double);
  if (need > lds) lds = need;
  if (a.nchunks <= 1)
    return record_or_launch(sk, K_FIN_FUSED, 0, 1, 1, lds, (const void*)finalize_fused_kernel, &a, sizeof(a));
  hipError_t e = record_or_launch(sk, K_GRAM_CHUNKS, 0, (unsigned)a.nchunks, 1, lds,
                                  (const void*)gram_chunks_kernel, &a, sizeof(a));
  if (e != hipSuccess) return e;
  return record_or_launch(sk, K_FIN_TAIL, 0, 1, 1, lds, (const void*)finalize_tail_kernel, &a, sizeof(a));
}

hipError_t finalize_launch(const FinalizeArgs& a, hipStream_t st) {
  Sink sk;
  sk.st = st;
  return finalize_launch(a, sk);
}


hipError_t init_model_launch(const double* lam_in, double* lam, double* lam_model, const double* G,
                             double* S, int N, int R, hipStream_t st) {
  hipLaunchKernelGGL(init_model_kernel, dim3(1), dim3(NT), 0, st, lam_in, lam, lam_model, G, S, N, R);
  return hipGetLastError();
}

hipError_t normalize_out_launch(float* W, int64_t I, int R, double* lam_self, hipStream_t st) {
  const int64_t n = I * R;
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(normalize_out_kernel, dim3(grid_for(n, NT, 4096)), dim3(NT), 0, st, W, I, R,
                     (const double*)lam_self);
  return hipGetLastError();
}

}  // namespace nncpk
