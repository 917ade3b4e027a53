// The FP32 partial-MTTKRP kernels' bodies with direct loads (left and right
// side); included by one translation unit per side, which instantiates them.
// Partial MTTKRP on MFMA for FP32 tensors: the root edges of the dimension tree
// (Section IV-A, Figure 2a), T = X_[L] * K (left node {1..s}) or
// T = X_[L]^T * K (right node {s+1..N}), where X_[L] is the tensor viewed as the
// column-major I_L x I_R matrix and K the Khatri-Rao product of the other
// side's factors (first contracted mode fastest).
//
// Design (gfx950, wave64):
//  * The reduction index is split as k = i1 + I1*j (i1: first contracted mode).
//    K(k, :) = H_1(i1, :) * Krest(j, :), so a work-group keeps the H_1 rows of
//    its i1 block in LDS (the MFMA B operand), and applies Krest(j, :) as a
//    per-column factor when it folds the FP32 MFMA sums into FP64 accumulators
//    (one v_fma_f64 per output). The Khatri-Rao product is never formed.
//  * X streams from HBM straight into VGPRs with vector loads (8 or 16 bytes per
//    lane), several k-steps ahead of the MFMAs (v_mfma_f32_16x16x4_f32), for any
//    shape: a load of padded i1 (>= I1) reads the next j's columns, which meet
//    zero rows of H_1 in LDS; a load of rows past the output reads into the next
//    column and only feeds outputs that are never stored; reads past the end of
//    the tensor are range-checked to zero (buffer loads).
//  * Precision: each MFMA chain covers at most `fold` k-steps (16 or 32 products
//    per output each) before it is added into FP64; split-K partials, the
//    cross-wave reduction and the output are FP64.
//  * Split-K over (i1 block, j block) pairs: each work-group writes an FP64
//    partial; a separate reduction kernel sums them in split order, so results
//    do not depend on scheduling and no cross-XCD fence is needed. A right node
//    with a tall output walks its i1 blocks inside the work-group instead
//    (restaging LDS), so it writes only its output.
#pragma once

#include "pm_common.hpp"

namespace nncpk {
namespace pm32 {

// How the tensor is loaded. LD_BUF, LD_BUFNT: range-checked buffer loads, which
// read zeros past the tensor's end, for shapes whose lane offsets fit 31 bits
// (pm_f32_buf): a lane's offsets are fixed per tile, so a step costs scalar address
// arithmetic only, and no branch stands between the loads and their use. LD_FAST:
// plain vector loads, where the shape guarantees that all of them lie inside the
// tensor (pm_f32_fast). LD_GEN: a uniform check per step and masked loads in the
// steps that reach the tensor's end; its branches make the compiler wait for all
// loads in flight once per ring round; it serves ragged tensors whose matricisation
// has columns of 34 MB and more on the right (67 at R > 32) or 143 MB on the left.
// The streaming (nontemporal) hint goes with LD_FAST and LD_BUFNT on the left,
// where a tensor's columns start on cache lines (and for the largest tensors,
// pm_left_stream): every line is then read once, by one load (128^4 left node 0.18 ms with the hint, 0.20 without; 1024^3 0.69 and
// 0.79). Everywhere else a line is read by two loads, of neighbouring rows or
// steps, or by a step's two halves on the right, and the hint drops it in between:
// right node of 1000x999x300 R = 20 401 -> 276 us without it, of 1024^3 R = 32
// 1036 -> 955, of 137x201x90 R = 16 24.1 -> 19.7.
enum : int { LD_GEN = 0, LD_FAST = 1, LD_BUF = 2, LD_BUFNT = 3 };
template <int L, bool NTL>
__device__ __forceinline__ f32v<L> buf_load(__amdgpu_buffer_rsrc_t rs, uint32_t off) {
  constexpr int aux = NTL ? kBufNt : 0;
  if constexpr (L == 4) return __builtin_bit_cast(f32v<4>, __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, aux));
  else return __builtin_bit_cast(f32v<2>, __builtin_amdgcn_raw_buffer_load_b64(rs, (int)off, 0, aux));
}

// Rows per left wave = 16 * left_tr(NB); columns per right wave = 16 * right_mc(NB).
// Chosen so that the FP64 accumulators (2 VGPRs per output) leave room for
// several k-steps of X in flight without spilling. PF = k-steps in flight.
constexpr int left_tr(int nb) { return nb >= 4 ? 2 : 4; }
constexpr int right_mc(int nb) { return nb >= 4 ? 2 : 4; }
constexpr int left_pf(int nb) { return nb == 2 ? 3 : 4; }
constexpr int right_pf(int nb) { return 3; }

// ----------------------------------------------------------------------------
// Left side: T(m, r) = sum_k X[m + IL*k] K(k, r); m is contiguous in X.
// A wave covers 16*TR rows m. In a k-step (16 consecutive i1 of one j), lane
// (li, lq) loads rows TR*li .. TR*li+TR-1 of the columns i1 = base + 4*lq + u,
// u = 0..3; MFMA chain tt uses row TR*li + tt of every load.
// ----------------------------------------------------------------------------
template <int NB, int D, int LD, bool MT, bool NTL>
__device__ __forceinline__ void pm_left_f32_body(const PmArgs& a, int bx, int by) {
  constexpr int RP = NB * 16;
  constexpr int TR = left_tr(NB);
  constexpr int KS = 16;
  constexpr int NACC = TR * NB;
  constexpr int WROWS = 16 * TR;
  using vT = f32v<TR>;
  extern __shared__ double lds_d[];
  const int hp = a.i1blk + 4;
  float* hs = (float*)lds_d;
  double* sc = lds_d + (RP * hp + 1) / 2;

  const int WM = a.wm, WK = 4 / WM;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wk = wave / WM;
  const int li = lane & 15, lq = lane >> 4;
  const int64_t Mtot = a.IL, Ktot = a.IR;
  const int mtile = WM * WROWS;
  // the group's M tiles tile0 .. tile0 + ntile - 1 (ntile > 1 only with WK == 1):
  // one continuous stream of k-steps per wave, the loads of a tile's first steps
  // issued while the previous tile's last steps are computed
  const int tile0 = MT ? bx * a.mper : bx;
  const int ntile = MT ? min(a.mper, a.mtiles - tile0) : 1;
  const int ib = by % a.n_i1blk, jb = by / a.n_i1blk;
  const int i1_0 = ib * a.i1blk;
  const int i1n = min(a.i1blk, a.I1pad - i1_0);
  const int64_t j0 = (int64_t)jb * a.jblk;
  const int jn = (int)min((int64_t)a.jblk, a.J - j0);
  const float* X = (const float*)a.X;

  const int S1 = i1n / KS;
  int sb, se;
  wave_range(S1 * jn, wk, WK, &sb, &se);
  se += (ntile - 1) * S1 * jn;

  double acc[NACC][4];
#pragma unroll
  for (int v = 0; v < NACC; ++v)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[v][e] = 0.0;

  // lane's first row in the tile being loaded; a row group wholly past the
  // output reads row 0
  int64_t m = (int64_t)tile0 * mtile + wm * WROWS + TR * li;
  int64_t mload = m < Mtot ? m : 0;
  const int ilim = a.I1 - i1_0;            // lane i1 offsets >= ilim are padding
  const float* zeros = (const float*)a.zeros;
  int64_t lane_col[4];                     // lane part of the address of column (colbase + 4*lq + u)
#pragma unroll
  for (int u = 0; u < 4; ++u) lane_col[u] = Mtot * (int64_t)(4 * lq + u);
  // LD_BUF: the resource of a step starts at the wave's first row of the step's
  // first column; lane byte offsets (rows past the output: none)
  const int64_t IX = Mtot * Ktot;
  uint32_t voff[4];
  auto set_voff = [&]() {
#pragma unroll
    for (int u = 0; u < 4; ++u) voff[u] = m < Mtot ? (uint32_t)((lane_col[u] + TR * li) * 4) : kBufNone;
  };
  set_voff();
  // The vector loads of a step read elements up to Mtot * (colbase + KS) + TR - 2
  // (row group start <= Mtot - 1, TR rows, in the step's last column): all of
  // them lie inside the tensor while Mtot * (colbase + KS) <= vec_lim.
  const int64_t vec_lim = Mtot * Ktot - (TR - 1);

  // load cursor (uniform): step = jl * S1 + tl. With one wave along K the group
  // starts at a j rotated by its M tile, so groups that share a split do not all
  // request the same addresses modulo the column stride at the same time.
  const int jrot = (WK == 1 && jn > 1) ? (int)(((unsigned)bx * 5u) % (unsigned)jn) : 0;
  int jcntL = sb / S1, tileL = 0;
  int jl = jcntL + jrot, tl = sb - jcntL * S1;
  if (jl >= jn) jl -= jn;  // an empty range (sb == S1 * jn) starts at the block's first j
  // The cursor stays inside the group's j block and tiles (it wraps), so loads
  // of steps past the wave's range read valid memory and are simply not used.
  auto load = [&](vT (&A)[4]) {
    const int64_t colbase = (int64_t)a.I1 * (j0 + jl) + i1_0 + KS * tl;
    const float* base = X + Mtot * colbase;
    if constexpr (LD == LD_BUF || LD == LD_BUFNT) {
      const int64_t e0 = Mtot * colbase + (int64_t)(tile0 + tileL) * mtile + wm * WROWS;
      const __amdgpu_buffer_rsrc_t rs = buf_rsrc<4>(X + e0, IX - e0);
#pragma unroll
      for (int u = 0; u < 4; ++u) A[u] = buf_load<TR, NTL>(rs, voff[u]);
    } else if (LD == LD_FAST || Mtot * (colbase + KS) <= vec_lim) {  // uniform
#pragma unroll
      for (int u = 0; u < 4; ++u) A[u] = tload<NTL>((const vT*)(base + lane_col[u] + mload));
    } else {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        // per lane: the whole row group of a real column in one vector load,
        // else element by element (rows past the output, padded i1: zero)
        const bool kv = (KS * tl + 4 * lq + u) < ilim;
        vT v;
        if (kv && m + TR <= Mtot) {
          v = *(const vT*)(base + lane_col[u] + m);
        } else {
#pragma unroll
          for (int e = 0; e < TR; ++e) {
            const float* p = (kv && m + e < Mtot) ? base + lane_col[u] + m + e : zeros;
            v[e] = *p;
          }
        }
        A[u] = v;
      }
    }
    if (++tl == S1) {
      tl = 0;
      if (++jl == jn) jl = 0;
      if (MT && ++jcntL == jn) {
        jcntL = 0;
        if (++tileL == ntile) tileL = 0;
        m = (int64_t)(tile0 + tileL) * mtile + wm * WROWS + TR * li;
        mload = m < Mtot ? m : 0;
        if constexpr (LD == LD_BUF || LD == LD_BUFNT) set_voff();
      }
    }
  };

  // The first D steps' loads of X go out before the LDS prologue, so that the
  // two round trips to memory overlap.
  vT A[D][4];
  const int jl0 = jl, tl0 = tl, jcnt0 = jcntL;
#pragma unroll
  for (int d = 0; d < D; ++d) load(A[d]);
  __builtin_amdgcn_sched_barrier(0);
  pm_prologue(a, hs, hp, sc, RP, i1_0, i1n, j0, jn);
  __syncthreads();

  // acc[tt*NB+nb][v]: row mw + TR*(4*lq + v) + tt, rank column 16nb + li.
  const bool direct = (a.nsplit == 1);
  const int64_t Mpad = (int64_t)a.mtiles * mtile;
  auto store_tile = [&](int64_t mw) {
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        double o[TR];
#pragma unroll
        for (int tt = 0; tt < TR; ++tt) o[tt] = acc[tt * NB + nb][v];
        pm_store_rows<TR>(a, direct, Mtot, Mpad, RP, by, 16 * nb + li, mw + TR * (4 * lq + v), o);
      }
  };

  // FP32 partial sums (one 16x16 block per (tt, nb)) live for `fold` k-steps and
  // are then added into the FP64 accumulators with the chunk's column scale.
  f4 c32[TR][NB];
#pragma unroll
  for (int tt = 0; tt < TR; ++tt)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) c32[tt][nb] = f4{0.f, 0.f, 0.f, 0.f};
  int jc = jl0, tc = tl0, jcntC = jcnt0, tileC = 0, fc = tl0 % a.fold, sc_left = se - sb;
  auto compute = [&](const vT (&A)[4]) {
    const int kk = KS * tc + 4 * lq;
    f4 B[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) B[nb] = *(const f4*)&hs[(16 * nb + li) * hp + kk];
    // u-major: consecutive MFMAs go to different accumulators
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
      for (int tt = 0; tt < TR; ++tt)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) c32[tt][nb] = mfma4(A[u][tt], B[nb][u], c32[tt][nb]);
    --sc_left;
    // fold every `fold` k-steps, at the end of each j (the last i1 block can be
    // shorter than the others, so fold need not divide its steps) and at the end
    if (++fc == a.fold || tc + 1 == S1 || sc_left == 0) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const double scl = sc[jc * RP + 16 * nb + li];
#pragma unroll
        for (int tt = 0; tt < TR; ++tt) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[tt * NB + nb][e] = __builtin_fma((double)c32[tt][nb][e], scl, acc[tt * NB + nb][e]);
          c32[tt][nb] = f4{0.f, 0.f, 0.f, 0.f};
        }
      }
      fc = 0;
    }
    if (++tc == S1) {
      tc = 0;
      if (++jc == jn) jc = 0;
      if (MT && ++jcntC == jn) {
        jcntC = 0;
        if (tileC + 1 < ntile) {  // a tile done (its last j folded above): store it, start the next
          store_tile((int64_t)(tile0 + tileC) * mtile + wm * WROWS);
#pragma unroll
          for (int v = 0; v < NACC; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[v][e] = 0.0;
          ++tileC;
        }
      }
    }
  };

  // D k-steps of X in flight: the loads of step s+D are issued right after step
  // s is consumed. sched_barrier keeps the compiler from sinking them. The first
  // D loads are issued unconditionally so every path into the loop has the same
  // loads in flight and the compiler's wait counts stay precise.
  int s = sb;
  for (; s + D - 1 < se; s += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      compute(A[d]);
      __builtin_amdgcn_sched_barrier(0);
      load(A[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int d = 0; d < D - 1; ++d)
    if (s + d < se) compute(A[d]);

  __syncthreads();  // LDS is reused by the cross-wave reduction
  wave_reduce_k<NACC>(acc, lds_d, wk, wm, WK);
  if (wk != 0) return;
  store_tile((int64_t)(tile0 + ntile - 1) * mtile + wm * WROWS);
}

// ----------------------------------------------------------------------------
// Right side: T(c, r) = sum_k X[k + IL*c] K(k, r); k is contiguous in X.
// A wave covers MC groups of 16 columns c. In a k-step (32 consecutive i1 of
// one j), lane (li, lq) loads k = base + 16h + 4*lq + u (u = 0..3 in one
// 16-byte load, h = 0..1) of column c = group + li. The work-group walks
// `istages` i1 blocks (j inside each), restaging LDS between them; istages > 1
// only with every wave on its own columns (WM = 4).
// ----------------------------------------------------------------------------
template <int NB, int D, int LD, bool MT, bool NTL>
__device__ __forceinline__ void pm_right_f32_body(const PmArgs& a, int bx, int by) {
  constexpr int RP = NB * 16;
  constexpr int MC = right_mc(NB);
  constexpr int KS = 32;
  constexpr int NACC = MC * NB;
  using vT = f32v<4>;
  extern __shared__ double lds_d[];
  const int hp = a.i1blk + 4;
  float* hs = (float*)lds_d;
  double* sc = lds_d + (RP * hp + 1) / 2;

  const int WM = a.wm, WK = 4 / WM;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = wave % WM, wk = wave / WM;
  const int li = lane & 15, lq = lane >> 4;
  const int64_t Mtot = a.IR, Ktot = a.IL;
  const int mtile = WM * 16 * MC;
  // the group's M tiles tile0 .. tile0 + ntile - 1 (ntile > 1 only with WK == 1
  // and istages == 1), streamed as one sequence of k-steps per wave
  const int tile0 = MT ? bx * a.mper : bx;
  const int ntile = MT ? min(a.mper, a.mtiles - tile0) : 1;
  const int n_i1grp = a.n_i1blk / a.istages;
  const int ib0 = (by % n_i1grp) * a.istages, jb = by / n_i1grp;
  const int64_t j0 = (int64_t)jb * a.jblk;
  const int jn = (int)min((int64_t)a.jblk, a.J - j0);
  const float* X = (const float*)a.X;

  // stage geometry: all stages have i1blk rows except possibly the last
  auto stage_rows = [&](int st) { return min(a.i1blk, a.I1pad - (ib0 + st) * a.i1blk); };

  int total = 0;
  for (int st = 0; st < a.istages; ++st) total += (stage_rows(st) / KS) * jn;
  int sb, se;
  wave_range(total, wk, WK, &sb, &se);  // istages > 1 implies WK == 1: the whole range
  se += (ntile - 1) * total;

  double acc[NACC][4];
#pragma unroll
  for (int v = 0; v < NACC; ++v)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[v][e] = 0.0;

  // Columns of the tile being loaded (columns past the output read column 0).
  // The vector loads of a step read elements up to Ktot * cmax + lbase + KS - 1
  // (cmax: the wave's last column that is read, lane offsets up to KS - 1): all
  // of them lie inside the tensor while lbase <= vec_lim. Only the steps that
  // run past the end of a column near the tensor's end fail this.
  const float* colp[MC];
  int64_t vec_lim;
  // LD_BUF: the resource of a step starts at the step's first element of the
  // wave's first column (cwk); lane byte offsets (columns past the output: none)
  const int64_t IX = Mtot * Ktot;
  int64_t cwk = 0;
  uint32_t voff[MC];
  auto set_tile = [&](int t) {
    const int64_t cw = (int64_t)(tile0 + t) * mtile + wm * 16 * MC;
    cwk = cw * Ktot;
#pragma unroll
    for (int g = 0; g < MC; ++g) {
      const int64_t c = cw + 16 * g + li;
      colp[g] = X + Ktot * (c < Mtot ? c : 0) + 4 * lq;
      voff[g] = c < Mtot ? (uint32_t)(((int64_t)(16 * g + li) * Ktot + 4 * lq) * 4) : kBufNone;
    }
    const int64_t cmax = min(cw + 16 * MC - 1, Mtot - 1);
    vec_lim = Mtot * Ktot - Ktot * cmax - KS;  // wave-uniform
  };
  set_tile(0);
  const float* zeros = (const float*)a.zeros;

  // cursor (stage, j, t): t over the stage's k-steps, j over the block (rotated
  // start with one wave along K), stages in order. The load cursor runs D steps
  // ahead and wraps to the start after the last step, so it stays in bounds.
  const int jrot = (WK == 1 && jn > 1) ? (int)(((unsigned)bx * 5u) % (unsigned)jn) : 0;
  int stL = 0, S1L = stage_rows(0) / KS, tileL = 0;
  int jcntL = sb / S1L;  // sb > 0 only when istages == 1
  int tl = sb - jcntL * S1L;
  int jl = jcntL + jrot;
  if (jl >= jn) jl -= jn;
  auto load = [&](vT (&A)[MC][2]) {
    const int i1s = (ib0 + stL) * a.i1blk;
    const int64_t lbase = (int64_t)a.I1 * (j0 + jl) + i1s + KS * tl;
    if constexpr (LD == LD_BUF || LD == LD_BUFNT) {
      const __amdgpu_buffer_rsrc_t rs = buf_rsrc<4>(X + cwk + lbase, IX - cwk - lbase);
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < MC; ++g) A[g][h] = buf_load<4, NTL>(rs, voff[g] + 64 * h);
    } else if (LD == LD_FAST || lbase <= vec_lim) {  // uniform
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int g = 0; g < MC; ++g) A[g][h] = tload<NTL>((const vT*)(colp[g] + lbase + 16 * h));
    } else {
      const int ilimL = a.I1 - i1s;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int off = KS * tl + 16 * h + 4 * lq;
#pragma unroll
        for (int g = 0; g < MC; ++g) {
          // per lane: four real k in one vector load, else element by element
          // (padded i1 reads zero)
          vT v;
          if (off + 4 <= ilimL) {
            v = *(const vT*)(colp[g] + lbase + 16 * h);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float* p = (off + e < ilimL) ? colp[g] + lbase + 16 * h + e : zeros;
              v[e] = *p;
            }
          }
          A[g][h] = v;
        }
      }
    }
    if (++tl == S1L) {
      tl = 0;
      if (++jl == jn) jl = 0;
      if (++jcntL == jn) {
        jcntL = 0;
        if (++stL == a.istages) {
          stL = 0;
          if (MT) {
            if (++tileL == ntile) tileL = 0;
            set_tile(tileL);
          }
        }
        S1L = stage_rows(stL) / KS;
      }
    }
  };

  // the first D steps' loads go out before the LDS prologue (see the left side)
  vT A[D][MC][2];
  const int S1C0 = S1L, jl0 = jl, tl0 = tl, jcnt0 = jcntL;
#pragma unroll
  for (int d = 0; d < D; ++d) load(A[d]);
  __builtin_amdgcn_sched_barrier(0);
  pm_prologue(a, hs, hp, sc, RP, ib0 * a.i1blk, stage_rows(0), j0, jn);
  __syncthreads();

  // acc[g*NB+nb][v]: column c = cw + 16g + 4*lq + v, rank column 16nb + li.
  const bool direct = (a.nsplit == 1);
  const int64_t Mpad = (int64_t)a.mtiles * mtile;
  auto store_tile = [&](int64_t cw) {
#pragma unroll
    for (int g = 0; g < MC; ++g)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        double o[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) o[v] = acc[g * NB + nb][v];
        pm_store_rows<4>(a, direct, Mtot, Mpad, RP, by, 16 * nb + li, cw + 16 * g + 4 * lq, o);
      }
  };

  f4 c32[MC][NB];
#pragma unroll
  for (int g = 0; g < MC; ++g)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) c32[g][nb] = f4{0.f, 0.f, 0.f, 0.f};
  int stC = 0, S1C = S1C0, jc = jl0, tc = tl0, jcntC = jcnt0, tileC = 0, fc = tl0 % a.fold, sc_left = se - sb;
  auto compute = [&](const vT (&A)[MC][2]) {
    const int kk = KS * tc + 4 * lq;
    f4 B[2][NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int h = 0; h < 2; ++h) B[h][nb] = *(const f4*)&hs[(16 * nb + li) * hp + kk + 16 * h];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int g = 0; g < MC; ++g)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) c32[g][nb] = mfma4(A[g][h][u], B[h][nb][u], c32[g][nb]);
    --sc_left;
    // fold every `fold` k-steps, at the end of each j (and so of each stage) and
    // at the end of the range
    if (++fc == a.fold || tc + 1 == S1C || sc_left == 0) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        const double scl = sc[jc * RP + 16 * nb + li];
#pragma unroll
        for (int g = 0; g < MC; ++g) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            acc[g * NB + nb][e] = __builtin_fma((double)c32[g][nb][e], scl, acc[g * NB + nb][e]);
          c32[g][nb] = f4{0.f, 0.f, 0.f, 0.f};
        }
      }
      fc = 0;
    }
    if (++tc == S1C) {
      tc = 0;
      if (++jc == jn) jc = 0;
      if (++jcntC == jn) {
        jcntC = 0;
        if (++stC < a.istages && sc_left > 0) {
          // next i1 block: every wave of the group gets here at the same step
          __syncthreads();
          pm_stage_h1(a, hs, hp, RP, (ib0 + stC) * a.i1blk, stage_rows(stC));
          __syncthreads();
          S1C = stage_rows(stC) / KS;
        } else if (MT && tileC + 1 < ntile) {  // a tile done (istages == 1): store it, start the next
          stC = 0;
          store_tile((int64_t)(tile0 + tileC) * mtile + wm * 16 * MC);
#pragma unroll
          for (int v = 0; v < NACC; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[v][e] = 0.0;
          ++tileC;
        }
      }
    }
  };

  int s = sb;
  for (; s + D - 1 < se; s += D) {
#pragma unroll
    for (int d = 0; d < D; ++d) {
      compute(A[d]);
      __builtin_amdgcn_sched_barrier(0);
      load(A[d]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int d = 0; d < D - 1; ++d)
    if (s + d < se) compute(A[d]);

  __syncthreads();
  wave_reduce_k<NACC>(acc, lds_d, wk, wm, WK);
  if (wk != 0) return;
  store_tile((int64_t)(tile0 + ntile - 1) * mtile + wm * 16 * MC);
}

// Stand-alone kernels: one work-group per (M tile group, split). MT: a group
// streams several M tiles (a separate form, so that the one-tile kernels keep
// their register budget). NTL: tensor loads with the streaming hint (above). The
// batched kernels load without it: several launches stream many small tensors at
// once, and with it 11.2 instead of 9.0 GB were fetched per tick of the 256-job
// batch (3.24 -> 2.56 ms). A batched right node keeps two k-steps in flight
// instead of three: its lanes' 128-byte runs start anywhere in a cache line, so a
// line is needed by two steps, and with three the lines in flight of a die's 32
// CUs (8 MB) pass its L2 (256-job tick 2.52 -> 2.48 ms).
template <int SIDE, int NB, int LD, bool MT, bool NTL, bool BATCH>
__device__ __forceinline__ void pm_f32_body(const PmArgs& a, int bx, int by) {
  if constexpr (SIDE == 0) pm_left_f32_body<NB, left_pf(NB), LD, MT, NTL>(a, bx, by);
  else pm_right_f32_body<NB, BATCH ? 2 : right_pf(NB), LD, MT, NTL>(a, bx, by);
}
template <int SIDE, int NB, int LD, bool MT>
__global__ __launch_bounds__(NT, 2) void pm_f32(PmArgs a) {
  pm_f32_body<SIDE, NB, LD, MT, SIDE == 0 && (LD == LD_FAST || LD == LD_BUFNT), false>(a, blockIdx.x, blockIdx.y);
}

// Persistent batched form of the same kernel: work-group b takes the items
// grp[0] + b, grp[0] + b + gridDim.x, ... below grp[0] + grp[1]; each item is one
// (M tile group, split) work-group of a recorded stand-alone launch of this variant.
template <int SIDE, int NB, int LD, bool MT>
__global__ __launch_bounds__(NT, 2) void pm_f32_items(const BItem* __restrict__ items, const int* __restrict__ grp,
                                                      const KOp* __restrict__ ops) {
  pm_walk_items(items, grp, ops, [](const PmArgs& a, int bx, int by) { pm_f32_body<SIDE, NB, LD, MT, false, true>(a, bx, by); });
}

template <int SIDE, int LD, bool MT>
const void* pick(int nb, bool batch) {
  switch (nb) {
    case 1: return batch ? (const void*)pm_f32_items<SIDE, 1, LD, MT> : (const void*)pm_f32<SIDE, 1, LD, MT>;
    case 2: return batch ? (const void*)pm_f32_items<SIDE, 2, LD, MT> : (const void*)pm_f32<SIDE, 2, LD, MT>;
    case 4: return batch ? (const void*)pm_f32_items<SIDE, 4, LD, MT> : (const void*)pm_f32<SIDE, 4, LD, MT>;
    default: return nullptr;
  }
}

template <bool MT>
const void* pick_nt(int nb) {
  switch (nb) {
    case 1: return (const void*)pm_f32<0, 1, LD_BUFNT, MT>;
    case 2: return (const void*)pm_f32<0, 2, LD_BUFNT, MT>;
    case 4: return (const void*)pm_f32<0, 4, LD_BUFNT, MT>;
    default: return nullptr;
  }
}

}  // namespace pm32

// Kernel of (column blocks, load form), stand-alone or batched, in the one-tile
// (MT false) or several-tile form.
template <int SIDE, bool MT>
const void* pm_f32_form(int nb, int ld, bool batch) {
  switch (ld) {
    case pm32::LD_FAST: return pm32::pick<SIDE, pm32::LD_FAST, MT>(nb, batch);
    case pm32::LD_BUF: return pm32::pick<SIDE, pm32::LD_BUF, MT>(nb, batch);
    case pm32::LD_BUFNT:  // stand-alone left nodes
      if (SIDE == 0 && !batch) return pm32::pick_nt<MT>(nb);
      return pm32::pick<SIDE, pm32::LD_BUF, MT>(nb, batch);
    default: return pm32::pick<SIDE, pm32::LD_GEN, MT>(nb, batch);
  }
}

}  // namespace nncpk
