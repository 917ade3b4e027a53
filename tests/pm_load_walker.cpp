// Host-side walk of the partial-MTTKRP kernels' tensor loads, in the form that the
// launcher picks for a plan (test infrastructure): plain, masked, range-checked or
// range-checked from dword starts, FP32 and 16-bit. For every work-group, wave,
// k-step and lane it follows the kernels' cursors and address arithmetic and checks
//  * that every element read lies inside the tensor (also by the loads a wave issues
//    past its range), and every byte offset of a buffer load below 2^31;
//  * that every element of a computed step that feeds a stored output arrives as
//    exactly that element of the tensor (through the range check's zeros, the dword
//    shift and the last element put in place).
// A plan of more than `kFull` elements is walked at its first, middle and last groups.
//
// stdin: "dtype IL IR I1_left I1_right R X_offset" per line (X_offset: elements past
// a dword); one "cover" line per case and side, a summary, exit status 1 on any violation.
#include <algorithm>
#include <cstdio>
#include <set>
#include <vector>
#include "nncp_internal.hpp"
using namespace nncpk;

enum { GEN = 0, FAST = 1, BUF = 2, BUF3 = 3 };  // BUF3: FP32 with the streaming hint; 16-bit from dword starts
static const int64_t kFull = 400000;
static long long bad = 0, nchk = 0;
static void need(bool ok, const char* what, long long a = 0, long long b = 0) {
  ++nchk;
  if (!ok && bad++ < 8) printf("  %s (%lld, %lld)\n", what, a, b);
}
constexpr int64_t kZero = -1;  // a value that is zero
constexpr int64_t kAny = -2;   // a value that must not be used

// One buffer load of w elements of esz bytes at byte offset `off` of a resource that
// starts at element e0: the elements that arrive. The check drops whole dwords.
static void buf_load(int64_t e0, int64_t off, int w, int esz, int64_t I, int64_t* out) {
  need(off >= 0 && off + (int64_t)w * esz <= ((int64_t)1 << 31), "offset past 31 bits", off);
  need(off % esz == 0, "offset inside an element", off);
  const int64_t rem = I - e0, cap = 0x7ffffffc / esz;
  const int64_t bytes = rem <= 0 ? 0 : (rem >= cap ? 0x7ffffffc : rem * esz);
  const int per = 4 / esz;  // elements per dword
  for (int d = 0; d < w / per; ++d) {
    const bool in = off + 4 * d + 4 <= bytes;
    for (int q = 0; q < per; ++q) {
      const int64_t e = e0 + off / esz + d * per + q;
      if (in) need(e >= 0 && e < I, "buffer load outside the tensor", e, I);
      out[d * per + q] = in ? e : kZero;
    }
  }
}
static void plain(int64_t e, int w, int64_t I, int64_t* out) {
  need(e >= 0 && e + w <= I, "plain load outside the tensor", e, I);
  for (int q = 0; q < w; ++q) out[q] = e + q;
}

static void range(int n, int wk, int WK, int* b, int* e) {
  const int per = (n + WK - 1) / WK;
  *b = std::min(wk * per, n);
  *e = std::min((wk + 1) * per, n);
}
static std::vector<int> pick(int n, bool all) {
  std::set<int> s;
  if (all) for (int i = 0; i < n; ++i) s.insert(i);
  else for (int i : {0, 1, n / 2, n - 2, n - 1}) if (i >= 0 && i < n) s.insert(i);
  return {s.begin(), s.end()};
}

struct Case {
  bool f32;
  int side, ld, xoff;
  int64_t IL, IR, I;
};

static void left(const Case& c, const PmLaunch& L) {
  const int TR = (c.f32 ? pm_f32_wave_rows(0, L.nb) : pm_16_wave_rows(0, L.nb)) / 16;
  const int KS = c.f32 ? pm_f32_kstep(0) : pm_16_kstep(0), NC = KS / 4, esz = c.f32 ? 4 : 2;
  const int D = c.f32 ? (L.nb == 2 ? 3 : 4) : 3;
  const int WM = L.wm, WK = 4 / WM, WROWS = 16 * TR;
  const int64_t Mtot = c.IL, Ktot = c.IR, vec_lim = Mtot * Ktot - (TR - 1);
  const bool all = c.I * L.nb <= kFull;
  for (int by : pick(L.nsplit, all)) for (int bx : pick(L.mgroups, all)) for (int wave = 0; wave < 4; ++wave) {
    const int wm = wave % WM, wk = wave / WM, tile0 = bx * L.mper, ntile = std::min(L.mper, L.mtiles - tile0);
    const int ib = by % L.n_i1blk, jb = by / L.n_i1blk, i1_0 = ib * L.i1blk, i1n = std::min(L.i1blk, L.I1pad - i1_0);
    const int64_t j0 = (int64_t)jb * L.jblk;
    const int jn = (int)std::min<int64_t>(L.jblk, L.J - j0), S1 = i1n / KS;
    int sb, se;
    range(S1 * jn, wk, WK, &sb, &se);
    se += (ntile - 1) * S1 * jn;
    const int jrot = (WK == 1 && jn > 1) ? (int)(((unsigned)bx * 5u) % (unsigned)jn) : 0;
    int jcnt = sb / S1, tile = 0, tl = sb - jcnt * S1, jl = jcnt + jrot;
    if (jl >= jn) jl -= jn;
    int loads = D;
    for (int s = sb; s + D - 1 < se; s += D) loads += D;
    const int ilim = L.I1 - i1_0;
    for (int q = 0; q < loads; ++q) {
      const int64_t colbase = (int64_t)L.I1 * (j0 + jl) + i1_0 + KS * tl;
      const int64_t mw = (int64_t)(tile0 + tile) * L.mtile + wm * WROWS;
      const bool computed = q < se - sb;
      const bool last = !c.f32 && c.ld == BUF && (Mtot & 1) && tl + 1 == S1 && j0 + jl + 1 == L.J && i1_0 + i1n == L.I1pad;
      for (int lane = 0; lane < 64; ++lane) for (int u = 0; u < NC; ++u) {
        const int li = lane & 15, cu = NC * (lane >> 4) + u;
        const int64_t m = mw + TR * li;
        int64_t v[8];
        std::fill(v, v + 8, kAny);
        if (c.ld == BUF || c.ld == BUF3) {
          if (m < Mtot) buf_load(Mtot * colbase + mw, (Mtot * cu + TR * li) * esz, TR, esz, c.I, v);
          if (last && m < Mtot && Mtot - m < TR && KS * tl + cu + 1 == ilim) {
            const int d = (int)(Mtot - m);
            for (int e = 0; e < TR; e += 2) if (d == e + 1) v[e] = c.I - 1;
          }
        } else if (c.ld == FAST || Mtot * (colbase + KS) <= vec_lim) {
          plain(Mtot * (colbase + cu) + (m < Mtot ? m : 0), TR, c.I, v);
        } else {
          const bool kv = KS * tl + cu < ilim;
          if (kv && m + TR <= Mtot) plain(Mtot * (colbase + cu) + m, TR, c.I, v);
          else for (int e = 0; e < TR; ++e) {
            v[e] = kZero;
            if (kv && m + e < Mtot) plain(Mtot * (colbase + cu) + m + e, 1, c.I, v + e);
          }
        }
        if (computed)
          for (int e = 0; e < TR; ++e)
            if (m + e < Mtot && KS * tl + cu < ilim) need(v[e] == Mtot * (colbase + cu) + m + e, "left: wrong element", v[e], Mtot * (colbase + cu) + m + e);
      }
      if (++tl == S1) {
        tl = 0;
        if (++jl == jn) jl = 0;
        if (L.mper > 1 && ++jcnt == jn) { jcnt = 0; if (++tile == ntile) tile = 0; }
      }
    }
  }
}

static void right(const Case& c, const PmLaunch& L) {
  const int MC = (c.f32 ? pm_f32_wave_rows(1, L.nb) : pm_16_wave_rows(1, L.nb, L.j1)) / 16;
  const int KS = c.f32 ? pm_f32_kstep(1) : pm_16_kstep(1), W = KS / 8, HS = KS / 2, esz = c.f32 ? 4 : 2;
  const bool shift = !c.f32 && c.ld == BUF3;
  const int D = !c.f32 && L.j1 ? (shift || L.nb >= 4 ? 2 : 3) : 3;
  const int WM = L.wm, WK = 4 / WM;
  const int64_t Mtot = c.IR, Ktot = c.IL;
  const int grp = L.n_i1blk / L.istages;
  const bool all = c.I * L.nb <= kFull;
  if (shift) need(c.xoff == 0, "dword starts of a tensor that is not on one");
  for (int by : pick(L.nsplit, all)) for (int bx : pick(L.mgroups, all)) for (int wave = 0; wave < 4; ++wave) {
    const int wm = wave % WM, wk = wave / WM, tile0 = bx * L.mper, ntile = std::min(L.mper, L.mtiles - tile0);
    const int ib0 = (by % grp) * L.istages, jb = by / grp;
    const int64_t j0 = (int64_t)jb * L.jblk;
    const int jn = (int)std::min<int64_t>(L.jblk, L.J - j0);
    auto rows = [&](int st) { return std::min(L.i1blk, L.I1pad - (ib0 + st) * L.i1blk); };
    int total = 0, sb, se;
    for (int st = 0; st < L.istages; ++st) total += rows(st) / KS * jn;
    range(total, wk, WK, &sb, &se);
    se += (ntile - 1) * total;
    const int jrot = (WK == 1 && jn > 1) ? (int)(((unsigned)bx * 5u) % (unsigned)jn) : 0;
    int st = 0, S1 = rows(0) / KS, tile = 0, jcnt = sb / S1, tl = sb - jcnt * S1, jl = jcnt + jrot;
    if (jl >= jn) jl -= jn;
    int loads = D;
    for (int s = sb; s + D - 1 < se; s += D) loads += D;
    for (int q = 0; q < loads; ++q) {
      const int i1s = (ib0 + st) * L.i1blk;
      const int64_t lbase = (int64_t)L.I1 * (j0 + jl) + i1s + KS * tl;
      const int64_t cw = (int64_t)(tile0 + tile) * L.mtile + wm * 16 * MC;
      const int64_t cmax = std::min(cw + 16 * MC - 1, Mtot - 1), vec_lim = Mtot * Ktot - Ktot * cmax - KS;
      const bool computed = q < se - sb;
      const bool last = !c.f32 && (c.ld == BUF || shift) && (L.I1 & 1) && tl + 1 == S1 && j0 + jl + 1 == L.J && ib0 + st + 1 == L.n_i1blk;
      for (int lane = 0; lane < 64; ++lane) for (int g = 0; g < MC; ++g) for (int h = 0; h < 2; ++h) {
        const int li = lane & 15, k = HS * h + W * (lane >> 4);
        const int64_t cc = cw + 16 * g + li;
        int64_t v[10];
        std::fill(v, v + 10, kAny);
        if (shift) {
          const int lodd = (int)(li & Ktot & 1), odd = (int)((j0 + jl) & 1), up = odd ? 4 * lodd : 0;
          if (cc < Mtot) {
            const int64_t e0 = cw * Ktot + lbase - odd, off = ((int64_t)(16 * g + li) * Ktot + W * (lane >> 4) - lodd) * 2 + up + 64 * h;
            need((e0 + off / 2) % 2 == 0 && off % 4 == 0, "a load that does not start on a dword", e0, off);
            buf_load(e0, off, 8, 2, c.I, v);
            if (lodd != odd) buf_load(e0, off + 16, 2, 2, c.I, v + 8);
            if (lodd ^ odd) for (int e = 0; e < 8; ++e) v[e] = v[e + 1];
          }
        } else if (c.ld == BUF || c.ld == BUF3) {
          if (cc < Mtot) buf_load(cw * Ktot + lbase, ((int64_t)(16 * g + li) * Ktot + k) * esz, W, esz, c.I, v);
        } else if (c.ld == FAST || lbase <= vec_lim) {
          plain(Ktot * (cc < Mtot ? cc : 0) + lbase + k, W, c.I, v);
        } else {
          const int64_t col = Ktot * (cc < Mtot ? cc : 0);
          const int lim = L.I1 - i1s - KS * tl - k;
          if (lim >= W) plain(col + lbase + k, W, c.I, v);
          else for (int e = 0; e < W; ++e) {
            v[e] = kZero;
            if (e < lim) plain(col + lbase + k + e, 1, c.I, v + e);
          }
        }
        if (last && cc + 1 == Mtot) {
          const int d = L.I1 - i1s - KS * tl - k;
          for (int e = 0; e < 8; e += 2) if (d == e + 1) v[e] = c.I - 1;
        }
        if (computed && cc < Mtot)
          for (int e = 0; e < W; ++e)
            if (i1s + KS * tl + k + e < L.I1) need(v[e] == Ktot * cc + lbase + k + e, "right: wrong element", v[e], Ktot * cc + lbase + k + e);
      }
      if (++tl == S1) {
        tl = 0;
        if (++jl == jn) jl = 0;
        if (++jcnt == jn) {
          jcnt = 0;
          if (++st == L.istages) {
            st = 0;
            if (L.mper > 1 && ++tile == ntile) tile = 0;
          }
          S1 = rows(st) / KS;
        }
      }
    }
  }
}

int main() {
  int dt, I1l, I1r, R, xoff, cases = 0;
  long long IL, IR;
  while (scanf("%d %lld %lld %d %d %d %d", &dt, &IL, &IR, &I1l, &I1r, &R, &xoff) == 7) {
    ++cases;
    for (int side = 0; side < 2; ++side) {
      const int I1 = side ? I1r : I1l;
      const PmLaunch L = pm_plan(side, dt, IL, IR, I1, R, 0);
      if (L.xs) continue;  // its loads are walked by pm_address_emulator.cpp
      Case c{dt == NNCP_F32, side, 0, xoff, IL, IR, (int64_t)IL * IR};
      const void* X = (const void*)(((uintptr_t)1 << 40) + xoff * (dt == NNCP_F32 ? 4 : 2));
      c.ld = c.f32 ? pm_f32_load_form(L, IL, IR, I1) : pm16_load_form(L, X, IL, IR, I1);
      const long long was = bad;
      const int form = c.ld;
      if (!c.f32 && c.ld == 4) c.ld = BUF;  // (the streaming hint changes no address)
      if (side) right(c, L);
      else left(c, L);
      printf("cover %s side %d form %d mt %d split %d j1 %d stages %d wm %d nb %d%s\n", c.f32 ? "f32" : "16", side, form, L.mper > 1,
             L.nsplit > 1, L.j1, L.istages > 1, L.wm, L.nb, bad > was ? " FAIL" : "");
      if (bad > was) printf("  ^ dtype %d IL %lld IR %lld I1 %d R %d offset %d\n", dt, IL, IR, I1, R, xoff);
    }
  }
  printf("%d cases, %lld checks, %lld bad\n", cases, nchk, bad);
  return bad ? 1 : 0;
}
