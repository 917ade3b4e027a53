// Host-side walk of the FP32 partial-MTTKRP kernels' range-checked loads (test
// infrastructure): for the plans the library makes, every lane's buffer offset
// stays below 2^31, every dword inside the range lies inside the tensor, and no
// element that feeds a stored output is cut off by the range.
//
// stdin: "IL IR I1_left I1_right R" per line; exit status 1 on any violation.
#include <algorithm>
#include <cstdio>
#include "nncp_internal.hpp"
using namespace nncpk;

static long long bad = 0, nchk = 0;
static void need(bool ok, const char* what) {
  ++nchk;
  if (!ok && bad++ < 5) printf("  %s\n", what);
}

// one lane load of `w` elements at offset `off` from element e0, of which `real` are needed
static void lane(int64_t e0, int64_t off, int w, int real, int64_t I) {
  need(off >= 0 && off * 4 + 4 * w <= ((int64_t)1 << 31), "offset past 31 bits");
  const int64_t rem = I - e0, n = rem <= 0 ? 0 : std::min<int64_t>(rem, 0x7ffffffc / 4);
  for (int e = 0; e < w; ++e) {
    const bool in = off + e < n;
    if (in) need(e0 + off + e >= 0 && e0 + off + e < I, "in range but outside the tensor");
    if (e < real) need(in, "a real element is cut off");
  }
}

static void side0(const PmLaunch& L, int64_t IL, int64_t IR) {
  const int wr = pm_f32_wave_rows(0, L.nb), TR = wr / 16, KS = pm_f32_kstep(0);
  for (int64_t m0 = 0; m0 < (int64_t)L.mtiles * L.mtile; m0 += wr)
    for (int64_t j = 0; j < L.J; ++j)
      for (int i1 = 0; i1 < L.I1pad; i1 += KS) {
        const int64_t col = (int64_t)L.I1 * j + i1, e0 = IL * col + m0;
        for (int ln = 0; ln < 64; ++ln)
          for (int u = 0; u < 4; ++u) {
            const int64_t m = m0 + TR * (ln & 15), c = 4 * (ln >> 4) + u;
            if (m >= IL) continue;  // reads nothing
            const int real = i1 + c < L.I1 ? (int)std::min<int64_t>(TR, IL - m) : 0;
            lane(e0, IL * c + TR * (ln & 15), TR, real, IL * IR);
          }
      }
}

static void side1(const PmLaunch& L, int64_t IL, int64_t IR) {
  const int wr = pm_f32_wave_rows(1, L.nb), KS = pm_f32_kstep(1);
  for (int64_t c0 = 0; c0 < (int64_t)L.mtiles * L.mtile; c0 += wr)
    for (int64_t j = 0; j < L.J; ++j)
      for (int i1 = 0; i1 < L.I1pad; i1 += KS) {
        const int64_t e0 = c0 * IL + (int64_t)L.I1 * j + i1;
        for (int ln = 0; ln < 64; ++ln)
          for (int g = 0; g < wr / 16; ++g)
            for (int h = 0; h < 2; ++h) {
              const int64_t c = c0 + 16 * g + (ln & 15);
              if (c >= IR) continue;
              const int k = 4 * (ln >> 4) + 16 * h;
              lane(e0, (16 * g + (ln & 15)) * IL + k, 4, std::max(0, std::min(4, L.I1 - (i1 + k))), IL * IR);
            }
      }
}

int main() {
  long long IL, IR;
  int a, b, R, cases = 0;
  while (scanf("%lld %lld %d %d %d", &IL, &IR, &a, &b, &R) == 5) {
    ++cases;
    for (int side = 0; side < 2; ++side) {
      const PmLaunch L = pm_plan(side, NNCP_F32, IL, IR, side ? b : a, R, 0);
      if (L.xs || !pm_f32_buf(side, IL, L.nb)) continue;
      if (side) side1(L, IL, IR);
      else side0(L, IL, IR);
    }
  }
  // the rule refuses exactly where an offset would pass 31 bits
  for (int side = 0; side < 2; ++side)
    for (int nb = 1; nb <= 4; nb *= 2) {
      const int64_t cols = side ? pm_f32_wave_rows(1, nb) : 15, lim = ((int64_t)1 << 29) / cols;
      need(pm_f32_buf(side, lim - 64, nb) && !pm_f32_buf(side, lim + 64, nb), "rule");
    }
  printf("%d cases, %lld checks, %lld bad\n", cases, nchk, bad);
  return bad ? 1 : 0;
}
