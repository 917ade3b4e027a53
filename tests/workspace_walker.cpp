// Host-side walk of a plan's workspace (test infrastructure): records one
// iteration of a plan whose workspace lies at a made-up address and checks that
// every region that the recorded launches write ends inside the workspace and
// before the next region that any launch of the iteration uses.
//
// stdin: "dtype R split no_tree wg_kib N dims..." per line; exit status 1 on any
// violation. "route" lines end with the kinds and variants of the launches.
#include <algorithm>
#include <cstdio>
#include <cstring>
#include <set>
#include <string>
#include <vector>
#include "nncp_internal.hpp"
using namespace nncpk;

static char* const kWs = (char*)((uintptr_t)1 << 46);

struct Extent {
  const char* b;
  size_t n;
  const char* what;
};

int main() {
  int cases = 0, failed = 0, dtype, R, split, no_tree, wg, N;
  while (scanf("%d %d %d %d %d %d", &dtype, &R, &split, &no_tree, &wg, &N) == 6) {
    int64_t dims[kMaxModes];
    for (int k = 0; k < N; ++k) {
      long long d;
      if (scanf("%lld", &d) != 1) return 2;
      dims[k] = d;
    }
    ++cases;
    nncp_options o{};
    o.split = split;
    o.no_tree = no_tree;
    o.pm_wg_kib = wg;
    float* H[kMaxModes];
    for (int k = 0; k < N; ++k) H[k] = (float*)(((uintptr_t)1 << 45) + ((uintptr_t)k << 40));
    std::vector<KOp> ops;
    size_t bytes = 0;
    const int st = record_iteration((const void*)((uintptr_t)1 << 44), dtype, N, dims, R, NNCP_HALS, H, &o, kWs, &bytes, &ops);
    if (st != NNCP_OK) {
      printf("FAIL status %d\n", st);
      ++failed;
      continue;
    }
    std::set<const char*> starts;
    std::vector<Extent> wr;
    auto uses = [&](const void* p) {
      if ((const char*)p >= kWs) starts.insert((const char*)p);
    };
    auto writes = [&](const void* p, size_t n, const char* what) {
      uses(p);
      wr.push_back({(const char*)p, n, what});
    };
    // `rows` x R columns of a temporary from column col0 on (the region starts at column 0)
    auto columns = [&](const void* T, int64_t rows, int col0, int R, int f64, const char* what) {
      uses(T);
      const size_t ld = (size_t)rows * (f64 ? 8 : 4);
      wr.push_back({(const char*)T + ld * col0, ld * R, what});
    };
    const size_t RR = (size_t)R * R;
    for (const KOp& k : ops) {
      const int side = (k.variant / 1000) % 10, nb = (k.variant / 100) % 10, big = (k.variant / 100000) % 10;
      switch (k.kind) {
        case K_SCTAB: writes(k.u.pm.sctab, (size_t)k.u.pm.J * k.variant * 8, "scale table"); break;
        case K_PACK16: {
          const int terms = pm16_terms(k.variant ? NNCP_BF16 : NNCP_F16);
          writes(k.u.pk.hscale, (size_t)k.u.pk.RP * 4, "pack scales");
          writes(k.u.pk.pack, (size_t)terms * k.u.pk.RP * k.u.pk.I1pad * 2, "pack");
          break;
        }
        case K_PM_F32: case K_PM_16: {
          const PmArgs& a = k.u.pm;
          const int64_t rows = side == 0 ? a.IL : a.IR;
          const int wr_rows = k.kind == K_PM_F32 ? pm_f32_wave_rows(side, nb, big) : pm_16_wave_rows(side, nb, big);
          uses(a.T);
          uses(a.zeros);
          if (a.nsplit > 1) writes(a.partial, (size_t)a.nsplit * 16 * nb * a.mtiles * a.wm * wr_rows * 8, "partials");
          else columns(a.T, rows, a.col0, a.R, a.t_f64, "T");
          break;
        }
        case K_PM_REDUCE: {
          const ReduceArgs& a = k.u.red;
          columns(a.T, a.Mtot, a.col0, a.R, a.t_f64, "reduced T");
          break;
        }
        case K_MTTV_TRAIL: case K_MTTV_LEAD: {
          const MttvArgs& a = k.u.mt;
          const int64_t rows = k.kind == K_MTTV_TRAIL ? a.Ia : a.J;
          uses(a.T);
          uses(a.out);
          if (k.kind == K_MTTV_TRAIL && a.nz > 1) writes(a.part, (size_t)a.nz * R * a.Ia * 8, "multi-TTV partials");
          else writes(a.out, (size_t)rows * R * (a.out_f64 ? 8 : 4), "multi-TTV");
          break;
        }
        case K_UPDATE: uses(k.u.up.M); break;
        default: {
          const FinalizeArgs& a = k.u.fin;
          writes(a.G, N * RR * 8, "G");
          writes(a.S, N * RR * 8, "S");
          writes(a.lam, (size_t)N * R * 8, "lambda");
          writes(a.lam_model, (size_t)R * 8, "model lambda");
          writes(a.fit_out, (size_t)a.fit_capacity * 8, "fit");
          uses(a.alpha);
          uses(a.iter_counter);
          if (a.nchunks > 1) writes(a.partial, (size_t)a.nchunks * (RR + 1) * 8, "Gram partials");
        }
      }
    }
    std::string bad;
    for (const Extent& e : wr) {
      const auto next = starts.upper_bound(e.b);
      const char* lim = next == starts.end() ? kWs + bytes : std::min<const char*>(*next, kWs + bytes);
      if (e.b < kWs || e.b + e.n > lim) {
        char line[160];
        snprintf(line, sizeof line, "  %s: %zu bytes at %zd, next region at %zd of %zu\n", e.what, e.n,
                 (ptrdiff_t)(e.b - kWs), (ptrdiff_t)(lim - kWs), bytes);
        if (bad.size() < 800) bad += line;
      }
    }
    printf("%s dtype %d R %d split %d no_tree %d wg %d:", bad.empty() ? "ok" : "FAIL", dtype, R, split, no_tree, wg);
    for (int k = 0; k < N; ++k) printf(" %lld", (long long)dims[k]);
    printf(" route");
    for (const KOp& k : ops) printf(" %d/%d", k.kind, k.variant);
    printf("\n%s", bad.c_str());
    failed += !bad.empty();
  }
  printf("%d cases, %d failed\n", cases, failed);
  return failed ? 1 : 0;
}
