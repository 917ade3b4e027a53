// Launch side of the BF16 / FP16 partial-MTTKRP kernels (pm16_body.hpp; the
// kernels themselves are instantiated per storage type in pm16_bf16.hip and
// pm16_f16.hip): the pack of the first contracted factor into hi + lo values,
// then the partial MTTKRP, launched or recorded for the batched executor.
#include "pm_common.hpp"

namespace nncpk {

extern template const void* pm16_kernel_form<NNCP_BF16, false>(int, int, int, int, bool);
extern template const void* pm16_kernel_form<NNCP_BF16, true>(int, int, int, int, bool);
extern template const void* pm16_kernel_form<NNCP_F16, false>(int, int, int, int, bool);
extern template const void* pm16_kernel_form<NNCP_F16, true>(int, int, int, int, bool);
extern template const void* pm16_pack_kernel<NNCP_BF16>(bool, int);
extern template const void* pm16_pack_kernel<NNCP_F16>(bool, int);

namespace {

constexpr int left_tr16(int nb) { return nb >= 4 ? 4 : 8; }
constexpr int right_mc16(int nb) { return 4; }
constexpr int right_mc16_j1(int nb) { return nb >= 4 ? 9 : 8; }

const void* kernel16(int dtype, int side, int nb, int j1, int ld, int mt, bool batch) {
  if (dtype == NNCP_BF16)
    return mt ? pm16_kernel_form<NNCP_BF16, true>(side, nb, j1, ld, batch)
              : pm16_kernel_form<NNCP_BF16, false>(side, nb, j1, ld, batch);
  return mt ? pm16_kernel_form<NNCP_F16, true>(side, nb, j1, ld, batch)
            : pm16_kernel_form<NNCP_F16, false>(side, nb, j1, ld, batch);
}

void allow_big_lds(const void* k) { pm_allow_lds(k, 160 * 1024); }

}  // namespace

int pm_16_wave_rows(int side, int nb, int j1) {
  return side == 0 ? 16 * left_tr16(nb) : 16 * (j1 ? right_mc16_j1(nb) : right_mc16(nb));
}
int pm_16_kstep(int side) { return side == 0 ? 32 : 64; }
bool pm16_fast(int side, int64_t IL, int I1, int nb) {
  if (I1 % pm_16_kstep(side) != 0) return false;
  return side == 1 || IL % left_tr16(nb) == 0;
}
// Lane offsets of the range-checked form (up to 31 columns of I_L elements and a
// row on the left, the wave's columns of I_L elements on the right) fit 31 bits.
bool pm16_buf(int side, int64_t IL, int nb, int j1) {
  const int64_t cols = side == 0 ? 31 : pm_16_wave_rows(1, nb, j1);
  return (cols * IL + 256) * 2 < ((int64_t)1 << 31);
}
size_t pm_16_reduce_lds(int side, int nb, int wm) {
  if (wm >= 4) return 0;  // (also every J == 1 launch: one wave per column range)
  const int nacc = side == 0 ? left_tr16(nb) * nb : right_mc16(nb) * nb;
  return (size_t)wm * nacc * 4 * 64 * sizeof(double);
}

// Which loads a launch uses (pm16_body.hpp: 0 masked, 1 plain, 2 range-checked, 3
// range-checked from dword starts, 4 range-checked with the streaming hint):
// plain ones for a right node, or a left node whose columns start on cache lines,
// if the shape allows them; range-checked for the rest, without the hint but for the
// largest tensors (pm_left_stream).
// F16 83x71x57x45 R = 24 left node 34.9 -> 28.7 us, BF16 200x180x220 R = 32 right
// node 39.9 -> 27.0, BF16 30012x1200x48 R = 10 right node 1361 -> 843 us against
// the masked loads with the hint (1338 range-checked with it).
// A right node of odd I_1 loads from dword starts (LD_BUFH) where the address unit is
// what its waves wait for: F16 83x71x57x45 R = 24 59 -> 31 us, BF16 301x40000 R = 10 30
// -> 19, 83x71x2565 R = 48 63 -> 45. Elsewhere the dword after each run is one more load
// to wait for, and the plain range-checked loads are the faster ones:
//  * columns below about 20 elements, 64 of which lie in a few cache lines (3x2x100000
//    R = 5 233 -> 199 us, 1x6x7000 R = 20 193 -> 166);
//  * few columns, as most lanes of a load are idle: up to 16 (R <= 16), 20 and 28 (R > 32;
//    363x3000x5 74 -> 52 us, R = 50 134 -> 108; equal at 17 to 40 columns, by rank);
//  * a small tensor's one group of four waves with columns for one of them or little
//    more (17x50x70 R = 20 54 -> 46 us; equal at about 100 columns, 190 at R > 32);
//  * four column blocks where most of a k-step is padding (15x20x40001 R = 40 84 -> 80;
//    but 31x5x40001 R = 48 66 -> 61 from dword starts).
static bool from_dwords(const PmLaunch& L, const void* X, int64_t IL, int64_t IR, int I1) {
  if (L.side != 1 || !(I1 & 1) || ((uintptr_t)X & 3) != 0) return false;
  if (IL <= 20 || IR <= 12 + 4 * L.nb) return false;
  if (L.wm == 4 && IR < (L.nb < 4 ? 96 : 192)) return false;
  return L.nb < 4 || I1 > 16;
}
int pm16_load_form(const PmLaunch& L, const void* X, int64_t IL, int64_t IR, int I1) {
  const bool fast = pm16_fast(L.side, IL, I1, L.nb);
  if (fast && (L.side == 1 || IL % 64 == 0)) return 1;
  if (pm16_buf(L.side, IL, L.nb, L.j1)) {
    if (L.side == 0) return pm_left_stream(IL, IR, 2) ? 4 : 2;
    return from_dwords(L, X, IL, IR, I1) ? 3 : 2;
  }
  return fast ? 1 : 0;
}

hipError_t pm_launch_16(const PmLaunch& L, const PmArgs& a, const Sink& sk) {
  const int RP = 16 * L.nb;
  if (!a.hpack || !a.hscale || !a.sctab) return hipErrorInvalidValue;
  const bool bf = L.dtype == NNCP_BF16;
  PackArgs pa{a.krp.f[0], a.I1, a.I1pad, a.R, a.col0, RP, a.hpack, a.hscale};
  const int wm = a.wm;
  const int ld = pm16_load_form(L, a.X, a.IL, a.IR, a.I1);
  const bool mt = L.mper > 1;
  // variant = j1*100000 + bf16*10000 + side*1000 + nb*100 + mt*10 + load form
  const int variant =
      (L.j1 ? 100000 : 0) + (bf ? 10000 : 0) + L.side * 1000 + L.nb * 100 + (mt ? 10 : 0) + ld;
  const void* k = kernel16(L.dtype, L.side, L.nb, L.j1, ld, mt, false);
  if (!k || (wm != 1 && wm != 4) || (L.j1 && wm != 4)) return hipErrorInvalidValue;
  size_t lds = L.lds_bytes;
  if (pm_16_reduce_lds(L.side, L.nb, wm) > lds) lds = pm_16_reduce_lds(L.side, L.nb, wm);
  if (lds > kPmMaxLds) return hipErrorInvalidValue;
  if (sk.rec) {
    KOp op{};
    op.kind = K_PACK16;
    op.variant = bf ? 1 : 0;
    op.gx = (unsigned)RP;
    op.gy = 1;
    op.u.pk = pa;
    hipError_t e = sink_record(sk, op);
    if (e != hipSuccess) return e;
    KOp pm{};
    pm.kind = K_PM_16;
    pm.variant = variant;
    pm.gx = (unsigned)L.mgroups;
    pm.gy = (unsigned)L.nsplit;
    pm.lds = (unsigned)lds;
    pm.u.pm = a;
    e = pm_scale_table_record(L, a, sk);
    return e == hipSuccess ? sink_record(sk, pm) : e;
  }
  {
    PmArgs sa = a;
    int64_t n = L.J * RP;
    void* pargs[] = {(void*)&pa, (void*)&sa, (void*)&n};
    // one group per column: 1024 threads for a long one (I_1 = 30012: 52 us with 256)
    const int pt = a.I1pad > 2048 ? 1024 : 256;
    hipError_t e = hipLaunchKernel(bf ? pm16_pack_kernel<NNCP_BF16>(false, pt) : pm16_pack_kernel<NNCP_F16>(false, pt),
                                   dim3((unsigned)(RP + (n + pt - 1) / pt)), dim3(pt), pargs, 0, sk.st);
    if (e != hipSuccess) return e;
  }
  allow_big_lds(k);
  void* args[] = {(void*)&a};
  return hipLaunchKernel(k, dim3(L.mgroups, L.nsplit), dim3(NT), args, lds, sk.st);
}

const void* pm16_batch_kernel(int variant) {
  const int j1 = variant >= 100000 ? 1 : 0;
  const int dtype = ((variant / 10000) % 10) ? NNCP_BF16 : NNCP_F16;
  const int side = (variant / 1000) % 10, nb = (variant / 100) % 10;
  const void* k = kernel16(dtype, side, nb, j1, variant % 10, (variant / 10) % 10, true);
  if (k) allow_big_lds(k);
  return k;
}

const void* pm16_pack_batch_kernel(int variant) {
  return variant ? pm16_pack_kernel<NNCP_BF16>(true, 256) : pm16_pack_kernel<NNCP_F16>(true, 256);
}

}  // namespace nncpk
