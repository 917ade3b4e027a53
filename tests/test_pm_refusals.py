"""The partial MTTKRP's launchers refuse, before any device work, arguments
without the buffers that the kernels read (host check; the launch is recorded, so a
launcher that let one pass would not reach a device either)."""

import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB_DIR = os.path.join(ROOT, "paper_1806_07985_amd", "lib")

SOURCE = r"""
#include <cstdio>
#include <vector>
#include "nncp_internal.hpp"
using namespace nncpk;
int main() {
  int bad = 0;
  for (int dt = 0; dt < 3; ++dt)
    for (int side = 0; side < 2; ++side)
      for (int drop = 0; drop < 4; ++drop) {
        const PmLaunch L = pm_plan(side, dt, 60, 35, side ? 60 : 35, 5);
        PmArgs a{};
        char* p = (char*)(1 << 20);
        a.X = p; a.IL = 60; a.IR = 35; a.R = 5; a.T = p; a.partial = (double*)p; a.zeros = p;
        a.krp.nm = 1; a.krp.f[0] = (const float*)p; a.krp.dim[0] = side ? 60 : 35;
        a.sctab = drop == 1 ? nullptr : (double*)p;
        a.hpack = drop == 2 ? nullptr : (unsigned short*)p;
        a.hscale = drop == 3 ? nullptr : (float*)p;
        pm_fill_args(L, a);
        std::vector<KOp> rec;
        Sink sk;
        sk.rec = &rec;
        const bool refuse = drop == 1 || (drop > 1 && dt != NNCP_F32);  // FP32 packs nothing
        const hipError_t e = pm_launch(L, a, sk);
        if ((e == hipErrorInvalidValue) != refuse || rec.empty() != refuse) { ++bad; printf("dtype %d side %d drop %d: %d\n", dt, side, drop, (int)e); }
      }
  printf("%d wrong\n", bad);
  return bad ? 1 : 0;
}
"""


def test_missing_buffers_are_refused(tmp_path):
    src, exe = tmp_path / "refuse.cpp", str(tmp_path / "refuse")
    src.write_text(SOURCE)
    cmd = [os.environ.get("HIPCC", "/opt/rocm/bin/hipcc"), "-O1", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
           os.path.join(ROOT, "paper_1806_07985_amd", "csrc"), str(src), "-o", exe, "-L", LIB_DIR, "-lnncp",
           f"-Wl,-rpath,{LIB_DIR}"]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "0 wrong" in r.stdout, r.stdout
