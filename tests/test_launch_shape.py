"""Launch shapes of the phases (csrc/launch_shape.cpp), built with g++ on its
own and driven by a small program: what the host gives a launch against what
its kernel takes from it."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2009_12849_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <cstring>
#include "kernels.h"
#include "launch_shape.h"
#include "plan_math.h"
using namespace monc;

static const Phase kX[] = {PH_XFWD, PH_XPRE, PH_XPRE_UPDATE, PH_RESID, PH_XINV, PH_XINV_P1, PH_XINV_CORR, PH_XINV_DOTS};

// x nx ny nz fp64 ex xpw: per x phase, threads a transform, workgroup, LDS bytes, workgroups
static void x_shapes() {
  int nx, ny, nz, fp64, ex, xpw;
  if (std::scanf("%d %d %d %d %d %d", &nx, &ny, &nz, &fp64, &ex, &xpw) != 6) return;
  MemberDesc d{};
  d.nx = nx;
  d.ny = ny;
  d.nz = nz;
  d.nxh = nx / 2 + 1;
  d.nrow = (long long)ny * nz;
  d.xpw = xpw;
  const bool ok = radix_plan(nx, d.fx) && fft_threads(d.fx, ex);
  const int nt = ct_supported(nx) ? ct_threads_host(nx, fp64 ? 8 : 4) : d.fx.nt;
  std::printf("x %d %d %d", ok ? 1 : 0, ct_supported(nx) ? 1 : 0, nt);
  for (Phase ph : kX) {
    if (!ok && !ct_supported(nx)) break;  // refused: more than 1024 threads a transform
    const Shape s = member_shape(d, ph, fp64 != 0);
    std::printf(" %d %zu %lld", s.block, s.lds, s.blocks);
  }
  std::printf("\n");
}

int main() {
  char what[32];
  while (std::scanf("%31s", what) == 1) {
    if (!std::strcmp(what, "x")) x_shapes();
  }
  return 0;
}
"""
X_PHASES = ["xfwd", "xpre", "xpre_update", "resid", "xinv", "xinv_p1", "xinv_corr", "xinv_dots"]


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    d = tmp_path_factory.mktemp("launch_shape")
    src = d / "driver.cpp"
    src.write_text(DRIVER)
    exe = d / "driver"
    subprocess.run([gxx, "-O1", "-std=c++17", f"-I{CSRC}", f"-I{os.path.join(ROOT, 'include')}", str(src),
                    os.path.join(CSRC, "launch_shape.cpp"), os.path.join(CSRC, "plan_math.cpp"), "-o", str(exe)],
                   check=True)

    def run(lines):
        out = subprocess.run([str(exe)], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True)
        return [l.split() for l in out.stdout.splitlines()]
    return run


def smooth(lo, hi):
    out = []
    for n in range(lo, hi + 1):
        r = n
        while r % 2 == 0:
            r //= 2
        while r % 3 == 0:
            r //= 3
        if r == 1:
            out.append(n)
    return out


def test_x_kernels_fit_the_lds_they_are_given(ask):
    """Every x length, type, elements per thread (runtime-length kernels) and
    transforms per workgroup (compile-time ones): the transforms of a
    workgroup fit its LDS, and in the kernels that end in a workgroup sum (the
    variable-density solver's residual update and inner products) so does the
    sum's double per thread."""
    cases = [(n, ny, nz, f64, ex, xpw) for n in smooth(1, 8192) for f64 in (0, 1)
             for ny, nz in ((36, 32),)
             for ex, xpw in ([(e, 0) for e in range(1, 9)] if n < 16 or n > 4096 else [(8, x) for x in range(0, 65)])]
    rows = ask([f"x {' '.join(map(str, c))}" for c in cases])
    assert len(rows) == len(cases)
    for (n, ny, nz, f64, ex, xpw), r in zip(cases, rows):
        ok, ct, nt = map(int, r[1:4])
        if not ok and not ct:
            continue                      # refused
        cb = 16 if f64 else 8
        for i, name in enumerate(X_PHASES):
            block, lds, blocks = map(int, r[4 + 3 * i:7 + 3 * i])
            case = (n, f64, ex, xpw, name, block, lds)
            ipw = block // nt
            assert 1 <= ipw and block <= (512 if ct else 1024), case
            assert blocks * ipw * 2 >= ny * nz, case
            assert ipw * n * cb <= lds, case
            if name in ("xpre_update", "xinv_dots"):
                assert block * 8 <= lds, case
