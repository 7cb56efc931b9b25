"""The column solve of FP32 storage on both of its kernels, at the lines of the
rule between them (csrc/launch_shape.cpp, tricol_shape) and with every row count
and wave count of the wave-per-chunk kernel. The shapes are checked against the
rule itself on the CPU, so that a moved line cannot leave an instance without a
case; on the GPU each is solved against the oracle."""
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
import oracle.projection
import synth
from tests.helpers import relerr
from tests.tolerances import p_tolerance

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2009_12849_amd", "csrc")

# (nx, ny, nz). 256 x 243 has 517 tiles of 64 columns (the last one ragged), 128 x 162
# 183, 16 x 2048 512, 16 x 4096 1024 and 32 x 4096 1536; spectra beyond the 256 MB
# Infinity Cache at 2048 x 486 from 67 levels on, at 2048 x 972 from 34.
SHAPES = [(256, 243, n) for n in (1, 2, *range(5, 34))] + [(16, 2048, 32), (128, 162, 97), (16, 4096, 97)] \
    + [(32, 4096, n) for n in (96, 97, 112, 113, 127, 128, 129, 160, 161, 177, 193, 208, 209, 224, 225, 241, 256, 257)] \
    + [(2048, 486, n) for n in (66, 67, 77, 85, 90, 96)] + [(2048, 972, n) for n in (33, 34, 37, 41, 46, 49, 54, 57, 61, 64)]
# neighbours on either side of a line: levels, tiles, size of the spectrum
LINES = [((256, 243, 32), (256, 243, 33)), ((16, 2048, 32), (256, 243, 32)), ((32, 4096, 96), (32, 4096, 97)),
         ((16, 4096, 97), (32, 4096, 97)), ((32, 4096, 128), (32, 4096, 129)), ((32, 4096, 160), (32, 4096, 161)),
         ((32, 4096, 256), (32, 4096, 257)), ((2048, 486, 66), (2048, 486, 67)), ((2048, 972, 33), (2048, 972, 34))]

DRIVER = r"""
#include <cstdio>
#include "launch_shape.h"
using namespace monc;
int main() {
  int nz, waves, rows;
  long long tiles;
  while (std::scanf("%d %lld", &nz, &tiles) == 2) {
    tricol_shape(nz, tiles, &waves, &rows);
    std::printf("%d %d\n", waves, rows);
  }
  return 0;
}
"""


def tiles(nx, ny):
    nxp = (nx // 2 + 1 + 7) // 8 * 8          # the padded spectral row
    return (ny * nxp + 63) // 64


def rule(tmp, shapes):
    """(waves, rows a wave) of each shape, (0, 0) on the lanes-per-column kernel."""
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    src = tmp / "driver.cpp"
    src.write_text(DRIVER)
    exe = tmp / "driver"
    subprocess.run(["g++", "-O1", "-std=c++17", f"-I{CSRC}", str(src), os.path.join(CSRC, "launch_shape.cpp"), "-o",
                    str(exe)], check=True)
    text = "\n".join(f"{nz} {tiles(nx, ny)}" for nx, ny, nz in shapes) + "\n"
    out = subprocess.run([str(exe)], input=text, capture_output=True, text=True, check=True).stdout
    return [tuple(map(int, l.split())) for l in out.splitlines()]


def test_shapes_cover_the_rule(tmp_path):
    """Every (waves, rows) that the rule gives any plan is in SHAPES, and both
    kernels are, on either side of each line."""
    kern = dict(zip(SHAPES, rule(tmp_path, SHAPES)))
    every = {r for nx, ny in ((256, 243), (32, 4096), (2048, 972))
             for r in rule(tmp_path, [(nx, ny, n) for n in range(1, 1025)])}
    assert every == set(kern.values()) and len(every) > 30
    for a, b in LINES:
        assert (kern[a] == (0, 0)) != (kern[b] == (0, 0)), (a, kern[a], b, kern[b])


@pytest.mark.gpu
@pytest.mark.parametrize("shape", SHAPES)
def test_columns_match_the_oracle(shape):
    """Random spectra through the solve stage of a mixed plan, against the oracle's
    elimination: all rows n of the small levels, the first and last eight and every
    37th of the others. The solve is FP64, its result rounded once (2^-24 a part);
    the elimination is backward stable (p_tolerance)."""
    torch = pytest.importorskip("torch")
    import paper_2009_12849_amd as monc
    nx, ny, nz = shape
    rng = np.random.default_rng(2100 + sum(shape))
    g = synth.random_grid(rng, nx, ny, nz, stretch=(1.0, min(1.1, 20.0 ** (1.0 / nz))))
    print(f"case columns {shape}", flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(sum(shape))
    B = torch.randn((nz, ny, nx // 2 + 1), dtype=torch.complex64, device="cuda:0", generator=gen)
    plan = monc.Plan.from_grid(g, "mixed")
    spec = plan.spectral_buffer()
    plan.spectral_set(spec, B)
    plan.debug_stage(monc.STAGE_SOLVE, [spec])
    rows = list(range(ny)) if ny <= 256 else sorted({*range(8), *range(0, ny, 37), *range(ny - 8, ny)})
    got = plan.spectral_get(spec)[:, rows].cpu().numpy().astype(np.complex128)
    plan.close()
    b = B[:, rows].cpu().numpy().astype(np.complex128)
    a, c = oracle.tridiag_coefficients(g.dz, g.rho0)
    lamx, lamy = oracle.modified_wavenumbers(nx, ny, g.dx, g.dy)
    lam = lamy[rows][:, None] + lamx[None, :]
    lam[0, 0] = 1.0                                            # the singular column, replaced below
    beta = (-(a + c))[:, None, None] - np.asarray(g.rho0)[:, None, None] * lam[None]
    ref = oracle.projection._thomas(a, beta, c, b)
    ref[:, 0, 0] = oracle.projection.solve_mean_column(b[:, 0, 0], g.dz, g.rho0)
    assert relerr(got, ref / (nx * ny)) <= p_tolerance(g) + 2.0 ** -23
