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
#include <vector>
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

// b fp64 n, then nx ny nz ex of each member: per launch of the forward x phase its
// workgroup and LDS bytes (as the launch takes them, the largest of its members)
// and each member's index and threads a transform
static void batch_shapes() {
  int fp64, n;
  if (std::scanf("%d %d", &fp64, &n) != 2) return;
  std::vector<MemberDesc> d(n);
  std::vector<const MemberDesc*> mem;
  for (MemberDesc& m : d) {
    int ex;
    if (std::scanf("%d %d %d %d", &m.nx, &m.ny, &m.nz, &ex) != 4) return;
    m.nxh = m.nx / 2 + 1;
    m.nrow = (long long)m.ny * m.nz;
    if (!radix_plan(m.nx, m.fx) || !fft_threads(m.fx, ex)) return;
    mem.push_back(&m);
  }
  for (const LaunchPart& p : launch_parts(mem, PH_XFWD, fp64 != 0)) {
    int block = 0;
    size_t lds = 0;
    for (int i : p.mem) {
      const Shape s = member_shape(d[i], PH_XFWD, fp64 != 0);
      block = s.block > block ? s.block : block;
      lds = s.lds > lds ? s.lds : lds;
    }
    std::printf("part %d %zu", block, lds);
    for (int i : p.mem) std::printf(" %d %d", i, ct_supported(d[i].nx) ? ct_threads_host(d[i].nx, fp64 ? 8 : 4) : d[i].fx.nt);
    std::printf("\n");
  }
  std::printf("end\n");
}

// t nz ny nxh: the column solve's tiles that the autotuner times, lanes and columns
// of each; after a bar the column counts of each
static void tri_tiles() {
  int nz, ny, nxh;
  if (std::scanf("%d %d %d", &nz, &ny, &nxh) != 3) return;
  std::printf("t");
  for (const TriTile& t : tri_lane_tiles(nz, ny, nxh)) std::printf(" %d %d", t.lanes, t.columns);
  for (const TriTile& t : tri_lane_tiles(nz, ny, nxh)) {
    std::printf(" |");
    for (int c : tri_column_values(ny, nxh, t.lanes)) std::printf(" %d", c);
  }
  std::printf("\n");
}

// c most n, then nx ny nz of each member: the chains they are dealt to
static void chains() {
  int most, n;
  if (std::scanf("%d %d", &most, &n) != 2) return;
  std::vector<MemberDesc> d(n);
  std::vector<const MemberDesc*> mem;
  for (MemberDesc& m : d) {
    if (std::scanf("%d %d %d", &m.nx, &m.ny, &m.nz) != 3) return;
    mem.push_back(&m);
  }
  std::printf("c");
  for (const std::vector<int>& c : deal_chains(mem, most)) {
    std::printf(" |");
    for (int i : c) std::printf(" %d", i);
  }
  std::printf("\n");
}

// l nz columns fp64: the automatic lanes
static void lanes() {
  int nz, columns, fp64;
  if (std::scanf("%d %d %d", &nz, &columns, &fp64) == 3) std::printf("l %d\n", tri_lanes(nz, columns, fp64 != 0));
}

int main() {
  char what[32];
  while (std::scanf("%31s", what) == 1) {
    if (!std::strcmp(what, "x")) x_shapes();
    if (!std::strcmp(what, "b")) batch_shapes();
    if (!std::strcmp(what, "t")) tri_tiles();
    if (!std::strcmp(what, "c")) chains();
    if (!std::strcmp(what, "l")) lanes();
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


@pytest.mark.parametrize("f64", [0, 1])
def test_members_that_share_an_x_launch_fit_its_lds(ask, f64):
    """A launch's workgroup is the largest of its members' and a kernel fills it
    with as many transforms of its member as it holds: their LDS is within what
    the launch has, for every pair of lengths (of the runtime-length kernels,
    whose workgroups differ from 256 threads above 4096 points) and for one batch
    of them all."""
    lengths = smooth(1, 15) + smooth(4097, 8192) + [16, 27, 96]
    batches = [[a, b] for a in lengths for b in lengths if a < b] + [lengths]
    rows = ask([f"b {f64} {len(b)} " + " ".join(f"{n} 36 32 8" for n in b) for b in batches])
    cb = 16 if f64 else 8
    it = iter(rows)
    for b in batches:
        seen = []
        for r in it:
            if r[0] == "end":
                break
            block, lds, members = int(r[1]), int(r[2]), list(map(int, r[3:]))
            for i, nt in zip(members[::2], members[1::2]):
                seen.append(i)
                assert block // nt * b[i] * cb <= lds, (b, b[i], block, lds)
        assert sorted(seen) == list(range(len(b)))


@pytest.mark.parametrize("ny,nx", [(4, 4), (32, 32), (256, 256), (1024, 1024)])
def test_autotuned_lane_counts_keep_the_threads_of_a_workgroup(ask, ny, nx):
    """The autotuner times every lane count that the kernel takes (2 rows a lane or
    more, at most 16), each with 128 or 256 threads a workgroup and so none refused
    (512 threads at most); the column counts timed for the lanes chosen include
    the automatic one."""
    nxh = nx // 2 + 1
    for nz, r in zip(range(1, 1025), ask([f"t {nz} {ny} {nxh}" for nz in range(1, 1025)])):
        head, *cols = " ".join(r[1:]).split("|")
        v = list(map(int, head.split()))
        tiles = list(zip(v[::2], v[1::2]))
        lanes = [1 << i for i in range(7)]
        assert [t[0] for t in tiles] == [P for P in lanes if -(-nz // P) <= 16 and (P == 1 or -(-nz // P) >= 2)], nz
        for (P, c), vals in zip(tiles, cols):
            assert P * c in (128, 256), (nz, P, c)
            assert c in map(int, vals.split()), (nz, P, c, vals)


@pytest.mark.parametrize("most", [1, 2, 3, 4])
def test_chains_of_a_batch(ask, most):
    """A batch's members are dealt to as many chains as asked for, to no more than
    there are pairs of nx and ny: each member once, in the members' order, those
    of one pair on one chain, and no chain more than a pair's points above the
    lightest. One chain is the members as they stand."""
    import random
    rng = random.Random(7)
    grids = [(64, 64, 64), (128, 128, 96), (192, 192, 128), (256, 256, 128), (64, 64, 20), (96, 64, 9), (64, 96, 9)]
    batches = [[rng.choice(grids) for _ in range(n)] for n in (1, 2, 3, 5, 8, 48) for _ in range(4)]
    rows = ask([f"c {most} {len(b)} " + " ".join(" ".join(map(str, g)) for g in b) for b in batches])
    for b, r in zip(batches, rows):
        chains = [list(map(int, c.split())) for c in " ".join(r[1:]).split("|")[1:]]
        pairs = {g[:2] for g in b}
        assert len(chains) == min(most, len(pairs)), (b, chains)
        assert sorted(i for c in chains for i in c) == list(range(len(b)))
        assert all(c == sorted(c) for c in chains)
        assert sum(len({b[i][:2] for i in c}) for c in chains) == len(pairs)
        points = [sum(b[i][0] * b[i][1] * b[i][2] for i in c) for c in chains]
        largest = max(sum(g[0] * g[1] * g[2] for g in b if g[:2] == p) for p in pairs)
        assert max(points) - min(points) <= largest


def fewest_lanes(nz):
    few = 1
    while -(-nz // few) > 6 and few < 64:
        few *= 2
    return few


def test_automatic_lanes(ask):
    """FP64 storage takes no more lanes a column than the fewest that leave at most
    six rows each (more put more of the elimination into the cyclic reduction,
    whose error in nearly singular columns is larger); a column count beside
    automatic lanes fits 512 threads with them wherever it does with those."""
    cases = [(nz, c, f) for nz in range(1, 1025) for c in (0, 1, 8, 32, 64, 128, 512) for f in (0, 1)]
    for (nz, c, f), r in zip(cases, ask([f"l {nz} {c} {f}" for nz, c, f in cases])):
        lanes, few = int(r[1]), fewest_lanes(nz)
        assert lanes in (1, 2, 4, 8, 16, 32, 64) and -(-nz // lanes) <= 16, (nz, c, f, lanes)
        if f:
            assert lanes <= few, (nz, c, lanes, few)
        assert (c * lanes <= 512) == (c * few <= 512), (nz, c, f, lanes, few)
