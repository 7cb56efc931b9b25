// Launch shapes (see launch_shape.h).
#include "launch_shape.h"

#include <algorithm>
#include <array>

#include "kernels.h"

namespace monc {

bool ct_supported(int n) {
  switch (n) {
#define MONC_CASE(N) case N:
#define MONC_GROUP_CASES(K) MONC_CT_GROUP_##K(MONC_CASE)
    MONC_FFT_GROUPS(MONC_GROUP_CASES)
#undef MONC_GROUP_CASES
#undef MONC_CASE
    return true;
    default:
      return false;
  }
}

bool pp_supported(int n) { return pp_length(n); }

bool is_xphase(Phase ph) {
  return ph == PH_XFWD || ph == PH_XPRE || ph == PH_XPRE_UPDATE || ph == PH_RESID || ph == PH_XINV ||
         ph == PH_XINV_P1 || ph == PH_XINV_CORR || ph == PH_XINV_DOTS;
}
bool is_yphase(Phase ph) { return ph == PH_YFWD || ph == PH_YINV; }
bool is_level_phase(Phase ph) { return ph >= PH_LEVEL_FWD; }

Shape member_shape(const MemberDesc& d, Phase ph, bool fp64) {
  const size_t cb = fp64 ? 16 : 8;
  Shape s;
  if (is_level_phase(ph)) {
    const int ntx = ct_threads_host(d.nx, (int)cb / 2), nty = ct_threads_y_host(d.ny, 8);
    s.variant = 1;
    const int threads = std::max(d.ny / 2 * ntx, d.nxh * nty), rounds = (threads + 511) / 512;
    s.block = ((threads + rounds - 1) / rounds + 63) / 64 * 64;
    // whole transforms and a partial one that fills the workgroup
    const size_t x = (size_t)((s.block + ntx - 1) / ntx) * xlds_len(d.nx, (int)cb);
    const size_t y = (size_t)((s.block + nty - 1) / nty) * d.ny;
    s.lds = std::max(x, y) * cb;
    s.blocks = d.nz;
  } else if (is_xphase(ph)) {
    const long long pairs = (d.nrow + 1) / 2;
    if (ct_supported(d.nx)) {
      const int nt = ct_threads_host(d.nx, (int)cb / 2);
      int ipw = d.xpw > 0 ? std::min(d.xpw, std::max(1, 512 / nt)) : std::max(1, 256 / nt);
      // the residual kernel at these lengths walks whole rows per wave: its
      // workgroups hold whole waves, the nearest multiple of m transforms
      // (up, unless that passes 512 threads; m nt <= 512, and at most 16
      // transforms of 256 to 1536 points stay within the LDS limit)
      if (ph == PH_RESID && xres_wave_rows(d.nx)) {
        const int m = wave_transforms(nt);
        ipw = (ipw + m - 1) / m * m;
        if (ipw * nt > 512) ipw -= m;
      }
      s.variant = d.nx;
      s.block = ipw * nt;
      s.lds = (size_t)ipw * xlds_len(d.nx, (int)cb) * cb;
      s.blocks = (pairs + ipw - 1) / ipw;
    } else {
      s.block = std::max(256, (d.fx.nt + 63) / 64 * 64);
      const int ipw = s.block / d.fx.nt;
      s.lds = (size_t)ipw * d.nx * cb;
      s.blocks = (pairs + ipw - 1) / ipw;
    }
    // group_sum: a double per thread, idle ones too (a runtime-length FP32 kernel
    // of one element a thread has fewer LDS values than threads)
    if (ph == PH_XPRE_UPDATE || ph == PH_XINV_DOTS) s.lds = std::max(s.lds, (size_t)s.block * sizeof(double));
  } else if (is_yphase(ph)) {
    if (ct_supported(d.ny) && d.yept == 32) {
      // the persistent kernel: a fixed number of columns per tile (ymt then
      // only sets the spectral column blocks)
      const int nt = ct_threads_y_host(d.ny, 32);
      const int mt = pp_columns(d.ny);
      s.variant = d.ny;
      s.block = mt * nt;
      s.lds = (size_t)d.ny * (mt + 1) * cb;  // the tile and the twiddle table
      s.blocks = (long long)d.nz * ((d.nxh + mt - 1) / mt);
      s.persistent = true;
    } else if (ct_supported(d.ny)) {
      const int nt = ct_threads_y_host(d.ny, d.yept);
      const int mt = std::max(1, std::min(d.ymt, 1024 / nt));
      s.variant = d.ny;
      s.block = mt * nt;
      s.lds = (size_t)d.ny * mt * cb;
      s.blocks = (long long)d.nz * ((d.nxh + mt - 1) / mt);
    } else {
      s.block = std::max(64, (d.ymt * d.fy.nt + 63) / 64 * 64);
      s.lds = (size_t)d.ny * d.ymt * cb;
      s.blocks = (long long)d.nz * ((d.nxh + d.ymt - 1) / d.ymt);
    }
  } else if (ph == PH_TRI && d.tcwaves) {
    s.variant = d.tcrows;
    s.sub = 2;
    s.block = 64 * d.tcwaves;
    s.lds = (size_t)tricol_lds(d.tcwaves) * sizeof(double);
    s.blocks = ((long long)d.ny * d.nxp + 63) / 64;
  } else if (ph == PH_TRI) {
    s.variant = d.tris;
    s.sub = tri_pairs(d.tris, d.tricw, !fp64) ? 1 : 0;
    s.block = d.tricw * d.triP;
    s.lds = (size_t)d.tricw * (d.triP * tri_lane_slots(d.tris, !fp64) + 1) * 16;  // matches the kernel's column stride
    s.blocks = ((long long)d.ny * d.nxp + d.tricw - 1) / d.tricw;  // over the padded plane
  } else {
    // points per thread: 16-byte field accesses on the mixed path (4 floats),
    // 2 doubles on the FP64 path; fewer when nx does not divide
    const int want = (ph == PH_GRAD_MIXED) ? 4 : 2;
    const int vec = (d.nx % want == 0) ? want : (d.nx % 2 == 0) ? 2 : 1;
    const long long nvec = (long long)d.nx * d.ny * d.nz / vec;
    s.variant = vec;
    s.blocks = (nvec + 255) / 256;
  }
  return s;
}

std::vector<LaunchPart> launch_parts(const std::vector<const MemberDesc*>& mem, Phase ph, bool fp64) {
  std::vector<LaunchPart> parts;
  std::vector<std::array<int, 3>> keys;
  for (int i = 0; i < (int)mem.size(); ++i) {
    const Shape s = member_shape(*mem[i], ph, fp64);
    // the compile-time kernels need blockDim to match each member exactly,
    // and the y kernels the member's elements per thread; the runtime-length x
    // kernels fill blockDim with transforms, of which the LDS holds those of the
    // member's own workgroup (8 beside 4374 points: 576 transforms of 8 where
    // the LDS of 4374 values holds 546)
    const std::array<int, 3> key{s.variant, s.variant || is_xphase(ph) ? s.block : 0,
                                 !s.variant ? 0 : is_yphase(ph) ? mem[i]->yept : s.sub};
    size_t pi = 0;
    while (pi < parts.size() && (keys[pi] != key || parts[pi].mem.size() >= (size_t)kMaxLaunchMembers)) ++pi;
    if (pi == parts.size()) {
      parts.push_back({s, {}});
      keys.push_back(key);
    }
    parts[pi].mem.push_back(i);
  }
  return parts;
}

// Members of one (nx, ny) share every launch. A phase is one launch per kernel
// instance, and an ensemble of uneven grids has one for most of its lengths: one
// after the other they leave a tail each, which for small members is most of
// their time (six members between 72 x 54 x 33 and 162 x 128 x 41 in FP64: 281 ->
// 204 us on chains).
std::vector<std::vector<int>> deal_chains(const std::vector<const MemberDesc*>& mem, int most) {
  struct Class {
    int nx, ny;
    double points;
    std::vector<int> mem;
  };
  std::vector<Class> cls;
  for (int i = 0; i < (int)mem.size(); ++i) {
    const MemberDesc& h = *mem[i];
    size_t c = 0;
    while (c < cls.size() && (cls[c].nx != h.nx || cls[c].ny != h.ny)) ++c;
    if (c == cls.size()) cls.push_back({h.nx, h.ny, 0.0, {}});
    cls[c].mem.push_back(i);
    cls[c].points += (double)h.nx * h.ny * h.nz;
  }
  std::stable_sort(cls.begin(), cls.end(), [](const Class& a, const Class& b) { return a.points > b.points; });
  const size_t nb = std::min<size_t>(cls.size(), std::max(1, most));
  std::vector<double> load(nb, 0.0);
  std::vector<std::vector<int>> out(nb);
  for (const Class& c : cls) {
    const size_t b = std::min_element(load.begin(), load.end()) - load.begin();
    load[b] += c.points;
    out[b].insert(out[b].end(), c.mem.begin(), c.mem.end());
  }
  for (auto& chain : out) std::sort(chain.begin(), chain.end());
  return out;
}

int tri_rows(int nz, int P) {
  const int s = std::max(2, (nz + P - 1) / P);
  if (s <= 8) return s;
  if (s <= 10) return 10;
  if (s <= 12) return 12;
  if (s <= kTriSmax) return kTriSmax;
  return 0;
}

// Sixteen lanes (one DPP row, the cheapest exchange) where that leaves 2 to 10
// rows a lane, four up to 16 levels, more lanes above 160. Against the fewest
// lanes of at most 6 rows, us (FP64): 256^2 x 128 36.5 -> 28.7 (32 -> 16), 128 x 128
// x 256 23.6 -> 20.4 (64 -> 32); but 1024 x 512 x 16 26 with four, 34 with 16.
// FP64 storage takes no more than those fewest: each lane ends the cyclic
// reduction with a division of its own, which in a nearly singular column (a
// horizontally long domain's lowest wavenumbers) puts an error of its own on each
// lane's part of the column, where the rows inside a lane follow from one another.
// The error of w against 64-bit sums, the default lanes with and without that
// bound (2-norm): 64 x 1024 x 8 4.0e-14 / 6.0e-13, 108 x 1024 x 24 4.6e-14 / 3.9e-13,
// 256 x 24 x 32 1.5e-14 / 4.7e-14 (u 5.9e-15 / 4.4e-14); the calls cost 32^3 22.2 / 21.7
// us, 128^2 x 40 42.7 / 41.7, 1024^2 x 32 971 / 975, 1024 x 512 x 8 128 / 132.
// A column count beside them is taken where the fewest lanes leave it room in
// 512 threads, and then with them where the others do not.
int tri_lanes(int nz, int columns, bool fp64) {
  int few = 1, lanes = nz <= 4 ? 1 : nz <= 16 ? 4 : 16;
  while ((nz + few - 1) / few > 6 && few < kTriPmax) few *= 2;
  while ((nz + lanes - 1) / lanes > 10 && lanes < kTriPmax) lanes *= 2;
  if (fp64) lanes = std::min(lanes, few);
  return (long long)columns * std::max(few, lanes) > 512 ? few : lanes;
}

// 256 threads, four waves, so that five workgroups fit a CU at ~100 registers per
// lane; half that where it leaves fewer than four workgroups a CU: 128^2 x 128 FP64
// 16.0 -> 15.4 us, but 1024^2 x 64 FP32 129 -> 185
int tri_columns(int ny, int nxh, int P) {
  const int threads = (long long)ny * nxh * P < 1024 * 256 ? 128 : 256;
  return std::max(1, threads / P);
}

std::vector<TriTile> tri_lane_tiles(int nz, int ny, int nxh) {
  std::vector<TriTile> out;
  for (int P = 1; P <= kTriPmax; P *= 2)
    if (tri_rows(nz, P) != 0 && (P == 1 || (nz + P - 1) / P >= 2)) out.push_back({P, tri_columns(ny, nxh, P)});
  return out;
}

std::vector<int> tri_column_values(int ny, int nxh, int P) {
  std::vector<int> out = {4, 8, 16, 32};
  const int automatic = tri_columns(ny, nxh, P);
  if (std::find(out.begin(), out.end(), automatic) == out.end()) out.push_back(automatic);
  return out;
}

// Measured (default tiles, us, lanes-per-column / wave-per-chunk):
//   above 96 levels from about 512^2 columns on: 128^2 x 128 13.3 / 14.0, 256^2 x 128
//   21.4 / 21.1, 512^2 x 128 54.7 / 53.1, 1024^2 x 100 211 / 160, 1024 x 512 x 128 128 /
//   104, 512^2 x 256 189 / 126, 1024^2 x 256 686 / 461; but not from 129 to 160, where
//   sixteen lanes still do and this kernel's sixteen waves have at most 10 rows
//   each: 512^2 x 160 59.6 / 84.8, 1024^2 x 160 284 / 325, 2048^2 x 160 1240 / 1292.
//   up to 32 levels over 512 tiles of 64 columns: 256^2 x 16 9.9 / 9.6, 512^2 x 32
//   21.4 / 17.9, 432^2 x 32 18.7 / 16.3, 1024 x 512 x 16 20.4 / 18.3.
//   between: 256^2 x 64 17.3 / 18.1, 512^2 x 96 41.9 / 43.2; beyond the 256 MB
//   Infinity Cache 129 / 110 (1024^2 x 64).
// Rows per wave: the fewest waves (2, 4, 8 or 16) with at most 16 rows. More rows
// mean fewer interface rows and more, smaller workgroups on a CU, whose loads
// overlap each other's elimination (512^2 x 128 8 waves of 16 rows 55 us, 16 of 8
// 75; 1024^2 x 64 4 of 16 109, 8 of 8 116, 16 of 4 196).
void tricol_shape(int nz, long long tiles, int* waves, int* rows) {
  *waves = *rows = 0;
  if (nz > kTriColMax) return;
  const bool beyond_cache = (double)tiles * 64 * nz * 8 > 256.0 * (1 << 20);
  const bool use = nz > 96 ? tiles > 1024 && (nz <= 128 || nz > 160) : nz <= 32 ? tiles > 512 : beyond_cache;
  if (!use) return;
  int P = 2;
  while (P < 16 && (nz + P - 1) / P > 16) P *= 2;
  *waves = P;
  *rows = std::max(2, (nz + P - 1) / P);
}

}  // namespace monc
