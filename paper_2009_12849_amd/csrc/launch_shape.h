// Launch shapes of the projection's phases, and the rules of the column
// kernels' tiles. Pure C++ (no HIP calls), so that what the host gives a kernel can be
// checked without a device.
#pragma once
#include <stddef.h>

#include <vector>

#include "monc_types.h"

namespace monc {

enum Phase {
  PH_XFWD, PH_XPRE, PH_XPRE_UPDATE, PH_RESID, PH_YFWD, PH_TRI, PH_YINV, PH_XINV, PH_XINV_P1, PH_XINV_CORR,
  PH_XINV_DOTS, PH_GRAD, PH_GRAD_MIXED,
  PH_LEVEL_FWD, PH_LEVEL_RESID, PH_LEVEL_INV, PH_LEVEL_INV_P1, PH_LEVEL_INV_CORR
};

bool is_xphase(Phase ph);
bool is_yphase(Phase ph);
bool is_level_phase(Phase ph);

// Launch shape of one member in one phase. Members whose shapes agree share
// a launch; `variant` identifies the kernel instance (compile-time length or
// the runtime-length kernel) and `block` its workgroup size.
struct Shape {
  int variant = 0;   // compile-time length, or 0 for the runtime-length kernel
  int sub = 0;       // kernel instance within the variant (tridiagonal: 1 column pairs, 2 wave per chunk)
  int block = 256;
  size_t lds = 0;
  long long blocks = 0;       // tiles of the phase
  bool persistent = false;    // the grid covers the CUs once and walks the tiles
};

Shape member_shape(const MemberDesc& d, Phase ph, bool fp64);

// The launches of one phase over several members: members of one kernel
// instance and workgroup size, up to kMaxLaunchMembers in each.
struct LaunchPart {
  Shape shape;           // of its first member
  std::vector<int> mem;  // indices of its members
};
std::vector<LaunchPart> launch_parts(const std::vector<const MemberDesc*>& mem, Phase ph, bool fp64);

// Members (their indices, in order) dealt to at most `most` independent chains of
// about equal points, members of one (nx, ny) together.
std::vector<std::vector<int>> deal_chains(const std::vector<const MemberDesc*>& mem, int most);

// Rows per lane of the lanes-per-column tridiagonal kernel for nz rows on P lanes:
// the smallest compiled row count (2..8, 10, 12, 16) that covers them, 0 if none.
int tri_rows(int nz, int P);
// Its automatic lanes per column beside a column count asked for (0: none), and
// its automatic columns per workgroup with P lanes a column.
int tri_lanes(int nz, int columns, bool fp64);
int tri_columns(int ny, int nxh, int P);
// Its tiles that the autotuner times: every lane count of at least two rows a lane
// with its automatic columns, then for the lanes chosen the column counts.
struct TriTile {
  int lanes, columns;
};
std::vector<TriTile> tri_lane_tiles(int nz, int ny, int nxh);
std::vector<int> tri_column_values(int ny, int nxh, int P);

// Waves and rows per wave of the wave-per-chunk tridiagonal kernel for a plan of
// FP32 storage with nz levels and `tiles` tiles of 64 columns, or 0 where the
// lanes-per-column kernel is the better one.
void tricol_shape(int nz, long long tiles, int* waves, int* rows);

}  // namespace monc
