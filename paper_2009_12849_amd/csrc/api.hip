// C ABI of the projection library: plans, the single and batched projection,
// stage-wise access, per-kernel profiling and the autotuner.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/monc.h"
#include "kernels.h"
#include "krylov.h"
#include "launch_shape.h"
#include "monc_types.h"
#include "plan_math.h"

using namespace monc;

// ---------------------------------------------------------------------------
// errors
// ---------------------------------------------------------------------------
static thread_local std::string g_err;

static int fail(int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  std::vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return code;
}

#define HIP_TRY(expr)                                                                    \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess) return fail(MONC_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

// ---------------------------------------------------------------------------
// profiler: HIP event pairs around the launches of selected kernels
// ---------------------------------------------------------------------------
struct Profiler {
  unsigned mask = 0;
  struct Rec {
    int id;
    hipEvent_t a, b;
  };
  std::vector<Rec> recs;
  std::vector<hipEvent_t> pool;
  std::mutex mu;

  hipEvent_t get() {
    if (!pool.empty()) {
      hipEvent_t e = pool.back();
      pool.pop_back();
      return e;
    }
    hipEvent_t e = nullptr;
    if (hipEventCreate(&e) != hipSuccess) return nullptr;
    return e;
  }
  ~Profiler() {
    for (auto& r : recs) {
      (void)hipEventDestroy(r.a);
      (void)hipEventDestroy(r.b);
    }
    for (auto e : pool) (void)hipEventDestroy(e);
  }
};

// ---------------------------------------------------------------------------
// plan
// ---------------------------------------------------------------------------
static std::atomic<unsigned long long> g_plan_ids{1};
static std::once_flag g_attr_once;

struct monc_plan {
  unsigned long long id = 0;
  unsigned long long version = 0;  // bumped when tile parameters change
  int nx = 0, ny = 0, nz = 0, dtype = 0, device = 0;
  double dx = 0, dy = 0;
  std::vector<double> dz, rho0;
  int ex = 8, ey = 8, ymt = 0, triP = 0, tricw = 0, xpw = 0, yept = 0;  // tile parameters (0 = automatic)
  MemberDesc h{};                          // host copy with device pointers
  MemberDesc* d_desc = nullptr;            // device copy
  void* d_tables = nullptr;
  void* d_spec = nullptr;
  float* d_s1 = nullptr;     // mixed path scratch: divergence, then the correction
  float* d_s2 = nullptr;     // mixed path scratch: first-pass pressure
  size_t spec_elems = 0;
  void* d_var = nullptr;     // work vectors of monc_project_var (allocated at its first call)
  MemberDesc h_pre{};        // the preconditioner's descriptor: h plus the solver's done flag
  Profiler prof;
};

static size_t elem_bytes(int dtype) { return dtype == MONC_FP64 ? 8 : 4; }
static size_t cplx_bytes(int dtype) { return 2 * elem_bytes(dtype); }

static int pow2_floor(int x) {
  int p = 1;
  while (p * 2 <= x) p *= 2;
  return p;
}

// Default y-FFT columns per workgroup: 128 bytes of a row below length 256. From
// there on the tile's LDS (columns * ny * cb) sets how many workgroups a CU holds,
// and four columns pay (whole projection, us, against 128 bytes: FP64 1024^2 x 96
// 3180 -> 3010, 432^2 x 32 185 -> 173, 256^2 x 128 237 -> 230, 128 x 768 x 32 112 ->
// 101, equal at 243^2 x 48 and 128^2 x 64, 32^3 25.5 -> 26.8; FP32 256^2 x 128 242 ->
// 234, 384 x 256 x 96 284 -> 280, 512^2 x 96 676 -> 673, 64^2 x 32 55.3 -> 56.7) until
// the shorter runs cost the x kernels and the column solve as much: FP32 from
// length 1024 on keeps eight (with four 1024^2 x 96 1.6 % slower, 2048^2 x 160 0.5 % faster)
// where these fill the CUs twice (96 x 2048 x 16 does not: 171 -> 157 with four).
static int y_columns(int nx, int ny, int nz, int cb) {
  if (ny < 256) return 128 / cb;
  if (cb == 16 || ny < 1024) return 4;
  return (long long)nz * ((nx / 2 + 8) / 8) >= 512 ? 8 : 4;
}

// Default transforms (of nt threads) per workgroup of the x kernels: 256 threads'
// worth; where that leaves fewer than eight workgroups a CU, the fewest that fill
// nine tenths of their waves (x kernels' sum, us, 256 threads -> these: 32^3 FP64
// 15.7 -> 14.6 and mixed 25.5 -> 22.9, 64^2 x 32 mixed 32.8 -> 28.9, 96^2 x 48 FP64
// 23.9 -> 20.6, 256^2 x 16 mixed 33.8 -> 32.1; equal at 256^2 x 128). A mixed plan
// whose residual walks whole rows per wave takes whole-wave counts (its workgroups
// would be rounded up to one: 384 x 256 x 96 63 -> 50 us).
static int x_transforms(int nx, long long pairs, int nt, bool fp64) {
  int m = std::max(1, 256 / nt);
  if (pairs < 2048LL * m)
    for (int k = 1; k < m; ++k)
      if (k * nt * 10 >= (k * nt + 63) / 64 * 64 * 9) m = k;
  const int w = wave_transforms(nt);
  return !fp64 && xres_wave_rows(nx) && m > w ? m / w * w : m;
}

// Derive FFT plans and tile parameters from (ex, ey, ymt, triP, tricw, xpw,
// yept); 0 = default.
static int configure_tiles(monc_plan* pl, int ex, int ey, int ymt, int triP, int tricw, int xpw, int yept) {
  MemberDesc& h = pl->h;
  FftPlan fx{}, fy{};
  if (!radix_plan(pl->nx, fx) || !radix_plan(pl->ny, fy))
    return fail(MONC_EUNSUPPORTED, "no radix plan for nx=%d ny=%d", pl->nx, pl->ny);
  if (ex <= 0) ex = pl->ex;
  if (ey <= 0) ey = pl->ey;
  if (ex > kGenericElems || ey > kGenericElems)
    return fail(MONC_EINVAL, "elements per thread must be <= %d (got %d, %d)", kGenericElems, ex, ey);
  if (!fft_threads(fx, ex) || !fft_threads(fy, ey))
    return fail(MONC_EUNSUPPORTED, "FFT of nx=%d or ny=%d needs more than 1024 threads", pl->nx, pl->ny);
  const size_t cb = cplx_bytes(pl->dtype);
  // elements per thread of the compile-time y-FFT (its radix plan): 8 or 16,
  // or 32 = the persistent FP32 kernel (mixed plans, lengths of
  // pp_supported)
  if (yept <= 0) yept = pl->yept;
  if (yept != 0 && yept != 8 && yept != 16 && yept != 32)
    return fail(MONC_EINVAL, "y-FFT elements per thread must be 8, 16 or 32 (got %d)", yept);
  if (yept == 32 && (pl->dtype == MONC_FP64 || !pp_supported(pl->ny)))
    return fail(MONC_EINVAL, "32 y-FFT elements per thread (the persistent kernel) need a mixed plan and ny of "
                             "1024, 1536, 2048 or 4096 (got ny=%d)", pl->ny);
  const int yeff = yept > 0 ? yept : ct_yept_default(pl->ny);
  // y-FFT columns per workgroup (also the width of the spectral column
  // blocks, up to 8): y_columns by default, bounded by the workgroup size
  // (1024) and 128 KB of LDS
  const int nty = ct_supported(pl->ny) ? ct_threads_y_host(pl->ny, yeff) : fy.nt;
  if (nty > 1024)
    return fail(MONC_EUNSUPPORTED, "a %d-point y-FFT with %d elements per thread needs more than 1024 threads", pl->ny,
                yeff);
  const int mt_cap = std::max(1, std::min(1024 / nty, (int)(131072 / (pl->ny * cb))));
  if (ymt <= 0) ymt = pl->ymt > 0 ? pl->ymt : y_columns(pl->nx, pl->ny, pl->nz, (int)cb);
  if (ymt > 64) return fail(MONC_EINVAL, "y-FFT columns per workgroup must be <= 64 (got %d)", ymt);
  ymt = std::max(1, std::min(ymt, mt_cap));
  const int nxh = pl->nx / 2 + 1;
  ymt = std::min(ymt, pow2_floor(nxh) * 2);
  // tridiagonal lanes per column and columns per workgroup (0 = automatic)
  if (triP <= 0) triP = pl->triP;
  if (tricw <= 0) tricw = pl->tricw;
  const int lanes = triP > 0 ? triP : tri_lanes(pl->nz, tricw, pl->dtype == MONC_FP64);
  if (lanes & (lanes - 1) || lanes > kTriPmax)
    return fail(MONC_EINVAL, "tridiagonal lanes per column must be a power of 2 <= %d (got %d)", kTriPmax, lanes);
  const int s = tri_rows(pl->nz, lanes);
  if (s == 0)
    return fail(MONC_EINVAL, "%d lanes leave %d rows per lane (max %d)", lanes, (pl->nz + lanes - 1) / lanes, kTriSmax);
  const int cw = tricw > 0 ? tricw : tri_columns(pl->ny, nxh, lanes);
  if (cw & (cw - 1) || cw * lanes > 512)
    return fail(MONC_EINVAL, "tridiagonal columns per workgroup must be a power of 2 with %d lanes <= 512 threads (got %d)",
                lanes, cw);
  // x transforms per workgroup of the compile-time x kernels (default:
  // x_transforms); at most 512 threads and 160 KB of LDS
  if (xpw <= 0) xpw = pl->xpw;
  int xeff = 1;
  if (ct_supported(pl->nx)) {
    const int nt = ct_threads_host(pl->nx, (int)cb / 2), ntr = ct_threads_x_request(pl->nx);
    const size_t per = (size_t)xlds_len(pl->nx, (int)cb) * cb;
    xeff = xpw > 0 ? xpw : x_transforms(pl->nx, ((long long)pl->ny * pl->nz + 1) / 2, nt, pl->dtype == MONC_FP64);
    // lengths with a radix plan of their own take any request, clamped
    if (ct_plan_index(pl->nx) >= 0)
      xeff = (int)std::min<size_t>(xeff, std::max<size_t>(1, std::min<size_t>(512 / nt, (160 * 1024) / per)));
    // the others as many as 512 threads of ct_threads_x_request hold, of which a
    // launch takes what its own 512 threads hold (512 threads of at most sixteen
    // elements are within the LDS)
    if (xeff * ntr > 512)
      return fail(MONC_EINVAL, "%d x transforms of %d points per workgroup exceed 512 threads or 160 KB of LDS", xeff,
                  pl->nx);
  }
  pl->ex = ex;
  pl->ey = ey;
  pl->ymt = ymt;
  pl->xpw = xpw;
  h.xpw = xeff;
  pl->yept = yept;
  h.yept = yeff;
  // spectral column blocks as wide as a y-FFT tile (up to kSpecBlockMax), so
  // that the tile is one contiguous run of each level
  h.sbw = std::min(kSpecBlockMax, pow2_floor(ymt));
  h.lbw = 0;
  while ((1 << h.lbw) < h.sbw) ++h.lbw;
  h.bst = pl->ny * h.sbw;
  div_magic((unsigned)h.bst, h.bst_mul, h.bst_shift);
  pl->triP = triP;
  pl->tricw = tricw;
  h.fx = fx;
  h.fy = fy;
  h.ymt = ymt;
  h.triP = lanes;
  h.tris = s;
  h.tricw = cw;
  h.tcwaves = h.tcrows = 0;
  if (pl->dtype != MONC_FP64)
    tricol_shape(pl->nz, ((long long)pl->ny * h.nxp + 63) / 64, &h.tcwaves, &h.tcrows);
  return MONC_OK;
}

static int upload_desc(monc_plan* pl) {
  HIP_TRY(hipMemcpy(pl->d_desc, &pl->h, sizeof(MemberDesc), hipMemcpyHostToDevice));
  return MONC_OK;
}

// ---------------------------------------------------------------------------
// tuning cache (flat JSON object: "arch:nx,ny,nz:dtype" -> [ex, ey, ymt, triP, tricw, xpw, yept];
// entries without the last value read it as 0, the default)
// ---------------------------------------------------------------------------
static std::mutex g_cache_mu;

static std::string cache_key(const monc_plan* pl) {
  char buf[128];
  std::snprintf(buf, sizeof buf, "gfx950:%d,%d,%d:%s", pl->nx, pl->ny, pl->nz,
                pl->dtype == MONC_FP64 ? "fp64" : "mixed");
  return buf;
}

static std::map<std::string, std::vector<int>> read_cache(const char* path) {
  std::map<std::string, std::vector<int>> out;
  FILE* f = std::fopen(path, "r");
  if (!f) return out;
  std::string s;
  char buf[4096];
  size_t n;
  while ((n = std::fread(buf, 1, sizeof buf, f)) > 0) s.append(buf, n);
  std::fclose(f);
  size_t pos = 0;
  while ((pos = s.find('"', pos)) != std::string::npos) {
    const size_t end = s.find('"', pos + 1);
    if (end == std::string::npos) break;
    std::string key = s.substr(pos + 1, end - pos - 1);
    const size_t lb = s.find('[', end), rb = s.find(']', end);
    if (lb == std::string::npos || rb == std::string::npos || rb < lb) break;
    std::vector<int> vals;
    const char* p = s.c_str() + lb + 1;
    while (p < s.c_str() + rb) {
      char* q = nullptr;
      long v = std::strtol(p, &q, 10);
      if (q == p) { ++p; continue; }
      vals.push_back((int)v);
      p = q;
    }
    out[key] = vals;
    pos = rb + 1;
  }
  return out;
}

static void write_cache(const char* path, const std::map<std::string, std::vector<int>>& m) {
  std::string tmp = std::string(path) + ".tmp";
  FILE* f = std::fopen(tmp.c_str(), "w");
  if (!f) return;
  std::fprintf(f, "{\n");
  size_t i = 0;
  for (auto& kv : m) {
    std::fprintf(f, "  \"%s\": [", kv.first.c_str());
    for (size_t j = 0; j < kv.second.size(); ++j) std::fprintf(f, "%s%d", j ? ", " : "", kv.second[j]);
    std::fprintf(f, "]%s\n", ++i < m.size() ? "," : "");
  }
  std::fprintf(f, "}\n");
  std::fclose(f);
  std::rename(tmp.c_str(), path);
}

// ---------------------------------------------------------------------------
// static workspace of the allocation-free entry point (monc_project_noalloc)
// ---------------------------------------------------------------------------
// One array per GPU, held until the process ends. In host code the name
// `scratch` only stands for the symbol: its device address (different on
// every device) comes from hipGetSymbolAddress, resolved once per device with
// that device current and kept in g_scratch_ptr.
static constexpr size_t kStaticScratchBytes = (size_t)128 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
static constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

// Device address of the static workspace on the current device.
static int static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return fail(MONC_EHIP, "hipGetDevice failed");
  if (dev < 0 || dev >= kMaxDevices) return fail(MONC_EUNSUPPORTED, "device %d is beyond the %d supported", dev, kMaxDevices);
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !ptr)
      return fail(MONC_EHIP, "hipGetSymbolAddress of the static workspace failed on device %d: %s", dev,
                  hipGetErrorString(e));
    g_scratch_ptr[dev] = ptr;
  }
  *out = g_scratch_ptr[dev];
  return MONC_OK;
}

// ---------------------------------------------------------------------------
// plan creation
// ---------------------------------------------------------------------------
extern "C" monc_plan* monc_plan_create(int nx, int ny, int nz, double dx, double dy, const double* dz,
                                       const double* rho0, int dtype) {
  std::string err;
  const int rc = check_plan_args(nx, ny, nz, dx, dy, dz, rho0, dtype, err);
  if (rc != MONC_OK) {
    g_err = err;
    return nullptr;
  }
  auto pl = std::make_unique<monc_plan>();
  pl->id = g_plan_ids.fetch_add(1);
  pl->nx = nx;
  pl->ny = ny;
  pl->nz = nz;
  pl->dx = dx;
  pl->dy = dy;
  pl->dtype = dtype;
  pl->dz.assign(dz, dz + nz);
  pl->rho0.assign(rho0, rho0 + nz);
  MemberDesc& h = pl->h;
  h.nx = nx;
  h.ny = ny;
  h.nz = nz;
  h.nxh = nx / 2 + 1;
  h.nxp = (h.nxh + kSpecBlockMax - 1) / kSpecBlockMax * kSpecBlockMax;
  h.dtype = dtype;
  h.nrow = (long long)nz * ny;
  div_magic((unsigned)nx, h.nx_mul, h.nx_shift);
  div_magic((unsigned)ny, h.ny_mul, h.ny_shift);
  div_magic((unsigned)nx * (unsigned)ny, h.nh_mul, h.nh_shift);
  // spectral level stride: an odd multiple of 256 bytes, so that the
  // tridiagonal solver's walk down a column does not revisit one HBM channel
  h.plane = (long long)ny * h.nxp;
  {
    const long long cbytes = (long long)cplx_bytes(dtype);
    if (((h.plane * cbytes) / 256) % 2 == 0) h.plane += 256 / cbytes;
  }
  h.rdx = 1.0 / dx;
  h.rdy = 1.0 / dy;
  h.inv_nxny = 1.0 / ((double)nx * (double)ny);
  // stencil kernels walk (8 level x J row pair) tiles once a level of one
  // field outgrows an XCD's L2 share (4 MB); smaller grids stay in row order.
  // The x-forward kernels take J row pairs of about 512 KB per level and
  // field (8 to 64 pairs: 64 at 1024 FP32 points a row, 32 at 2048 FP32 or
  // 1024 FP64, 16 at 2048 FP64 or 4096 FP32, 8 at 4096 FP64), the gradient
  // J = 8 rows: each workgroup writes its spectral bins as short runs spread
  // over the level, which a tile whose J pairs run at about the same time
  // turns into longer runs, while the neighbour rows its stencil re-reads
  // must still meet in L2. At 2048^2 x 160 (mixed) 32 pairs against 8: the
  // divergence 2.47 -> 2.31 ms and the residual 3.45 -> 3.30 ms; 64 pairs
  // were as fast but re-read 15-20 % more from HBM (traffic over
  // algorithmic bytes 1.21 / 1.60 against 1.07 / 1.34).
  h.ptk = ((double)nx * ny * elem_bytes(dtype) >= 4.0 * (1 << 20)) ? 8 : 1;
  {
    const double pair_bytes = 2.0 * nx * elem_bytes(dtype);
    int j = 8;
    while (j < 64 && 2 * j * pair_bytes <= (double)(1 << 19)) j *= 2;
    h.ptj = j;
  }
  h.rdxf = (float)h.rdx;
  h.rdyf = (float)h.rdy;
  // tile parameters (cached tuning first)
  int ex = 0, ey = 0, ymt = 0, triP = 0, tricw = 0, xpw = 0, yept = 0;
  if (const char* path = std::getenv("MONC_TUNE_CACHE")) {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto m = read_cache(path);
    auto it = m.find(cache_key(pl.get()));
    if (it != m.end() && (it->second.size() == MONC_NPARAMS || it->second.size() == MONC_NPARAMS - 1)) {
      ex = it->second[0];
      ey = it->second[1];
      ymt = it->second[2];
      triP = it->second[3];
      tricw = it->second[4];
      xpw = it->second[5];
      yept = it->second.size() > 6 ? it->second[6] : 0;
    }
  }
  if (configure_tiles(pl.get(), ex, ey, ymt, triP, tricw, xpw, yept) != MONC_OK &&
      configure_tiles(pl.get(), 8, 8, 0, 0, 0, 0, 0) != MONC_OK)
    return nullptr;

  // host tables
  VerticalTables vt = vertical_tables(nz, dz, rho0);
  h.rH = vt.rH;
  {
    double sr = 0.0, cmax = 0.0;
    for (int k = 0; k < nz; ++k) {
      sr += dz[k] * rho0[k];
      cmax = std::max(cmax, (vt.ta[k] + vt.tc[k]) / rho0[k]);
    }
    h.rSr = 1.0 / sr;
    // a column with lam >= 1e-4 max_k (a_k + c_k)/rho0_k has a condition
    // number below ~1e4 and gains nothing from the deflation
    h.lamdef = 1e-4 * cmax;
  }
  std::vector<double> lamx = modified_wavenumbers(nx, h.nxh, dx);
  std::vector<double> lamy = modified_wavenumbers(ny, ny, dy);
  std::vector<double> twx = twiddles(nx), twy = twiddles(ny);

  // one device blob for the tables: 3 FP64 vertical, the packed metrics,
  // lamx, lamy, twiddles in the storage precision
  const size_t eb = elem_bytes(dtype);
  auto al = [](size_t x) { return (x + 255) / 256 * 256; };
  size_t off = 0;
  const size_t o_v64 = off; off += al(3 * (size_t)nz * 8);
  const size_t o_lev = off; off += al((size_t)kLev64 * nz * 8);
  const size_t o_levf = off; off += al((size_t)kLev32 * nz * 4);
  const size_t o_lx = off; off += al((size_t)h.nxh * 8);
  const size_t o_ly = off; off += al((size_t)ny * 8);
  const size_t o_tx = off; off += al((size_t)nx * 2 * eb);
  const size_t o_ty = off; off += al((size_t)ny * 2 * eb);
  const size_t o_tr = off; off += al(3 * (size_t)(nz + kTriPmax) * 8);
  const size_t tables_bytes = off;
  std::vector<unsigned char> blob(tables_bytes, 0);
  double* v64 = reinterpret_cast<double*>(blob.data() + o_v64);
  const std::vector<double>* cols[3] = {&vt.rdz, &vt.rdzc, &vt.dz};
  for (int t = 0; t < 3; ++t) std::memcpy(v64 + (size_t)t * nz, cols[t]->data(), (size_t)nz * 8);
  double* lev = reinterpret_cast<double*>(blob.data() + o_lev);
  float* levf = reinterpret_cast<float*>(blob.data() + o_levf);
  for (int k = 0; k < nz; ++k) {
    const double l[kLev64] = {vt.rho0[k], vt.rdz[k], vt.rhow[k], k ? vt.rhow[k - 1] : 0.0,
                              vt.rdzc[k], k ? vt.rdzc[k - 1] : 0.0};
    for (int i = 0; i < kLev64; ++i) lev[kLev64 * k + i] = l[i];
    for (int i = 0; i < kLev32; ++i) levf[kLev32 * k + i] = (float)l[i];
  }
  std::memcpy(blob.data() + o_lx, lamx.data(), lamx.size() * 8);
  std::memcpy(blob.data() + o_ly, lamy.data(), lamy.size() * 8);
  auto put_tw = [&](size_t o, const std::vector<double>& tw) {
    if (dtype == MONC_FP64) {
      std::memcpy(blob.data() + o, tw.data(), tw.size() * 8);
    } else {
      float* f = reinterpret_cast<float*>(blob.data() + o);
      for (size_t i = 0; i < tw.size(); ++i) f[i] = (float)tw[i];
    }
  };
  put_tw(o_tx, twx);
  put_tw(o_ty, twy);
  {
    const size_t nt = (size_t)nz + kTriPmax;
    double* tr = reinterpret_cast<double*>(blob.data() + o_tr);
    for (size_t k = 0; k < nt; ++k) {
      const bool in = k < (size_t)nz;
      tr[k] = in ? vt.ta[k] : 1.0;
      tr[nt + k] = in ? vt.tc[k] : 0.0;
      tr[2 * nt + k] = in ? vt.rho0[k] : 0.0;
    }
  }

  // device side
  std::call_once(g_attr_once, [] { init_kernel_attributes(); });
  init_fft_attributes(nx);
  init_fft_attributes(ny);
  if (hipGetDevice(&pl->device) != hipSuccess) {
    fail(MONC_EHIP, "hipGetDevice failed (no usable HIP device)");
    return nullptr;
  }
  {
    // set-up of the allocation-free entry point on this device (its first
    // call retries and reports a failure)
    void* unused = nullptr;
    (void)static_scratch(&unused);
  }
  pl->spec_elems = (size_t)nz * h.plane;
  auto release = [&]() {
    if (pl->d_tables) (void)hipFree(pl->d_tables);
    if (pl->d_spec) (void)hipFree(pl->d_spec);
    if (pl->d_s1) (void)hipFree(pl->d_s1);
    if (pl->d_s2) (void)hipFree(pl->d_s2);
    if (pl->d_desc) (void)hipFree(pl->d_desc);
  };
  if (hipMalloc(&pl->d_tables, tables_bytes) != hipSuccess ||
      hipMalloc(&pl->d_spec, pl->spec_elems * cplx_bytes(dtype)) != hipSuccess ||
      hipMalloc((void**)&pl->d_desc, sizeof(MemberDesc)) != hipSuccess ||
      (dtype == MONC_MIXED &&
       (hipMalloc((void**)&pl->d_s1, (size_t)nx * ny * nz * sizeof(float)) != hipSuccess ||
        hipMalloc((void**)&pl->d_s2, (size_t)nx * ny * nz * sizeof(float)) != hipSuccess))) {
    (void)hipGetLastError();
    release();
    fail(MONC_ENOMEM, "device allocation failed for a %dx%dx%d plan", nx, ny, nz);
    return nullptr;
  }
  if (hipMemcpy(pl->d_tables, blob.data(), tables_bytes, hipMemcpyHostToDevice) != hipSuccess) {
    release();
    fail(MONC_EHIP, "table upload failed");
    return nullptr;
  }
  unsigned char* base = reinterpret_cast<unsigned char*>(pl->d_tables);
  const double* d64 = reinterpret_cast<const double*>(base + o_v64);
  h.rdz = d64;
  h.rdzc = d64 + nz;
  h.dz = d64 + 2 * (size_t)nz;
  h.tra = reinterpret_cast<const double*>(base + o_tr);
  h.trc = h.tra + nz + kTriPmax;
  h.trr = h.trc + nz + kTriPmax;
  h.lev = reinterpret_cast<const double*>(base + o_lev);
  h.levf = reinterpret_cast<const float*>(base + o_levf);
  h.lamx = reinterpret_cast<const double*>(base + o_lx);
  h.lamy = reinterpret_cast<const double*>(base + o_ly);
  h.twx = base + o_tx;
  h.twy = base + o_ty;
  h.spec = pl->d_spec;
  if (upload_desc(pl.get()) != MONC_OK) {
    release();
    return nullptr;
  }
  g_err.clear();
  return pl.release();
}

static void drop_batch_cache_for(unsigned long long plan_id);

extern "C" void monc_plan_destroy(monc_plan* pl) {
  if (!pl) return;
  drop_batch_cache_for(pl->id);
  if (pl->d_tables) (void)hipFree(pl->d_tables);
  if (pl->d_spec) (void)hipFree(pl->d_spec);
  if (pl->d_s1) (void)hipFree(pl->d_s1);
  if (pl->d_s2) (void)hipFree(pl->d_s2);
  if (pl->d_desc) (void)hipFree(pl->d_desc);
  if (pl->d_var) (void)hipFree(pl->d_var);
  delete pl;
}

extern "C" const char* monc_last_error(void) { return g_err.c_str(); }

extern "C" size_t monc_spectral_layout(const monc_plan* pl, int* row_len, int* col_block, long long* plane_len,
                                       int* eb) {
  if (!pl) return 0;
  if (row_len) *row_len = pl->h.nxp;
  if (col_block) *col_block = pl->h.sbw;
  if (plane_len) *plane_len = pl->h.plane;
  if (eb) *eb = (int)cplx_bytes(pl->dtype);
  return pl->spec_elems;
}

extern "C" const char* monc_kernel_name(int id) {
  static const char* names[MONC_K_COUNT] = {"div_fftx", "ffty_fwd",  "tridiag",    "ffty_inv",
                                            "ifftx",    "grad",      "resid_fftx", "grad_final"};
  if (id < 0 || id >= MONC_K_COUNT) return "";
  return names[id];
}

// ---------------------------------------------------------------------------
// grouped launches
// ---------------------------------------------------------------------------
struct GroupMember {
  const MemberDesc* h;  // host copy
  const MemberDesc* d;  // device copy
  IoPtrs io;
};

struct Group {
  std::vector<GroupMember> mem;
  bool fp64 = true;
};

static int phase_kernel_id(Phase ph) {
  switch (ph) {
    case PH_XFWD: case PH_XPRE: case PH_XPRE_UPDATE: case PH_LEVEL_FWD: return MONC_K_DIV_FFTX;
    case PH_RESID: case PH_LEVEL_RESID: return MONC_K_RESID_FFTX;
    case PH_YFWD: return MONC_K_FFTY_FWD;
    case PH_TRI: return MONC_K_TRIDIAG;
    case PH_YINV: return MONC_K_FFTY_INV;
    case PH_XINV: case PH_XINV_P1: case PH_XINV_CORR: case PH_XINV_DOTS: return MONC_K_IFFTX;
    case PH_LEVEL_INV: case PH_LEVEL_INV_P1: case PH_LEVEL_INV_CORR: return MONC_K_IFFTX;
    case PH_GRAD: return MONC_K_GRAD;
    case PH_GRAD_MIXED: return MONC_K_GRAD_FINAL;
  }
  return 0;
}


// compute units of the current device (queried once per device)
static int cu_count() {
  static std::atomic<int> cache[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cache[dev].load();
  if (n <= 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cache[dev].store(n);
  }
  return n;
}

// The n members idx of the group in one launch (sh: the first one's shape).
static int launch_one(const Group& g, const int* idx, int n, Phase ph, const Shape& sh, void* stream,
                      Profiler* prof) {
  LaunchArgs a;  // entries past the members are not read
  a.nmem = n;
  long long blocks = 0;
  size_t lds = 0;
  int block = sh.block;
  for (int t = 0; t < n; ++t) {
    const GroupMember& m = g.mem[idx[t]];
    const Shape s = t == 0 ? sh : member_shape(*m.h, ph, g.fp64);
    a.mem[t] = m.d;
    a.io[t] = m.io;
    a.block_start[t] = (int)blocks;
    blocks += s.blocks;
    lds = std::max(lds, s.lds);
    block = std::max(block, s.block);
    if (blocks > (1LL << 31) - 1) return fail(MONC_EUNSUPPORTED, "grid too large");
  }
  a.block_start[n] = (int)blocks;
  if (block > 1024) return fail(MONC_EUNSUPPORTED, "launch needs %d threads per workgroup", block);
  if (lds > 160 * 1024) return fail(MONC_EUNSUPPORTED, "phase needs %zu bytes of LDS", lds);
  if (blocks == 0) return MONC_OK;
  // a persistent kernel takes one workgroup per CU slot its LDS leaves
  const long long slots = (long long)cu_count() * (long long)std::max<size_t>(1, (160 * 1024) / std::max<size_t>(lds, 1));
  const int grid = sh.persistent ? (int)std::min(blocks, slots) : (int)blocks;
  const int kid = phase_kernel_id(ph);
  hipEvent_t e0 = nullptr, e1 = nullptr;
  const bool timed = prof && (prof->mask >> kid & 1u);
  if (timed) {
    std::lock_guard<std::mutex> lk(prof->mu);
    e0 = prof->get();
    e1 = prof->get();
    if (e0) (void)hipEventRecord(e0, (hipStream_t)stream);
  }
  const int v = sh.variant;
  switch (ph) {
    case PH_XFWD: launch_xfwd(a, grid, block, lds, g.fp64, 0, v, stream); break;
    case PH_XPRE: launch_xfwd(a, grid, block, lds, g.fp64, 2, v, stream); break;
    case PH_XPRE_UPDATE: launch_xfwd(a, grid, block, lds, g.fp64, 3, v, stream); break;
    case PH_RESID: launch_xfwd(a, grid, block, lds, false, 1, v, stream); break;
    case PH_YFWD: launch_ffty(a, grid, block, lds, g.fp64, false, v, g.mem[idx[0]].h->yept, stream); break;
    case PH_YINV: launch_ffty(a, grid, block, lds, g.fp64, true, v, g.mem[idx[0]].h->yept, stream); break;
    case PH_TRI:
      if (sh.sub == 2) launch_tricol(a, grid, block, lds, v, stream);
      else launch_tridiag(a, grid, block, lds, g.fp64, v, sh.sub != 0, stream); break;
    case PH_XINV: launch_xinv(a, grid, block, lds, g.fp64, 0, v, stream); break;
    case PH_LEVEL_FWD: launch_level_fwd(a, grid, block, lds, g.fp64, 0, stream); break;
    case PH_LEVEL_RESID: launch_level_fwd(a, grid, block, lds, false, 1, stream); break;
    case PH_LEVEL_INV: launch_level_inv(a, grid, block, lds, g.fp64, 0, stream); break;
    case PH_LEVEL_INV_P1: launch_level_inv(a, grid, block, lds, false, 2, stream); break;
    case PH_LEVEL_INV_CORR: launch_level_inv(a, grid, block, lds, false, 1, stream); break;
    case PH_XINV_P1: launch_xinv(a, grid, block, lds, false, 2, v, stream); break;
    case PH_XINV_DOTS: launch_xinv(a, grid, block, lds, g.fp64, 3, v, stream); break;
    case PH_XINV_CORR: launch_xinv(a, grid, block, lds, false, 1, v, stream); break;
    case PH_GRAD:
    case PH_GRAD_MIXED: {
      // per-level reductions of the outputs when the caller asked for them
      bool red = false;
      for (int t = 0; t < n; ++t)
        if (a.io[t].stats) {
          launch_stats_init(a.io[t].stats, g.mem[idx[t]].h->nz, stream);
          red = true;
        }
      launch_grad(a, grid, ph == PH_GRAD && g.fp64, v, red, stream);
      break;
    }
  }
  hipError_t le = hipGetLastError();
  if (timed) {
    std::lock_guard<std::mutex> lk(prof->mu);
    if (e1) (void)hipEventRecord(e1, (hipStream_t)stream);
    if (e0 && e1) prof->recs.push_back({kid, e0, e1});
  }
  if (le != hipSuccess) return fail(MONC_EHIP, "launch of %s failed: %s", monc_kernel_name(kid), hipGetErrorString(le));
  return MONC_OK;
}

// One phase for every member of the group, a launch per part.
static int launch_phase(const Group& g, Phase ph, void* stream, Profiler* prof) {
  if (g.mem.size() == 1) {
    const int only = 0;
    return launch_one(g, &only, 1, ph, member_shape(*g.mem[0].h, ph, g.fp64), stream, prof);
  }
  std::vector<const MemberDesc*> mem;
  for (const GroupMember& m : g.mem) mem.push_back(m.h);
  for (const LaunchPart& part : launch_parts(mem, ph, g.fp64)) {
    const int rc = launch_one(g, part.mem.data(), (int)part.mem.size(), ph, part.shape, stream, prof);
    if (rc != MONC_OK) return rc;
  }
  return MONC_OK;
}

static int run_phases(const std::vector<Group>& groups, const std::vector<Phase>& phases, void* stream,
                      Profiler* prof) {
  for (Phase ph : phases)
    for (const auto& g : groups) {
      const int rc = launch_phase(g, ph, stream, prof);
      if (rc != MONC_OK) return rc;
    }
  return MONC_OK;
}

static const std::vector<Phase>& full_sequence(bool fp64) {
  static const std::vector<Phase> f64 = {PH_XFWD, PH_YFWD, PH_TRI, PH_YINV, PH_XINV, PH_GRAD};
  // mixed: the first solve leaves p1 in s2; the residual D(u*) - L p1
  // (FP64) is solved for the correction delta (into s1); the gradient kernel
  // forms p1 + delta in FP64, corrects u, v, w with it and writes p
  static const std::vector<Phase> mixed = {PH_XFWD, PH_YFWD, PH_TRI, PH_YINV, PH_XINV_P1, PH_RESID,
                                           PH_YFWD, PH_TRI,  PH_YINV, PH_XINV_CORR, PH_GRAD_MIXED};
  return fp64 ? f64 : mixed;
}

// Whether one workgroup a level does both transforms of a plan (k_level_fwd,
// k_level_inv): FP32 up to 64 x 64 points, FP64 up to 1536 points a level, where
// the launches that it saves outweigh the CUs that it leaves idle. GPU time of a
// projection, us, separate / level kernels: mixed 16^3 36.5 / 32.0, 32^3 36.5 / 32.8,
// 48^3 44.6 / 41.5, 64^2 x 32 46.4 / 39.8, 64^2 x 256 82.8 / 65.7, but 72^2 x 32 47.5 /
// 50.8, 96^2 x 48 57 / 87; FP64 16^3 22.0 / 19.2, 32^3 22.0 / 20.7, 24 x 48 x 32 26.4 /
// 25.8, 32^2 x 512 40.6 / 37.6, but 54 x 36 x 20 24.6 / 29.1, 48^3 28.5 / 30.3, 64^2 x
// 32 23.8 / 27.2.
static bool level_fused(const MemberDesc& d, bool fp64) {
  return d.ny % 2 == 0 && level_length(d.nx, false) && level_length(d.ny, true) &&
         (!fp64 || d.nx * d.ny <= 1536) && (ct_plan_index(d.ny) >= 0 || d.yept == 8);
}

// The launches of one plan's projection: with the level kernels where these are
// the better ones, but each kernel by itself while its times are recorded (the
// results' bits are the same).
static const std::vector<Phase>& plan_sequence(const MemberDesc& d, bool fp64, const Profiler* prof) {
  static const std::vector<Phase> f64 = {PH_LEVEL_FWD, PH_TRI, PH_LEVEL_INV, PH_GRAD};
  static const std::vector<Phase> mixed = {PH_LEVEL_FWD, PH_TRI,            PH_LEVEL_INV_P1, PH_LEVEL_RESID,
                                           PH_TRI,       PH_LEVEL_INV_CORR, PH_GRAD_MIXED};
  if (prof || !level_fused(d, fp64)) return full_sequence(fp64);
  return fp64 ? f64 : mixed;
}

// The launch pointers of one member: caller fields, the plan's spectral
// workspace and (mixed plans) its two scratch fields.
static IoPtrs plan_io(const monc_plan* pl, void* u, void* v, void* w, void* p) {
  IoPtrs io;
  io.u = u;
  io.v = v;
  io.w = w;
  io.p = p;
  io.spec = pl->d_spec;
  io.s1 = pl->d_s1;
  io.s2 = pl->d_s2;
  return io;
}

// ---------------------------------------------------------------------------
// pointer checks
// ---------------------------------------------------------------------------
static int check_fields(const monc_plan* pl, void* const* ptrs, int n, const char* what) {
  const size_t bytes = (size_t)pl->nx * pl->ny * pl->nz * elem_bytes(pl->dtype);
  for (int i = 0; i < n; ++i) {
    if (!ptrs[i]) return fail(MONC_EINVAL, "%s: pointer %d is null", what, i);
    if (reinterpret_cast<uintptr_t>(ptrs[i]) % 16 != 0)
      return fail(MONC_EINVAL, "%s: pointer %d is not 16-byte aligned", what, i);
  }
  for (int i = 0; i < n; ++i)
    for (int j = i + 1; j < n; ++j) {
      const uintptr_t a = reinterpret_cast<uintptr_t>(ptrs[i]), b = reinterpret_cast<uintptr_t>(ptrs[j]);
      if (a < b + bytes && b < a + bytes) return fail(MONC_EINVAL, "%s: arrays %d and %d overlap", what, i, j);
    }
  return MONC_OK;
}

static int check_device(const monc_plan* pl) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return fail(MONC_EHIP, "hipGetDevice failed");
  if (dev != pl->device)
    return fail(MONC_EINVAL, "plan was created on device %d but device %d is current", pl->device, dev);
  return MONC_OK;
}

// ---------------------------------------------------------------------------
// single projection
// ---------------------------------------------------------------------------
extern "C" int monc_project(monc_plan* pl, void* u, void* v, void* w, void* p, void* stream) {
  if (!pl) return fail(MONC_EINVAL, "plan is null");
  void* ptrs[4] = {u, v, w, p};
  int rc = check_fields(pl, ptrs, 4, "monc_project");
  if (rc != MONC_OK) return rc;
  rc = check_device(pl);
  if (rc != MONC_OK) return rc;
  std::vector<Group> groups(1);
  Group& g = groups[0];
  g.fp64 = pl->dtype == MONC_FP64;
  g.mem.push_back({&pl->h, pl->d_desc, plan_io(pl, u, v, w, p)});
  Profiler* const prof = pl->prof.mask ? &pl->prof : nullptr;
  return run_phases(groups, plan_sequence(pl->h, g.fp64, prof), stream, prof);
}

extern "C" int monc_project_reduce(monc_plan* pl, void* u, void* v, void* w, void* p, double* stats,
                                   void* stream) {
  if (!pl) return fail(MONC_EINVAL, "plan is null");
  if (!stats || reinterpret_cast<uintptr_t>(stats) % 8 != 0) return fail(MONC_EINVAL, "stats is null or misaligned");
  void* ptrs[4] = {u, v, w, p};
  int rc = check_fields(pl, ptrs, 4, "monc_project_reduce");
  if (rc != MONC_OK) return rc;
  {
    const uintptr_t s0 = reinterpret_cast<uintptr_t>(stats), s1 = s0 + 8 * sizeof(double) * pl->nz;
    const size_t bytes = (size_t)pl->nx * pl->ny * pl->nz * elem_bytes(pl->dtype);
    for (int i = 0; i < 4; ++i) {
      const uintptr_t a = reinterpret_cast<uintptr_t>(ptrs[i]);
      if (a < s1 && s0 < a + bytes) return fail(MONC_EINVAL, "monc_project_reduce: stats overlaps array %d", i);
    }
  }
  rc = check_device(pl);
  if (rc != MONC_OK) return rc;
  std::vector<Group> groups(1);
  Group& g = groups[0];
  g.fp64 = pl->dtype == MONC_FP64;
  IoPtrs io = plan_io(pl, u, v, w, p);
  io.stats = stats;
  g.mem.push_back({&pl->h, pl->d_desc, io});
  Profiler* const prof = pl->prof.mask ? &pl->prof : nullptr;
  return run_phases(groups, plan_sequence(pl->h, g.fp64, prof), stream, prof);
}

// ---------------------------------------------------------------------------
// allocation-free projection
// ---------------------------------------------------------------------------
static size_t align256(size_t x);

extern "C" int monc_project_noalloc(monc_plan* pl, void* u, void* v, void* w, void* p, void* stream) {
  if (!pl) return fail(MONC_EINVAL, "plan is null");
  void* ptrs[4] = {u, v, w, p};
  int rc = check_fields(pl, ptrs, 4, "monc_project_noalloc");
  if (rc != MONC_OK) return rc;
  rc = check_device(pl);
  if (rc != MONC_OK) return rc;
  const bool fp64 = pl->dtype == MONC_FP64;
  const size_t spec = align256(pl->spec_elems * cplx_bytes(pl->dtype));
  const size_t field = align256((size_t)pl->nx * pl->ny * pl->nz * sizeof(float));
  const size_t need = spec + (fp64 ? 0 : 2 * field);
  if (need > kStaticScratchBytes)
    return fail(MONC_EUNSUPPORTED,
                "monc_project_noalloc: a %dx%dx%d %s plan needs %zu bytes of workspace, above the static %zu",
                pl->nx, pl->ny, pl->nz, fp64 ? "FP64" : "MIXED", need, kStaticScratchBytes);
  void* base = nullptr;
  rc = static_scratch(&base);
  if (rc != MONC_OK) return rc;
  // the plan's own workspace is not touched: every kernel takes its
  // workspace pointers from the launch arguments
  unsigned char* b = static_cast<unsigned char*>(base);
  IoPtrs io = plan_io(pl, u, v, w, p);
  io.spec = b;
  io.s1 = fp64 ? nullptr : reinterpret_cast<float*>(b + spec);
  io.s2 = fp64 ? nullptr : reinterpret_cast<float*>(b + spec + field);
  std::vector<Group> groups(1);
  groups[0].fp64 = fp64;
  groups[0].mem.push_back({&pl->h, pl->d_desc, io});
  return run_phases(groups, plan_sequence(pl->h, fp64, nullptr), stream, nullptr);  // no profiling events
}

// ---------------------------------------------------------------------------
// variable-density projection: preconditioned conjugate gradients
// ---------------------------------------------------------------------------
static constexpr int kVarMaxIt = 10000;

// Work vectors of one plan, carved from one allocation: r, d, q (FP64
// fields), z (storage type), two partial-sum arrays, the scalars (status
// row and one row per iteration), the vertical interpolation weights za, zb and
// the preconditioner's device descriptor.
struct VarWs {
  double *r, *d, *q, *part0, *part1, *scal, *za, *zb;
  void* z;
  MemberDesc* desc;
};

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static int var_workspace(monc_plan* pl, VarWs* ws) {
  const size_t n = (size_t)pl->nx * pl->ny * pl->nz;
  // partial sums: of the stencil kernels, the pointwise ones, and the x kernels
  // (at most one workgroup per row pair, whatever the tile parameters)
  const size_t nparts = (size_t)std::max({var_stencil_parts(pl->nx, pl->ny, pl->nz), var_point_parts(pl->nx, pl->ny, pl->nz),
                                          (pl->h.nrow + 1) / 2});
  constexpr int kParts = 10;
  const size_t sizes[kParts] = {n * 8, n * 8, n * 8, n * elem_bytes(pl->dtype), nparts * 8, nparts * 8,
                                (size_t)(kVarMaxIt + 2) * kVarSlots * 8, (size_t)pl->nz * 8, (size_t)pl->nz * 8,
                                sizeof(MemberDesc)};
  size_t off[kParts], total = 0;
  for (int i = 0; i < kParts; ++i) {
    off[i] = total;
    total += align256(sizes[i]);
  }
  if (!pl->d_var) {
    if (hipMalloc(&pl->d_var, total) != hipSuccess) {
      pl->d_var = nullptr;
      (void)hipGetLastError();
      return fail(MONC_ENOMEM, "monc_project_var: cannot allocate %zu bytes of work vectors", total);
    }
    std::vector<double> za, zb;
    face_weights(pl->nz, pl->dz.data(), za, zb);
    char* b = static_cast<char*>(pl->d_var);
    if (hipMemcpy(b + off[7], za.data(), pl->nz * 8, hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(b + off[8], zb.data(), pl->nz * 8, hipMemcpyHostToDevice) != hipSuccess) {
      (void)hipFree(pl->d_var);
      pl->d_var = nullptr;
      return fail(MONC_EHIP, "monc_project_var: upload of the interpolation weights failed");
    }
  }
  char* b = static_cast<char*>(pl->d_var);
  ws->r = reinterpret_cast<double*>(b + off[0]);
  ws->d = reinterpret_cast<double*>(b + off[1]);
  ws->q = reinterpret_cast<double*>(b + off[2]);
  ws->z = b + off[3];
  ws->part0 = reinterpret_cast<double*>(b + off[4]);
  ws->part1 = reinterpret_cast<double*>(b + off[5]);
  ws->scal = reinterpret_cast<double*>(b + off[6]);
  ws->za = reinterpret_cast<double*>(b + off[7]);
  ws->zb = reinterpret_cast<double*>(b + off[8]);
  ws->desc = reinterpret_cast<MemberDesc*>(b + off[9]);
  return MONC_OK;
}

static int read_scalars(const double* dev, double* host, int n, void* stream) {
  if (hipMemcpyAsync(host, dev, n * sizeof(double), hipMemcpyDeviceToHost, (hipStream_t)stream) != hipSuccess ||
      hipStreamSynchronize((hipStream_t)stream) != hipSuccess)
    return fail(MONC_EHIP, "monc_project_var: reading the solver's status failed: %s",
                hipGetErrorString(hipGetLastError()));
  return MONC_OK;
}

static int var_launched(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(MONC_EHIP, "monc_project_var: launch of %s failed: %s", what, hipGetErrorString(e));
  return MONC_OK;
}

extern "C" int monc_project_var(monc_plan* pl, const double* rho, double* u, double* v, double* w, double* p,
                                double tol, int maxit, int* iters, double* relres, void* stream) {
  if (!pl) return fail(MONC_EINVAL, "plan is null");
  if (!(tol >= 0.0) || !std::isfinite(tol)) return fail(MONC_EINVAL, "monc_project_var: tol must be finite and >= 0");
  if (maxit < 1 || maxit > kVarMaxIt)
    return fail(MONC_EINVAL, "monc_project_var: maxit must be in [1, %d], got %d", kVarMaxIt, maxit);
  {
    void* ptrs[5] = {const_cast<double*>(rho), u, v, w, p};
    const size_t bytes = (size_t)pl->nx * pl->ny * pl->nz * sizeof(double);
    for (int i = 0; i < 5; ++i) {
      if (!ptrs[i]) return fail(MONC_EINVAL, "monc_project_var: pointer %d is null", i);
      if (reinterpret_cast<uintptr_t>(ptrs[i]) % 16 != 0)
        return fail(MONC_EINVAL, "monc_project_var: pointer %d is not 16-byte aligned", i);
    }
    for (int i = 0; i < 5; ++i)
      for (int j = i + 1; j < 5; ++j) {
        const uintptr_t a = reinterpret_cast<uintptr_t>(ptrs[i]), b = reinterpret_cast<uintptr_t>(ptrs[j]);
        if (a < b + bytes && b < a + bytes) return fail(MONC_EINVAL, "monc_project_var: arrays %d and %d overlap", i, j);
      }
  }
  int rc = check_device(pl);
  if (rc != MONC_OK) return rc;
  VarWs ws;
  rc = var_workspace(pl, &ws);
  if (rc != MONC_OK) return rc;
  const MemberDesc& h = pl->h;
  VarGrid g;
  g.nx = pl->nx;
  g.ny = pl->ny;
  g.nz = pl->nz;
  g.rdx = 1.0 / pl->dx;
  g.rdy = 1.0 / pl->dy;
  g.rdx2 = g.rdx * g.rdx;
  g.rdy2 = g.rdy * g.rdy;
  g.rho = rho;
  g.dz = h.dz;
  g.rdz = h.rdz;
  g.rdzc = h.rdzc;
  g.za = ws.za;
  g.zb = ws.zb;
  const long long np_st = var_stencil_parts(pl->nx, pl->ny, pl->nz);  // partials of the stencil kernels
  const long long np_pt = var_point_parts(pl->nx, pl->ny, pl->nz);    // partials of the pointwise kernels
  const bool z64 = pl->dtype == MONC_FP64;
  Profiler* prof = pl->prof.mask ? &pl->prof : nullptr;

  // preconditioner z = M^-1 r: the plan's spectral solve with r as its
  // source, through a copy of the plan's descriptor that carries the
  // solver's done flag (queued iterations past convergence then cost only
  // their launches). Its first kernel also takes the residual's step and sums
  // <r, r>, its last one the inner products of z.
  pl->h_pre = pl->h;
  pl->h_pre.skip = ws.scal + kVarDone;
  if (hipMemcpyAsync(ws.desc, &pl->h_pre, sizeof(MemberDesc), hipMemcpyHostToDevice, (hipStream_t)stream) !=
      hipSuccess)
    return fail(MONC_EHIP, "monc_project_var: descriptor upload failed");
  std::vector<Group> pre(1);
  pre[0].fp64 = z64;
  pre[0].mem.push_back({&pl->h_pre, ws.desc, IoPtrs()});
  IoPtrs& pio = pre[0].mem[0].io;
  pio.u = ws.r;
  pio.p = ws.z;
  pio.spec = pl->d_spec;
  const long long np_up = member_shape(pl->h, PH_XPRE_UPDATE, z64).blocks;  // partials of the x kernels
  const long long np_dot = member_shape(pl->h, PH_XINV_DOTS, z64).blocks;
  const double tol2 = tol * tol;
  static const std::vector<Phase> source_seq = {PH_XPRE}, update_seq = {PH_XPRE_UPDATE},
                                  solve_seq = {PH_YFWD, PH_TRI, PH_YINV}, dots_seq = {PH_XINV_DOTS};
  // r_it = r_{it-1} - alpha q and its norm (sets the done flag), on the way
  // into the preconditioner's first transform; r_0 as it is
  auto residual = [&](int i) {
    if (i == 0) return run_phases(pre, source_seq, stream, prof);
    pio.v = ws.q;
    pio.w = ws.scal + var_slot(i - 1, kVarRZ);
    pio.stats = ws.part0;
    const int e = run_phases(pre, update_seq, stream, prof);
    if (e != MONC_OK) return e;
    launch_var_finish_rr(ws.part0, np_up, ws.scal, i, tol2, stream);
    return var_launched("the residual norm");
  };
  // the rest of z_it = M^-1 r_it, with <r_it, z_it> and <z_it, q_{it-1}>, then
  // p_it and d_it
  auto direction = [&](int i) {
    int e = run_phases(pre, solve_seq, stream, prof);
    if (e != MONC_OK) return e;
    // <z, q> only for the flexible update (FP32 preconditioner)
    const bool flex = i > 0 && !z64;
    pio.v = flex ? ws.q : nullptr;
    pio.w = ws.part1;
    pio.stats = ws.part0;
    if ((e = run_phases(pre, dots_seq, stream, prof)) != MONC_OK) return e;
    launch_var_finish(ws.part0, flex ? ws.part1 : nullptr, np_dot, ws.scal, var_slot(i, kVarRZ), var_slot(i, kVarZQ),
                      true, stream);
    if ((e = var_launched("the partial-sum reduction")) != MONC_OK) return e;
    launch_var_dir(g, ws.scal, i, ws.z, z64, ws.d, p, stream);
    return var_launched("the direction update");
  };
  // q = L d_it and <d_it, q>, then r_{it+1}
  auto step = [&](int i) {
    launch_var_apply(g, ws.scal, ws.d, ws.q, ws.part0, stream);
    int e = var_launched("the operator");
    if (e != MONC_OK) return e;
    launch_var_finish(ws.part0, nullptr, np_st, ws.scal, var_slot(i, kVarDQ), 0, true, stream);
    if ((e = var_launched("the partial-sum reduction")) != MONC_OK) return e;
    return residual(i + 1);
  };

  launch_var_zero(ws.scal, (maxit + 2) * kVarSlots, stream);
  launch_var_div(g, u, v, w, ws.r, p, ws.part0, stream);
  if ((rc = var_launched("the divergence")) != MONC_OK) return rc;
  // <r_0, r_0>, through the residual-norm reduction of iteration 0: it sets
  // the done flag when the input is already divergence-free (or tol >= 1) and
  // flags a non-finite input, so the host needs no read before the first
  // batch; a done flag makes the queued work of that batch return at once
  launch_var_finish_rr(ws.part0, np_st, ws.scal, 0, tol2, stream);
  if ((rc = var_launched("the partial-sum reduction")) != MONC_OK) return rc;
  int it = 0;
  double rel = 0.0;
  if ((rc = residual(0)) != MONC_OK || (rc = direction(0)) != MONC_OK) return rc;
  // Iterations are queued in batches and the status read once per batch;
  // the next batch's length is the iteration count that the convergence rate
  // seen so far predicts (at least 1, at most 32).
  int queued = 0, batch = 3;
  double rel_prev = 1.0;
  for (;;) {
    const int nb = std::min(batch, maxit - queued);
    for (int b = 0; b < nb; ++b, ++queued) {
      if ((rc = step(queued)) != MONC_OK) return rc;
      if (queued + 1 < maxit && (rc = direction(queued + 1)) != MONC_OK) return rc;
    }
    // the status row and iteration 0's row (<r_0, r_0>) in one read
    double st[2 * kVarSlots];
    if ((rc = read_scalars(ws.scal, st, 2 * kVarSlots, stream)) != MONC_OK) return rc;
    const double rr0 = st[var_slot(0, kVarRR)];
    it = (int)st[kVarLast];
    if (st[kVarDone] == 2.0) {
      if (it == 0) return fail(MONC_EINVAL, "monc_project_var: the divergence of the input is not finite");
      return fail(MONC_EINVAL, "monc_project_var: breakdown at iteration %d (is rho positive everywhere?)", it);
    }
    rel = rr0 > 0.0 ? std::sqrt(st[kVarLastRR] / rr0) : 0.0;
    if (st[kVarDone] != 0.0 || queued >= maxit) break;
    batch = krylov_batch(rel, rel_prev, nb, tol, 32);
    rel_prev = rel;
  }
  // the last step of p, then the gauge in FP64: subtract the dz-weighted mean of p (the constants are
  // the operator's null space, so the residual does not change; an FP32
  // preconditioner's rounding would otherwise leave a small mean in p)
  if (it > 0) {
    double wsum = 0.0;
    for (int k = 0; k < pl->nz; ++k) wsum += pl->dz[k];
    launch_var_wsum(g, ws.scal, it, ws.d, p, ws.part0, stream);
    if ((rc = var_launched("the gauge sum")) != MONC_OK) return rc;
    launch_var_finish(ws.part0, nullptr, np_pt, ws.scal, kVarGauge, 0, false, stream);
    if ((rc = var_launched("the partial-sum reduction")) != MONC_OK) return rc;
    launch_var_shift(g, ws.scal, kVarGauge, 1.0 / ((double)pl->nx * pl->ny * wsum), p, stream);
    if ((rc = var_launched("the gauge shift")) != MONC_OK) return rc;
  }
  if (iters) *iters = it;
  if (relres) *relres = rel;
  // u = u* - G p, w = 0 on the lid: the FP64 gradient kernel
  Group gr;
  gr.fp64 = true;
  gr.mem.push_back({&pl->h, pl->d_desc, plan_io(pl, u, v, w, p)});
  const std::vector<Group> grad_groups{gr};
  static const std::vector<Phase> grad_seq = {PH_GRAD};
  return run_phases(grad_groups, grad_seq, stream, prof);
}

// ---------------------------------------------------------------------------
// stage-wise access
// ---------------------------------------------------------------------------
extern "C" int monc_debug_stage(monc_plan* pl, int stage, void* const* bufs, int nbufs, void* stream) {
  if (!pl) return fail(MONC_EINVAL, "plan is null");
  if (!bufs) return fail(MONC_EINVAL, "bufs is null");
  int rc = check_device(pl);
  if (rc != MONC_OK) return rc;
  const bool fp64 = pl->dtype == MONC_FP64;
  auto need = [&](int n) { return nbufs == n ? MONC_OK : fail(MONC_EINVAL, "stage %d takes %d buffers (got %d)", stage, n, nbufs); };
  for (int i = 0; i < nbufs; ++i)
    if (!bufs[i] || reinterpret_cast<uintptr_t>(bufs[i]) % 16) return fail(MONC_EINVAL, "buffer %d is null or misaligned", i);
  IoPtrs io;
  std::vector<Phase> seq;
  switch (stage) {
    case MONC_STAGE_FORWARD:
      if ((rc = need(4))) return rc;
      io.u = bufs[0];
      io.v = bufs[1];
      io.w = bufs[2];
      io.spec = bufs[3];
      seq = {PH_XFWD, PH_YFWD};
      break;
    case MONC_STAGE_SOLVE:
      if ((rc = need(1))) return rc;
      io.spec = bufs[0];
      seq = {PH_TRI};
      break;
    case MONC_STAGE_INVERSE:
      if ((rc = need(2))) return rc;
      io.spec = bufs[0];
      io.p = bufs[1];
      seq = {PH_YINV, PH_XINV};
      break;
    case MONC_STAGE_GRADIENT:
      if ((rc = need(4))) return rc;
      if (!fp64) return fail(MONC_EINVAL, "the gradient stage takes an FP64 pressure (FP64 plans only)");
      io.u = bufs[1];
      io.v = bufs[2];
      io.w = bufs[3];
      io.p = bufs[0];
      seq = {PH_GRAD};
      break;
    case MONC_STAGE_RESIDUAL:
      if ((rc = need(5))) return rc;
      if (fp64) return fail(MONC_EINVAL, "the residual stage exists on MIXED plans only");
      io.u = bufs[0];
      io.v = bufs[1];
      io.w = bufs[2];
      io.s2 = static_cast<float*>(bufs[3]);
      io.spec = bufs[4];
      seq = {PH_RESID, PH_YFWD};
      break;
    default:
      return fail(MONC_EINVAL, "unknown stage %d", stage);
  }
  Group g;
  g.fp64 = fp64;
  g.mem.push_back({&pl->h, pl->d_desc, io});
  return run_phases({g}, seq, stream, nullptr);
}

// ---------------------------------------------------------------------------
// batched projection: grouped launches captured in a HIP graph
// ---------------------------------------------------------------------------
struct BatchEntry {
  std::vector<unsigned long long> key;
  std::vector<unsigned long long> plan_ids;
  hipGraphExec_t exec = nullptr;
  hipGraph_t graph = nullptr;
  unsigned long long last_use = 0;
  ~BatchEntry() {
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
  }
};

static std::mutex g_batch_mu;
static std::vector<std::unique_ptr<BatchEntry>> g_batches;
static unsigned long long g_batch_clock = 0;
static const size_t kBatchCacheSize = 8;

static void drop_batch_cache_for(unsigned long long plan_id) {
  std::lock_guard<std::mutex> lk(g_batch_mu);
  g_batches.erase(std::remove_if(g_batches.begin(), g_batches.end(),
                                 [&](const std::unique_ptr<BatchEntry>& e) {
                                   return std::find(e->plan_ids.begin(), e->plan_ids.end(), plan_id) !=
                                          e->plan_ids.end();
                                 }),
                  g_batches.end());
}

// ---------------------------------------------------------------------------
// batch schedule: member order and grouping (tuned by monc_autotune)
// ---------------------------------------------------------------------------
// order 0 puts the largest members first (their workgroups start first, the
// small ones fill the tail), order 1 the smallest first. budget_mb 0 runs
// every phase over all members (one launch per kernel instance and phase);
// otherwise members, in order, are packed into groups whose working set
// (fields, spectral workspace, scratch) stays under budget_mb MB, and the
// groups run one after the other, all phases of a group before the next, so
// that a group's intermediates can stay in the 256 MB Infinity Cache.
struct BatchSchedule {
  int order = 0;
  int budget_mb = 0;
  // most independent graph branches: of the groups with a budget, of the members
  // without (deal_chains); 0 (the default): one with a budget, MONC_MAX_BRANCHES without
  int branches = 0;
};

static std::mutex g_sched_mu;
static std::map<std::string, BatchSchedule> g_sched;

// Key of a batch for the tuned schedule: the multiset of member grids and
// the dtype (FNV-1a hash of the sorted grid list).
static std::string batch_key(monc_plan* const* plans, int count) {
  std::vector<std::string> grids;
  for (int i = 0; i < count; ++i) {
    char b[64];
    std::snprintf(b, sizeof b, "%d,%d,%d;", plans[i]->nx, plans[i]->ny, plans[i]->nz);
    grids.push_back(b);
  }
  std::sort(grids.begin(), grids.end());
  unsigned long long h = 1469598103934665603ull;
  for (const auto& g : grids)
    for (char c : g) {
      h ^= (unsigned char)c;
      h *= 1099511628211ull;
    }
  char key[128];
  std::snprintf(key, sizeof key, "gfx950:batch:%d:%016llx:%s", count, h,
                plans[0]->dtype == MONC_FP64 ? "fp64" : "mixed");
  return key;
}

static BatchSchedule lookup_schedule(monc_plan* const* plans, int count) {
  const std::string key = batch_key(plans, count);
  {
    std::lock_guard<std::mutex> lk(g_sched_mu);
    auto it = g_sched.find(key);
    if (it != g_sched.end()) return it->second;
  }
  BatchSchedule sc;
  if (const char* path = std::getenv("MONC_TUNE_CACHE")) {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto m = read_cache(path);
    auto it = m.find(key);
    // [order, budget_mb] or [order, budget_mb, branches]
    if (it != m.end() && (it->second.size() == 2 || it->second.size() == 3) &&
        (it->second[0] == 0 || it->second[0] == 1) && it->second[1] >= 0 &&
        (it->second.size() == 2 || (it->second[2] >= 1 && it->second[2] <= MONC_MAX_BRANCHES))) {
      sc.order = it->second[0];
      sc.budget_mb = it->second[1];
      // a file names the branches that a schedule has: one group's chains, dealt
      // automatically, are one where its members share their lengths
      sc.branches = it->second.size() == 3 && (sc.budget_mb > 0 || it->second[2] > 1) ? it->second[2] : 0;
    }
  }
  std::lock_guard<std::mutex> lk(g_sched_mu);
  g_sched[key] = sc;
  return sc;
}

static size_t member_bytes(const monc_plan* pl) {
  const size_t n = (size_t)pl->nx * pl->ny * pl->nz;
  return 4 * n * elem_bytes(pl->dtype) + pl->spec_elems * cplx_bytes(pl->dtype) +
         (pl->dtype == MONC_FP64 ? 0 : 2 * n * sizeof(float));
}

static std::vector<int> batch_order(monc_plan* const* plans, int count, int order) {
  std::vector<int> ord(count);
  for (int i = 0; i < count; ++i) ord[i] = i;
  std::stable_sort(ord.begin(), ord.end(), [&](int a, int b) {
    const long long pa = (long long)plans[a]->nx * plans[a]->ny * plans[a]->nz;
    const long long pb = (long long)plans[b]->nx * plans[b]->ny * plans[b]->nz;
    return order == 0 ? pa > pb : pa < pb;
  });
  return ord;
}

static void build_groups(monc_plan* const* plans, int count, void* const* u, void* const* v, void* const* w,
                         void* const* p, const std::vector<int>& ord, const BatchSchedule& sc, std::vector<Group>& groups) {
  groups.clear();
  const size_t budget = (size_t)sc.budget_mb << 20;
  Group g;
  g.fp64 = plans[0]->dtype == MONC_FP64;
  size_t used = 0;
  for (int t = 0; t < count; ++t) {
    const int i = ord[t];
    const size_t mb = member_bytes(plans[i]);
    if (budget && !g.mem.empty() && used + mb > budget) {
      groups.push_back(std::move(g));
      g = Group();
      g.fp64 = plans[0]->dtype == MONC_FP64;
      used = 0;
    }
    g.mem.push_back({&plans[i]->h, plans[i]->d_desc, plan_io(plans[i], u[i], v[i], w[i], p[i])});
    used += mb;
  }
  groups.push_back(std::move(g));
}

// The group's members as its chains.
static std::vector<Group> chain_groups(const Group& g, int most) {
  std::vector<const MemberDesc*> mem;
  for (const GroupMember& m : g.mem) mem.push_back(m.h);
  std::vector<Group> out;
  for (const std::vector<int>& chain : deal_chains(mem, most)) {
    out.emplace_back();
    out.back().fp64 = g.fp64;
    for (int i : chain) out.back().mem.push_back(g.mem[i]);
  }
  return out;
}

// The graph branches that the schedule asks for (of groups) or has (of chains).
static int schedule_branches(monc_plan* const* plans, int count, const BatchSchedule& sc) {
  if (sc.branches > 0) return sc.branches;
  if (sc.budget_mb > 0) return 1;
  std::vector<const MemberDesc*> mem;
  for (int i = 0; i < count; ++i) mem.push_back(&plans[i]->h);
  return (int)deal_chains(mem, MONC_MAX_BRANCHES).size();
}

// All phases of each group in turn. With side streams (a capture in progress
// on `stream`), group g goes to branch g mod (1 + side.size()): the captured
// graph then holds that many independent chains, which the device runs
// concurrently, so that one chain's small launches fill the tails and gaps
// another leaves. Without, the groups run one after the other on `stream`.
static int run_batch(const std::vector<Group>& groups, const std::vector<Phase>& seq, void* stream, Profiler* prof,
                     const std::vector<hipStream_t>& side = {}) {
  const size_t nb = 1 + std::min(side.size(), groups.size() ? groups.size() - 1 : 0);
  std::vector<hipEvent_t> ev;
  auto cleanup = [&]() {
    for (hipEvent_t e : ev) (void)hipEventDestroy(e);
  };
  if (nb > 1) {  // fork: the side streams start after what the main one holds
    hipEvent_t fork = nullptr;
    if (hipEventCreateWithFlags(&fork, hipEventDisableTiming) != hipSuccess)
      return fail(MONC_EHIP, "batch: event creation failed");
    ev.push_back(fork);
    bool ok = hipEventRecord(fork, (hipStream_t)stream) == hipSuccess;
    for (size_t b = 1; b < nb && ok; ++b) ok = hipStreamWaitEvent(side[b - 1], fork, 0) == hipSuccess;
    if (!ok) {
      cleanup();
      return fail(MONC_EHIP, "batch: fork of the graph branches failed");
    }
  }
  for (size_t gi = 0; gi < groups.size(); ++gi) {
    void* st = (gi % nb) ? (void*)side[gi % nb - 1] : stream;
    for (Phase ph : seq) {
      const int rc = launch_phase(groups[gi], ph, st, prof);
      if (rc != MONC_OK) {
        cleanup();
        return rc;
      }
    }
  }
  for (size_t b = 1; b < nb; ++b) {  // join
    hipEvent_t join = nullptr;
    if (hipEventCreateWithFlags(&join, hipEventDisableTiming) != hipSuccess) {
      cleanup();
      return fail(MONC_EHIP, "batch: event creation failed");
    }
    ev.push_back(join);
    if (hipEventRecord(join, side[b - 1]) != hipSuccess || hipStreamWaitEvent((hipStream_t)stream, join, 0) != hipSuccess) {
      cleanup();
      return fail(MONC_EHIP, "batch: join of the graph branches failed");
    }
  }
  cleanup();
  return MONC_OK;
}

static int check_batch(monc_plan* const* plans, int count, const char* what) {
  if (!plans) return fail(MONC_EINVAL, "%s: plans is null", what);
  if (count < 1 || count > MONC_MAX_BATCH)
    return fail(MONC_EINVAL, "%s: count must be in [1, %d] (got %d)", what, MONC_MAX_BATCH, count);
  for (int i = 0; i < count; ++i) {
    if (!plans[i]) return fail(MONC_EINVAL, "%s: plans[%d] is null", what, i);
    if (plans[i]->dtype != plans[0]->dtype) return fail(MONC_EINVAL, "batch mixes dtypes (member %d)", i);
    if (plans[i]->device != plans[0]->device) return fail(MONC_EINVAL, "batch spans devices (member %d)", i);
    for (int j = 0; j < i; ++j)
      if (plans[j] == plans[i]) return fail(MONC_EINVAL, "plan of member %d repeats member %d (one workspace per plan)", i, j);
  }
  return MONC_OK;
}

// The streams that batches are captured on (nothing runs on them): created
// once per device and used under g_batch_mu.
static hipStream_t g_capture[kMaxDevices][MONC_MAX_BRANCHES] = {};

static int capture_streams(int branches, hipStream_t* first, std::vector<hipStream_t>& side) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return fail(MONC_EHIP, "hipGetDevice failed");
  for (int b = 0; b < std::max(1, branches); ++b) {
    hipStream_t& s = g_capture[dev][b];
    if (!s && hipStreamCreateWithFlags(&s, hipStreamNonBlocking) != hipSuccess) {
      s = nullptr;
      return fail(MONC_EHIP, "batch: stream creation failed");
    }
    if (b == 0) *first = s;
    else side.push_back(s);
  }
  return MONC_OK;
}

// After a failed capture: its streams may be left in a broken state.
static void drop_capture_streams() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return;
  for (hipStream_t& s : g_capture[dev]) {
    if (s) (void)hipStreamDestroy(s);
    s = nullptr;
  }
}

extern "C" int monc_project_batched(monc_plan* const* plans, int count, void* const* u, void* const* v,
                                    void* const* w, void* const* p, void* stream) {
  if (!plans || !u || !v || !w || !p) return fail(MONC_EINVAL, "null argument array");
  int rc = check_batch(plans, count, "monc_project_batched");
  if (rc != MONC_OK) return rc;
  for (int i = 0; i < count; ++i) {
    void* ptrs[4] = {u[i], v[i], w[i], p[i]};
    char what[64];
    std::snprintf(what, sizeof what, "batch member %d", i);
    rc = check_fields(plans[i], ptrs, 4, what);
    if (rc != MONC_OK) return rc;
  }
  rc = check_device(plans[0]);
  if (rc != MONC_OK) return rc;
  const bool fp64 = plans[0]->dtype == MONC_FP64;
  Profiler* prof = plans[0]->prof.mask ? &plans[0]->prof : nullptr;
  const BatchSchedule sc = lookup_schedule(plans, count);
  const std::vector<int> ord = batch_order(plans, count, sc.order);

  // key: schedule, plan ids, versions and field pointers
  std::vector<unsigned long long> key;
  key.reserve(6 * count + 2);
  key.push_back((unsigned long long)sc.order);
  key.push_back((unsigned long long)sc.budget_mb);
  key.push_back((unsigned long long)sc.branches);
  for (int i = 0; i < count; ++i) {
    key.push_back(plans[i]->id);
    key.push_back(plans[i]->version);
    key.push_back((unsigned long long)(uintptr_t)u[i]);
    key.push_back((unsigned long long)(uintptr_t)v[i]);
    key.push_back((unsigned long long)(uintptr_t)w[i]);
    key.push_back((unsigned long long)(uintptr_t)p[i]);
  }
  std::lock_guard<std::mutex> lk(g_batch_mu);
  BatchEntry* ent = nullptr;
  for (auto& e : g_batches)
    if (e->key == key) ent = e.get();
  // A graph pays for its capture (0.3 to 0.8 ms for a few members) only when it
  // is replayed, so the first call over new pointers launches its phases
  // directly: a batch that is called once, or on fields that move, never
  // captures. So does a call while the caller captures the stream.
  const bool first = !ent;
  if (first) {
    auto e = std::make_unique<BatchEntry>();
    e->key = key;
    for (int i = 0; i < count; ++i) e->plan_ids.push_back(plans[i]->id);
    if (g_batches.size() >= kBatchCacheSize) {
      auto oldest = std::min_element(g_batches.begin(), g_batches.end(),
                                     [](const std::unique_ptr<BatchEntry>& a, const std::unique_ptr<BatchEntry>& b) {
                                       return a->last_use < b->last_use;
                                     });
      g_batches.erase(oldest);
    }
    ent = e.get();
    g_batches.push_back(std::move(e));
  }
  ent->last_use = ++g_batch_clock;
  std::vector<Group> groups;
  build_groups(plans, count, u, v, w, p, ord, sc, groups);
  const auto& seq = full_sequence(fp64);
  bool eager = prof || first;  // kernels are timed around direct launches
  if (!eager) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    eager = hipStreamIsCapturing((hipStream_t)stream, &cap) != hipSuccess || cap != hipStreamCaptureStatusNone;
    if (eager) (void)hipGetLastError();
  }
  if (eager) {
    if (sc.budget_mb == 0) return run_phases(groups, seq, stream, prof);
    return run_batch(groups, seq, stream, prof);
  }
  if (!ent->exec) {
    int branches = std::max(1, sc.branches);
    if (sc.budget_mb == 0) {  // one group: its chains
      groups = chain_groups(groups[0], sc.branches > 0 ? sc.branches : MONC_MAX_BRANCHES);
      branches = (int)groups.size();
    }
    // side streams of the capture: forked from the first and joined back into
    // it, so they record into the same graph
    std::vector<hipStream_t> side;
    hipStream_t cs = nullptr;
    rc = capture_streams(branches, &cs, side);
    if (rc != MONC_OK) return rc;
    hipError_t e = hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
      drop_capture_streams();
      return fail(MONC_EHIP, "hipStreamBeginCapture failed: %s", hipGetErrorString(e));
    }
    rc = run_batch(groups, seq, cs, nullptr, side);
    hipGraph_t graph = nullptr;
    e = hipStreamEndCapture(cs, &graph);
    if (rc != MONC_OK || e != hipSuccess) drop_capture_streams();
    if (rc != MONC_OK) {
      if (graph) (void)hipGraphDestroy(graph);
      return rc;
    }
    if (e != hipSuccess) return fail(MONC_EHIP, "hipStreamEndCapture failed: %s", hipGetErrorString(e));
    ent->graph = graph;
    HIP_TRY(hipGraphInstantiate(&ent->exec, graph, nullptr, nullptr, 0));
  }
  HIP_TRY(hipGraphLaunch(ent->exec, (hipStream_t)stream));
  return MONC_OK;
}

extern "C" int monc_batch_schedule(monc_plan* const* plans, int count, int* out) {
  int rc = check_batch(plans, count, "monc_batch_schedule");
  if (rc != MONC_OK) return rc;
  if (!out) return fail(MONC_EINVAL, "monc_batch_schedule: out is null");
  const BatchSchedule sc = lookup_schedule(plans, count);
  const std::vector<int> ord = batch_order(plans, count, sc.order);
  size_t used = 0;
  int ngroups = 1;
  const size_t budget = (size_t)sc.budget_mb << 20;
  for (int t = 0, n = 0; t < count; ++t, ++n) {
    const size_t mb = member_bytes(plans[ord[t]]);
    if (budget && n > 0 && used + mb > budget) {
      ++ngroups;
      used = 0;
    }
    used += mb;
  }
  out[0] = sc.order;
  out[1] = sc.budget_mb;
  out[2] = ngroups;
  out[3] = schedule_branches(plans, count, sc);
  return MONC_OK;
}

extern "C" int monc_batch_set_schedule(monc_plan* const* plans, int count, int order, int budget_mb,
                                       int branches) {
  int rc = check_batch(plans, count, "monc_batch_set_schedule");
  if (rc != MONC_OK) return rc;
  if (order != 0 && order != 1) return fail(MONC_EINVAL, "monc_batch_set_schedule: order must be 0 or 1 (got %d)", order);
  if (budget_mb < 0) return fail(MONC_EINVAL, "monc_batch_set_schedule: budget_mb must be >= 0 (got %d)", budget_mb);
  if (branches < 1 || branches > MONC_MAX_BRANCHES)
    return fail(MONC_EINVAL, "monc_batch_set_schedule: branches must be in [1, %d] (got %d)", MONC_MAX_BRANCHES,
                branches);
  BatchSchedule sc;
  sc.order = order;
  sc.budget_mb = budget_mb;
  sc.branches = branches;
  std::lock_guard<std::mutex> lk(g_sched_mu);
  g_sched[batch_key(plans, count)] = sc;
  return MONC_OK;
}

// ---------------------------------------------------------------------------
// profiling
// ---------------------------------------------------------------------------
extern "C" int monc_profile_enable(monc_plan* pl, unsigned mask) {
  if (!pl) return fail(MONC_EINVAL, "plan is null");
  std::lock_guard<std::mutex> lk(pl->prof.mu);
  pl->prof.mask = mask;
  return MONC_OK;
}

extern "C" int monc_profile_read(monc_plan* pl, double* ms, int* launches) {
  if (!pl) return fail(MONC_EINVAL, "plan is null");
  std::lock_guard<std::mutex> lk(pl->prof.mu);
  int rc = MONC_OK;
  for (auto& r : pl->prof.recs) {
    float t = 0.0f;
    if (hipEventSynchronize(r.b) != hipSuccess || hipEventElapsedTime(&t, r.a, r.b) != hipSuccess) {
      rc = fail(MONC_EHIP, "profiling event query failed");
    } else {
      if (ms) ms[r.id] += t;
      if (launches) launches[r.id] += 1;
    }
    pl->prof.pool.push_back(r.a);
    pl->prof.pool.push_back(r.b);
  }
  pl->prof.recs.clear();
  return rc;
}

// ---------------------------------------------------------------------------
// tile parameters and autotuning
// ---------------------------------------------------------------------------
extern "C" int monc_plan_params(const monc_plan* pl, int* out) {
  if (!pl || !out) return fail(MONC_EINVAL, "null argument");
  out[0] = pl->ex;
  out[1] = pl->ey;
  out[2] = pl->ymt;
  out[3] = pl->h.triP;
  out[4] = pl->h.tricw;
  out[5] = pl->h.xpw;
  out[6] = pl->h.yept;
  return MONC_OK;
}

extern "C" int monc_plan_set_params(monc_plan* pl, const int* in) {
  if (!pl || !in) return fail(MONC_EINVAL, "null argument");
  for (int i = 0; i < MONC_NPARAMS; ++i)
    if (in[i] < 0) return fail(MONC_EINVAL, "parameter %d is negative", i);
  const MemberDesc saved = pl->h;
  const int sv[MONC_NPARAMS] = {pl->ex, pl->ey, pl->ymt, pl->triP, pl->tricw, pl->xpw, pl->yept};
  int rc = configure_tiles(pl, in[0], in[1], in[2], in[3], in[4], in[5], in[6]);
  if (rc != MONC_OK) {
    pl->h = saved;
    pl->ex = sv[0]; pl->ey = sv[1]; pl->ymt = sv[2]; pl->triP = sv[3]; pl->tricw = sv[4]; pl->xpw = sv[5];
    pl->yept = sv[6];
    return rc;
  }
  HIP_TRY(hipDeviceSynchronize());  // in-flight work may still read the old descriptor
  rc = upload_desc(pl);
  if (rc == MONC_OK) ++pl->version;
  return rc;
}

// Tile parameters of one plan: time every candidate value of one parameter,
// all else fixed, one parameter after the other.
static int tune_plan(monc_plan* pl, void* stream) {
  int rc = check_device(pl);
  if (rc != MONC_OK) return rc;
  const size_t bytes = (size_t)pl->nx * pl->ny * pl->nz * elem_bytes(pl->dtype);
  void* buf[4] = {nullptr, nullptr, nullptr, nullptr};
  for (auto& b : buf) {
    if (hipMalloc(&b, bytes) != hipSuccess) {
      for (auto& c : buf) if (c) (void)hipFree(c);
      return fail(MONC_ENOMEM, "autotune scratch allocation failed");
    }
    (void)hipMemset(b, 0, bytes);
  }
  hipStream_t st = (hipStream_t)stream;
  const unsigned saved_mask = pl->prof.mask;
  // time every candidate value of one parameter, all else fixed; the cost of
  // a candidate is the summed time of the kernels that parameter shapes over
  // `reps` projections (enough for a few milliseconds of kernel time, so that
  // small grids are not ranked on noise)
  int reps = 4;
  auto measure = [&](const int* prm, unsigned kmask, double& cost) -> int {
    int r = monc_plan_set_params(pl, prm);
    if (r != MONC_OK) return r;
    pl->prof.mask = kmask;
    for (int it = 0; it < 2; ++it)
      if ((r = monc_project(pl, buf[0], buf[1], buf[2], buf[3], st)) != MONC_OK) return r;
    double ms[MONC_K_COUNT] = {0};
    int cnt[MONC_K_COUNT] = {0};
    monc_profile_read(pl, nullptr, nullptr);  // drop warm-up records
    for (int it = 0; it < reps; ++it)
      if ((r = monc_project(pl, buf[0], buf[1], buf[2], buf[3], st)) != MONC_OK) return r;
    if ((r = monc_profile_read(pl, ms, cnt)) != MONC_OK) return r;
    cost = 0.0;
    for (int k = 0; k < MONC_K_COUNT; ++k) cost += ms[k];
    return MONC_OK;
  };
  int best[MONC_NPARAMS] = {pl->ex, pl->ey, pl->ymt, pl->h.triP, pl->h.tricw, pl->h.xpw, pl->h.yept};
  {
    double whole = 0.0;
    const int r = measure(best, (1u << MONC_K_COUNT) - 1, whole);
    if (r != MONC_OK) {
      pl->prof.mask = saved_mask;
      for (auto& b : buf) (void)hipFree(b);
      return r;
    }
    const double per = whole / reps;  // ms per projection
    reps = per > 0.0 ? (int)std::min(64.0, std::max(4.0, std::ceil(3.0 / per))) : 4;
  }
  const unsigned xmask = (1u << MONC_K_DIV_FFTX) | (1u << MONC_K_IFFTX) | (1u << MONC_K_RESID_FFTX);
  const unsigned ymask = (1u << MONC_K_FFTY_FWD) | (1u << MONC_K_FFTY_INV);
  const unsigned tmask = 1u << MONC_K_TRIDIAG;
  struct Axis {
    int idx;
    std::vector<int> vals;
    unsigned mask;
  };
  // elements per thread only shape the runtime-length FFT kernels
  std::vector<Axis> axes;
  if (!ct_supported(pl->nx)) axes.push_back({0, {2, 4, 8}, xmask});
  if (!ct_supported(pl->ny)) axes.push_back({1, {2, 4, 8}, ymask});
  // the radix plan of the compile-time y-FFT (8 or 16 elements per thread;
  // on mixed plans of the lengths it covers also 32, the persistent kernel),
  // timed together with the y tile width, which it bounds (threads per
  // workgroup) and which sets the spectral column blocks that shape the x
  // kernels' spectral traffic
  if (ct_supported(pl->ny) && pl->ny >= 16) {
    if (pl->dtype != MONC_FP64 && pp_supported(pl->ny)) axes.push_back({6, {8, 16, 32}, ymask | xmask});
    else axes.push_back({6, {8, 16}, ymask | xmask});
  }
  axes.push_back({2, {1, 2, 4, 8, 16, 32}, ymask | xmask});
  std::vector<int> lanes;
  std::map<int, int> lane_columns;
  if (!pl->h.tcwaves) {  // the lanes-per-column tridiagonal kernel
    // each lane count with the columns of its automatic tile: a fixed column
    // count would time the others with more or fewer threads a workgroup, or
    // refuse them
    for (const TriTile& t : tri_lane_tiles(pl->nz, pl->ny, pl->h.nxh)) {
      lanes.push_back(t.lanes);
      lane_columns[t.lanes] = t.columns;
    }
    axes.push_back({3, lanes, tmask});
    axes.push_back({4, {}, tmask});  // its values follow from the lanes chosen
  }
  if (ct_supported(pl->nx)) axes.push_back({5, {1, 2, 4}, xmask});
  for (const auto& ax : axes) {
    double best_cost = 1e300;
    int best_val = best[ax.idx];
    for (int val : ax.idx == 4 ? tri_column_values(pl->ny, pl->h.nxh, best[3]) : ax.vals) {
      int prm[MONC_NPARAMS];
      std::copy(best, best + MONC_NPARAMS, prm);
      prm[ax.idx] = val;
      if (ax.idx == 3) prm[4] = lane_columns[val];
      double cost = 0.0;
      if (measure(prm, ax.mask, cost) != MONC_OK) continue;
      int eff[MONC_NPARAMS];
      monc_plan_params(pl, eff);
      if (eff[ax.idx] != val) continue;  // clamped to another candidate
      if (cost < best_cost) {
        best_cost = cost;
        best_val = val;
      }
    }
    best[ax.idx] = best_val;
    if (ax.idx == 3 && lane_columns.count(best_val)) best[4] = lane_columns[best_val];
  }
  pl->prof.mask = saved_mask;
  for (auto& b : buf) (void)hipFree(b);
  rc = monc_plan_set_params(pl, best);
  if (rc != MONC_OK) return rc;
  if (const char* path = std::getenv("MONC_TUNE_CACHE")) {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto m = read_cache(path);
    m[cache_key(pl)] = {pl->ex, pl->ey, pl->ymt, pl->triP, pl->tricw, pl->h.xpw, pl->h.yept};
    write_cache(path, m);
  }
  return MONC_OK;
}

// The batch schedule: every candidate (member order x grouping budget x
// branches of the groups; one group is dealt to its chains automatically) is
// captured and replayed on scratch fields; the fastest replays win.
static int tune_schedule(monc_plan* const* plans, int count, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  const size_t eb = elem_bytes(plans[0]->dtype);
  std::vector<void*> bufs;
  auto release = [&]() {
    for (void* b : bufs) (void)hipFree(b);
    bufs.clear();
  };
  std::vector<void*> f[4];
  for (int i = 0; i < count; ++i) {
    const size_t bytes = (size_t)plans[i]->nx * plans[i]->ny * plans[i]->nz * eb;
    for (int t = 0; t < 4; ++t) {
      void* b = nullptr;
      if (hipMalloc(&b, bytes) != hipSuccess) {
        (void)hipGetLastError();
        release();
        return fail(MONC_ENOMEM, "autotune: scratch fields for the batch do not fit");
      }
      (void)hipMemset(b, 0, bytes);
      bufs.push_back(b);
      f[t].push_back(b);
    }
  }
  hipEvent_t e0 = nullptr, e1 = nullptr;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    release();
    return fail(MONC_EHIP, "autotune: event creation failed");
  }
  size_t total = 0;
  for (int i = 0; i < count; ++i) total += member_bytes(plans[i]);
  const int budgets[] = {0, 1024, 512, 256, 128, 64};
  const int branch_counts[] = {1, 2, 4};
  auto store = [&](const BatchSchedule& sc) {
    std::lock_guard<std::mutex> lk(g_sched_mu);
    g_sched[batch_key(plans, count)] = sc;
  };
  BatchSchedule best;
  double best_ms = 1e300;
  int rc = MONC_OK;
  for (int order = 0; order < 2 && rc == MONC_OK; ++order)
    for (int budget : budgets)
      for (int branches : branch_counts) {
        if (rc != MONC_OK) break;
        if (budget && ((size_t)budget << 20) >= total) continue;  // one group anyway
        if (branches > 1 && !budget) continue;                     // one group: its chains
        if (branches > 1 && ((size_t)budget << 20) * (size_t)(branches - 1) >= total)
          continue;  // fewer groups than branches
        BatchSchedule sc;
        sc.order = order;
        sc.budget_mb = budget;
        sc.branches = budget ? branches : 0;
        store(sc);
        for (int r = 0; r < 3 && rc == MONC_OK; ++r)  // direct launches, capture and launch, one warm replay
          rc = monc_project_batched(plans, count, f[0].data(), f[1].data(), f[2].data(), f[3].data(), stream);
        if (rc != MONC_OK) break;
        const int reps = 5;
        (void)hipEventRecord(e0, st);
        for (int r = 0; r < reps && rc == MONC_OK; ++r)
          rc = monc_project_batched(plans, count, f[0].data(), f[1].data(), f[2].data(), f[3].data(), stream);
        (void)hipEventRecord(e1, st);
        float ms = 0.0f;
        if (rc == MONC_OK && (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess))
          rc = fail(MONC_EHIP, "autotune: event timing failed");
        if (rc == MONC_OK && ms < best_ms) {
          best_ms = ms;
          best = sc;
        }
      }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  // the candidates' graphs hold the scratch pointers: drop them with the fields
  if (hipStreamSynchronize(st) != hipSuccess && rc == MONC_OK) rc = fail(MONC_EHIP, "autotune: stream failed");
  for (int i = 0; i < count; ++i) drop_batch_cache_for(plans[i]->id);
  release();
  if (rc != MONC_OK) return rc;
  store(best);
  if (const char* path = std::getenv("MONC_TUNE_CACHE")) {
    std::lock_guard<std::mutex> lk(g_cache_mu);
    auto m = read_cache(path);
    m[batch_key(plans, count)] = {best.order, best.budget_mb, schedule_branches(plans, count, best)};
    write_cache(path, m);
  }
  return MONC_OK;
}

extern "C" int monc_autotune(monc_plan* const* plans, int count, void* stream) {
  int rc = check_batch(plans, count, "monc_autotune");
  if (rc != MONC_OK) return rc;
  // tile parameters: the first plan of every distinct grid is tuned, the
  // others of that grid take its parameters
  for (int i = 0; i < count; ++i) {
    int j = 0;
    while (j < i && !(plans[j]->nx == plans[i]->nx && plans[j]->ny == plans[i]->ny && plans[j]->nz == plans[i]->nz))
      ++j;
    if (j == i) {
      rc = tune_plan(plans[i], stream);
    } else {
      int prm[MONC_NPARAMS];
      monc_plan_params(plans[j], prm);
      rc = monc_plan_set_params(plans[i], prm);
    }
    if (rc != MONC_OK) return rc;
  }
  if (count == 1) return MONC_OK;
  return tune_schedule(plans, count, stream);
}
