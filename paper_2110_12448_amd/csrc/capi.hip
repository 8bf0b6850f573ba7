// capi.hip -- the C ABI of include/pf.h: parameter validation, workspace
// layout, state upload/download and the per-step launch sequence.
#include <float.h>
#include <math.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <memory>
#include <new>
#include <string>
#include <thread>
#include <tuple>
#include <utility>
#include <vector>

#include "pf_device.hpp"
#include "pf_internal.hpp"

using namespace pf;

namespace {

thread_local std::string g_err;

int fail(int code, const std::string &msg) {
  g_err = msg;
  return code;
}

}  // namespace

namespace pf {
int report_error(int code, const char *msg) { return fail(code, msg); }
}  // namespace pf

namespace {

#define PF_HIP(call)                                                          \
  do {                                                                        \
    hipError_t e_ = (call);                                                   \
    if (e_ != hipSuccess)                                                     \
      return fail(PF_ERR_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

// Run f(begin, end) over the pieces of [0, n) on up to kHostThreads threads
// (the caller's among them), at least `grain` items each; fewer than `least`
// pieces run in the calling thread alone.  The hand-over of the
// fields between the caller's FP64 arrays and the device's is bound by one
// core's conversions, page faults and tanh: with 8 threads pf_read_fields of
// 1024x2048 FP32 takes 3.9 ms instead of 11.0.  f must not throw.  A thread that cannot be
// started leaves its piece to the caller's.
constexpr size_t kHostThreads = 8;
template <typename F>
void host_parallel(size_t n, size_t grain, size_t least, F f) {
  size_t k = std::min(kHostThreads, n / grain);
  if (k < least) k = 1;
  if (k > 1) k = std::min<size_t>(k, std::max(1u, std::thread::hardware_concurrency()));
  if (k == 1) return f(0, n);
  auto piece = [&](size_t i) { f(n * i / k, n * (i + 1) / k); };
  std::thread th[kHostThreads];
  size_t started = 0;
  try {
    for (; started + 1 < k; ++started) th[started] = std::thread(piece, started);
  } catch (...) {  // no more threads: the rest runs here
  }
  for (size_t i = started; i < k; ++i) piece(i);
  for (size_t i = 0; i < started; ++i) th[i].join();
}
// Cells a thread takes at least: reading back writes fresh pages and evaluates
// tanh (448^2 404 -> 272 us with 3 threads); creation only converts and checks,
// where starting threads for less costs more than they save (700^2 with 7
// threads of 64k cells 640 -> 780 us).
constexpr size_t kHostGrain = 1 << 16, kHostGrainIn = 1 << 18;
// and pieces it takes at least.  pf_create in us, in the calling thread alone /
// in pieces (some runs put two threads where they share little and take half as
// long again): FP32 760^2 815 / 2 pieces 850, 900^2 1230 / 3 pieces 1130; FP64
// 760^2 950 / 2 pieces 1360, 900^2 1430 / 3 pieces 1600, 1024^2 2200 / 4 pieces
// 2200 (after a read-back by threads 2450 / 2010).
constexpr size_t least_pieces_in(size_t elem) { return elem == 4 ? 3 : 4; }

// thin-interface constant a2 = 47/75 (Sec. 2.1): default lambda = D~ / a2
constexpr double kA2 = 47.0 / 75.0;
// Default 2D geometry, -k: k waves per SIMD, so that the launch fills whole
// rounds of the device (a fraction of a round leaves the SIMDs that hold one
// wave more to finish alone).  Each segment recomputes about 1.5 rows of
// work below it, so fewer, longer segments cost less, while more waves per
// SIMD hide more latency.  With R = strips * ny / SIMDs rows per SIMD, k =
// round(R^0.4) in FP32 and round(0.75 R^0.4) in FP64 (at most 3 waves of
// the FP64 kernel fit a SIMD), within [1, 64]: fitted to sweeps of k on
// 256^2 .. 8192^2 lattices (1024x2048: 4 waves per SIMD); on the lattices
// measured it is within 3.5% of the fastest k, which pf_autotune finds.
int default_seg2d(int nx, int ny, int precision, int ncu) {
  const double strips = (nx + 59) / 60;
  const double R = strips * ny / (4.0 * std::max(1, ncu));
  const double k = (precision == PF_F64 ? 0.75 : 1.0) * std::pow(R, 0.4);
  return -std::min(64, std::max(1, (int)std::lround(k)));
}
// Batched members keep segments of at least 8 rows: the batch fills the chip
// by itself.  A segment repeats about 3 rows of work, so members that nobody
// tuned (by pf_tune or pf_autotune) take 20 rows from 60 strip rows per SIMD in
// the whole batch on, and 32 from 160 on; below 60 that would leave SIMDs idle.
// us a step with 8 / 20 / 32 rows, FP32 (FP64), sides and strip rows R per SIMD:
//    16 of 100-400,  R  20:  12.8 /  16.6 /  19.5  (23.9 / 29.3 / 29.0)
//    16 of 150-600,  R  43:  20.4 /  22.5 /  24.7  (38.3 / 39.5 / 42.3)
//     8 of 256-1024, R  62:  26.6 /  26.7 /  31.3  (52.8 / 50.2 / 56.2)
//    16 of 200-800,  R  75:  28.8 /  27.0 /  31.8  (58.5 / 50.4 / 56.6)
//    12 of 300-900,  R  78:  30.6 /  31.7 /  31.8  (62.4 / 59.8 / 57.1)
//    16 of 256-1024, R 122:  41.1 /  40.4 /  45.3  (96.4 / 84.6 / 88.6)
//    32 of 256-1024, R 242:  77.7 /  70.5 /  73.6  (207.6 / 167.1 / 164.9)
//    64 of 256-1024, R 483: 172.5 / 147.0 / 142.1  (399.0 / 324.0 / 312.6)
constexpr int kMinSegBatch2D = 8;
int batch_rows2d(double R) { return R < 60.0 ? kMinSegBatch2D : R < 160.0 ? 20 : 32; }
constexpr size_t kMaxLds3DBytes = 163840;  // LDS one gfx950 workgroup may allocate
constexpr size_t kMaxLds3D = kMaxLds3DBytes;
// Default 3D geometry.  z rows per wide workgroup: 14, 6 or 2 in FP32 (16, 8
// or 4 waves; 16 is the most one workgroup holds, ring rows costing 16/14),
// 6 or 2 in FP64 (its launch bound is 8 waves), with the segment count that
// minimises the estimated time rounds x (rows + 2.5) x (1 + 0.43 w): rounds of
// resident workgroups, a segment's prologue costing about 2.5 rows, and w
// waves per SIMD on a CU of the fullest round (a row takes 1.8 us at one wave
// per SIMD, 2.15 at two and 3.4 at four in FP32: on a lattice that leaves CUs
// idle, more and smaller workgroups finish sooner).  The rows of a column are
// split evenly.  Fewer z rows are taken only for 5% by that estimate, so that
// large lattices keep the fewest ring rows: 256^3 FP32 (4 wide strips of 19 z
// tiles and a thin strip of 6) takes 14 and 3 segments of 85-86 rows (the
// thin strip 4 of 64), 252 workgroups in one round.  33x29x17 FP32: 28.6 us a
// step with 14 z rows, 14.8 with 2; 64^3 26.1 and 18.7 with 6; 128^3 57.9
// with 14 and 63.1 with 6.  pf_autotune refines it per lattice.
std::pair<int, int> default_geom3d(const pf_params *p, int ncu) {
  const bool f64 = p->precision == PF_F64;
  const long long cus = std::max(1, ncu);
  int best = p->ny, best_zt = 1;
  double best_cost = 1e300;
  int last = 0;
  for (int want : {14, 6, 2}) {
    if (f64 && want > 6) continue;
    const int zt = std::min(want, std::max(1, p->nz));
    if (zt == last) continue;
    last = zt;
    const int nw = zt + 2;
    const size_t lds = step3d_lds_bytes(p->nx, zt, f64 ? 8 : 4);
    const int by_waves = std::max(1, (f64 ? 8 : 16) / nw);
    const int by_lds = std::max(1, (int)(kMaxLds3DBytes / lds));
    const long long per_cu = std::min(by_waves, by_lds);
    int rows_zt = p->ny;
    double cost_zt = 1e300;
    for (int n = 1; n <= std::max(1, p->ny / 4); ++n) {
      const int rows = (p->ny + n - 1) / n;
      const long long blocks = geom3d(p->nx, p->ny, p->nz, rows, zt).blocks;
      const long long rounds = (blocks + cus * per_cu - 1) / (cus * per_cu);
      const double w = (double)(std::min(per_cu, (blocks + cus - 1) / cus) * nw) / 4.0;
      const double cost = (double)rounds * (rows + 2.5) * (1.0 + 0.43 * w);
      if (cost < cost_zt - 1e-9) {
        cost_zt = cost;
        rows_zt = rows;
      }
    }
    if (cost_zt < 0.95 * best_cost) {
      best_cost = cost_zt;
      best = rows_zt;
      best_zt = zt;
    }
  }
  return {best, best_zt};
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

size_t cells(const pf_params *p) {
  return (size_t)p->nx * (size_t)p->ny * (size_t)(p->dim == 3 ? p->nz : 1);
}

void weights_of(const pf_params *p, double w[3]) {
  if (p->scheme == PF_SCHEME_STD) {
    w[0] = 1.0; w[1] = 0.0; w[2] = 0.0;
  } else if (p->scheme == PF_SCHEME_WEIGHTS) {
    double s = p->weights[0] + p->weights[1] + (p->dim == 3 ? p->weights[2] : 0.0);
    w[0] = p->weights[0] / s;
    w[1] = p->weights[1] / s;
    w[2] = p->dim == 3 ? p->weights[2] / s : 0.0;
  } else if (p->dim == 2) {
    w[0] = 2.0 / 3.0; w[1] = 1.0 / 3.0; w[2] = 0.0;
  } else {
    w[0] = 1.0 / 3.0; w[1] = 2.0 / 3.0; w[2] = 0.0;
  }
}

// smallest F1 of Eq. Thermal_F1 over the lattice rows for the zeta offset
// off = s h - y0 - Vp t (zeta = y + off is linear in y, so the extreme rows
// bound it); 1 if isothermal
double f1_min_at(const pf_params *p, double off) {
  if (!(p->lT > 0.0)) return 1.0;
  double zmax = (p->ny - 1) * p->h + off;
  double zmin = off;
  double a = 1.0 - (1.0 - p->k) * zmax / p->lT;
  double b = 1.0 - (1.0 - p->k) * zmin / p->lT;
  return a < b ? a : b;
}

// at t = 0 with no frame shift
double f1_min(const pf_params *p) { return f1_min_at(p, -p->y0); }

// explicit limit h^2 / (2 dim max(D~, 1/F1_min))
double stable_dt_for(const pf_params *p, double f1) {
  return p->h * p->h / (2.0 * p->dim * std::max(p->D, 1.0 / f1));
}

struct Layout {
  size_t psi[2], U[2], grain, grain2, rot, frame[3], partials, result, total;
};

Layout layout_of(const pf_params *p) {
  Layout L;
  size_t es = p->precision == PF_F64 ? 8 : 4;
  size_t n = cells(p);
  size_t o = 0;
  // Fields beyond the 256 MB last-level cache start 33 x 256 bytes further apart:
  // a step reads and writes the same cell of all four at a time, and where their
  // starts are equal modulo a large power of two these accesses meet in the same
  // memory banks (8192^2 FP32 at its default geometry with the frame 280-312 us a
  // step, 255-258 apart; without it 274-301 and 250; pf_step_diffusion 273 and
  // 265).  Within the cache it gains nothing (4096^2 with grains 104.8 and 106.0).
  const size_t apart = 4 * n * es > ((size_t)256 << 20) ? 33 * 256 : 0;
  for (int i = 0; i < 2; ++i) { L.psi[i] = o; o += align256(n * es) + apart; }
  for (int i = 0; i < 2; ++i) { L.U[i] = o; o += align256(n * es) + apart; }
  L.grain = o; o += align256(p->n_grains > 1 ? n : 1);
  L.grain2 = o; o += align256(p->dynamic_grains ? n : 1);  // the next level's map
  L.rot = o; o += align256((size_t)(p->n_grains > 0 ? p->n_grains : 1) * 9 * es);
  for (int i = 0; i < 3; ++i) { L.frame[i] = o; o += 256; }
  // one partial per workgroup of the reduction
  int nb = reduce_blocks(p->nx, p->ny, p->dim == 3 ? p->nz : 1);
  L.partials = o; o += align256((size_t)(nb + 64) * tip_acc_bytes());
  L.result = o; o += 256;
  L.total = o;
  return L;
}

int validate(const pf_params *p) {
  if (!p) return fail(PF_ERR_ARG, "params is NULL");
  if (p->dim != 2 && p->dim != 3) return fail(PF_ERR_ARG, "dim must be 2 or 3");
  if (p->nx < 4 || p->ny < 4 || (p->dim == 3 && p->nz < 4))
    return fail(PF_ERR_ARG, "every lattice side must be >= 4");
  if ((double)p->nx * p->ny * (p->dim == 3 ? p->nz : 1) > 4.0e9)
    return fail(PF_ERR_ARG, "lattice larger than 4e9 cells");
  if ((long long)p->nx * p->ny > 2147483647LL / 2 ||
      (long long)p->ny * (p->dim == 3 ? p->nz : 1) > 2147483647LL / 2)
    return fail(PF_ERR_ARG, "x-y plane or y-z plane too large");
  if (p->precision != PF_F32 && p->precision != PF_F64)
    return fail(PF_ERR_ARG, "precision must be PF_F32 or PF_F64");
  if (p->scheme < PF_SCHEME_ISO || p->scheme > PF_SCHEME_WEIGHTS)
    return fail(PF_ERR_ARG, "unknown scheme");
  if (p->scheme == PF_SCHEME_WEIGHTS) {
    double s = p->weights[0] + p->weights[1] + (p->dim == 3 ? p->weights[2] : 0.0);
    if (!(fabs(s) > 1e-12)) return fail(PF_ERR_ARG, "shell weights sum to zero");
    if (p->dim == 2 && p->weights[2] != 0.0)
      return fail(PF_ERR_ARG, "2D has two shells: weights[2] must be 0");
  }
  if (p->antitrapping != PF_AT_APPROX && p->antitrapping != PF_AT_FULL)
    return fail(PF_ERR_ARG, "antitrapping must be PF_AT_APPROX or PF_AT_FULL");
  if (p->divergence != PF_DIV_SHELLS && p->divergence != PF_DIV_TWO_POINT)
    return fail(PF_ERR_ARG, "divergence must be PF_DIV_SHELLS or PF_DIV_TWO_POINT");
  if (p->dim == 3 && (p->antitrapping != PF_AT_APPROX || p->divergence != PF_DIV_SHELLS))
    return fail(PF_ERR_ARG, "3D runs the approximated current with shell divergences only");
  if (!(p->k > 0.0 && p->k < 1.0)) return fail(PF_ERR_ARG, "k must lie in (0, 1)");
  if (!(p->eps4 >= 0.0 && p->eps4 < 1.0 / 15.0))
    return fail(PF_ERR_ARG, "eps4 must lie in [0, 1/15)");
  if (!(p->D > 0.0)) return fail(PF_ERR_ARG, "D must be > 0");
  if (!(p->h > 0.0)) return fail(PF_ERR_ARG, "h must be > 0");
  if (!isfinite(p->lambda) || !isfinite(p->dt) || !isfinite(p->Vp) || !isfinite(p->lT) ||
      !isfinite(p->y0))
    return fail(PF_ERR_ARG, "non-finite scalar parameter");
  for (int a = 0; a < 3; ++a)
    if (p->bc[a] != PF_BC_NOFLUX && p->bc[a] != PF_BC_PERIODIC)
      return fail(PF_ERR_ARG, "bc must be PF_BC_NOFLUX or PF_BC_PERIODIC");
  if (p->frame) {
    if (p->bc[1] != PF_BC_NOFLUX) return fail(PF_ERR_ARG, "the moving frame needs no-flux y walls");
    if (p->shift_row < 1 || p->shift_row > p->ny - 2)
      return fail(PF_ERR_ARG, "shift_row must lie in [1, ny-2]");
  }
  if (p->n_grains < 1 || p->n_grains > 127) return fail(PF_ERR_ARG, "n_grains must be 1..127");
  if (p->dynamic_grains != 0 && p->dynamic_grains != 1)
    return fail(PF_ERR_ARG, "dynamic_grains must be 0 or 1");
  if (p->dynamic_grains && p->n_grains < 2)
    return fail(PF_ERR_ARG, "dynamic grains need n_grains >= 2");
  if (!p->grain_rot) return fail(PF_ERR_ARG, "grain_rot is NULL");
  for (int g = 0; g < p->n_grains; ++g) {
    const double *R = p->grain_rot + 9 * g;
    for (int i = 0; i < 9; ++i)
      if (!isfinite(R[i])) return fail(PF_ERR_ARG, "non-finite rotation entry");
    for (int i = 0; i < 3; ++i)
      for (int j = 0; j < 3; ++j) {
        double d = 0.0;
        for (int m = 0; m < 3; ++m) d += R[m * 3 + i] * R[m * 3 + j];
        if (fabs(d - (i == j ? 1.0 : 0.0)) > 1e-9)
          return fail(PF_ERR_ARG, "grain rotation is not orthonormal");
      }
    double det = R[0] * (R[4] * R[8] - R[5] * R[7]) - R[1] * (R[3] * R[8] - R[5] * R[6]) +
                 R[2] * (R[3] * R[7] - R[4] * R[6]);
    if (det < 0.0) return fail(PF_ERR_ARG, "grain rotation is improper (det < 0)");
    if (p->dim == 2 && (fabs(R[2]) > 1e-12 || fabs(R[5]) > 1e-12 || fabs(R[6]) > 1e-12 ||
                        fabs(R[7]) > 1e-12))
      return fail(PF_ERR_ARG, "2D grain rotations must be rotations about z");
  }
  if (p->lT > 0.0 && !(f1_min(p) > 0.0))
    return fail(PF_ERR_ARG, "F1 = 1 - (1-k) zeta / lT is not positive over the lattice");
  return PF_OK;
}

}  // namespace

struct pf_solver {
  pf_params p;
  std::vector<double> rot;
  double w[3];
  double lambda, dt;
  size_t n;
  hipStream_t stream;
  char *ws;
  size_t ws_bytes;
  bool own;
  Layout L;
  int cur;    // current field buffers
  int fcur;   // current frame record (0..2, advances with the frame on)
  long long step;
  int seg, ztile;  // launch geometry (2D seg < 0: -(waves per SIMD))
  bool tuned;      // seg was set by pf_tune or pf_autotune
  int ncu;         // compute units of the device the solver was created on
  bool have_prev;
  double prev_t, prev_y;
};

namespace {

// The library's launch geometry of a problem nobody tuned: (rows per segment or
// -(waves per SIMD), z rows per workgroup).
std::pair<int, int> default_geom(const pf_params *p, int ncu) {
  if (p->dim == 2) return {default_seg2d(p->nx, p->ny, p->precision, ncu), 1};
  return default_geom3d(p, ncu);
}

// Waves of one step launch at the geometry (seg, ztile).
int64_t solo_waves(const pf_params &p, int seg, int ztile, int ncu) {
  if (p.dim == 2) {
    const Geom2D g = geom2d(p.nx, p.ny, seg, ncu, true);
    return (int64_t)g.nstrips * g.nsegs;
  }
  const Geom3D g = geom3d(p.nx, p.ny, p.nz, seg, ztile);
  return (int64_t)g.blocks * (g.threads / 64);
}

// Geometry of a batch member whose own is seg: its rows per segment (the longest
// segment when it asks for waves per SIMD), but at least min_rows.
Geom2D member_geom2d(const pf_params &p, int seg, int ncu, int min_rows) {
  int rows = seg;
  if (seg < 0) {
    const Geom2D g = geom2d(p.nx, p.ny, seg, ncu, true);
    rows = g.segbase + (g.segrem ? 1 : 0);
  }
  return geom2d(p.nx, p.ny, std::max(rows, min_rows), 0, true);
}

template <typename T>
T *field(pf_solver *s, size_t off) {
  return reinterpret_cast<T *>(s->ws + off);
}

template <typename T>
Coef<T> coef_of(const pf_solver *s) {
  const pf_params &p = s->p;
  const double h = p.h, h2 = h * h;
  Coef<T> c = {};
  c.dt = (T)s->dt;
  c.k = (T)p.k;
  c.omk = (T)(1.0 - p.k);
  c.eps4 = (T)p.eps4;
  c.an0 = (T)(1.0 - 3.0 * p.eps4);
  c.an4 = (T)(4.0 * p.eps4);
  c.an16 = (T)(16.0 * p.eps4);
  c.D = (T)p.D;
  c.lambda = (T)s->lambda;
  c.h = (T)h;
  // the psi equation times h^2, with L and G by their prefactors (2D: Eqs.
  // 2D_L10, 2D_L01, Grad_10, Grad_11; 3D: Eqs. 3D_L100, 3D_L110, 3D_L111,
  // Grad_100, Grad_110, Grad_111); the eps4 remainder holds -s1 / h^2
  const double pl = p.dim == 2 ? 2.0 : 4.0, pg = p.dim == 2 ? 8.0 : 16.0;
  c.rA1 = (T)(s->w[0] - 1.0);
  c.rA2 = (T)(s->w[1] / pl);
  c.rA3 = (T)(s->w[2] / pl);
  c.rB1 = (T)(-sqrt(2.0) * s->w[0] / 4.0);
  c.rB2 = (T)(-sqrt(2.0) * s->w[1] / pg);
  c.rB3 = (T)(-sqrt(2.0) * s->w[2] / pg);
  c.rK = (T)(sqrt(2.0) * h2);
  c.h2 = (T)h2;
  c.omkh2 = (T)((1.0 - p.k) * h2);
  c.hT = (T)(p.lT > 0.0 ? h / p.lT : 0.0);
  if (p.dim == 2) {
    // D_{1,0}: fluxes carry the 4-point alpha sum, /(4h^2); D_{0,1}: plaquette
    // means times dbeta, /(2h^2) (Eqs. flux_10, flux_11); the kernel's link
    // alphas carry another factor 4
    c.cD1 = (T)(s->w[0] / (16.0 * h2));
    c.cD2 = (T)(s->w[1] / (8.0 * h2));
    // two-point faces carry (alpha_0 + alpha_e) dbeta: /(2h^2); links of the
    // full current carry h / |h grad psi| and enter with a factor h
    c.cT = (T)(1.0 / (2.0 * h2));
    c.at_eps = (T)(1e-12 * h2);
    c.ac_eps = (T)(4e-12 * h2);
    c.an1 = (T)(1.0 + p.eps4);
    c.an2 = (T)(2.0 * p.eps4);
    c.an8 = (T)(8.0 * p.eps4);
    c.rC1 = (T)(s->w[0] / h2);
    c.rC2 = (T)(s->w[1] / (2.0 * h2));
    c.rG1 = (T)(s->w[0] / (4.0 * h2));
    c.rG2 = (T)(s->w[1] / (8.0 * h2));
    c.rStd = (T)(1.0 / h2);
    c.inv_lT = (T)(p.lT > 0.0 ? 1.0 / p.lT : 0.0);
  } else {
    // D_{1,0,0} = sum abar dbeta / h^2; D_{0,1,0}, D_{0,0,1} = / (4h^2); the
    // kernel's averages are 16, 32 and 8 times abar
    c.kA = (T)(s->w[0] / h2 / 16.0);
    c.kB = (T)(s->w[1] / (4.0 * h2) / 32.0);
    c.kC = (T)(s->w[2] / (4.0 * h2) / 8.0);
    c.ac_eps = (T)(4e-12 * h2);
    c.f3_eps = (T)(16e-12 * h2);
  }
  return c;
}

// 2D grains may be turned over (R_zz = -1, a half turn about an in-plane axis):
// the step kernels take the rotation's angle about z, so such a grain is first
// turned about the crystal's own x axis, which leaves the cubic form unchanged.
void upright_2d(std::vector<double> &rot) {
  for (size_t g = 0; g + 9 <= rot.size(); g += 9)
    if (rot[g + 8] < 0.0)
      for (int i = 0; i < 9; i += 3) {
        rot[g + i + 1] = -rot[g + i + 1];
        rot[g + i + 2] = -rot[g + i + 2];
      }
}

// cos and sin of twice the angle of a rotation about z (row-major 3 x 3)
void double_angle(const double *R, double *c2, double *s2) {
  *c2 = R[0] * R[4] + R[1] * R[3];
  *s2 = R[3] * R[0] - R[1] * R[4];
}

template <typename T>
int upload(pf_solver *s, const pf_init *init) {
  const size_t n = s->n;
  std::unique_ptr<T[]> buf(new (std::nothrow) T[n]);
  if (!buf) return fail(PF_ERR_OOM, "host allocation failed");
  T *tmp = buf.get();
  // FP32 in the calling thread alone: whole lines are written before the
  // conversions store into them, because after a read-back by threads the
  // buffer's lines are in other cores' caches (pf_create of 512^2 then 570 us
  // without, 525 with; of 512^2 otherwise 505 and 512).  FP64 ran up to 4%
  // slower with it, also after a read-back.
  if (sizeof(T) == 4 && n < least_pieces_in(sizeof(T)) * kHostGrainIn)
    memset(tmp, 0, n * sizeof(T));
  for (int k = 0; k < 2; ++k) {
    const double *src = k == 0 ? init->psi : init->U;
    host_parallel(n, kHostGrainIn, least_pieces_in(sizeof(T)), [&](size_t b, size_t e) {
      for (size_t i = b; i < e; ++i) tmp[i] = (T)src[i];
    });
    PF_HIP(hipMemcpy(field<T>(s, k == 0 ? s->L.psi[0] : s->L.U[0]), tmp, n * sizeof(T),
                     hipMemcpyHostToDevice));
  }
  // rotation table: 2D (cos, sin of twice the angle) per grain, then (r00, r01,
  // r10, r11) per grain; 3D all 9
  const int ng = s->p.n_grains;
  std::vector<T> rt((size_t)ng * 9, (T)0);
  for (int g = 0; g < ng; ++g) {
    const double *R = s->rot.data() + 9 * g;
    if (s->p.dim == 2) {
      double c2, s2;
      double_angle(R, &c2, &s2);
      rt[2 * g + 0] = (T)c2;
      rt[2 * g + 1] = (T)s2;
      for (int i = 0; i < 4; ++i) rt[2 * ng + 4 * g + i] = (T)R[i < 2 ? i : i + 1];
    } else {
      for (int i = 0; i < 9; ++i) rt[9 * g + i] = (T)R[i];
    }
  }
  PF_HIP(hipMemcpy(s->ws + s->L.rot, rt.data(), rt.size() * sizeof(T), hipMemcpyHostToDevice));
  return PF_OK;
}

// Grain map k (0, 1): the static map, or the two levels of a dynamic one
// (the current level is the solver's buffer parity, like psi and U).
int8_t *grain_buf(pf_solver *s, int k) {
  return reinterpret_cast<int8_t *>(s->ws + (k == 0 || !s->p.dynamic_grains ? s->L.grain
                                                                            : s->L.grain2));
}

// Argument block of the 2D step of solver s (pointers set per launch).
template <typename T>
void fill2d(pf_solver *s, Step2DArgs<T> &a, const Geom2D &g) {
  const pf_params &p = s->p;
  memset(&a, 0, sizeof(a));
  a.grain = p.n_grains > 1 ? grain_buf(s, s->cur) : nullptr;
  a.grain_out = p.dynamic_grains ? grain_buf(s, 1 - s->cur) : nullptr;
  a.rot = field<T>(s, s->L.rot);
  a.axes = a.rot + 2 * std::max(p.n_grains, 1);
  double c2, s2;
  double_angle(s->rot.data(), &c2, &s2);
  a.c2 = (T)c2; a.s2 = (T)s2;
  a.nx = p.nx; a.ny = p.ny; a.bcx = p.bc[0]; a.bcy = p.bc[1];
  a.wout = g.wout; a.nstrips = g.nstrips; a.nsegs = g.nsegs;
  a.segbase = g.segbase; a.segrem = g.segrem;
  a.strip_rcp = (unsigned)std::min<unsigned long long>((1ULL << 32) / g.nstrips, 0xffffffffULL);
  a.nshared = g.nshared; a.sharedsegs = g.sharedsegs;
  a.c = coef_of<T>(s);
  a.hd = p.h; a.y0 = p.y0; a.Vp = p.Vp; a.dtd = s->dt;
  a.inv_lTd = p.lT > 0.0 ? 1.0 / p.lT : 0.0;
  a.frame = p.frame; a.shift_row = p.shift_row;
}

template <typename T>
int step_impl(pf_solver *s, long long nsteps, bool diffusion_only = false) {
  const pf_params &p = s->p;
  const bool frozen = p.lT > 0.0;
  const bool reduce = p.frame != 0;
  const bool multi = p.n_grains > 1;
  const Coef<T> c = coef_of<T>(s);
  auto frec = [&](int i) { return reinterpret_cast<FrameState *>(s->ws + s->L.frame[i % 3]); };
  if (p.dim == 2) {
    Step2DArgs<T> a;
    const Geom2D g = geom2d(p.nx, p.ny, s->seg, s->ncu, !diffusion_only);
    fill2d<T>(s, a, g);
    (void)c;
    const bool two = p.divergence == PF_DIV_TWO_POINT;
    const int at = diffusion_only ? kAtDiffusionOnly
                   : p.antitrapping == PF_AT_FULL ? (two ? kAtFullTwoPoint : kAtFullShells)
                                                  : (two ? kAtApproxTwoPoint : kAtApproxShells);
    for (long long i = 0; i < nsteps; ++i) {
      a.psi_in = field<T>(s, s->L.psi[s->cur]);
      a.U_in = field<T>(s, s->L.U[s->cur]);
      a.psi_out = field<T>(s, s->L.psi[1 - s->cur]);
      a.U_out = field<T>(s, s->L.U[1 - s->cur]);
      if (multi) a.grain = grain_buf(s, s->cur);
      if (p.dynamic_grains) a.grain_out = grain_buf(s, 1 - s->cur);
      a.frame_in = frec(s->fcur);
      a.frame_out = frec(s->fcur + 1);
      a.frame_clear = frec(s->fcur + 2);
      a.step = s->step;
      PF_HIP(launch_step2d<T>(a, g, frozen, reduce, multi, at, s->stream));
      s->cur = 1 - s->cur;
      if (reduce) s->fcur = (s->fcur + 1) % 3;
      s->step += 1;
    }
  } else {
    Step3DArgs<T> a;
    memset(&a, 0, sizeof(a));
    Geom3D g = geom3d(p.nx, p.ny, p.nz, s->seg, s->ztile);
    a.grain = multi ? grain_buf(s, s->cur) : nullptr;
    a.grain_out = p.dynamic_grains ? grain_buf(s, 1 - s->cur) : nullptr;
    a.rot = field<T>(s, s->L.rot);
    for (int i = 0; i < 9; ++i) a.R[i] = (T)s->rot[i];
    a.nx = p.nx; a.ny = p.ny; a.nz = p.nz;
    a.bcx = p.bc[0]; a.bcy = p.bc[1]; a.bcz = p.bc[2];
    a.wout = g.wout; a.nstrips = g.nstrips; a.nzt = g.nzt; a.nsegs = g.nsegs; a.seg = g.seg;
    a.ztile = g.ztile;
    a.segbase = g.segbase; a.segrem = g.segrem;
    a.ncols = g.ncols; a.ncols_wide = g.ncols_wide;
    a.thin_g = g.thin_g; a.thin_G = g.thin_G; a.thin_wout = g.thin_wout;
    a.thin_nzt = g.thin_nzt; a.thin_segbase = g.thin_segbase; a.thin_segrem = g.thin_segrem;
    a.c = c;
    a.hd = p.h; a.y0 = p.y0; a.Vp = p.Vp; a.dtd = s->dt;
    a.inv_lTd = p.lT > 0.0 ? 1.0 / p.lT : 0.0;
    a.frame = p.frame; a.shift_row = p.shift_row;
    for (long long i = 0; i < nsteps; ++i) {
      a.psi_in = field<T>(s, s->L.psi[s->cur]);
      a.U_in = field<T>(s, s->L.U[s->cur]);
      a.psi_out = field<T>(s, s->L.psi[1 - s->cur]);
      a.U_out = field<T>(s, s->L.U[1 - s->cur]);
      if (multi) a.grain = grain_buf(s, s->cur);
      if (p.dynamic_grains) a.grain_out = grain_buf(s, 1 - s->cur);
      a.frame_in = frec(s->fcur);
      a.frame_out = frec(s->fcur + 1);
      a.frame_clear = frec(s->fcur + 2);
      a.step = s->step;
      PF_HIP(launch_step3d<T>(a, g, frozen, reduce, multi, s->stream));
      s->cur = 1 - s->cur;
      if (reduce) s->fcur = (s->fcur + 1) % 3;
      s->step += 1;
    }
  }
  return PF_OK;
}

template <typename T>
int reduce_impl(pf_solver *s, TipResult *res, FrameState *fr) {
  ReduceArgs<T> a;
  a.psi = field<T>(s, s->L.psi[s->cur]);
  a.U = field<T>(s, s->L.U[s->cur]);
  a.nx = s->p.nx; a.ny = s->p.ny; a.nz = s->p.dim == 3 ? s->p.nz : 1;
  a.hd = s->p.h;
  a.rows = 0;  // set by the launcher
  a.frame = reinterpret_cast<const FrameState *>(s->ws + s->L.frame[s->fcur]);
  a.pending = 0;
  a.red = Reduce{reinterpret_cast<TipAcc *>(s->ws + s->L.partials),
                 reinterpret_cast<TipResult *>(s->ws + s->L.result)};
  PF_HIP(launch_reduce<T>(a, s->stream));
  // the result record carries a copy of the frame record the reduction read
  PF_HIP(hipMemcpyAsync(res, a.red.result, sizeof(TipResult), hipMemcpyDeviceToHost, s->stream));
  PF_HIP(hipStreamSynchronize(s->stream));
  *fr = res->frame;
  return PF_OK;
}

template <typename T>
int read_impl(pf_solver *s, double *phi, double *U, double *psi) {
  const pf_params &p = s->p;
  const size_t n = s->n;
  FrameState fr;
  PF_HIP(hipStreamSynchronize(s->stream));
  PF_HIP(hipMemcpy(&fr, s->ws + s->L.frame[s->fcur], sizeof(fr), hipMemcpyDeviceToHost));
  std::unique_ptr<T[]> bp(new (std::nothrow) T[n]), bu(new (std::nothrow) T[n]);
  if (!bp || !bu) return fail(PF_ERR_OOM, "host allocation failed");
  const T *hp = bp.get(), *hu = bu.get();
  PF_HIP(hipMemcpy(bp.get(), field<T>(s, s->L.psi[s->cur]), n * sizeof(T), hipMemcpyDeviceToHost));
  PF_HIP(hipMemcpy(bu.get(), field<T>(s, s->L.U[s->cur]), n * sizeof(T), hipMemcpyDeviceToHost));
  const size_t nx = p.nx, ny = p.ny, nz = p.dim == 3 ? p.nz : 1;
  host_parallel(ny * nz, std::max<size_t>(1, kHostGrain / nx), 2, [&](size_t b, size_t e) {
    for (size_t row = b; row < e; ++row) {
      const size_t j = row % ny, jp = fr.pending ? std::min(j + 1, ny - 1) : j;
      const size_t dst = row * nx, src = (row - j + jp) * nx;
      for (size_t i = 0; i < nx; ++i) {
        const double vp = (double)hp[src + i];
        if (psi) psi[dst + i] = vp;
        if (phi) phi[dst + i] = tanh(vp / sqrt(2.0));
        if (U) U[dst + i] = (double)hu[src + i];
      }
    }
  });
  return PF_OK;
}

}  // namespace

struct pf_batch {
  std::vector<pf_solver *> s;
  int precision;
  bool frozen, frame, multi;
  hipStream_t stream;
  void *table;  // device BatchSolve2D<T>[n]
  int2 *map;    // device workgroup map
  int blocks;
  std::vector<long long> expect;  // solver steps the device table assumes
  std::vector<int> seg;           // batch_key of the members the table was built with
  long long waves;                // waves of one launch
  int graph_steps;
  int seg_fixed;  // > 0: rows per segment of every member (pf_batch_autotune)
  hipStream_t cap;
  hipGraph_t graph;
  hipGraphExec_t gexec;
};

namespace {

int xcd_remap_host(int b, int nb) {
  const int X = 8;
  int q = nb / X, r = nb % X, x = b % X;
  return x * q + (x < r ? x : r) + b / X;
}

// What the batch's geometry takes from a member: the segment length it was tuned
// to, 0 if nobody tuned it.
int batch_key(const pf_solver *s) { return s->tuned ? s->seg : 0; }

// (Re)build the device table and workgroup map from the solvers' state.
template <typename T>
int batch_build(pf_batch *b) {
  const int n = (int)b->s.size();
  std::vector<BatchSolve2D<T>> tab(n);
  std::vector<int2> list;
  double R = 0.0;  // strip rows per SIMD
  for (const pf_solver *s : b->s)
    R += (double)((s->p.nx + 59) / 60) * s->p.ny / (4.0 * std::max(1, s->ncu));
  const int rows = batch_rows2d(R);
  long long waves = 0;
  for (int i = 0; i < n; ++i) {
    pf_solver *s = b->s[i];
    BatchSolve2D<T> &e = tab[i];
    memset(&e, 0, sizeof(e));
    const Geom2D g = b->seg_fixed > 0
                         ? geom2d(s->p.nx, s->p.ny, b->seg_fixed, 0, true)
                         : member_geom2d(s->p, s->seg, s->ncu, s->tuned ? kMinSegBatch2D : rows);
    fill2d<T>(s, e.a, g);
    for (int k = 0; k < 2; ++k) {
      e.psi[k] = field<T>(s, s->L.psi[k]);
      e.U[k] = field<T>(s, s->L.U[k]);
    }
    for (int k = 0; k < 3; ++k) e.frames[k] = reinterpret_cast<FrameState *>(s->ws + s->L.frame[k]);
    e.n0 = s->step;
    e.par0 = s->cur;
    e.f0 = s->fcur;
    for (int lb = 0; lb < g.blocks; ++lb) list.push_back(int2{i, lb});
    waves += (long long)g.nstrips * g.nsegs;
    b->expect[i] = s->step;
    b->seg[i] = batch_key(s);
  }
  const int total = (int)list.size();
  std::vector<int2> map(total);
  for (int k = 0; k < total; ++k) map[k] = list[xcd_remap_host(k, total)];
  PF_HIP(hipStreamSynchronize(b->stream));
  if (b->table) (void)hipFree(b->table);
  if (b->map) (void)hipFree(b->map);
  b->table = nullptr;
  b->map = nullptr;
  PF_HIP(hipMalloc(&b->table, sizeof(BatchSolve2D<T>) * n));
  PF_HIP(hipMalloc((void **)&b->map, sizeof(int2) * total));
  PF_HIP(hipMemcpy(b->table, tab.data(), sizeof(BatchSolve2D<T>) * n, hipMemcpyHostToDevice));
  PF_HIP(hipMemcpy(b->map, map.data(), sizeof(int2) * total, hipMemcpyHostToDevice));
  b->blocks = total;
  b->waves = waves;
  return PF_OK;
}

void batch_drop_graph(pf_batch *b) {
  if (b->gexec) (void)hipGraphExecDestroy(b->gexec);
  if (b->graph) (void)hipGraphDestroy(b->graph);
  b->gexec = nullptr;
  b->graph = nullptr;
}

template <typename T>
int batch_capture(pf_batch *b) {
  batch_drop_graph(b);
  if (b->graph_steps <= 0) return PF_OK;
  auto *tab = reinterpret_cast<BatchSolve2D<T> *>(b->table);
  PF_HIP(hipStreamBeginCapture(b->cap, hipStreamCaptureModeRelaxed));
  for (int k = 0; k < b->graph_steps; ++k)
    (void)launch_batch2d<T>(tab, b->map, b->blocks, k, b->frozen, b->frame, b->multi, b->cap);
  (void)launch_batch2d_advance<T>(tab, (int)b->s.size(), b->graph_steps, b->frame, b->cap);
  PF_HIP(hipStreamEndCapture(b->cap, &b->graph));
  PF_HIP(hipGraphInstantiate(&b->gexec, b->graph, nullptr, nullptr, 0));
  return PF_OK;
}

// Rebuild the table (and the graph) if a member was stepped or tuned on its own.
template <typename T>
int batch_refresh(pf_batch *b) {
  bool stale = false;
  for (size_t i = 0; i < b->s.size(); ++i)
    if (b->s[i]->step != b->expect[i] || batch_key(b->s[i]) != b->seg[i]) stale = true;
  if (!stale) return PF_OK;
  const int rc = batch_build<T>(b);
  return rc != PF_OK ? rc : batch_capture<T>(b);
}

template <typename T>
int batch_step(pf_batch *b, long long nsteps) {
  const int rc = batch_refresh<T>(b);
  if (rc != PF_OK) return rc;
  auto *tab = reinterpret_cast<BatchSolve2D<T> *>(b->table);
  long long done = 0;
  if (b->gexec) {
    for (; done + b->graph_steps <= nsteps; done += b->graph_steps)
      PF_HIP(hipGraphLaunch(b->gexec, b->stream));
  }
  const int rem = (int)(nsteps - done);
  if (rem > 0) {
    for (int k = 0; k < rem; ++k)
      PF_HIP(launch_batch2d<T>(tab, b->map, b->blocks, k, b->frozen, b->frame, b->multi,
                               b->stream));
    PF_HIP(launch_batch2d_advance<T>(tab, (int)b->s.size(), rem, b->frame, b->stream));
  }
  for (size_t i = 0; i < b->s.size(); ++i) {
    pf_solver *s = b->s[i];
    s->step += nsteps;
    s->cur = (int)((s->cur + nsteps) & 1);
    if (b->frame) s->fcur = (int)((s->fcur + nsteps) % 3);
    b->expect[i] = s->step;
  }
  return PF_OK;
}

}  // namespace

namespace {

// Seconds of `steps` steps of `run` on `st` (after 2 warm-up steps), or a
// negative value when a HIP call failed.
template <typename F>
double time_steps(hipStream_t st, int steps, F run) {
  hipEvent_t e0 = nullptr, e1 = nullptr;
  double out = -1.0;
  float ms = 0.f;
  if (hipEventCreate(&e0) == hipSuccess && hipEventCreate(&e1) == hipSuccess && run(2) == PF_OK &&
      hipEventRecord(e0, st) == hipSuccess && run(steps) == PF_OK &&
      hipEventRecord(e1, st) == hipSuccess && hipEventSynchronize(e1) == hipSuccess &&
      hipEventElapsedTime(&ms, e0, e1) == hipSuccess)
    out = ms * 1e-3;
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  return out;
}

// Longest trial a caller may ask for: the confirming passes run four times as
// many steps, which must stay within an int.
constexpr int kMaxTrialSteps = 1 << 20;

// Index of the fastest of n candidates timed by trial(i, m) (seconds of m
// times the trial's base step count, negative on failure; -1 returned then).
// Candidate 0 is the geometry in use: each candidate is timed in two
// interleaved passes and keeps its better time.  A candidate more than 3%
// faster than candidate 0 is then confirmed against it in three interleaved
// passes four times as long, and replaces it only when it is still more than
// 2% faster there: a short trial can misjudge near-equal geometries, and the
// choice should not flip from run to run on timing noise.
template <typename F>
int pick_fastest(int n, F trial) {
  std::vector<double> best(n, 1e300);
  for (int pass = 0; pass < 2; ++pass)
    for (int i = 0; i < n; ++i) {
      double sec = trial(i, 1);
      if (sec < 0.0) return -1;
      best[i] = std::min(best[i], sec);
    }
  int k = 0;
  for (int i = 1; i < n; ++i)
    if (best[i] < best[k]) k = i;
  if (!(best[k] < 0.97 * best[0])) return 0;
  double b0 = 1e300, bk = 1e300;
  for (int pass = 0; pass < 3; ++pass) {
    const double s0 = trial(0, 4), sk = trial(k, 4);
    if (s0 < 0.0 || sk < 0.0) return -1;
    b0 = std::min(b0, s0);
    bk = std::min(bk, sk);
  }
  return bk < 0.98 * b0 ? k : 0;
}

// A copy of solver s whose workspace is a fresh device copy of s's (the
// caller frees clone.ws).  Stepping the copy leaves s untouched.
int clone_solver(pf_solver *s, pf_solver &clone) {
  void *d = nullptr;
  PF_HIP(hipStreamSynchronize(s->stream));
  if (hipMalloc(&d, s->L.total) != hipSuccess)
    return fail(PF_ERR_OOM, "autotune scratch allocation of " + std::to_string(s->L.total) +
                                " bytes failed");
  if (hipMemcpy(d, s->ws, s->L.total, hipMemcpyDeviceToDevice) != hipSuccess) {
    (void)hipFree(d);
    return fail(PF_ERR_DEVICE, "autotune scratch copy failed");
  }
  clone = *s;
  clone.ws = reinterpret_cast<char *>(d);
  clone.ws_bytes = s->L.total;
  clone.own = false;
  return PF_OK;
}

template <typename T>
int autotune_impl(pf_solver *s, int steps) {
  pf_solver t;
  int rc = clone_solver(s, t);
  if (rc != PF_OK) return rc;
  // (rows per segment, z rows per workgroup); the geometry in use first
  std::vector<std::pair<int, int>> cand = {{s->seg, s->ztile}};
  auto add = [&](int seg, int zt) {
    if (seg != s->seg || zt != s->ztile) cand.push_back({seg, zt});
  };
  if (s->p.dim == 2) {
    // waves per SIMD; counts that give the same segments as one already
    // listed are skipped
    std::vector<int> nsegs = {geom2d(s->p.nx, s->p.ny, s->seg, s->ncu, true).nsegs};
    for (int k : {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 20, 24, 32}) {
      const int n = geom2d(s->p.nx, s->p.ny, -k, s->ncu, true).nsegs;
      if (std::find(nsegs.begin(), nsegs.end(), n) != nsegs.end()) continue;
      nsegs.push_back(n);
      add(-k, s->ztile);
    }
  } else {
    // rows per segment, each candidate kept only when it gives a segment
    // count not listed yet for its z rows (the rows are split evenly)
    const int zmax = s->p.precision == PF_F64 ? 6 : 14;
    for (int zt : {1, 2, 4, 6, 8, 10, 12, 14}) {
      std::vector<int> seen;
      if (zt == s->ztile) seen.push_back(geom3d(s->p.nx, s->p.ny, s->p.nz, s->seg, zt).nsegs);
      for (int seg : {8, 12, 16, 24, 32, 43, 64, 86, 128, 256}) {
        if (zt > zmax || zt > s->p.nz || seg > std::max(8, s->p.ny) ||
            step3d_lds_bytes(s->p.nx, zt, sizeof(T)) > kMaxLds3D)
          continue;
        const int ns = geom3d(s->p.nx, s->p.ny, s->p.nz, seg, zt).nsegs;
        if (std::find(seen.begin(), seen.end(), ns) != seen.end()) continue;
        seen.push_back(ns);
        add(seg, zt);
      }
    }
  }
  const int k = pick_fastest((int)cand.size(), [&](int i, int m) {
    t.seg = cand[i].first;
    t.ztile = cand[i].second;
    return time_steps(s->stream, steps * m, [&](int n) { return step_impl<T>(&t, n); });
  });
  (void)hipStreamSynchronize(s->stream);
  (void)hipFree(t.ws);
  if (k < 0) return fail(PF_ERR_DEVICE, "autotune trial failed");
  s->seg = cand[k].first;
  s->ztile = cand[k].second;
  s->tuned = true;
  return PF_OK;
}

template <typename T>
int batch_autotune_impl(pf_batch *b, int steps) {
  PF_HIP(hipStreamSynchronize(b->stream));
  const int n = (int)b->s.size();
  std::vector<pf_solver> clones(n);
  int made = 0, rc = PF_OK;
  for (; made < n && rc == PF_OK; ++made) rc = clone_solver(b->s[made], clones[made]);
  if (rc != PF_OK) --made;
  pf_batch tb;
  tb.precision = b->precision;
  tb.frozen = b->frozen;
  tb.frame = b->frame;
  tb.multi = b->multi;
  tb.stream = b->stream;
  tb.table = nullptr;
  tb.map = nullptr;
  tb.graph_steps = 0;
  tb.cap = nullptr;
  tb.graph = nullptr;
  tb.gexec = nullptr;
  for (int i = 0; i < made; ++i) tb.s.push_back(&clones[i]);
  tb.expect.assign(made, -1);
  tb.seg.assign(made, 0);
  // candidate 0: the segment length in use (0 = each member's own)
  std::vector<int> cand = {b->seg_fixed};
  for (int seg : {4, 6, 8, 12, 16, 24, 32})
    if (seg != b->seg_fixed) cand.push_back(seg);
  int bseg = b->seg_fixed;
  if (rc == PF_OK) {
    const int k = pick_fastest((int)cand.size(), [&](int i, int mult) {
      tb.seg_fixed = cand[i];
      tb.expect.assign(made, -1);  // rebuild with this segment length
      return time_steps(b->stream, steps * mult, [&](int m) { return batch_step<T>(&tb, m); });
    });
    if (k < 0)
      rc = fail(PF_ERR_DEVICE, "batch autotune trial failed");
    else
      bseg = cand[k];
  }
  (void)hipStreamSynchronize(b->stream);
  if (tb.table) (void)hipFree(tb.table);
  if (tb.map) (void)hipFree(tb.map);
  for (int i = 0; i < made; ++i) (void)hipFree(clones[i].ws);
  if (rc != PF_OK) return rc;
  b->seg_fixed = bseg;
  rc = batch_build<T>(b);
  if (rc != PF_OK) return rc;
  return batch_capture<T>(b);
}

}  // namespace

extern "C" {

int pf_batch_create(pf_solver *const *solvers, int32_t n, pf_batch **out) {
  if (!solvers || n < 1 || !out) return fail(PF_ERR_ARG, "need n >= 1 solvers and an out pointer");
  for (int i = 0; i < n; ++i)
    if (!solvers[i]) return fail(PF_ERR_ARG, "solver is NULL");
  const pf_solver *s0 = solvers[0];
  for (int i = 0; i < n; ++i) {
    const pf_solver *s = solvers[i];
    if (s->p.dim != 2) return fail(PF_ERR_ARG, "batched stepping is 2D only");
    if (s->p.antitrapping != PF_AT_APPROX || s->p.divergence != PF_DIV_SHELLS)
      return fail(PF_ERR_ARG, "batched stepping runs the approximated current on shell divergences");
    if (s->p.dynamic_grains) return fail(PF_ERR_ARG, "batched stepping takes static grain maps");
    if (s->p.precision != s0->p.precision) return fail(PF_ERR_ARG, "mixed precisions in a batch");
    if ((s->p.lT > 0.0) != (s0->p.lT > 0.0) || (s->p.frame != 0) != (s0->p.frame != 0) ||
        (s->p.n_grains > 1) != (s0->p.n_grains > 1))
      return fail(PF_ERR_ARG, "a batch needs one kind: all frozen or all isothermal, all with or "
                              "without frame, all single- or all multi-grain");
    if (s->stream != s0->stream) return fail(PF_ERR_ARG, "solvers of a batch share one stream");
    for (int j = 0; j < i; ++j)
      if (solvers[j] == s) return fail(PF_ERR_ARG, "a solver appears twice in the batch");
  }
  pf_batch *b = new (std::nothrow) pf_batch();
  if (!b) return fail(PF_ERR_OOM, "host allocation failed");
  b->s.assign(solvers, solvers + n);
  b->precision = s0->p.precision;
  b->frozen = s0->p.lT > 0.0;
  b->frame = s0->p.frame != 0;
  b->multi = s0->p.n_grains > 1;
  b->stream = s0->stream;
  b->table = nullptr;
  b->map = nullptr;
  b->expect.assign(n, -1);
  b->seg.assign(n, 0);
  b->graph_steps = 0;
  b->seg_fixed = 0;
  b->graph = nullptr;
  b->gexec = nullptr;
  if (hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking) != hipSuccess) {
    delete b;
    return fail(PF_ERR_DEVICE, "capture stream creation failed");
  }
  int rc = b->precision == PF_F64 ? batch_build<double>(b) : batch_build<float>(b);
  if (rc != PF_OK) {
    pf_batch_destroy(b);
    return rc;
  }
  *out = b;
  return PF_OK;
}

int pf_batch_step(pf_batch *b, int64_t nsteps) {
  if (!b) return fail(PF_ERR_ARG, "batch is NULL");
  if (nsteps < 0) return fail(PF_ERR_ARG, "nsteps must be >= 0");
  return b->precision == PF_F64 ? batch_step<double>(b, nsteps) : batch_step<float>(b, nsteps);
}

int pf_batch_launch_waves(pf_batch *b, int64_t *waves) {
  if (!b || !waves) return fail(PF_ERR_ARG, "batch or waves is NULL");
  const int rc = b->precision == PF_F64 ? batch_refresh<double>(b) : batch_refresh<float>(b);
  if (rc != PF_OK) return rc;
  *waves = b->waves;
  return PF_OK;
}

int pf_batch_use_graph(pf_batch *b, int32_t steps_per_graph) {
  if (!b) return fail(PF_ERR_ARG, "batch is NULL");
  if (steps_per_graph < 0) return fail(PF_ERR_ARG, "steps_per_graph must be >= 0");
  if (steps_per_graph > 0 && steps_per_graph % (b->frame ? 6 : 2) != 0)
    return fail(PF_ERR_ARG, "steps_per_graph must be a multiple of 2 (6 with the moving frame)");
  b->graph_steps = steps_per_graph;
  PF_HIP(hipStreamSynchronize(b->stream));
  int rc = b->precision == PF_F64 ? batch_build<double>(b) : batch_build<float>(b);
  if (rc != PF_OK) return rc;
  return b->precision == PF_F64 ? batch_capture<double>(b) : batch_capture<float>(b);
}

void pf_batch_destroy(pf_batch *b) {
  if (!b) return;
  (void)hipStreamSynchronize(b->stream);
  batch_drop_graph(b);
  if (b->table) (void)hipFree(b->table);
  if (b->map) (void)hipFree(b->map);
  if (b->cap) (void)hipStreamDestroy(b->cap);
  delete b;
}

int pf_autotune(pf_solver *s, int32_t steps_per_trial, int32_t *seg, int32_t *ztile) {
  if (!s) return fail(PF_ERR_ARG, "solver is NULL");
  if (steps_per_trial < 1 || steps_per_trial > kMaxTrialSteps)
    return fail(PF_ERR_ARG, "steps_per_trial must be in [1, 2^20]");
  int rc = s->p.precision == PF_F64 ? autotune_impl<double>(s, steps_per_trial)
                                    : autotune_impl<float>(s, steps_per_trial);
  if (rc != PF_OK) return rc;
  if (seg) *seg = s->seg;
  if (ztile) *ztile = s->p.dim == 3 ? s->ztile : 1;
  return PF_OK;
}

int pf_batch_autotune(pf_batch *b, int32_t steps_per_trial, int32_t *seg) {
  if (!b) return fail(PF_ERR_ARG, "batch is NULL");
  if (steps_per_trial < 1 || steps_per_trial > kMaxTrialSteps)
    return fail(PF_ERR_ARG, "steps_per_trial must be in [1, 2^20]");
  int rc = b->precision == PF_F64 ? batch_autotune_impl<double>(b, steps_per_trial)
                                  : batch_autotune_impl<float>(b, steps_per_trial);
  if (rc != PF_OK) return rc;
  if (seg) *seg = b->seg_fixed;
  return PF_OK;
}

int pf_version(void) { return PF_VERSION; }

const char *pf_last_error(void) { return g_err.c_str(); }

double pf_stable_dt(const pf_params *p) {
  if (validate(p) != PF_OK) return -1.0;
  return stable_dt_for(p, f1_min(p));
}

size_t pf_workspace_bytes(const pf_params *p) {
  if (validate(p) != PF_OK) return 0;
  return layout_of(p).total;
}

int pf_create(const pf_params *p, const pf_init *init, void *workspace, size_t workspace_bytes,
              void *stream, pf_solver **out) {
  int rc = validate(p);
  if (rc != PF_OK) return rc;
  if (!init || !init->psi || !init->U) return fail(PF_ERR_ARG, "init arrays are NULL");
  if (!out) return fail(PF_ERR_ARG, "out is NULL");
  const size_t n = cells(p);
  const size_t least = least_pieces_in(p->precision == PF_F64 ? 8 : 4);
  std::atomic<bool> bad{false};
  host_parallel(n, kHostGrainIn, least, [&](size_t b, size_t e) {
    const double *psi = init->psi, *U = init->U;
    int any = 0;  // no branch on a cell, so the loop vectorises (half the time)
    for (size_t i = b; i < e; ++i)
      any |= (int)!(fabs(psi[i]) <= DBL_MAX) | (int)!(fabs(U[i]) <= DBL_MAX);
    if (any) bad.store(true, std::memory_order_relaxed);
  });
  if (bad.load()) return fail(PF_ERR_NONFINITE, "initial psi or U holds NaN or Inf");
  if (init->grain) {
    host_parallel(n, kHostGrainIn, least, [&](size_t b, size_t e) {
      const int8_t *g = init->grain;
      const int ng = p->n_grains;
      int any = 0;
      for (size_t i = b; i < e; ++i) any |= (int)(g[i] < 0) | (int)(g[i] >= ng);
      if (any) bad.store(true, std::memory_order_relaxed);
    });
    if (bad.load()) return fail(PF_ERR_ARG, "grain index outside [0, n_grains)");
    if (p->frame && !p->dynamic_grains) {  // a static map does not shift with the frame
      const int nx = p->nx, ny = p->ny, nz = p->dim == 3 ? p->nz : 1;
      for (int l = 0; l < nz; ++l)
        for (int j = 1; j < ny; ++j)
          for (int i = 0; i < nx; ++i)
            if (init->grain[((size_t)l * ny + j) * nx + i] != init->grain[(size_t)l * ny * nx + i])
              return fail(PF_ERR_ARG, "with the moving frame the grain map must not vary along y");
    }
  }
  double lambda = p->lambda > 0.0 ? p->lambda : p->D / kA2;
  double dtmax = pf_stable_dt(p);
  double dt = p->dt > 0.0 ? p->dt : 0.8 * dtmax;
  if (dt > dtmax * (1.0 + 1e-12))
    return fail(PF_ERR_UNSTABLE_DT, "dt = " + std::to_string(dt) + " exceeds the stability limit " +
                                        std::to_string(dtmax));
  Layout L = layout_of(p);
  pf_solver *s = new (std::nothrow) pf_solver();
  if (!s) return fail(PF_ERR_OOM, "host allocation failed");
  s->p = *p;
  s->rot.assign(p->grain_rot, p->grain_rot + 9 * p->n_grains);
  if (p->dim == 2) upright_2d(s->rot);
  s->p.grain_rot = s->rot.data();
  weights_of(p, s->w);
  s->lambda = lambda;
  s->dt = dt;
  s->n = n;
  s->stream = reinterpret_cast<hipStream_t>(stream);
  s->L = L;
  s->cur = 0;
  s->fcur = 0;
  s->step = 0;
  s->have_prev = false;
  s->tuned = false;
  if (workspace) {
    if (workspace_bytes < L.total || (reinterpret_cast<uintptr_t>(workspace) & 255u)) {
      delete s;
      return fail(PF_ERR_OOM, "workspace smaller than pf_workspace_bytes() or not 256-byte aligned");
    }
    s->ws = reinterpret_cast<char *>(workspace);
    s->ws_bytes = workspace_bytes;
    s->own = false;
  } else {
    void *d = nullptr;
    if (hipMalloc(&d, L.total) != hipSuccess) {
      delete s;
      return fail(PF_ERR_OOM, "hipMalloc of " + std::to_string(L.total) + " bytes failed");
    }
    s->ws = reinterpret_cast<char *>(d);
    s->ws_bytes = L.total;
    s->own = true;
  }
  int r2 = PF_OK;
  {
    int dev = 0;
    s->ncu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&s->ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        s->ncu < 1)
      r2 = fail(PF_ERR_DEVICE, "cannot read the device's compute unit count");
  }
  std::tie(s->seg, s->ztile) = default_geom(p, s->ncu);
  if (r2 == PF_OK)
    r2 = p->precision == PF_F64 ? upload<double>(s, init) : upload<float>(s, init);
  if (r2 == PF_OK && p->n_grains > 1) {
    std::vector<int8_t> g(n, 0);
    if (init->grain) memcpy(g.data(), init->grain, n);
    if (hipMemcpy(s->ws + L.grain, g.data(), n, hipMemcpyHostToDevice) != hipSuccess)
      r2 = fail(PF_ERR_DEVICE, "grain upload failed");
  }
  if (r2 == PF_OK) {
    FrameState z{0, 0, 0};
    if (hipMemcpy(s->ws + L.frame[0], &z, sizeof(z), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(s->ws + L.frame[1], &z, sizeof(z), hipMemcpyHostToDevice) != hipSuccess ||
        hipMemcpy(s->ws + L.frame[2], &z, sizeof(z), hipMemcpyHostToDevice) != hipSuccess)
      r2 = fail(PF_ERR_DEVICE, "state initialisation failed");
  }
  if (r2 != PF_OK) {
    if (s->own) (void)hipFree(s->ws);
    delete s;
    return r2;
  }
  *out = s;
  return PF_OK;
}

int pf_step(pf_solver *s, int64_t nsteps) {
  if (!s) return fail(PF_ERR_ARG, "solver is NULL");
  if (nsteps < 0) return fail(PF_ERR_ARG, "nsteps must be >= 0");
  return s->p.precision == PF_F64 ? step_impl<double>(s, nsteps) : step_impl<float>(s, nsteps);
}

int pf_step_diffusion(pf_solver *s, int64_t nsteps) {
  if (!s) return fail(PF_ERR_ARG, "solver is NULL");
  if (nsteps < 0) return fail(PF_ERR_ARG, "nsteps must be >= 0");
  if (s->p.dim != 2) return fail(PF_ERR_ARG, "the diffusion-only step is 2D only");
  if (s->p.divergence != PF_DIV_SHELLS)
    return fail(PF_ERR_ARG, "the diffusion-only step uses the shell divergence");
  return s->p.precision == PF_F64 ? step_impl<double>(s, nsteps, true)
                                  : step_impl<float>(s, nsteps, true);
}

int pf_synchronize(pf_solver *s) {
  if (!s) return fail(PF_ERR_ARG, "solver is NULL");
  PF_HIP(hipStreamSynchronize(s->stream));
  return PF_OK;
}

int pf_read_fields(pf_solver *s, double *phi, double *U, double *psi, int8_t *grain) {
  if (!s) return fail(PF_ERR_ARG, "solver is NULL");
  int rc = s->p.precision == PF_F64 ? read_impl<double>(s, phi, U, psi)
                                    : read_impl<float>(s, phi, U, psi);
  if (rc != PF_OK) return rc;
  if (grain) {
    if (s->p.dynamic_grains) {
      // the current level's map, with the frame shift it may still owe
      FrameState fr;
      PF_HIP(hipMemcpy(&fr, s->ws + s->L.frame[s->fcur], sizeof(fr), hipMemcpyDeviceToHost));
      std::vector<int8_t> hg(s->n);
      PF_HIP(hipMemcpy(hg.data(), grain_buf(s, s->cur), s->n, hipMemcpyDeviceToHost));
      const int nx = s->p.nx, ny = s->p.ny, nz = s->p.dim == 3 ? s->p.nz : 1;
      for (int l = 0; l < nz; ++l)
        for (int j = 0; j < ny; ++j) {
          int jp = (s->p.frame && fr.pending) ? std::min(j + 1, ny - 1) : j;
          memcpy(grain + ((size_t)l * ny + j) * nx, hg.data() + ((size_t)l * ny + jp) * nx, nx);
        }
    } else if (s->p.n_grains > 1) {
      PF_HIP(hipMemcpy(grain, s->ws + s->L.grain, s->n, hipMemcpyDeviceToHost));
    } else {
      memset(grain, 0, s->n);
    }
  }
  return PF_OK;
}

int pf_tip_state(pf_solver *s, pf_tip *out) {
  if (!s || !out) return fail(PF_ERR_ARG, "solver or out is NULL");
  TipResult r;
  FrameState fr;
  int rc = s->p.precision == PF_F64 ? reduce_impl<double>(s, &r, &fr)
                                    : reduce_impl<float>(s, &r, &fr);
  if (rc != PF_OK) return rc;
  const pf_params &p = s->p;
  pf_tip t;
  memset(&t, 0, sizeof(t));
  t.step = s->step;
  t.t = (double)s->step * s->dt;
  t.found = r.found;
  t.nonfinite = r.bad ? 1 : 0;
  t.frame_shift = fr.base + fr.pending;
  t.solid_fraction = r.fs_sum / (double)s->n;
  if (r.found) {
    const long long nx = p.nx, ny = p.ny;
    t.index = r.idx;
    t.x = (double)(r.idx % nx) * p.h;
    t.z = p.dim == 3 ? (double)(r.idx / (nx * ny)) * p.h : 0.0;
    t.y_frame = r.y;
    t.y_lab = r.y + (double)t.frame_shift * p.h;
    if (s->have_prev && t.t > s->prev_t) t.velocity = (t.y_lab - s->prev_y) / (t.t - s->prev_t);
    s->have_prev = true;
    s->prev_t = t.t;
    s->prev_y = t.y_lab;
  } else {
    t.index = -1;
  }
  *out = t;
  if (r.bad) return fail(PF_ERR_NONFINITE, "state holds NaN or Inf values");
  if (p.lT > 0.0) {
    // the thermal coordinate has moved with the frame shift and the clock:
    // F1 must stay positive and dt within the limit it sets
    const double f1 = f1_min_at(&p, (double)t.frame_shift * p.h - p.y0 - p.Vp * t.t);
    if (!(f1 > 0.0))
      return fail(PF_ERR_UNSTABLE_DT, "F1 = 1 - (1-k) zeta / lT is no longer positive over the "
                                      "lattice (frame shift " + std::to_string(t.frame_shift) +
                                      ", t = " + std::to_string(t.t) + ")");
    const double dtmax = stable_dt_for(&p, f1);
    if (s->dt > dtmax * (1.0 + 1e-12))
      return fail(PF_ERR_UNSTABLE_DT, "dt = " + std::to_string(s->dt) +
                                          " now exceeds the stability limit " +
                                          std::to_string(dtmax) + " (F1 min " +
                                          std::to_string(f1) + ")");
  }
  return PF_OK;
}

int pf_device_fields(pf_solver *s, void **psi, void **U) {
  if (!s) return fail(PF_ERR_ARG, "solver is NULL");
  if (psi) *psi = s->ws + s->L.psi[s->cur];
  if (U) *U = s->ws + s->L.U[s->cur];
  return PF_OK;
}

int pf_frame_state(pf_solver *s, int64_t *shift, int32_t *pending) {
  if (!s) return fail(PF_ERR_ARG, "solver is NULL");
  FrameState fr;
  PF_HIP(hipStreamSynchronize(s->stream));
  PF_HIP(hipMemcpy(&fr, s->ws + s->L.frame[s->fcur], sizeof(fr), hipMemcpyDeviceToHost));
  if (shift) *shift = fr.base + fr.pending;
  if (pending) *pending = fr.pending;
  return PF_OK;
}

int pf_tune(pf_solver *s, int32_t rows_per_segment, int32_t z_tile) {
  if (!s) return fail(PF_ERR_ARG, "solver is NULL");
  if (s->p.dim == 2 && rows_per_segment >= -64 && rows_per_segment <= -1) {
    s->seg = rows_per_segment;  // -k: k waves per SIMD
    s->tuned = true;
    return PF_OK;
  }
  if (rows_per_segment < 4 || rows_per_segment > 256)
    return fail(PF_ERR_ARG, s->p.dim == 2 ? "rows_per_segment must lie in [4, 256] or [-64, -1]"
                                          : "rows_per_segment must lie in [4, 256]");
  if (s->p.dim == 3 && (z_tile < 1 || z_tile > 14))
    return fail(PF_ERR_ARG, "z_tile must lie in [1, 14]");
  if (s->p.dim == 3 && s->p.precision == PF_F64 && z_tile > 6)
    return fail(PF_ERR_ARG, "FP64 3D workgroups hold at most 6 z rows (8 waves)");
  if (s->p.dim == 3 &&
      step3d_lds_bytes(s->p.nx, z_tile, s->p.precision == PF_F64 ? 8 : 4) > kMaxLds3D)
    return fail(PF_ERR_ARG, "z_tile too large for the LDS of one workgroup at this precision");
  s->seg = rows_per_segment;
  s->tuned = true;
  if (s->p.dim == 3) s->ztile = z_tile;
  return PF_OK;
}

int pf_launch_waves(pf_solver *s, int64_t *waves) {
  if (!s || !waves) return fail(PF_ERR_ARG, "solver or waves is NULL");
  *waves = solo_waves(s->p, s->seg, s->ztile, s->ncu);
  return PF_OK;
}

int pf_default_waves(const pf_params *p, int32_t cus, double batch_load, int64_t *waves) {
  const int rc = validate(p);
  if (rc != PF_OK) return rc;
  if (!waves || cus < 1) return fail(PF_ERR_ARG, "need cus >= 1 and a waves pointer");
  const auto geo = default_geom(p, cus);
  if (!(batch_load >= 0.0)) {
    *waves = solo_waves(*p, geo.first, geo.second, cus);
    return PF_OK;
  }
  if (p->dim != 2) return fail(PF_ERR_ARG, "batched stepping is 2D only");
  const Geom2D g = member_geom2d(*p, geo.first, cus, batch_rows2d(batch_load));
  *waves = (int64_t)g.nstrips * g.nsegs;
  return PF_OK;
}

int pf_geometry(pf_solver *s, int32_t *rows_per_segment, int32_t *z_tile) {
  if (!s) return fail(PF_ERR_ARG, "solver is NULL");
  if (rows_per_segment) *rows_per_segment = s->seg;
  if (z_tile) *z_tile = s->p.dim == 3 ? s->ztile : 1;
  return PF_OK;
}

void pf_destroy(pf_solver *s) {
  if (!s) return;
  (void)hipStreamSynchronize(s->stream);
  if (s->own) (void)hipFree(s->ws);
  delete s;
}

}  // extern "C"
