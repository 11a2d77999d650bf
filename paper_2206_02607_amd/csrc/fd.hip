// Full-order explicit finite-difference heat solver in FP64 (Sec.
// "Thermodynamics / Full-order Model": 3-point Laplacian; Sec. "Image
// Processing / Full-order Model": 5-point Laplacian; forward Euler; zero
// Dirichlet boundary).  It generates training snapshots, judges reduced-order
// rollouts and is the fallback when a latent step fails.
//
// Grids are batched: `n_grid` independent fields of the same shape, one
// after another.  1D fields take one launch per substep; 2D fields advance
// many substeps per launch in registers, except many small or narrow fields
// and single substeps, which take one launch each too.
#include "common.hpp"

// Evaluate exactly in the written order (no fused multiply-add), so that the
// solver reproduces a plain double-precision evaluation of the same formula.
#pragma clang fp contract(off)

namespace crom {

// One substep on a batch of 1D fields [n_grid][n]: u_out = u + dt nu Lap u,
// end nodes held at 0.
__global__ void fd1d_kernel(const double* __restrict__ u, double* __restrict__ v,
                            const double* __restrict__ nu, int nu_per_node, int64_t n, int64_t n_grid,
                            double dt, double dx2) {
  const int64_t total = n * n_grid;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < total;
       k += (int64_t)gridDim.x * blockDim.x) {
    const int64_t gidx = k / n, i = k - gidx * n;
    double out = 0.0;
    if (i > 0 && i < n - 1) {
      // boundary nodes count as 0 whatever the input holds there
      const double c = u[k];
      const double l = i - 1 > 0 ? u[k - 1] : 0.0;
      const double r = i + 1 < n - 1 ? u[k + 1] : 0.0;
      const double lap = ((l + r) - 2.0 * c) / dx2;
      const double nv = nu_per_node ? nu[k] : nu[gidx];
      out = c + (dt * nv) * lap;
    }
    v[k] = out;
  }
}

// One substep on a batch of 2D fields [n_grid][nx][ny] (index [i_x][i_y]).
__global__ void fd2d_step_kernel(const double* __restrict__ u, double* __restrict__ v, const double* __restrict__ nu,
                                 int nu_per_node, int64_t nx, int64_t ny, int64_t n_grid, double dt, double dx2) {
  const int64_t plane = nx * ny, total = plane * n_grid;
  for (int64_t k = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; k < total; k += (int64_t)gridDim.x * blockDim.x) {
    const int64_t gidx = k / plane, r = k - gidx * plane;
    const int64_t i = r / ny, j = r - i * ny;
    double out = 0.0;
    if (i > 0 && i < nx - 1 && j > 0 && j < ny - 1) {
      const double c = u[k];
      const double xm = i - 1 > 0 ? u[k - ny] : 0.0, xp = i + 1 < nx - 1 ? u[k + ny] : 0.0;
      const double ym = j - 1 > 0 ? u[k - 1] : 0.0, yp = j + 1 < ny - 1 ? u[k + 1] : 0.0;
      const double lap = ((((xm + xp) + ym) + yp) - 4.0 * c) / dx2;
      const double nv = nu_per_node ? nu[k] : nu[gidx];
      out = c + (dt * nv) * lap;
    }
    v[k] = out;
  }
}

// 2D fields, `sub` substeps per launch.
//
// A launch per substep was bound by the launch, not by memory: 40 fields of
// 128 x 128 (10 MB read and written) took 6.3 us a substep, where the copy
// rate would allow 2.  So a workgroup takes a tile of FD_ROWS x FD_COLS
// nodes into registers and advances it `sub` substeps before it writes those
// nodes back that are at least `halo` >= sub away from the tile's open
// edges (sides that are not the field's boundary); the rest of the tile is
// recomputed by its neighbours.  A wave holds FD_R whole rows, two columns
// per lane: x neighbours are the lane's own registers, y neighbours come
// from the adjacent lanes (whole-wave DPP shifts), and only each wave's
// first and last row pass through LDS, double-buffered, one barrier per
// substep.  What bounds it then is the FP64 vector rate: ten operations and
// two shifts per node and substep (a resident tile takes 0.89 us a substep,
// of which those operations fill 0.74).  The 5,000 substeps of 40 fields of
// 128 x 128 went from 34.2 to 5.6 ms (same box).  Four rows per wave: with eight, the
// two copies of the loop body spill at four waves per SIMD (1.76 us a
// substep against 1.39, halo 16).
//
// The division by dx^2 is the longest part of the formula.  Its exact result
// comes from the reciprocal in two parts (yh + yl = 1/dx^2 to 2^-106):
// q = a yh + a yl is the quotient to less than one ulp, so its residual
// a - q dx^2 is exact and q + residual yh is the correctly rounded quotient
// (Markstein, "Computation of elementary functions on the IBM RISC System/
// 6000 processor", 1990).  That needs a clear of the underflow and overflow
// thresholds: the field is carried times 2^400 (exact), and a tile that ends
// with a non-finite value (or a dx^2 beyond 2^+-200) is done again from its input with the division
// itself and no scaling (EXACT).  Only results in the denormal range can
// differ from the plain evaluation, by their last places.
constexpr int FD_R = 4, FD_WAVES = 16, FD_ROWS = FD_R * FD_WAVES, FD_COLS = 128;

struct Fd2dArgs {
  const double* u;
  double* v;
  const double* nu;
  int64_t nx, ny;
  uint32_t nty, per_field, tiles;  // per_field = ntx * nty, tiles = per_field * n_grid
  int sub, halo;
  int plain;  // the division itself throughout
  int pairs;  // 16-byte accesses of two columns
  double dt, dx2, yh, yl;
};

// Lane l's neighbour value (l - 1: CTRL 0x138, l + 1: CTRL 0x130), 0 past the wave.
template <int CTRL>
__device__ __forceinline__ double fd_lane(double v) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(v);
  const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
  const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Tile t of one axis with n nodes and T nodes per tile: its first node, and
// the range [lo, hi) of tile positions it writes back.
__device__ __forceinline__ void fd_tile(int64_t n, int T, int halo, int64_t t, int64_t& x0, int& lo, int& hi) {
  x0 = t * (T - 2 * halo);
  if (x0 + T > n) x0 = n > T ? n - T : 0;
  lo = x0 > 0 ? halo : 0;
  hi = x0 + T < n ? T - halo : (int)(n - x0);
}

// The tile's rows r0 .. r0 + FD_R - 1 and columns c0, c0 + 1 of this lane,
// loaded and advanced a.sub substeps.  Row r sits in slot r + 1 of u before
// an even substep and in slot r before an odd one: with one spare slot and
// the rows taken upwards, then downwards, a new row takes the place of one
// that is no longer needed, and no registers are copied.
template <bool PN, bool EXACT>
__device__ __forceinline__ void fd2d_advance(const Fd2dArgs& a, int64_t g, int64_t r0, int64_t c0,
                                             double (&u)[FD_R + 1][2], double (*edge)[FD_WAVES][2][FD_COLS]) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const double scale = EXACT ? 1.0 : 0x1p400;
  bool cin[2], rin[FD_R];  // interior columns and rows: other nodes are held at 0
  double k[PN ? FD_R : 1][2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    cin[e] = c0 + e > 0 && c0 + e < a.ny - 1;
    if constexpr (!PN) k[0][e] = cin[e] ? a.dt * a.nu[g] : 0.0;
  }
#pragma unroll
  for (int r = 0; r < FD_R; ++r) {  // clamped, branch-free: all loads issue at once
    const int64_t i = r0 + r, row = (g * a.nx + (i < a.nx ? i : a.nx - 1)) * a.ny;
    rin[r] = i > 0 && i < a.nx - 1;
    if (a.pairs) {  // ny even: both columns or neither, 16-byte aligned
      const double2 v = *reinterpret_cast<const double2*>(&a.u[row + (c0 < a.ny ? c0 : 0)]);
      u[r + 1][0] = v.x;
      u[r + 1][1] = v.y;
    } else {
#pragma unroll
      for (int e = 0; e < 2; ++e) u[r + 1][e] = a.u[row + (c0 + e < a.ny ? c0 + e : a.ny - 1)];
    }
    if constexpr (PN) {
#pragma unroll
      for (int e = 0; e < 2; ++e) k[r][e] = a.dt * a.nu[row + (c0 + e < a.ny ? c0 + e : a.ny - 1)];
    }
  }
#pragma unroll
  for (int r = 0; r < FD_R; ++r)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      u[r + 1][e] = cin[e] && rin[r] ? u[r + 1][e] * scale : 0.0;
      if constexpr (PN) k[r][e] = cin[e] && rin[r] ? k[r][e] : 0.0;
    }
  // one substep; ROWS: every row of the wave is interior
  auto advance = [&](auto rows, auto up) {
    constexpr bool ROWS = decltype(rows)::value, UP = decltype(up)::value;
    constexpr int S = UP ? 1 : 0;  // row r: slot r + S before, r + 1 - S after
    double(*eb)[2][FD_COLS] = edge[S];
    *reinterpret_cast<double2*>(&eb[wave][0][2 * lane]) = double2{u[S][0], u[S][1]};
    *reinterpret_cast<double2*>(&eb[wave][1][2 * lane]) = double2{u[FD_R - 1 + S][0], u[FD_R - 1 + S][1]};
    __syncthreads();
    double2 lo = {0.0, 0.0}, hi = {0.0, 0.0};  // the rows below r0 and above r0 + FD_R - 1
    if (wave > 0) lo = *reinterpret_cast<const double2*>(&eb[wave - 1][1][2 * lane]);
    if (wave < FD_WAVES - 1) hi = *reinterpret_cast<const double2*>(&eb[wave + 1][0][2 * lane]);
#pragma unroll
    for (int t = 0; t < FD_R; ++t) {
      const int r = UP ? t : FD_R - 1 - t;
      const double v0 = u[r + S][0], v1 = u[r + S][1];
      const double ym[2] = {fd_lane<0x138>(v1), v0}, yp[2] = {v1, fd_lane<0x130>(v0)};
      double o[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const double c = u[r + S][e];
        const double xm = r > 0 ? u[r > 0 ? r - 1 + S : 0][e] : (e ? lo.y : lo.x);
        const double xp = r + 1 < FD_R ? u[r + 1 < FD_R ? r + 1 + S : 0][e] : (e ? hi.y : hi.x);
        const double n4 = ((xm + xp) + ym[e]) + yp[e];
        const double kk = k[PN ? r : 0][e];
        if constexpr (EXACT) {
          o[e] = c + kk * ((n4 - 4.0 * c) / a.dx2);
        } else {
          const double d = fma(-4.0, c, n4);  // 4 c is exact
          const double q = fma(d, a.yh, d * a.yl);
          o[e] = c + kk * fma(fma(-q, a.dx2, d), a.yh, q);  // boundary columns: 0 + 0 lap
        }
        if constexpr (EXACT) o[e] = cin[e] ? o[e] : 0.0;
        if constexpr (EXACT || !ROWS) o[e] = rin[r] ? o[e] : 0.0;
      }
      u[r + 1 - S][0] = o[0];
      u[r + 1 - S][1] = o[1];
    }
  };
  auto sweep = [&](auto rows) {
    int s = 0;
    for (; s + 1 < a.sub; s += 2) {
      advance(rows, std::true_type{});
      advance(rows, std::false_type{});
    }
    if (s < a.sub) {
      advance(rows, std::true_type{});
#pragma unroll
      for (int r = FD_R; r > 0; --r)
#pragma unroll
        for (int e = 0; e < 2; ++e) u[r][e] = u[r - 1][e];
    }
  };
  if (!EXACT && __builtin_amdgcn_readfirstlane((int)(r0 > 0 && r0 + FD_R < a.nx))) sweep(std::true_type{});
  else sweep(std::false_type{});
}

template <bool PN>
__global__ __launch_bounds__(FD_WAVES * 64) __attribute__((amdgpu_waves_per_eu(4))) void fd2d_kernel(Fd2dArgs a) {
  __shared__ __align__(16) double edge[2][FD_WAVES][2][FD_COLS];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (uint32_t t = blockIdx.x; t < a.tiles; t += gridDim.x) {
    const uint32_t g = t / a.per_field, ti = t - g * a.per_field, tx = ti / a.nty, ty = ti - tx * a.nty;
    int64_t x0, y0;
    int xlo, xhi, ylo, yhi;
    fd_tile(a.nx, FD_ROWS, a.halo, tx, x0, xlo, xhi);
    fd_tile(a.ny, FD_COLS, a.halo, ty, y0, ylo, yhi);
    const int64_t r0 = x0 + wave * FD_R, c0 = y0 + 2 * lane;
    double u[FD_R + 1][2];
    fd2d_advance<PN, false>(a, g, r0, c0, u, edge);
    const int i0 = wave * FD_R, j0 = 2 * lane;
    const bool col[2] = {j0 >= ylo && j0 < yhi, j0 + 1 >= ylo && j0 + 1 < yhi};  // written back
    bool bad = a.plain != 0;
#pragma unroll
    for (int r = 0; r < FD_R; ++r)
#pragma unroll
      for (int e = 0; e < 2; ++e)
        bad |= col[e] && i0 + r >= xlo && i0 + r < xhi && !(fabs(u[r + 1][e]) < 0x1p1000);
    double scale = 0x1p-400;
    if (__syncthreads_or(bad)) {  // nothing is written yet: the input is still there, in place too
      fd2d_advance<PN, true>(a, g, r0, c0, u, edge);
      scale = 1.0;
    }
#pragma unroll
    for (int r = 0; r < FD_R; ++r)
      if (i0 + r >= xlo && i0 + r < xhi) {
        double* v = &a.v[(g * a.nx + r0 + r) * a.ny + c0];
        if (a.pairs && col[0] && col[1]) {
          *reinterpret_cast<double2*>(v) = double2{u[r + 1][0] * scale, u[r + 1][1] * scale};
        } else {
#pragma unroll
          for (int e = 0; e < 2; ++e)
            if (col[e]) v[e] = u[r + 1][e] * scale;
        }
      }
    __syncthreads();  // the edge rows are read before the next tile writes them
  }
}

// Tiles along one axis of n nodes for tiles of T nodes with `halo` open nodes.
static int64_t fd_tiles(int64_t n, int T, int halo) {
  return n <= T ? 1 : (n - T + (T - 2 * halo) - 1) / (T - 2 * halo) + 1;
}

// Launches of the tile kernel for a number of substeps: between tiles they
// alternate u -> scratch -> u, an even number of them.
static int64_t fd2d_launches(int halo, int64_t steps) {
  return halo == 0 ? (steps + 4095) / 4096 : ((steps + halo - 1) / halo + 1) / 2 * 2;
}

// Halo of the tiles (0: a field is one tile), or -1 where a launch per substep
// is faster.  Either kind of launch takes about 4 us and 4 us per million
// nodes (loads and stores); tiles add 0.89 us per substep for each round of
// tiles over the 256 compute units, however few of a tile's nodes there are.
// Measured, us a substep by launches and by tiles: 16,384 fields of 16 x 16
// 18.2 and 58.7, 4,096 of 32 x 32 17.3 and 14.5; 2,048 of 8 x 8 3.8 and 7.5,
// 300 of 16 x 16 3.9 and 1.9; one field of 100,000 x 8 6.0 and 12.0.  Two
// substeps of 200 fields of 128 x 128: 32 and 40 us, three: 59 and 42.
static int fd2d_halo(int64_t nx, int64_t ny, int64_t n_grid, int64_t steps) {
  auto tiles = [&](int h) { return (double)fd_tiles(nx, FD_ROWS, h) * (double)fd_tiles(ny, FD_COLS, h) * (double)n_grid; };
  auto rounds = [&](int h) { return ceil(tiles(h) / 256.0); };
  // Substeps per launch: more of them share one launch, but widen the
  // recomputed halo and so the number of tiles.  A field that is one tile
  // needs no halo and runs its substeps in place, up to 4,096 per launch.
  int halo = 0;
  if (fd_tiles(nx, FD_ROWS, 0) * fd_tiles(ny, FD_COLS, 0) > 1) {
    double best = 0.0;
    for (int h : {8, 12, 16, 20, 24, 28}) {
      const double cost = 0.89 * rounds(h) + 8.0 / h;
      if (halo == 0 || cost < best) {
        best = cost;
        halo = h;
      }
    }
  }
  const double launch = 4.0 + 4e-6 * (double)nx * (double)ny * (double)n_grid;
  const double by_tiles = (double)fd2d_launches(halo, steps) * launch + 0.89 * rounds(halo) * (double)steps;
  const double by_steps = (double)(steps + steps % 2) * launch;  // an odd number ends with a copy
  return by_tiles <= by_steps && tiles(halo) < 2147483648.0 ? halo : -1;
}

static crom_status fd2d_run(int halo, int64_t nx, int64_t ny, int64_t n_grid, const double* nu, int nu_per_node, double dx2,
                            double dt, int64_t steps, double* u, double* scratch, hipStream_t st) {
  Fd2dArgs a{};
  a.nu = nu;
  a.nx = nx;
  a.ny = ny;
  const int64_t nty = fd_tiles(ny, FD_COLS, halo), per_field = fd_tiles(nx, FD_ROWS, halo) * nty;
  a.nty = (uint32_t)nty;
  a.per_field = (uint32_t)per_field;
  a.tiles = (uint32_t)(per_field * n_grid);
  a.pairs = ny % 2 == 0 && (reinterpret_cast<uintptr_t>(u) | reinterpret_cast<uintptr_t>(scratch)) % 16 == 0;
  a.halo = halo;
  a.plain = !(dx2 > 0x1p-200 && dx2 < 0x1p200);
  a.dt = dt;
  a.dx2 = dx2;
  a.yh = 1.0 / dx2;
  a.yl = fma(-a.yh, dx2, 1.0) / dx2;
  const uint32_t grid = a.tiles < 65536 ? a.tiles : 65536;
  const int64_t launches = fd2d_launches(halo, steps);  // the substeps shared out evenly
  for (int64_t l = 0; l < launches; ++l) {
    a.u = halo == 0 || l % 2 == 0 ? u : scratch;
    a.v = halo == 0 || l % 2 == 1 ? u : scratch;
    a.sub = (int)(steps / launches + (l < steps % launches ? 1 : 0));
    if (nu_per_node) hipLaunchKernelGGL(fd2d_kernel<true>, dim3(grid), dim3(FD_WAVES * 64), 0, st, a);
    else hipLaunchKernelGGL(fd2d_kernel<false>, dim3(grid), dim3(FD_WAVES * 64), 0, st, a);
  }
  return hip_check(hipGetLastError(), "fd launch");
}

}  // namespace crom

using namespace crom;

extern "C" {

crom_status crom_fd_heat(int32_t dim, const int64_t* shape, int64_t n_grid, const double* nu,
                         int32_t nu_per_node, double dx, double dt, int64_t steps, double* u,
                         double* scratch, void* stream) {
  if (dim != 1 && dim != 2) return fail(CROM_ERR_INVALID_ARG, "dim must be 1 or 2");
  if (!shape) return fail(CROM_ERR_INVALID_ARG, "shape is NULL");
  const int64_t nx = shape[0], ny = dim == 2 ? shape[1] : 1;
  if (nx < 1 || ny < 1 || n_grid < 0 || steps < 0) return fail(CROM_ERR_INVALID_ARG, "negative size");
  if (!(dx > 0.0) || !(dt >= 0.0)) return fail(CROM_ERR_INVALID_ARG, "dx must be positive, dt non-negative");
  const int64_t total = nx * ny * n_grid;
  if (total == 0 || steps == 0) return CROM_OK;
  if (!u || !scratch || !nu) return fail(CROM_ERR_INVALID_ARG, "u, scratch and nu are required");
  hipStream_t st = static_cast<hipStream_t>(stream);
  const double dx2 = dx * dx;
  if (dim == 2) {
    const int halo = fd2d_halo(nx, ny, n_grid, steps);
    if (halo >= 0) return fd2d_run(halo, nx, ny, n_grid, nu, nu_per_node, dx2, dt, steps, u, scratch, st);
  }
  const int threads = 256;
  int64_t blocks = (total + threads - 1) / threads;
  if (blocks > 65536) blocks = 65536;
  double* a = u;
  double* b = scratch;
  for (int64_t s = 0; s < steps; ++s) {
    if (dim == 1)
      hipLaunchKernelGGL(fd1d_kernel, dim3((unsigned)blocks), dim3(threads), 0, st, a, b, nu, nu_per_node, nx, n_grid,
                         dt, dx2);
    else
      hipLaunchKernelGGL(fd2d_step_kernel, dim3((unsigned)blocks), dim3(threads), 0, st, a, b, nu, nu_per_node, nx, ny,
                         n_grid, dt, dx2);
    double* t = a;
    a = b;
    b = t;
  }
  crom_status s = hip_check(hipGetLastError(), "fd launch");
  if (s != CROM_OK) return s;
  if (a != u) s = hip_check(hipMemcpyAsync(u, a, total * sizeof(double), hipMemcpyDeviceToDevice, st), "copy");
  return s;
}

}  // extern "C"
