// Direct solution of the periodic 7-point Poisson problem by Hartley
// transforms along the three axes (spectral.h).
//
// Why: the discrete problem A psi = b has constant coefficients on a periodic
// box (uniform permittivity, also inside solids), so its exact solution costs
// a fixed handful of passes over the field, where a multigrid solve to 1e-8
// from the time loop's extrapolated start takes two to three cycles of about
// ten passes (and a dozen launches) each.
//
// One cycle is: the residual r = b + shift - A x (with its norms) transformed
// along x and y; along z, divided by the eigenvalues, and back along z; back
// along y and x and added to x.  On the start it reduces the residual to
// rounding, so the time loop takes one cycle; a tolerance below that is met
// by iterative refinement or reported.
//
// Layout: lines are transformed in LDS.  Where a whole plane of the grid fits
// there (up to 128 x 128), x and y go in one kernel, a workgroup per plane,
// and a cycle reads and writes the field three times (bound by the launches
// on the boxes whose field is cache resident).  Larger planes take x in
// tiles of 16 rows and y in tiles of 16 columns (128-byte segments): five
// passes, bound by HBM.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <type_traits>
#include <vector>

#include "ek_context.h"
#include "reduce.h"
#include "spectral.h"

using namespace ek;

namespace {

constexpr int TILE = 16;             // rows or columns of a tile (8 complex lines)
constexpr int TILE_PS = TILE / 2 + 1;   // odd row length: the passes' strided writes spread over the banks
constexpr size_t PLANE_LDS_MAX = 150 * 1024;

struct SpecArgs {
  int nx, ny, nz;
  DhtPlan px, py, pz;
  const double2 *tx, *ty, *tz;
  const double *lx, *ly, *lz;
  double* hat;
  double h2, inv_n;
  const SpecItem* items;       // several problems: this block's is items[blockIdx.y]
};

SpecArgs args_of(const Spectral& s, const SpecItem* items) {
  return SpecArgs{s.nx, s.ny, s.nz, s.px, s.py, s.pz, s.tx, s.ty, s.tz, s.lx, s.ly, s.lz, s.hat,
                  s.h2, 1.0 / (double(s.nx) * s.ny * s.nz), items};
}

// Workgroup -> item, so that each XCD (which takes every eighth workgroup)
// holds a contiguous share of them: neighbouring planes meet in one L2.
__device__ __forceinline__ int xcd_order(int b, int n) {
  return (n & 7) == 0 ? (b & 7) * (n >> 3) + (b >> 3) : b;
}

__device__ __forceinline__ void load_twiddles(double2* dst, const double2* src, int n, int tid,
                                              int nthr) {
  for (int k = tid; k < n; k += nthr) dst[k] = src[k];
}

// Right-hand side at site (x, y, z): with the iterate its residual (and its
// terms of the norms), without it f.
template <bool RES>
__device__ __forceinline__ double spec_rhs(const double* __restrict__ x,
                                           const double* __restrict__ f, double shift, int ix,
                                           int iy, int iz, const SpecArgs& a, double (&acc)[3]) {
  const long long nxy = (long long)a.nx * a.ny;
  const long long row = iz * nxy + (long long)iy * a.nx;
  if constexpr (!RES) {
    return f[row + ix];
  } else {
    const int xm = ix == 0 ? a.nx - 1 : ix - 1, xp = ix == a.nx - 1 ? 0 : ix + 1;
    const int ym = iy == 0 ? a.ny - 1 : iy - 1, yp = iy == a.ny - 1 ? 0 : iy + 1;
    const int zm = iz == 0 ? a.nz - 1 : iz - 1, zp = iz == a.nz - 1 ? 0 : iz + 1;
    const double c = x[row + ix];
    const double lap = x[row + xm] + x[row + xp] + x[iz * nxy + (long long)ym * a.nx + ix] +
                       x[iz * nxy + (long long)yp * a.nx + ix] +
                       x[zm * nxy + (long long)iy * a.nx + ix] +
                       x[zp * nxy + (long long)iy * a.nx + ix] - 6.0 * c;
    const double rhs = f[row + ix] + shift;
    const double res = rhs - lap;
    acc[0] += res * res;
    acc[1] += rhs * rhs;
    acc[2] += c;
    return res;
  }
}

// x and y of a whole plane, a workgroup per plane.
template <int EPT, int MAXT, bool PRIME, bool RES>
__global__ __launch_bounds__(MAXT) void k_spec_plane(const double* __restrict__ x,
                                                     const double* __restrict__ f,
                                                     const PoissonScalars* __restrict__ ps,
                                                     double* __restrict__ partials, SpecArgs a) {
  extern __shared__ __align__(16) double D[];
  if (a.items) {
    const SpecItem& it = a.items[blockIdx.y];
    x = it.x; f = it.f; ps = it.ps; partials = it.partials; a.hat = it.hat;
  }
  if (ps->done) return;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int z = xcd_order(blockIdx.x, gridDim.x), ld = a.nx + 1;
  double2* twx = (double2*)(D + (((size_t)a.ny * ld + 1) & ~size_t(1)));
  double2* twy = twx + a.nx;
  const double shift = RES ? ps->shift : 0.0;
  const float inv_nx = 1.0f / a.nx;
  const int sites = a.nx * a.ny;
  double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll 4
  for (int t = tid; t < sites; t += nthr) {
    int ix;
    const int iy = divide(t, a.nx, inv_nx, ix);
    D[iy * ld + ix] = spec_rhs<RES>(x, f, shift, ix, iy, z, a, acc);
  }
  load_twiddles(twx, a.tx, a.nx, tid, nthr);
  load_twiddles(twy, a.ty, a.ny, tid, nthr);
  __syncthreads();
  const Lines rows{a.ny / 2, ld, 1, (a.ny / 2) * ld}, cols{a.nx / 2, 1, ld, a.nx / 2};
#pragma unroll 1
  for (int axis = 0; axis < 2; ++axis) {   // one copy of the code for both axes
    fft_lines<EPT, PRIME>(D, axis ? twy : twx, axis ? a.py : a.px, axis ? cols : rows, tid, nthr);
    separate_lines(D, axis ? a.ny : a.nx, axis ? cols : rows, tid, nthr);
  }
  double* out = a.hat + (long long)z * sites;
  for (int t = tid; t < sites; t += nthr) {
    int ix;
    const int iy = divide(t, a.nx, inv_nx, ix);
    out[t] = D[iy * ld + ix];
  }
  if constexpr (RES) block_partials<3>(acc, partials, blockIdx.x, gridDim.x);
}

// The way back of a plane: y, then x, then x_out += or =.
template <int EPT, int MAXT, bool PRIME, bool ADD>
__global__ __launch_bounds__(MAXT) void k_spec_plane_back(double* __restrict__ x,
                                                          const PoissonScalars* __restrict__ ps,
                                                          SpecArgs a) {
  extern __shared__ __align__(16) double D[];
  if (a.items) {
    const SpecItem& it = a.items[blockIdx.y];
    x = it.x; ps = it.ps; a.hat = it.hat;
  }
  if (ps->done) return;
  const double gauge = a.items ? ps->psum * a.inv_n : 0.0;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int z = xcd_order(blockIdx.x, gridDim.x), ld = a.nx + 1;
  double2* twx = (double2*)(D + (((size_t)a.ny * ld + 1) & ~size_t(1)));
  double2* twy = twx + a.nx;
  const float inv_nx = 1.0f / a.nx;
  const int sites = a.nx * a.ny;
  const double* in = a.hat + (long long)z * sites;
#pragma unroll 4
  for (int t = tid; t < sites; t += nthr) {
    int ix;
    const int iy = divide(t, a.nx, inv_nx, ix);
    D[iy * ld + ix] = in[t];
  }
  load_twiddles(twx, a.tx, a.nx, tid, nthr);
  load_twiddles(twy, a.ty, a.ny, tid, nthr);
  __syncthreads();
  const Lines rows{a.ny / 2, ld, 1, (a.ny / 2) * ld}, cols{a.nx / 2, 1, ld, a.nx / 2};
#pragma unroll 1
  for (int axis = 1; axis >= 0; --axis) {
    fft_lines<EPT, PRIME>(D, axis ? twy : twx, axis ? a.py : a.px, axis ? cols : rows, tid, nthr);
    separate_lines(D, axis ? a.ny : a.nx, axis ? cols : rows, tid, nthr);
  }
  double* out = x + (long long)z * sites;
#pragma unroll 4
  for (int t = tid; t < sites; t += nthr) {
    int ix;
    const int iy = divide(t, a.nx, inv_nx, ix);
    const double v = D[iy * ld + ix];
    out[t] = ADD ? out[t] + (v - gauge) : v;
  }
}

// x of 16 rows of a plane (larger planes).
template <int EPT, int MAXT, bool PRIME, bool RES>
__global__ __launch_bounds__(MAXT) void k_spec_rows(const double* __restrict__ x,
                                                    const double* __restrict__ f,
                                                    const PoissonScalars* __restrict__ ps,
                                                    double* __restrict__ partials, SpecArgs a) {
  extern __shared__ __align__(16) double D[];
  if (a.items) {
    const SpecItem& it = a.items[blockIdx.y];
    x = it.x; f = it.f; ps = it.ps; partials = it.partials; a.hat = it.hat;
  }
  if (ps->done) return;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int nty = (a.ny + TILE - 1) / TILE;
  const int b = xcd_order(blockIdx.x, gridDim.x), z = b / nty, y0 = (b - z * nty) * TILE;
  const int ld = a.nx + 1, ny = min(TILE, a.ny - y0);
  double2* tw = (double2*)(D + TILE * ld);
  const double shift = RES ? ps->shift : 0.0;
  const float inv_nx = 1.0f / a.nx;
  double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll 4
  for (int t = tid; t < TILE * a.nx; t += nthr) {
    int ix;
    const int j = divide(t, a.nx, inv_nx, ix);
    D[j * ld + ix] = j < ny ? spec_rhs<RES>(x, f, shift, ix, y0 + j, z, a, acc) : 0.0;
  }
  load_twiddles(tw, a.tx, a.nx, tid, nthr);
  __syncthreads();
  const Lines rows{TILE / 2, ld, 1, (TILE / 2) * ld};
  fft_lines<EPT, PRIME>(D, tw, a.px, rows, tid, nthr);
  separate_lines(D, a.nx, rows, tid, nthr);
  double* out = a.hat + ((long long)z * a.ny + y0) * a.nx;
  for (int t = tid; t < ny * a.nx; t += nthr) {
    int ix;
    const int j = divide(t, a.nx, inv_nx, ix);
    out[t] = D[j * ld + ix];
  }
  if constexpr (RES) block_partials<3>(acc, partials, blockIdx.x, gridDim.x);
}

template <int EPT, int MAXT, bool PRIME, bool ADD>
__global__ __launch_bounds__(MAXT) void k_spec_rows_back(double* __restrict__ x,
                                                         const PoissonScalars* __restrict__ ps,
                                                         SpecArgs a) {
  extern __shared__ __align__(16) double D[];
  if (a.items) {
    const SpecItem& it = a.items[blockIdx.y];
    x = it.x; ps = it.ps; a.hat = it.hat;
  }
  if (ps->done) return;
  const double gauge = a.items ? ps->psum * a.inv_n : 0.0;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int nty = (a.ny + TILE - 1) / TILE;
  const int b = xcd_order(blockIdx.x, gridDim.x), z = b / nty, y0 = (b - z * nty) * TILE;
  const int ld = a.nx + 1, ny = min(TILE, a.ny - y0);
  double2* tw = (double2*)(D + TILE * ld);
  const float inv_nx = 1.0f / a.nx;
  const long long first = ((long long)z * a.ny + y0) * a.nx;
#pragma unroll 4
  for (int t = tid; t < TILE * a.nx; t += nthr) {
    int ix;
    const int j = divide(t, a.nx, inv_nx, ix);
    D[j * ld + ix] = j < ny ? a.hat[first + t] : 0.0;
  }
  load_twiddles(tw, a.tx, a.nx, tid, nthr);
  __syncthreads();
  const Lines rows{TILE / 2, ld, 1, (TILE / 2) * ld};
  fft_lines<EPT, PRIME>(D, tw, a.px, rows, tid, nthr);
  separate_lines(D, a.nx, rows, tid, nthr);
#pragma unroll 4
  for (int t = tid; t < ny * a.nx; t += nthr) {
    int ix;
    const int j = divide(t, a.nx, inv_nx, ix);
    const double v = D[j * ld + ix];
    x[first + t] = ADD ? x[first + t] + (v - gauge) : v;
  }
}

// Lines across the rows of the work field, 16 columns of x at a time, in
// place: along y (Z = false), or along z with the division by the
// eigenvalues and the way back along z (Z = true).
template <int EPT, int MAXT, bool PRIME, bool Z>
__global__ __launch_bounds__(MAXT) void k_spec_cols(const PoissonScalars* __restrict__ ps,
                                                    SpecArgs a) {
  extern __shared__ __align__(16) double D[];
  if (a.items) {
    const SpecItem& it = a.items[blockIdx.y];
    ps = it.ps; a.hat = it.hat;
  }
  if (ps->done) return;
  const int tid = threadIdx.x, nthr = blockDim.x;
  const int ntx = (a.nx + TILE - 1) / TILE;
  const int b = xcd_order(blockIdx.x, gridDim.x), o = b / ntx, x0 = (b - o * ntx) * TILE;
  const int n = Z ? a.nz : a.ny, nx = min(TILE, a.nx - x0);
  const long long nxy = (long long)a.nx * a.ny;
  const long long step = Z ? nxy : a.nx;
  double* base = a.hat + (Z ? (long long)o * a.nx : o * nxy) + x0;
  double2* tw = (double2*)(D + n * 2 * TILE_PS);
  const Lines cols{TILE / 2, 1, TILE_PS, n * TILE_PS};
  const int c = tid % TILE;
  double* dc = D + (c < TILE / 2 ? c : c - TILE / 2 + cols.im);
#pragma unroll 4
  for (int j = tid / TILE; j < n; j += nthr / TILE)
    dc[j * TILE_PS] = c < nx ? base[j * step + c] : 0.0;
  load_twiddles(tw, Z ? a.tz : a.ty, n, tid, nthr);
  __syncthreads();
  const DhtPlan& plan = Z ? a.pz : a.py;
#pragma unroll 1
  for (int back = Z ? 0 : 1; back < 2; ++back) {
    fft_lines<EPT, PRIME>(D, tw, plan, cols, tid, nthr);
    // separated; on the way there along z also divided by the eigenvalue (the
    // same at k and n - k), which joins the lines again as they lie
    const double ly = Z ? a.ly[o] : 0.0;
    const int half = n / 2 + 1;
    for (int it = tid; it < half * (TILE / 2); it += nthr) {
      const int l = it % (TILE / 2), k = it / (TILE / 2), kn = k == 0 ? 0 : n - k;
      double* z = D + l + k * TILE_PS;
      double* zn = D + l + kn * TILE_PS;
      HartleyPair h = hartley({z[0], z[cols.im]}, {zn[0], zn[cols.im]});
      if (!back) {
        const int xa = x0 + l, xb = xa + TILE / 2;
        const double lyz = ly + a.lz[k];
        const double ea = xa < a.nx ? a.lx[xa] + lyz : 1.0, eb = xb < a.nx ? a.lx[xb] + lyz : 1.0;
        const double sa = ea == 0.0 ? 0.0 : a.h2 * a.inv_n / ea;
        const double sb = eb == 0.0 ? 0.0 : a.h2 * a.inv_n / eb;
        h = {h.a * sa, h.an * sa, h.b * sb, h.bn * sb};
      }
      z[0] = h.a;
      z[cols.im] = h.b;
      zn[0] = h.an;
      zn[cols.im] = h.bn;
    }
    __syncthreads();
  }
#pragma unroll 4
  for (int j = tid / TILE; j < n; j += nthr / TILE)
    if (c < nx) base[j * step + c] = dc[j * TILE_PS];
}

// Launch shapes: threads and complex values per thread (a radix-8 pass takes
// one butterfly of 8 all the same), in order of preference.  Few values per
// thread leave room for two workgroups per compute unit, which hide each
// other's barriers: the y and z passes of 256 x 256 x 512 take 811 us with
// 512 threads of 4 values, 857 with 256 of 8, 1,019 with 256 of 8 held to 128
// registers.  Plans with a prime factor from 7 on take the second or the last
// (fewer instances).
struct Shape {
  int threads, ept;
};
constexpr Shape SHAPES[] = {{256, 4}, {512, 4}, {1024, 4}, {1024, 8}};
constexpr int NSHAPES = 4;

// Index of the first shape from `first` on that holds the lines of the plans,
// or -1.
int shape_for(const DhtPlan& p, int lines_p, const DhtPlan* q, int lines_q, int first, bool prime) {
  for (int k = first; k < NSHAPES; ++k) {
    if (prime && k % 2 == 0) continue;
    if (fft_fits(p, lines_p, SHAPES[k].ept, SHAPES[k].threads) &&
        (!q || fft_fits(*q, lines_q, SHAPES[k].ept, SHAPES[k].threads)))
      return k;
  }
  return -1;
}

// Calls go(values per thread, threads, prime) with the constants of shape k.
template <typename F>
void with_shape(int k, bool prime, F go) {
  constexpr std::integral_constant<int, 4> e4{};
  constexpr std::integral_constant<int, 8> e8{};
  constexpr std::integral_constant<int, 256> t256{};
  constexpr std::integral_constant<int, 512> t512{};
  constexpr std::integral_constant<int, 1024> t1024{};
  if (prime) {
    if (k == 1) go(e4, t512, std::true_type{});
    else go(e8, t1024, std::true_type{});
    return;
  }
  switch (k) {
    case 0: go(e4, t256, std::false_type{}); break;
    case 1: go(e4, t512, std::false_type{}); break;
    case 2: go(e4, t1024, std::false_type{}); break;
    default: go(e8, t1024, std::false_type{}); break;
  }
}

size_t plane_lds(int nx, int ny) {
  return (((size_t)ny * (nx + 1) + 1) & ~size_t(1)) * 8 + (size_t)(nx + ny) * 16;
}
size_t rows_lds(int nx) { return (size_t)TILE * (nx + 1) * 8 + (size_t)nx * 16; }
size_t cols_lds(int n) { return (size_t)n * 2 * TILE_PS * 8 + (size_t)n * 16; }

size_t al256(size_t b) { return (b + 255) & ~size_t(255); }

bool allow_lds(const void* kernel, size_t bytes) {
  if (bytes <= 64 * 1024) return true;
  if (hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes) == hipSuccess)
    return true;
  (void)hipGetLastError();
  return false;
}

}  // namespace

bool ek::dht_plan(int n, DhtPlan& plan) {
  plan = DhtPlan{};
  if (n < 2 || n > DHT_MAX_N || (n & 1)) return false;
  plan.n = n;
  auto pass = [&](int code) { plan.code |= (unsigned long long)code << (4 * plan.count++); };
  for (const int r : {8, 4, 2, 3, 5})
    for (; n % r == 0; n /= r) pass(r);
  for (int r = 7; n > 1; r += 2)
    for (; n % r == 0; n /= r) {
      plan.prime[plan.primes++] = r;
      pass(PRIME_PASS);
    }
  return true;
}

size_t ek::spectral_table_bytes(int nx, int ny, int nz) {
  DhtPlan p;
  if (!dht_plan(nx, p) || !dht_plan(ny, p) || !dht_plan(nz, p)) return 0;
  return al256((size_t)(nx + ny + nz) * 24);
}

size_t ek::spectral_bytes(int nx, int ny, int nz) {
  const size_t tables = spectral_table_bytes(nx, ny, nz);
  return tables ? al256((size_t)nx * ny * nz * 8) + tables + 256 : 0;
}

void ek::spectral_setup(Spectral& s, char* mem, int nx, int ny, int nz, double h2,
                        bool own_field) {
  s = Spectral{};
  if (!dht_plan(nx, s.px) || !dht_plan(ny, s.py) || !dht_plan(nz, s.pz)) return;
  s.nx = nx;
  s.ny = ny;
  s.nz = nz;
  s.h2 = h2;
  s.hat = own_field ? (double*)mem : nullptr;
  const int m = nx + ny + nz;
  std::vector<double> host((size_t)3 * m);
  double* lam = host.data() + 2 * (size_t)m;
  int at = 0;
  for (const int n : {nx, ny, nz})
    for (int k = 0; k < n; ++k, ++at) {
      // octant-exact angles: the symmetric modes get equal eigenvalues
      const int kk = k > n / 2 ? n - k : k;
      const double c = std::cos(2.0 * M_PI * kk / n), sn = std::sin(2.0 * M_PI * kk / n);
      host[2 * at] = c;
      host[2 * at + 1] = kk == k ? -sn : sn;
      // 2 cos t - 2 = -4 sin(t / 2)^2, without the cancellation
      const double h = std::sin(M_PI * kk / n);
      lam[at] = -4.0 * h * h;
    }
  char* tab = mem + (own_field ? al256((size_t)nx * ny * nz * 8) : 0);
  if (hipMemcpy(tab, host.data(), host.size() * 8, hipMemcpyHostToDevice) != hipSuccess) {
    (void)hipGetLastError();
    return;
  }
  s.tx = (const double2*)tab;
  s.ty = s.tx + nx;
  s.tz = s.ty + ny;
  s.lx = (const double*)(s.tz + nz);
  s.ly = s.lx + nx;
  s.lz = s.ly + ny;
  bool ok = true;
  s.plane_prime = s.px.primes > 0 || s.py.primes > 0;
  s.row_prime = s.px.primes > 0;
  s.col_prime = s.py.primes > 0;
  s.z_prime = s.pz.primes > 0;
  s.plane_shape = plane_lds(nx, ny) <= PLANE_LDS_MAX
                      ? shape_for(s.px, ny / 2, &s.py, nx / 2, nx * ny >= 1024 ? 1 : 0, s.plane_prime)
                      : -1;
  if (s.plane_shape < 0) {
    s.row_shape = shape_for(s.px, TILE / 2, nullptr, 0, nx > 128 ? 1 : 0, s.row_prime);
    s.col_shape = shape_for(s.py, TILE / 2, nullptr, 0, ny > 128 ? 1 : 0, s.col_prime);
    ok = s.row_shape >= 0 && s.col_shape >= 0;
  }
  s.z_shape = shape_for(s.pz, TILE / 2, nullptr, 0, nz > 128 ? 1 : 0, s.z_prime);
  ok = ok && s.z_shape >= 0;
  if (!ok) return;
  if (s.plane_shape >= 0) {
    with_shape(s.plane_shape, s.plane_prime, [&](auto e, auto t, auto pr) {
      constexpr int E = decltype(e)::value, T = decltype(t)::value;
      constexpr bool P = decltype(pr)::value;
      const size_t b = plane_lds(nx, ny);
      ok = allow_lds((const void*)k_spec_plane<E, T, P, true>, b) &&
           allow_lds((const void*)k_spec_plane<E, T, P, false>, b) &&
           allow_lds((const void*)k_spec_plane_back<E, T, P, true>, b) &&
           allow_lds((const void*)k_spec_plane_back<E, T, P, false>, b);
    });
  } else {
    with_shape(s.row_shape, s.row_prime, [&](auto e, auto t, auto pr) {
      constexpr int E = decltype(e)::value, T = decltype(t)::value;
      constexpr bool P = decltype(pr)::value;
      const size_t b = rows_lds(nx);
      ok = allow_lds((const void*)k_spec_rows<E, T, P, true>, b) &&
           allow_lds((const void*)k_spec_rows<E, T, P, false>, b) &&
           allow_lds((const void*)k_spec_rows_back<E, T, P, true>, b) &&
           allow_lds((const void*)k_spec_rows_back<E, T, P, false>, b);
    });
    with_shape(s.col_shape, s.col_prime, [&](auto e, auto t, auto pr) {
      constexpr int E = decltype(e)::value, T = decltype(t)::value;
      constexpr bool P = decltype(pr)::value;
      ok = ok && allow_lds((const void*)k_spec_cols<E, T, P, false>, cols_lds(ny));
    });
  }
  with_shape(s.z_shape, s.z_prime, [&](auto e, auto t, auto pr) {
    constexpr int E = decltype(e)::value, T = decltype(t)::value;
    constexpr bool P = decltype(pr)::value;
    ok = ok && allow_lds((const void*)k_spec_cols<E, T, P, true>, cols_lds(nz));
  });
  s.ok = ok;
}

int ek::spectral_blocks(const Spectral& s) {
  return s.plane_shape >= 0 ? s.nz : s.nz * ((s.ny + TILE - 1) / TILE);
}

int ek::launch_spectral_forward(const Spectral& s, const double* x, const double* f,
                                const PoissonScalars* ps, double* partials, hipStream_t st,
                                const SpecItem* items, int count) {
  const SpecArgs a = args_of(s, items);
  const int nb = spectral_blocks(s);
  const bool res = x || items;
  if (s.plane_shape >= 0) {
    with_shape(s.plane_shape, s.plane_prime, [&](auto e, auto t, auto pr) {
      constexpr int E = decltype(e)::value, T = decltype(t)::value;
      constexpr bool P = decltype(pr)::value;
      const size_t lds = plane_lds(s.nx, s.ny);
      if (res)
        hipLaunchKernelGGL((k_spec_plane<E, T, P, true>), dim3(nb, count), dim3(T), lds, st, x, f, ps,
                           partials, a);
      else
        hipLaunchKernelGGL((k_spec_plane<E, T, P, false>), dim3(nb, count), dim3(T), lds, st, x, f, ps,
                           partials, a);
    });
    return nb;
  }
  with_shape(s.row_shape, s.row_prime, [&](auto e, auto t, auto pr) {
    constexpr int E = decltype(e)::value, T = decltype(t)::value;
    constexpr bool P = decltype(pr)::value;
    const size_t lds = rows_lds(s.nx);
    if (res)
      hipLaunchKernelGGL((k_spec_rows<E, T, P, true>), dim3(nb, count), dim3(T), lds, st, x, f, ps, partials, a);
    else
      hipLaunchKernelGGL((k_spec_rows<E, T, P, false>), dim3(nb, count), dim3(T), lds, st, x, f, ps, partials, a);
  });
  return nb;
}

void ek::launch_spectral_solve(const Spectral& s, double* x, bool add, const PoissonScalars* ps,
                               hipStream_t st, const SpecItem* items, int count) {
  const SpecArgs a = args_of(s, items);
  const int nb = spectral_blocks(s), ntx = (s.nx + TILE - 1) / TILE;
  auto along_y = [&] {
    with_shape(s.col_shape, s.col_prime, [&](auto e, auto t, auto pr) {
      constexpr int E = decltype(e)::value, T = decltype(t)::value;
      constexpr bool P = decltype(pr)::value;
      hipLaunchKernelGGL((k_spec_cols<E, T, P, false>), dim3(ntx * s.nz, count), dim3(T), cols_lds(s.ny), st,
                         ps, a);
    });
  };
  if (s.plane_shape < 0) along_y();
  with_shape(s.z_shape, s.z_prime, [&](auto e, auto t, auto pr) {
    constexpr int E = decltype(e)::value, T = decltype(t)::value;
    constexpr bool P = decltype(pr)::value;
    hipLaunchKernelGGL((k_spec_cols<E, T, P, true>), dim3(ntx * s.ny, count), dim3(T), cols_lds(s.nz), st, ps,
                       a);
  });
  if (s.plane_shape < 0) along_y();
  if (s.plane_shape >= 0) {
    with_shape(s.plane_shape, s.plane_prime, [&](auto e, auto t, auto pr) {
      constexpr int E = decltype(e)::value, T = decltype(t)::value;
      constexpr bool P = decltype(pr)::value;
      const size_t lds = plane_lds(s.nx, s.ny);
      if (add)
        hipLaunchKernelGGL((k_spec_plane_back<E, T, P, true>), dim3(nb, count), dim3(T), lds, st, x, ps, a);
      else
        hipLaunchKernelGGL((k_spec_plane_back<E, T, P, false>), dim3(nb, count), dim3(T), lds, st, x, ps, a);
    });
    return;
  }
  with_shape(s.row_shape, s.row_prime, [&](auto e, auto t, auto pr) {
    constexpr int E = decltype(e)::value, T = decltype(t)::value;
    constexpr bool P = decltype(pr)::value;
    const size_t lds = rows_lds(s.nx);
    if (add)
      hipLaunchKernelGGL((k_spec_rows_back<E, T, P, true>), dim3(nb, count), dim3(T), lds, st, x, ps, a);
    else
      hipLaunchKernelGGL((k_spec_rows_back<E, T, P, false>), dim3(nb, count), dim3(T), lds, st, x, ps, a);
  });
}

// ---------------------------------------------------------------------------
// The time loop's solve.
// ---------------------------------------------------------------------------
void ek_ctx::spectral_cycle(const double* bb, double* x, bool start) {
  const int nb = launch_spectral_forward(spec, x, bb, ps, partials, stream);
  if (start) launch_residual_final(partials, nb, p.poisson_tol, 0, 1, ps, stream);
  launch_spectral_solve(spec, x, true, ps, stream);
}

// The first cycle, with the start's test, without waiting for its result.
// That is written to host memory by the kernel that finds it: a copy of its
// own and an event behind it left the device idle for 15 us.
ek_status ek_ctx::spectral_begin(const double* bb, double* x) {
  spectral_cycle(bb, x, true);
  const int nr = residual_launch(bb, x);
  launch_residual_final(partials, nr, p.poisson_tol, 1, 0, ps, stream, look, ++look_seq);
  if (!defer_shift) launch_psi_shift(x, ps, 1.0 / double(dims.n), dims, stream);
  return EK_OK;
}

// Waits for the result of spectral_begin's cycle.  Once the stream has ended
// it is there; a failed stream ends the wait.
ek_status ek_ctx::spectral_look(PoissonScalars& h) {
  for (unsigned n = 1; __atomic_load_n(&look->seq, __ATOMIC_ACQUIRE) != look_seq; ++n) {
    if (n % 1024 != 0) continue;
    const hipError_t e = hipStreamQuery(stream);
    if (e == hipErrorNotReady) continue;
    if (e != hipSuccess) return fail(EK_EHIP, std::string("hipStreamQuery: ") + hipGetErrorString(e));
    if (__atomic_load_n(&look->seq, __ATOMIC_ACQUIRE) != look_seq)
      return fail(EK_EHIP, "the solve's result did not arrive");
  }
  h = look->s;
  return EK_OK;
}

// Cycles from the start x until the residual, taken by a pass of its own
// after each, meets the tolerance.  With start_norms the first cycle also
// tests the start (its residual is formed there anyway; `begun`: it has been
// enqueued); the other kernels of the solve skip themselves once the flag is
// set.
ek_status ek_ctx::spectral_solve(const double* bb, double* x, PoissonScalars h, int& iters,
                                 double& res, double& res0, bool start_norms, bool begun) {
  int it = 0;
  ek_status st = EK_OK;
  if (start_norms) {
    if (!begun) st = spectral_begin(bb, x);
    if (!st) st = spectral_look(h);
    if (st) return st;
    it = 1;
  }
  if (it < p.poisson_max_iter) neutralize(h);
  while (!h.done && it < p.poisson_max_iter) {
    ++it;
    spectral_cycle(bb, x, false);
    const int nr = residual_launch(bb, x);
    launch_residual_final(partials, nr, p.poisson_tol, it, 0, ps, stream);
    st = read_scalars(&h);
    if (st) return st;
  }
  res0 = h.rel0;
  res = h.rel;
  if (!h.done) {
    iters = it;
    char buf[160];
    std::snprintf(buf, sizeof buf, "the Poisson solve did not reach %.3g in %d cycles (residual %.3e)",
                  p.poisson_tol, p.poisson_max_iter, h.rel);
    return fail(EK_ENOCONV, buf);
  }
  iters = h.iters;
  if (defer_shift) shift_pending = true;
  else if (!start_norms || it > 1) launch_psi_shift(x, ps, 1.0 / double(dims.n), dims, stream);
  return EK_OK;
}
