// The ensemble's time step as launches over all replicas.
//
// Every kernel takes the whole ensemble: blockIdx.y (or x, where a workgroup
// owns a replica) picks the replica, whose descriptor (ensemble.h) holds its
// pointers, its current buffer and its state; the host enqueues steps without
// looking.  The site loops run at the rate of HBM (charge pass and lattice
// step are read and written once), and the Poisson solve is the direct one of
// kernels_spectral.hip, three passes over the field in place of two or three
// multigrid cycles of about ten.  The persistent kernel, whose workgroups
// meet at barriers of their own, spends its step waiting on memory instead
// (2,048 threads a replica): 5.9 ms per step of 64 replicas of 48x48x96, of
// which 3.8 were multigrid; the launches take 2.6 (charge pass 0.55, Poisson
// 0.61, chain 0.2, lattice step 1.25).
//
// A replica whose solve misses the tolerance after the first cycle pauses
// (its kernels skip it) until the host has seen to it; the others go on.
#include "ensemble.h"
#include "lb_site.h"
#include "reduce.h"

namespace ek {

namespace {

constexpr int SPT = 4;   // sites per thread of the site loops: a block sums 1,024 sites at once
constexpr int SITES = SPT * BLOCK;

int site_blocks(const Dims& d) { return int((d.n + SITES - 1) / SITES); }

// Whether a replica takes part in the launches made for status `want`.
__device__ __forceinline__ bool runs(const RepDev& R, int want) {
  return R.status == want && R.todo > 0;
}

// End of phase ph of the replica's step (one thread).
__device__ inline void lap(RepDev& R, int ph) {
  const unsigned long long now = wall_clock64();
  R.phase_ticks[ph] += now - R.phase_mark;
  R.phase_mark = now;
}

__device__ __forceinline__ void site_of_index(long long t, const Dims& d, int& x, int& y, int& z) {
  const unsigned row = unsigned(t) / unsigned(d.nx);   // n < 2^31
  x = int(unsigned(t) - row * unsigned(d.nx));
  z = int(row / unsigned(d.ny));
  y = int(row - unsigned(z) * unsigned(d.ny));
}

__device__ __forceinline__ BeadTableView table_of(const RepDev& R) {
  BeadTableView bt;
  bt.keys = R.keys;
  bt.vals = R.vals;
  bt.bits = ENS_TABLE_BITS;
  return bt;
}

// Bead charges of time t: a workgroup per replica.
__global__ __launch_bounds__(1024) void k_rep_deposit(RepDev* reps, Dims d) {
  RepDev& R = reps[blockIdx.x];
  if (!runs(R, ST_OK)) return;
  if (threadIdx.x == 0) R.phase_mark = wall_clock64();
  if (R.n_beads == 0) return;
  table_clear_items(R.keys, R.vals, R.mask, d.n, ENS_TABLE_BITS, threadIdx.x, blockDim.x);
  __syncthreads();
  deposit_items(R.bs, R.n_beads, R.keys, R.vals, R.mask, d, ENS_TABLE_BITS, threadIdx.x, blockDim.x);
}

// Charge pass, with the extrapolated start of the solve (as the persistent
// kernel's) where the replica holds a history.
template <typename I>
__global__ __launch_bounds__(BLOCK) void k_rep_charge(const RepDev* __restrict__ reps,
                                                      const double* __restrict__ wall_q,
                                                      double inv_eps, double* __restrict__ part,
                                                      size_t part_stride, Dims d) {
  const RepDev& R = reps[blockIdx.y];
  if (!runs(R, ST_OK)) return;
  const float* f = (const float*)R.f[R.cur];
  const LBParams lp = R.lp;
  const BeadTableView bt = table_of(R);
  double* b = R.b;
  double* psi = R.psi;
  double* old = R.psi_old;
  const int hist = old ? R.psi_hist : 0;
  double acc[1] = {0.0};
  const long long t0 = (long long)blockIdx.x * SITES + threadIdx.x;
#pragma unroll 1
  for (int k = 0; k < SPT; ++k) {
    const long long t = t0 + k * BLOCK;
    if (t >= d.n) break;
    int x, y, z;
    site_of_index(t, d, x, y, z);
    const double rho = charge_site<float, I>(f, R.mask, wall_q, lp, bt, x, y, z, d);
    b[t] = -rho * inv_eps;
    acc[0] += rho;
    if (hist > 0) {
      const double p = psi[t];
      if (hist >= 2) psi[t] = 2.0 * p - old[t];
      old[t] = p;
    }
  }
  block_partials<1>(acc, part + blockIdx.y * part_stride, blockIdx.x, gridDim.x);
}

// Mean charge and the flags of the solve: a workgroup per replica.
__global__ __launch_bounds__(BLOCK) void k_rep_shift(RepDev* reps, PoissonScalars* pss,
                                                     const double* __restrict__ part,
                                                     size_t part_stride, int nb, double inv_eps,
                                                     Dims d) {
  RepDev& R = reps[blockIdx.x];
  PoissonScalars* ps = pss + blockIdx.x;
  if (!runs(R, ST_OK)) {
    if (threadIdx.x == 0) ps->done = 1;   // the solve's kernels skip the replica
    return;
  }
  const double rho = block_sum_256(part + blockIdx.x * part_stride, nb);
  if (threadIdx.x == 0) {
    ps->shift = rho / double(d.n) * inv_eps;
    ps->done = 0;
    ps->zero_rhs = 0;
    ps->iters = 0;
    if (R.psi_old) R.psi_hist = R.psi_hist < 2 ? R.psi_hist + 1 : 2;
    lap(R, 0);
  }
}

// Norms of the start: a workgroup per replica.
__global__ __launch_bounds__(1024) void k_rep_start(PoissonScalars* pss,
                                                    const double* __restrict__ part,
                                                    size_t part_stride, int nb, double tol) {
  PoissonScalars* ps = pss + blockIdx.x;
  if (ps->done) return;
  double v[3];
  block_sums_1024<3>(part + blockIdx.x * part_stride, nb, v);
  if (threadIdx.x == 0) {
    ps->b2 = v[1];
    ps->psum = v[2];
    ps->rel0 = v[1] > 0.0 ? sqrt(v[0] / v[1]) : (v[0] == 0.0 ? 0.0 : INFINITY);
    ps->rel = ps->rel0;
    if (v[1] == 0.0) ps->zero_rhs = 1;
    if (v[1] == 0.0 || ps->rel0 <= tol) ps->done = 1;
  }
}

// Residual and sum of the iterate.
__global__ __launch_bounds__(BLOCK) void k_rep_residual(const RepDev* __restrict__ reps,
                                                        const PoissonScalars* __restrict__ pss,
                                                        double* __restrict__ part,
                                                        size_t part_stride, Dims d) {
  const PoissonScalars* ps = pss + blockIdx.y;
  if (ps->done) return;
  const RepDev& R = reps[blockIdx.y];
  const double* __restrict__ psi = R.psi;
  const double* __restrict__ b = R.b;
  const double shift = ps->shift;
  const int nxy = d.nx * d.ny, n = int(d.n);
  double acc[3] = {0.0, 0.0, 0.0};
  const long long t0 = (long long)blockIdx.x * SITES + threadIdx.x;
#pragma unroll
  for (int k = 0; k < SPT; ++k) {
    const long long tt = t0 + k * BLOCK;
    if (tt >= d.n) break;
    const int t = int(tt);
    int x, y, z;
    site_of_index(t, d, x, y, z);
    const double c = psi[t];
    const double lap = psi[x == 0 ? t + d.nx - 1 : t - 1] + psi[x == d.nx - 1 ? t - x : t + 1] +
                       psi[y == 0 ? t + nxy - d.nx : t - d.nx] +
                       psi[y == d.ny - 1 ? t - nxy + d.nx : t + d.nx] +
                       psi[z == 0 ? t + n - nxy : t - nxy] +
                       psi[z == d.nz - 1 ? t - n + nxy : t + nxy] - 6.0 * c;
    const double rhs = b[t] + shift;
    const double res = rhs - lap;
    acc[0] += res * res;
    acc[1] += rhs * rhs;
    acc[2] += c;
  }
  block_partials<3>(acc, part + blockIdx.y * part_stride, blockIdx.x, gridDim.x);
}

// What the cycle reached: a workgroup per replica.  A replica over the
// tolerance pauses; a vanishing right-hand side has the potential zero.
__global__ __launch_bounds__(1024) void k_rep_verdict(RepDev* reps, PoissonScalars* pss,
                                                      const double* __restrict__ part,
                                                      size_t part_stride, int nb, double tol,
                                                      int want, Dims d) {
  RepDev& R = reps[blockIdx.x];
  PoissonScalars* ps = pss + blockIdx.x;
  if (!runs(R, want)) return;
  const bool cycled = !ps->done;
  double v[3] = {0.0, 0.0, 0.0};
  if (cycled) block_sums_1024<3>(part + blockIdx.x * part_stride, nb, v);
  if (!cycled && ps->zero_rhs)
    for (long long t = threadIdx.x; t < d.n; t += blockDim.x) R.psi[t] = 0.0;
  __syncthreads();   // every thread has read the flag
  if (threadIdx.x == 0) {
    if (cycled) {
      ps->iters += 1;
      ps->psum = v[2];
      ps->rel = v[1] > 0.0 ? sqrt(v[0] / v[1]) : (v[0] == 0.0 ? 0.0 : INFINITY);
      ps->done = 1;
      if (!(ps->rel <= tol)) R.status = ST_PAUSED;
    }
    R.last_cycles = ps->iters;
    R.last_res = ps->rel;
    R.last_res0 = ps->rel0;
    lap(R, 1);
  }
}

// Lets the solve's kernels go on with the paused replicas over the tolerance.
__global__ __launch_bounds__(64) void k_rep_rearm(const RepDev* __restrict__ reps,
                                                  PoissonScalars* pss, int n_rep, double tol) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rep) return;
  if (runs(reps[r], ST_PAUSED) && reps[r].last_res > tol) pss[r].done = 0;
}

// Fields around the beads: a workgroup per bead.
__global__ __launch_bounds__(BLOCK) void k_rep_box(const RepDev* __restrict__ reps, int want, Dims d) {
  const RepDev& R = reps[blockIdx.y];
  if (int(blockIdx.x) >= R.n_beads || !runs(R, want)) return;
  for (int t = threadIdx.x; t < WallGeom<1>::ITEMS; t += BLOCK)
    bead_box_item(R.bs, blockIdx.x, t, (const float*)R.f[R.cur], R.mask, R.psi, R.lp, d);
}

// The chains' substeps: a workgroup per replica, eight lanes per bead, pair
// lists with room for every partner.
__global__ __launch_bounds__(512) void k_rep_chain(RepDev* reps, int want, Dims d) {
  extern __shared__ __align__(16) unsigned char smem[];
  RepDev& R = reps[blockIdx.x];
  if (!runs(R, want)) return;
  if (R.n_beads > 0)
    md_chain<true, 8, SMALL_CHAIN / 8, 1, false>(R.bs, R.mp, R.keys, R.vals, R.mask, d,
                                                 ENS_TABLE_BITS, 16 * R.n_beads, smem);
  if (threadIdx.x == 0) lap(R, 2);
}

// Fused collide-and-stream.
template <typename I>
__global__ __launch_bounds__(BLOCK) void k_rep_lb(const RepDev* __restrict__ reps,
                                                  double* __restrict__ part, size_t part_stride,
                                                  int want, Dims d) {
  const RepDev& R = reps[blockIdx.y];
  if (!runs(R, want)) return;
  const float* fsrc = (const float*)R.f[R.cur];
  float* fdst = (float*)R.f[R.cur ^ 1];
  const LBParams lp = R.lp;
  const BeadTableView bt = table_of(R);
  double acc[6] = {0, 0, 0, 0, 0, 0};
  const long long t0 = (long long)blockIdx.x * SITES + threadIdx.x;
#pragma unroll 1
  for (int k = 0; k < SPT; ++k) {
    const long long t = t0 + k * BLOCK;
    if (t >= d.n) break;
    int x, y, z;
    site_of_index(t, d, x, y, z);
    lb_site<float, I>(fsrc, fdst, R.mask, R.psi, lp, bt, x, y, z, d, acc);
  }
  block_partials<6>(acc, part + blockIdx.y * part_stride, blockIdx.x, gridDim.x);
}

// End of the step: sums, state, the other buffer: a workgroup per replica.
__global__ __launch_bounds__(1024) void k_rep_end(RepDev* reps, SpecItem* items,
                                                  const double* __restrict__ part,
                                                  size_t part_stride, int nb, int want) {
  RepDev& R = reps[blockIdx.x];
  if (!runs(R, want)) return;
  double acc[6];
  block_sums_1024<6>(part + blockIdx.x * part_stride, nb, acc);
  if (threadIdx.x != 0) return;
  for (int c = 0; c < 6; ++c) R.stats[c] = acc[c];
  R.steps += 1;
  R.todo -= 1;
  items[blockIdx.x].hat = (double*)R.f[R.cur];   // free from now on
  R.cur ^= 1;
  int status = ST_OK;
  for (int sp = 0; sp < 3; ++sp)
    if (!(acc[sp] >= 0.0) || !isfinite(acc[sp])) status = ST_UNSTABLE;
  if (R.n_beads > 0 && *R.bs.err) status = ST_UNSTABLE;
  R.status = status;
  lap(R, 3);
}

// The direct solve's view of the replicas (the work field is the buffer that
// the lattice step writes afterwards).
__global__ __launch_bounds__(64) void k_rep_items(const RepDev* __restrict__ reps, SpecItem* items,
                                                  PoissonScalars* pss, double* part,
                                                  size_t part_stride, int n_rep) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= n_rep) return;
  const RepDev& R = reps[r];
  items[r] = SpecItem{R.psi, R.b, pss + r, part + r * part_stride, (double*)R.f[R.cur ^ 1]};
}

size_t al256(size_t x) { return (x + 255) & ~size_t(255); }

size_t part_doubles(const Spectral& s, const Dims& d) {
  const size_t sites = 6 * (size_t)site_blocks(d);
  const size_t spec = 3 * (size_t)s.nz * ((s.ny + 15) / 16);   // rows of 16, or fewer blocks
  return (sites > spec ? sites : spec) + 32;
}

hipError_t cycle(const RepBatch& b, bool start, int want, hipStream_t s) {
  const int nb = launch_spectral_forward(b.spec, nullptr, nullptr, nullptr, nullptr, s, b.items, b.n_rep);
  if (start)
    hipLaunchKernelGGL(k_rep_start, dim3(b.n_rep), dim3(1024), 0, s, b.ps, b.part, b.part_stride, nb,
                       b.tol);
  launch_spectral_solve(b.spec, nullptr, true, nullptr, s, b.items, b.n_rep);
  const int sb = site_blocks(b.d);
  hipLaunchKernelGGL(k_rep_residual, dim3(sb, b.n_rep), dim3(BLOCK), 0, s, b.reps, b.ps, b.part,
                     b.part_stride, b.d);
  hipLaunchKernelGGL(k_rep_verdict, dim3(b.n_rep), dim3(1024), 0, s, b.reps, b.ps, b.part,
                     b.part_stride, sb, b.tol, want, b.d);
  return hipGetLastError();
}

// LDS of a chain of n beads: positions, node table of 16 slots a bead, lists.
int chain_threads(int n) { return ((8 * n + 63) / 64) * 64; }
size_t chain_lds(int n) {
  return (((size_t)n * 24 + 15) & ~size_t(15)) + (size_t)16 * n * (9 * 8 + 4) +
         md_list_bytes(chain_threads(n), SMALL_CHAIN / 8);
}

hipError_t advance(const RepBatch& b, int want, hipStream_t s) {
  if (b.beads > 0) {
    hipLaunchKernelGGL(k_rep_box, dim3(b.beads, b.n_rep), dim3(BLOCK), 0, s, b.reps, want, b.d);
    const size_t lds = chain_lds(b.beads);
    if (lds > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute((const void*)k_rep_chain,
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k_rep_chain, dim3(b.n_rep), dim3(chain_threads(b.beads)), lds, s, b.reps, want,
                       b.d);
  } else {
    hipLaunchKernelGGL(k_rep_chain, dim3(b.n_rep), dim3(64), 0, s, b.reps, want, b.d);
  }
  const int sb = site_blocks(b.d);
  const dim3 grid(sb, b.n_rep);
  if (fits_idx32<float>(b.d.n))
    hipLaunchKernelGGL(k_rep_lb<uint32_t>, grid, dim3(BLOCK), 0, s, b.reps, b.part, b.part_stride, want, b.d);
  else
    hipLaunchKernelGGL(k_rep_lb<long long>, grid, dim3(BLOCK), 0, s, b.reps, b.part, b.part_stride, want, b.d);
  hipLaunchKernelGGL(k_rep_end, dim3(b.n_rep), dim3(1024), 0, s, b.reps, b.items, b.part, b.part_stride,
                     sb, want);
  return hipGetLastError();
}

}  // namespace

size_t replicas_bytes(int nx, int ny, int nz, int n_rep) {
  const size_t tables = spectral_table_bytes(nx, ny, nz);
  const long long n = (long long)nx * ny * nz;
  if (!tables || n > INT_MAX / 2) return 0;
  Spectral s;
  s.ny = ny;
  s.nz = nz;
  return tables + al256(n_rep * sizeof(SpecItem)) + al256(n_rep * sizeof(PoissonScalars)) +
         al256(n_rep * part_doubles(s, Dims{nx, ny, nz, n}) * 8);
}

void replicas_setup(RepBatch& b, char* mem, int nx, int ny, int nz, int n_rep) {
  b.n_rep = n_rep;
  b.d = Dims{nx, ny, nz, (long long)nx * ny * nz};
  if (replicas_bytes(nx, ny, nz, n_rep) == 0) return;
  spectral_setup(b.spec, mem, nx, ny, nz, 1.0, false);
  char* p = mem + spectral_table_bytes(nx, ny, nz);
  b.items = (SpecItem*)p;
  p += al256(n_rep * sizeof(SpecItem));
  b.ps = (PoissonScalars*)p;
  p += al256(n_rep * sizeof(PoissonScalars));
  b.part = (double*)p;
  b.part_stride = part_doubles(b.spec, b.d);
}

hipError_t replicas_begin(const RepBatch& b, hipStream_t s) {
  hipLaunchKernelGGL(k_rep_items, dim3((b.n_rep + 63) / 64), dim3(64), 0, s, b.reps, b.items, b.ps,
                     b.part, b.part_stride, b.n_rep);
  return hipGetLastError();
}

hipError_t replicas_step(const RepBatch& b, hipStream_t s) {
  const int sb = site_blocks(b.d);
  hipLaunchKernelGGL(k_rep_deposit, dim3(b.n_rep), dim3(1024), 0, s, b.reps, b.d);
  const dim3 grid(sb, b.n_rep);
  if (fits_idx32<float>(b.d.n))
    hipLaunchKernelGGL(k_rep_charge<uint32_t>, grid, dim3(BLOCK), 0, s, b.reps, b.wall_q, b.inv_eps,
                       b.part, b.part_stride, b.d);
  else
    hipLaunchKernelGGL(k_rep_charge<long long>, grid, dim3(BLOCK), 0, s, b.reps, b.wall_q, b.inv_eps,
                       b.part, b.part_stride, b.d);
  hipLaunchKernelGGL(k_rep_shift, dim3(b.n_rep), dim3(BLOCK), 0, s, b.reps, b.ps, b.part,
                     b.part_stride, sb, b.inv_eps, b.d);
  const hipError_t e = cycle(b, true, ST_OK, s);
  return e != hipSuccess ? e : advance(b, ST_OK, s);
}

hipError_t replicas_cycle(const RepBatch& b, hipStream_t s) {
  hipLaunchKernelGGL(k_rep_rearm, dim3((b.n_rep + 63) / 64), dim3(64), 0, s, b.reps, b.ps, b.n_rep,
                     b.tol);
  return cycle(b, false, ST_PAUSED, s);
}

hipError_t replicas_finish(const RepBatch& b, hipStream_t s) { return advance(b, ST_PAUSED, s); }

}  // namespace ek
