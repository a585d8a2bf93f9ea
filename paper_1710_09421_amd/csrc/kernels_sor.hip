// Red-black SOR (Sec. II.C) of lattices that the chip's LDS holds: batches of
// iterations in one launch, the potential kept in LDS and only the tiles' faces
// exchanged.
//
// What bounds the iteration: a 64x64x128 lattice is 4 MB, so one launch per
// half sweep and two per residual test are bound by their launches and by the
// caches' latency (17 us an iteration, 22 with insulating walls).  Here
// a workgroup owns a tile of whole x-rows (ty rows by tz planes) for a whole
// batch, and what bounds it is the trip of its boundary rows through the
// memory side of the chip to its neighbours.  There is one such trip an
// iteration: a workgroup also relaxes the red sites of the ring around its
// tile, for which it needs the black values of two rings, and after the black
// half sweep it takes those from its eight neighbours.  (Sending each colour's
// ring after its half sweep relaxes nothing twice but makes two trips, some 1.1
// us more an iteration.)  An iteration takes 2.0 us at 32^3, 2.4 at 64^3, 3.0 at
// 64x64x128; a solve of 64x64x128 to 1e-8 from zero 1.42 ms (6.9 by single
// launches), two steps of the 48x48x64 insulating pore with their read-out 4.1
// to 4.8 (33), of the 32^3 box to 1e-10 1.18 (3.5).
//
// Exchange: every value travels as one 64-bit device-scope store into a slot of
// the receiver's mailbox, which the receiver polls (sor_mail.h).
//
// The launch is cooperative, so the device has room for all its workgroups at
// once; kernels of other queues may still keep some of them from starting for a
// while, and a wait is bounded.  When one gives up, or a launch is refused, the
// solve goes on with single launches from the iterate that the last batch
// started from (its input is whole whatever became of its result), with the same
// bits, and the context takes single launches from then on.
//
// Convergence: every tested iteration's sum of squared residuals costs no
// reads of its own (at a colour-1 site from its update's neighbours and the
// new value, at a colour-0 site from the next update's neighbours and the old
// value).  The next launch begins with the verdict, which each of its
// workgroups takes for itself from the same sums.  When an iteration inside
// the batch met the tolerance, the batch is run again from its start for
// exactly that many iterations, so the result is the iterate of the iteration
// that converged, as with one test after another.  Otherwise the residual's
// rate tells how long the next batch should be: it stops a little before the
// expected end, and a short one then crosses it, so that little is run twice.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <type_traits>

#include "ek_context.h"
#include "reduce.h"
#include "sor_mail.h"

using namespace ek;

namespace {

constexpr int SOR_THREADS = 512;
constexpr int SOR_WAVES = SOR_THREADS / 64;
constexpr int SOR_MAX_BATCH = 256;
constexpr int SOR_NEAR = 12;          // iterations left within which a batch crosses the end
constexpr int SOR_SHORT = 4;          // else it stops this many before the expected end
constexpr int SOR_AFTER = 24;         // iterations expected after single launches
constexpr int SOR_MAX_ITEMS = 4;      // sites of a colour per thread
constexpr int SOR_MAX_TAKE = 8;       // values a thread takes per iteration
constexpr int SOR_MAX_GROUPS = 256;   // one workgroup per compute unit
constexpr size_t SOR_LDS_MAX = 150 * 1024;

enum : int { SOR_START = 0, SOR_RAN = 1, SOR_REPLAYED = 2, SOR_FINAL = 3, SOR_LIMIT = 4 };

}  // namespace

// What the last launch of a solve left (device memory, two of them in turn).
struct ek::SorControl {
  int state;
  int cur;            // RAN, REPLAYED: the buffer it started from (0 the caller's, 1 the
                      // scratch one), its result is in the other; FINAL, LIMIT: the result
  int base, n;        // iterations before it, and of it
  int found;          // iteration that met the tolerance
  int aborted;        // a wait ran into its limit: cur and base hold, no result
  double omega;       // relaxation factor of its first half sweep
  double omega_next;  // ... of the half sweep after it
};

namespace {

struct SorArgs {
  double* buf[2];
  const double* b;
  const uint32_t* mask;
  const PoissonScalars* ps;
  SorControl* ctl;    // [2]: read at launch & 1, written at the other
  uint64_t* mail;     // [bank][set][workgroup][row][x / 2]
  int bank;           // of this launch
  int spin_limit;     // looks in vain after which a wait gives up
  double* part;       // [2][iteration of the batch][workgroup]: likewise
  int launch;
  int start;          // iterations that the caller has run
  double omega;       // relaxation factor of the half sweep after them
  int first;          // length of the first batch
  int nx, ny, nz, ty, tz, gy, gz;
  int max_iter, every;
  double rj;
  double tol;
};

__device__ __forceinline__ bool tested(const SorArgs& a, int it) {
  return it % a.every == 0 || it == a.max_iter;
}

// The relaxation factors' recursion, rounded as the host rounds it (no fused
// multiply-add).
__device__ inline double chebyshev_first(double rj) {
#pragma clang fp contract(off)
  const double h = 0.5 * rj;
  const double t = h * rj;
  return 1.0 / (1.0 - t);
}
__device__ inline double chebyshev_next(double rj, double omega) {
#pragma clang fp contract(off)
  const double q = 0.25 * rj;
  const double t = q * rj;
  const double v = t * omega;
  return 1.0 / (1.0 - v);
}

// What this launch runs, from what the last one left: base, n, cur and omega
// of its batch, state = REPLAYED where the batch is the last one again (with
// `found`), or FINAL / LIMIT and nothing to run.  `rel` is scratch.
__device__ inline SorControl sor_verdict(const SorArgs& a, double* rel) {
  SorControl c = a.ctl[a.launch & 1];
  if (c.aborted) c.state = SOR_LIMIT;
  if (c.state == SOR_START) {
    c.state = SOR_RAN;
    c.cur = 0;
    c.base = a.start;
    c.n = a.first;
    c.omega = a.omega;
    return c;
  }
  if (c.state == SOR_REPLAYED) {
    c.state = SOR_FINAL;
    c.cur ^= 1;
  }
  if (c.state >= SOR_FINAL) return c;
  const int W = gridDim.x, lane = threadIdx.x & 63;
  const double* part = a.part + (size_t)(a.launch & 1) * SOR_MAX_BATCH * W;
  const double b2 = a.ps->b2;
  for (int it = 1 + (threadIdx.x >> 6); it <= c.n; it += SOR_WAVES) {
    double s = 0.0;
    if (tested(a, c.base + it))
#pragma unroll 4
      for (int k = lane; k < W; k += 64) s += part[(size_t)(it - 1) * W + k];
    s = wave_sum(s);
    if (lane == 0) rel[it - 1] = sqrt(s / b2);
  }
  __syncthreads();
  int last = 0, before = 0;          // the last two tested iterations a quarter of it apart
  for (int it = 1; it <= c.n; ++it) {
    if (!tested(a, c.base + it)) continue;
    if (rel[it - 1] <= a.tol) {
      c.found = c.base + it;
      if (it == c.n) {
        c.state = SOR_FINAL;
        c.cur ^= 1;
      } else {
        c.state = SOR_REPLAYED;
        c.n = it;
      }
      return c;
    }
    last = it;
    if (before == 0 || 4 * it <= 3 * c.n) before = it;
  }
  int n = SOR_MAX_BATCH;
  if (last > before) {
    const double rate = log(rel[last - 1] / rel[before - 1]) / (last - before);
    const double left = log(a.tol / rel[last - 1]) / rate + (last - c.n);
    if (rate < 0.0 && left < double(SOR_MAX_BATCH + SOR_SHORT)) {
      const int k = max(1, int(ceil(left)));
      n = k > SOR_NEAR ? k - SOR_SHORT : k + 2;
    }
  } else {
    n = max(a.every, 8);
  }
  c.base += c.n;
  c.n = min(min(n, SOR_MAX_BATCH), a.max_iter - c.base);
  c.cur ^= 1;
  c.omega = c.omega_next;
  c.state = c.n > 0 ? SOR_RAN : SOR_LIMIT;
  return c;
}

// NEU: insulating walls (fluid sites only, the link words' bits 1..6 mark the
// solid face neighbours, see kernels_poisson.hip).  U: sites of a colour per
// thread, of the tile and of its ring.  TAKE: values a thread takes after an
// iteration.  Colour 0 is red here, colour 1 black.
template <bool NEU, int U, int TAKE>
__global__ __launch_bounds__(SOR_THREADS) void k_sor_team(SorArgs a) {
  extern __shared__ double P[];      // [colour][row of the tile and two rings][x / 2]
  __shared__ int s_abort;
  __shared__ double s_rel[SOR_MAX_BATCH];
  __shared__ double s_sum[SOR_WAVES];
  {
    // the next launch's bank of this workgroup's slots
    const int box = (4 * (a.ty + a.tz) + 4) * (a.nx / 2);
    for (int t = threadIdx.x; t < SOR_SETS * box; t += SOR_THREADS) {
      const int half = t >= box;
      uint64_t* to = a.mail + ((size_t)((a.bank ^ 1) * SOR_SETS + half) * gridDim.x + blockIdx.x) * box;
      __hip_atomic_store(to + t - half * box, SOR_UNSENT, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  const SorControl c = sor_verdict(a, s_rel);
  if (c.state >= SOR_FINAL) {
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctl[(a.launch & 1) ^ 1] = c;
    return;
  }
  const int n_it = c.n;
  const int tid = threadIdx.x, w = blockIdx.x, W = gridDim.x;
  const int ty = a.ty, tz = a.tz, hx = a.nx / 2, ry = ty + 4;
  const int plane = ry * (tz + 4) * hx;
  const int wy = w % a.gy, wz = w / a.gy, y0 = wy * ty, z0 = wz * tz;
  const double* in = a.buf[c.cur];
  double* out = a.buf[c.cur ^ 1];
  const double shift = a.ps->shift;
  if (tid == 0) s_abort = 0;
  // LDS index of row (yy, zz) of the tile, rings at -2, -1 and ty, ty + 1
  auto row_at = [&](int yy, int zz) { return ((zz + 2) * ry + yy + 2) * hx; };
  // the tile and its rings (of the corners only the inner rows are read)
  for (int t = tid; t < ry * (tz + 4) * a.nx; t += SOR_THREADS) {
    const int row = t / a.nx, x = t - row * a.nx;
    const int zz = row / ry - 2, yy = row % ry - 2;
    const int y = (y0 + yy + a.ny) % a.ny, z = (z0 + zz + a.nz) % a.nz;
    P[((x + y + z) & 1) * plane + row * hx + (x >> 1)] =
        in[((long long)z * a.ny + y) * a.nx + x];
  }
  // this thread's sites: rows on the tile's faces first, so that what the
  // neighbours wait for is sent before the inner rows are relaxed
  const int rows = ty * tz, items = rows * hx, ring_items = 2 * (ty + tz) * hx;
  // LDS index o of a site, and o2 of the neighbour in x that is not at o in the
  // other colour's array
  int own[U], own2[2][U], yz[U];     // yz: yy | zz << 16
  int ring[U], ring2[U];             // the red sites of the ring that it relaxes too
  double rhs[2][U], ring_rhs[U];
  int open[2][U], ring_open[U];      // NEU: bits 1..6 open neighbours (1 at o, 2 at o2), bit 0 fluid
  auto beside = [&](int o, int i, bool right) {   // right: x = 2 i + 1
    return right ? (i == hx - 1 ? o - hx + 1 : o + 1) : (i == 0 ? o + hx - 1 : o - 1);
  };
  auto site_of = [&](int yy, int zz, int x) {
    const int y = (y0 + yy + a.ny) % a.ny, z = (z0 + zz + a.nz) % a.nz;
    return ((long long)z * a.ny + y) * a.nx + x;
  };
  auto neighbours_of = [&](long long s, bool right) {
    if constexpr (NEU) {
      const uint32_t m = a.mask[s];
      const int n = int(~m & 126u) | (m & MASK_SOLID ? 0 : 1);   // bit 1: x - 1, bit 2: x + 1
      return right ? n : (n & ~6) | (n & 2) << 1 | (n & 4) >> 1;
    } else {
      return 127;
    }
  };
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int ez = 2, ey = 2, mid = tz - 2, inner = max(ty - 2, 1);
    int t = min(tid + u * SOR_THREADS, items - 1);
    int r = t / hx, i = t - r * hx, yy, zz;
    if (r < ez * ty) {
      zz = r < ty ? 0 : tz - 1;
      yy = r % ty;
    } else if ((r -= ez * ty) < mid * ey) {
      zz = 1 + r / ey;
      yy = r % ey ? ty - 1 : 0;
    } else {
      r -= mid * ey;
      zz = 1 + r / inner;
      yy = 1 + r % inner;
    }
    own[u] = row_at(yy, zz) + i;
    yz[u] = yy | zz << 16;
    int odd = (y0 + yy + z0 + zz) & 1;           // x of red = 2 i + odd
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const long long s = site_of(yy, zz, 2 * i + (odd ^ k));
      own2[k][u] = beside(own[u], i, (odd ^ k) != 0);
      rhs[k][u] = a.b[s] + shift;
      open[k][u] = neighbours_of(s, (odd ^ k) != 0);
    }
    t = min(tid + u * SOR_THREADS, ring_items - 1);
    r = t / hx;
    i = t - r * hx;
    if (r < 2 * tz) {
      yy = r < tz ? -1 : ty;
      zz = r % tz;
    } else {
      r -= 2 * tz;
      zz = r < ty ? -1 : tz;
      yy = r % ty;
    }
    // sides are even: a wrap keeps the colours
    ring[u] = row_at(yy, zz) + i;
    odd = (y0 + yy + z0 + zz) & 1;
    const long long s = site_of(yy, zz, 2 * i + odd);
    ring2[u] = beside(ring[u], i, odd != 0);
    ring_rhs[u] = a.b[s] + shift;
    ring_open[u] = neighbours_of(s, odd != 0);
  }
  // The black values this workgroup takes after every iteration, by rows of
  // its mailbox: 2 tz rows below and above in y (yy = -1 - d and ty + d at
  // d tz + zz), 2 ty rows below and above in z, four corner rows.
  const int box_rows = 4 * (ty + tz) + 4, box = box_rows * hx;
  // (a thread with fewer than TAKE values takes its first one again, or none in
  // place of the last)
  int from[TAKE], dst[TAKE]; // value of the mailbox, LDS index
#pragma unroll
  for (int v = 0; v < TAKE; ++v) {
    const int own_value = tid + v * SOR_THREADS, t = own_value < box ? own_value : min(tid, box - 1);
    from[v] = t;
    int k = t / hx, yy, zz;
    const int i = t - k * hx;
    if (k < 2 * tz) {
      yy = -1 - k / tz;
      zz = k % tz;
    } else if ((k -= 2 * tz) < 2 * tz) {
      yy = ty + k / tz;
      zz = k % tz;
    } else if ((k -= 2 * tz) < 2 * ty) {
      zz = -1 - k / ty;
      yy = k % ty;
    } else if ((k -= 2 * ty) < 2 * ty) {
      zz = tz + k / ty;
      yy = k % ty;
    } else {
      k -= 2 * ty;
      yy = k & 1 ? ty : -1;
      zz = k & 2 ? tz : -1;
    }
    dst[v] = row_at(yy, zz) + i;
  }
  // the mailboxes of the eight neighbours
  const int wyl = wy == 0 ? a.gy - 1 : wy - 1, wyh = wy == a.gy - 1 ? 0 : wy + 1;
  const int wzl = wz == 0 ? a.gz - 1 : wz - 1, wzh = wz == a.gz - 1 ? 0 : wz + 1;
  const size_t set = (size_t)W * box;
  uint64_t* const mail = a.mail + a.bank * SOR_SETS * set;
  auto mail_of = [&](int y, int z) { return mail + (size_t)(z * a.gy + y) * box; };
  const uint64_t* const mine = mail_of(wy, wz);
  constexpr int LAST = TAKE - 1;
  const bool has_last = tid + LAST * SOR_THREADS < box;
  // the words of the last two iterations: received, and sent (the same to all)
  uint64_t got[2][TAKE], gave[2][U];
#pragma unroll
  for (int k = 0; k < TAKE; ++k) got[0][k] = got[1][k] = SOR_UNSENT;
#pragma unroll
  for (int u = 0; u < U; ++u) gave[0][u] = gave[1][u] = SOR_UNSENT;
  // takes the values sent after iteration it into the rings
  auto take = [&](int it) {
    const uint64_t* words = mine + (it & 1) * set;
    uint64_t v[TAKE];
    int spins = 0;
    bool waits;
    // The values cannot be there before a trip through the memory side; a
    // look before that comes back empty only after the next could have come
    // back full (64x48x48: 2.55 us an iteration after a pause of 256 clocks,
    // 2.43 of 512, 2.23 of 768, 2.29 of 1024; 64x64x128: 3.09, 3.02, 3.03, 3.11).
    __builtin_amdgcn_s_sleep(12);
    if (tid >= box) return;
    do {
      // a branch for the last value only: each would wait for the load before
      // it (a branch per value: 2.45 instead of 2.00 us at 32^3)
#pragma unroll
      for (int k = 0; k < LAST; ++k)
        v[k] = __hip_atomic_load(words + from[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      v[LAST] = ~got[0][LAST];
      if (has_last)
        v[LAST] = __hip_atomic_load(words + from[LAST], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      waits = false;
#pragma unroll
      for (int k = 0; k < TAKE; ++k) waits |= v[k] == got[0][k];
      if (waits && ++spins > a.spin_limit) {
        s_abort = 1;
        break;
      }
    } while (waits);
#pragma unroll
    for (int k = 0; k < TAKE; ++k) {
      if (k < LAST || has_last)
        P[plane + dst[k]] = __longlong_as_double((long long)sor_value(v[k], got[0][k]));
      got[0][k] = got[1][k];
      got[1][k] = v[k];
    }
  };
  const double rj = a.rj;
  // this iteration's factors of red and black; the next ones are computed
  // while the neighbours' values are on their way
  double omega = c.omega, omega_black;
  omega_black = c.base == 0 ? chebyshev_first(rj) : chebyshev_next(rj, omega);
  double acc = 0.0;
  // sum over the face neighbours (of the other colour) of the site of colour
  // k at LDS index o; the two in x commute
  auto around = [&](int k, int o, int o2, int m) -> double {
    const double* q = P + (k ^ 1) * plane;
    const double x1 = q[o], x2 = q[o2];
    const double ym = q[o - hx], yp = q[o + hx], zm = q[o - ry * hx], zp = q[o + ry * hx];
    if constexpr (NEU) {
      double s = 0.0;
      s += m & 2 ? x1 : 0.0;
      s += m & 4 ? x2 : 0.0;
      s += m & 8 ? ym : 0.0;
      s += m & 16 ? yp : 0.0;
      s += m & 32 ? zm : 0.0;
      s += m & 64 ? zp : 0.0;
      return s;
    } else {
      return x1 + x2 + ym + yp + zm + zp;
    }
  };
  auto relaxed = [&](double w_sor, double old, double s, double f, int m) {
    if constexpr (NEU) return old + w_sor * ((s - f) / double(__builtin_popcount(m & 126)) - old);
    else return old + w_sor * ((s - f) * (1.0 / 6.0) - old);
  };
  // squared residual at a site with neighbour sum s and value v
  auto square = [&](int k, int u, double s, double v) {
    const double d = NEU ? double(__builtin_popcount(open[k][u] & 126)) : 6.0;
    const double lap = s - d * v;
    const double r = rhs[k][u] - lap;
    return r * r;
  };
  // the workgroup's sum of iteration it: by waves, and after the next barrier
  // over the waves
  auto sum_waves = [&] {
    const double s = wave_sum(acc);
    if ((tid & 63) == 0) s_sum[tid >> 6] = s;
    acc = 0.0;
  };
  double* part = a.part + (size_t)((a.launch & 1) ^ 1) * SOR_MAX_BATCH * W;
  auto store_part = [&](int it) {
    if (tid == 0) {
      double s = s_sum[0];
      for (int k = 1; k < SOR_WAVES; ++k) s += s_sum[k];
      part[(size_t)(it - 1) * W + w] = s;
    }
  };
  auto give_up = [&] {
    if (tid != 0) return;
    // the same values from every workgroup that gives up, or ends (w == 0)
    SorControl* o = a.ctl + ((a.launch & 1) ^ 1);
    __hip_atomic_store(&o->cur, c.cur, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&o->base, c.base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&o->aborted, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  bool test = false;
  int since = c.base % a.every;          // iterations since the last multiple of `every`
  for (int it = 1; it <= n_it; ++it) {
    const bool prev = test;
    since = since + 1 == a.every ? 0 : since + 1;
    test = since == 0 || c.base + it == a.max_iter;
    if (it > 1) take(it - 1);
    __syncthreads();
    if (s_abort) return give_up();
    // red, in the tile and in the ring around it
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (tid + u * SOR_THREADS < items && (!NEU || (open[0][u] & 1))) {
        double* p = P + own[u];
        const double old = *p, s = around(0, own[u], own2[0][u], open[0][u]);
        if (prev) acc += square(0, u, s, old);
        *p = relaxed(omega, old, s, rhs[0][u], open[0][u]);
      }
      if (tid + u * SOR_THREADS < ring_items && (!NEU || (ring_open[u] & 1))) {
        double* p = P + ring[u];
        *p = relaxed(omega, *p, around(0, ring[u], ring2[u], ring_open[u]), ring_rhs[u], ring_open[u]);
      }
    }
    if (prev) sum_waves();
    __syncthreads();
    if (prev) store_part(it - 1);
    // black, and to the neighbours
    const size_t at = (it & 1) * set;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (tid + u * SOR_THREADS >= items) continue;
      double* p = P + plane + own[u];
      double v = *p;
      if (!NEU || (open[1][u] & 1)) {
        const double s = around(1, own[u], own2[1][u], open[1][u]);
        v = relaxed(omega_black, v, s, rhs[1][u], open[1][u]);
        if (test) acc += square(1, u, s, v);
        *p = v;
      }
      const int yy = yz[u] & 0xffff, zz = yz[u] >> 16, i = own[u] - row_at(yy, zz);
      const uint64_t m = sor_word((uint64_t)__double_as_longlong(v), gave[0][u]);
      gave[0][u] = gave[1][u];
      gave[1][u] = m;
      auto put = [&](uint64_t* to, int row) {
        __hip_atomic_store(to + at + row * hx + i, m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      };
      const bool yl = yy == 0, yh = yy == ty - 1, zl = zz == 0, zh = zz == tz - 1;
      if (yy < 2) put(mail_of(wyl, wz), 2 * tz + yy * tz + zz);
      if (yy >= ty - 2) put(mail_of(wyh, wz), (ty - 1 - yy) * tz + zz);
      if (zz < 2) put(mail_of(wy, wzl), 4 * tz + 2 * ty + zz * ty + yy);
      if (zz >= tz - 2) put(mail_of(wy, wzh), 4 * tz + (tz - 1 - zz) * ty + yy);
      const int corner = 4 * (ty + tz);
      if (yl && zl) put(mail_of(wyl, wzl), corner + 3);
      if (yh && zl) put(mail_of(wyh, wzl), corner + 2);
      if (yl && zh) put(mail_of(wyl, wzh), corner + 1);
      if (yh && zh) put(mail_of(wyh, wzh), corner);
    }
    omega = chebyshev_next(rj, omega_black);
    omega_black = chebyshev_next(rj, omega);
  }
  take(n_it);
  __syncthreads();
  if (s_abort) return give_up();
  if (test) {
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (tid + u * SOR_THREADS < items && (!NEU || (open[0][u] & 1)))
        acc += square(0, u, around(0, own[u], own2[0][u], open[0][u]), P[own[u]]);
    sum_waves();
    __syncthreads();
    store_part(n_it);
  }
  for (int t = tid; t < rows * a.nx; t += SOR_THREADS) {
    const int r = t / a.nx, x = t - r * a.nx;
    const int zz = r / ty, yy = r - zz * ty, y = y0 + yy, z = z0 + zz;
    out[((long long)z * a.ny + y) * a.nx + x] =
        P[((x + y + z) & 1) * plane + row_at(yy, zz) + (x >> 1)];
  }
  if (w == 0 && tid == 0) {
    SorControl* o = a.ctl + ((a.launch & 1) ^ 1);
    o->state = c.state;
    __hip_atomic_store(&o->cur, c.cur, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(&o->base, c.base, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    o->n = c.n;
    o->found = c.found;
    o->omega = c.omega;
    o->omega_next = omega;
  }
}

__global__ void k_sor_reset(SorControl* c) {
  if (threadIdx.x < 2) c[threadIdx.x] = SorControl{SOR_START, 0, 0, 0, 0, 0, 1.0, 1.0};
}

__global__ __launch_bounds__(256) void k_mail_fill(uint64_t* mail, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) mail[i] = SOR_UNSENT;
}

size_t al256(size_t b) { return (b + 255) & ~size_t(255); }

size_t tile_lds(int nx, int ty, int tz) { return (size_t)(ty + 4) * (tz + 4) * nx * 8; }
int box_rows(int ty, int tz) { return 4 * (ty + tz) + 4; }
size_t mail_words(const SorPlan& p, int nx) {
  return (size_t)SOR_BANKS * SOR_SETS * p.gy * p.gz * box_rows(p.ty, p.tz) * (nx / 2);
}

}  // namespace

// The tile of whole x-rows: the most workgroups up to one per compute unit
// (the shortest half sweep), and of equal counts the least face.
bool ek::sor_plan(int nx, int ny, int nz, SorPlan& p) {
  p = SorPlan{};
  const int hx = nx / 2;
  for (int ty = 2; ty <= ny; ++ty) {
    if (ny % ty) continue;
    for (int tz = 2; tz <= nz; ++tz) {
      if (nz % tz) continue;
      const int groups = (ny / ty) * (nz / tz);
      const long long items = std::max((long long)ty * tz, 2LL * (ty + tz)) * hx;
      if (groups > SOR_MAX_GROUPS || items > (long long)SOR_MAX_ITEMS * SOR_THREADS ||
          (long long)box_rows(ty, tz) * hx > (long long)SOR_MAX_TAKE * SOR_THREADS ||
          tile_lds(nx, ty, tz) > SOR_LDS_MAX)
        continue;
      const int best = p.gy * p.gz;
      if (groups > best || (groups == best && ty + tz < p.ty + p.tz)) {
        p.ty = ty;
        p.tz = tz;
        p.gy = ny / ty;
        p.gz = nz / tz;
      }
    }
  }
  return p.ty > 0;
}

size_t ek::sor_bytes(int nx, int ny, int nz) {
  SorPlan p;
  if (!sor_plan(nx, ny, nz, p)) return 0;
  const size_t groups = (size_t)p.gy * p.gz;
  return al256((size_t)nx * ny * nz * 8) + al256(mail_words(p, nx) * 8) +
         al256((size_t)2 * SOR_MAX_BATCH * groups * 8) + 256;
}

void ek_ctx::sor_setup(char* mem) {
  if (!sor_plan(p.nx, p.ny, p.nz, sor)) return;
  const size_t groups = (size_t)sor.gy * sor.gz;
  sor.tmp = (double*)mem;
  mem += al256((size_t)dims.n * 8);
  sor.mail = (uint64_t*)mem;
  mem += al256(mail_words(sor, p.nx) * 8);
  sor.part = (double*)mem;
  mem += al256((size_t)2 * SOR_MAX_BATCH * groups * 8);
  sor.ctl = (SorControl*)mem;
  const size_t words = mail_words(sor, p.nx);
  hipLaunchKernelGGL(k_mail_fill, dim3(int((words + 255) / 256)), dim3(256), 0, stream, sor.mail,
                     words);
  sor.ok = true;
}

extern "C" void ek_test_sor_batches(ek_ctx* ctx, int spin_limit, int limit_from, int refuse_at) {
  ctx->sor.spin_limit = spin_limit;
  ctx->sor.limit_from = limit_from;
  ctx->sor.refuse_at = refuse_at;
}

// The solve of sor_solve by batches in one launch each; false (and x as it
// was) where that is not possible here.  `it` iterations are in x, with `omega`
// for the half sweep after them, and `it` of them afterwards; the caller goes on
// from there where h says that the solve is not done.
bool ek_ctx::sor_team_solve(const double* bb, double* x, PoissonScalars& h, int& it, double omega,
                            ek_status& st) {
  st = EK_OK;
  if (!sor.ok) return false;
  SorArgs a{};
  a.buf[0] = x;
  a.buf[1] = sor.tmp;
  a.b = bb;
  a.mask = mask;
  a.ps = ps;
  a.ctl = sor.ctl;
  a.mail = sor.mail;
  a.part = sor.part;
  a.nx = p.nx;
  a.ny = p.ny;
  a.nz = p.nz;
  a.ty = sor.ty;
  a.tz = sor.tz;
  a.gy = sor.gy;
  a.gz = sor.gz;
  a.start = it;
  a.omega = omega;
  a.max_iter = p.poisson_max_iter;
  a.every = p.poisson_check_every;
  a.rj = jacobi_radius();
  a.tol = p.poisson_tol;
  const int groups = sor.gy * sor.gz;
  const int items = std::max(sor.ty * sor.tz, 2 * (sor.ty + sor.tz)) * (p.nx / 2);
  const size_t lds = tile_lds(p.nx, sor.ty, sor.tz);
  auto launch = [&](auto kernel) -> bool {
    if (lds > 64 * 1024 &&
        hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    if (a.launch == sor.refuse_at) return false;
    a.spin_limit = a.launch >= sor.limit_from ? sor.spin_limit : SOR_SPIN_LIMIT;
    a.bank = sor.bank;
    void* args[] = {(void*)&a};
    if (hipLaunchCooperativeKernel((const void*)kernel, dim3(groups), dim3(SOR_THREADS), args,
                                   (unsigned)lds, stream) != hipSuccess) {
      (void)hipGetLastError();
      return false;
    }
    sor.bank ^= 1;
    return true;
  };
  const int u = (items + SOR_THREADS - 1) / SOR_THREADS;
  const int take = (box_rows(sor.ty, sor.tz) * (p.nx / 2) + SOR_THREADS - 1) / SOR_THREADS;
  // the smallest instance (the ring has two sites a row and the mailbox four
  // values, and a corner's rows: take <= 2 u + 1 up to 64 sites along x)
  auto run_as = [&](auto neu) -> bool {
    constexpr bool NEU = decltype(neu)::value;
    if (u == 1 && take == 1) return launch(k_sor_team<NEU, 1, 1>);
    if (u == 1 && take == 2) return launch(k_sor_team<NEU, 1, 2>);
    if (u == 1 && take == 3) return launch(k_sor_team<NEU, 1, 3>);
    if (u == 1 && take <= 4) return launch(k_sor_team<NEU, 1, 4>);
    if (u <= 2 && take <= 4) return launch(k_sor_team<NEU, 2, 4>);
    if (u <= 2) return launch(k_sor_team<NEU, 2, 8>);
    return launch(k_sor_team<NEU, 4, 8>);
  };
  auto run = [&] { return insulating() ? run_as(std::true_type{}) : run_as(std::false_type{}); };
  hipLaunchKernelGGL(k_sor_reset, dim3(1), dim3(64), 0, stream, sor.ctl);
  SorControl c{};
  // full batches, the two that end the solve, its second run and the verdict
  // on that (a launch with nothing left to run ends at once)
  const int expect = it > 0 ? SOR_AFTER : last_iters > 0 ? last_iters : 200;
  a.first = std::min({expect > SOR_NEAR ? expect - SOR_SHORT : expect + 2, SOR_MAX_BATCH,
                      p.poisson_max_iter - it});
  int ahead = expect / SOR_MAX_BATCH + 4;
  bool refused = false;
  while (c.state < SOR_FINAL && !c.aborted && !refused) {
    for (int k = 0; k < ahead && !refused; ++k) {
      refused = !run();
      if (refused && a.launch == 0) {
        sor.ok = false;
        return false;
      }
      if (!refused) ++a.launch;
    }
    ahead = 2;
    if (hipMemcpyAsync(pinned, sor.ctl + (a.launch & 1), sizeof c, hipMemcpyDeviceToHost, stream) !=
        hipSuccess) {
      st = fail(EK_EHIP, "reading the solve's state failed");
      return true;
    }
    st = sync();
    if (st) return true;
    std::memcpy(&c, pinned, sizeof c);
  }
  // without a result of its own: from what the last launch started from
  const bool left = c.aborted || c.state < SOR_FINAL;
  if (c.aborted || refused) sor.ok = false;
  if (c.cur == 1 &&
      hipMemcpyAsync(x, sor.tmp, dims.n * 8, hipMemcpyDeviceToDevice, stream) != hipSuccess) {
    st = fail(EK_EHIP, "copying the iterate failed");
    return true;
  }
  if (left) {
    it = c.base;
    return true;
  }
  // the residual of the result as the single launches take it
  it = c.state == SOR_FINAL ? c.found : c.base;
  const int nr = residual_launch(bb, x);
  launch_residual_final(partials, nr, p.poisson_tol, it, 0, ps, stream);
  st = read_scalars(&h);
  return true;
}
