// Discrete Hartley transforms of lines held in LDS, and the direct solution of
// the periodic 7-point problem that they give.
//
// The Hartley transform H_k = sum_j x_j cas(2 pi j k / n), cas = cos + sin, is
// real, is its own inverse up to 1/n, and its basis vectors are eigenvectors
// of the periodic second difference with eigenvalue 2 cos(2 pi k / n) - 2.
// Applied along x, y and z it therefore turns
//   (sum of the 6 neighbours - 6 x) / h^2 = f
// into a division by the sum of three such eigenvalues (the constant mode,
// whose eigenvalue is 0, is set to 0).
//
// Two real lines a, b are transformed as one complex line a + i b by a
// mixed-radix Stockham FFT (radices 2, 3, 4, 5, 8 and any larger prime), in
// place in LDS (every thread holds its butterflies in registers over a
// barrier), and separated afterwards:
//   H_a[k] = ((Zr[k] + Zr[-k]) - (Zi[k] - Zi[-k])) / 2
//   H_b[k] = ((Zi[k] + Zi[-k]) + (Zr[k] - Zr[-k])) / 2
#pragma once

#include <hip/hip_runtime.h>

#include "ek_internal.h"

namespace ek {

constexpr int DHT_MAX_N = 960;       // longest line: its tile of 16 columns fits LDS

// Radices of a line of n sites, packed so that a kernel keeps them in scalar
// registers: four bits a pass in `code`, the radix itself for 2, 3, 4, 5 and
// 8, PRIME_PASS for the next of `prime` (up to three primes from 7 on).
constexpr int PRIME_PASS = 7;
struct DhtPlan {
  unsigned long long code = 0;
  int n = 0;
  int count = 0;
  int primes = 0;
  int prime[3] = {0, 0, 0};
};

// The plan of n, or false where n is odd or too long.
bool dht_plan(int n, DhtPlan& plan);

struct Cx {
  double r, i;
};
__device__ __forceinline__ Cx cadd(Cx a, Cx b) { return {a.r + b.r, a.i + b.i}; }
__device__ __forceinline__ Cx csub(Cx a, Cx b) { return {a.r - b.r, a.i - b.i}; }
__device__ __forceinline__ Cx cmul(Cx a, Cx b) { return {a.r * b.r - a.i * b.i, a.r * b.i + a.i * b.r}; }
// -i a
__device__ __forceinline__ Cx cnegi(Cx a) { return {a.i, -a.r}; }

// cos and sin of 2 pi m / R for the odd radices 3 and 5.
template <int R>
__device__ __forceinline__ constexpr double dht_cos(int m) {
  constexpr double c3[] = {1.0, -0.5};
  constexpr double c5[] = {1.0, 0.30901699437494742410, -0.80901699437494742410};
  const int k = m % R, h = k > R / 2 ? R - k : k;
  return R == 3 ? c3[h] : c5[h];
}
template <int R>
__device__ __forceinline__ constexpr double dht_sin(int m) {
  constexpr double s3[] = {0.0, 0.86602540378443864676};
  constexpr double s5[] = {0.0, 0.95105651629515357212, 0.58778525229247312917};
  const int k = m % R, h = k > R / 2 ? R - k : k;
  const double s = R == 3 ? s3[h] : s5[h];
  return k > R / 2 ? -s : s;
}

// Forward DFT of R values: v_k <- sum_j v_j exp(-2 pi i j k / R).
template <int R>
__device__ __forceinline__ void butterfly(Cx (&v)[R]) {
  if constexpr (R == 2) {
    const Cx a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
  } else if constexpr (R == 4) {
    const Cx t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    const Cx t2 = cadd(v[1], v[3]), t3 = cnegi(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, t3);
    v[3] = csub(t1, t3);
  } else if constexpr (R == 8) {
    constexpr double h = 0.70710678118654752440;
    Cx e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
    butterfly<4>(e);
    butterfly<4>(o);
    const Cx w1 = {h * (o[1].r + o[1].i), h * (o[1].i - o[1].r)};
    const Cx w2 = cnegi(o[2]);
    const Cx w3 = {h * (o[3].i - o[3].r), -h * (o[3].r + o[3].i)};
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], w1);
    v[5] = csub(e[1], w1);
    v[2] = cadd(e[2], w2);
    v[6] = csub(e[2], w2);
    v[3] = cadd(e[3], w3);
    v[7] = csub(e[3], w3);
  } else {
    constexpr int H = R / 2;
    Cx p[H], m[H];
#pragma unroll
    for (int j = 0; j < H; ++j) {
      p[j] = cadd(v[j + 1], v[R - 1 - j]);
      m[j] = csub(v[j + 1], v[R - 1 - j]);
    }
    const Cx z = v[0];
#pragma unroll
    for (int j = 0; j < H; ++j) v[0] = cadd(v[0], p[j]);
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      Cx a = z, b = {0.0, 0.0};
#pragma unroll
      for (int j = 0; j < H; ++j) {
        const double c = dht_cos<R>((j + 1) * k), s = dht_sin<R>((j + 1) * k);
        a.r += c * p[j].r;
        a.i += c * p[j].i;
        b.r += s * m[j].i;
        b.i -= s * m[j].r;
      }
      v[k] = cadd(a, b);
      v[R - k] = csub(a, b);
    }
  }
}

// t / d and t - d (t / d) for 0 <= t < 2^24 (the float quotient is off by at
// most one).
__device__ __forceinline__ int divide(int t, int d, float inv_d, int& rem) {
  int q = int(float(t) * inv_d);
  rem = t - q * d;
  if (rem < 0) { --q; rem += d; }
  else if (rem >= d) { ++q; rem -= d; }
  return q;
}

// Lines in LDS: element j of complex line l has its real part at
// D[l * ls + j * ps] and its imaginary part `im` further on.
struct Lines {
  int count, ls, ps, im;
};

// One radix-R pass over all lines, s = the product of the radices before it.
// A thread takes up to U butterflies (U R complex values in registers);
// n / R * count <= U * nthr.
template <int R, int U>
__device__ __forceinline__ void dht_pass(double* D, const double2* tw, int n, int s, const Lines& L,
                                         int tid, int nthr) {
  const int nb = n / R, items = nb * L.count, m = nb / s;
  const float inv_l = 1.0f / L.count, inv_s = 1.0f / s;
  Cx v[U][R];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int it = tid + u * nthr;
    if (it < items) {
      int l;
      const int t = divide(it, L.count, inv_l, l);
      const double* src = D + l * L.ls + t * L.ps;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        v[u][j].r = src[j * nb * L.ps];
        v[u][j].i = src[j * nb * L.ps + L.im];
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int it = tid + u * nthr;
    if (it < items) {
      int l, q;
      const int t = divide(it, L.count, inv_l, l);
      const int p = divide(t, s, inv_s, q);
      butterfly<R>(v[u]);
      if (m > 1) {
#pragma unroll
        for (int j = 1; j < R; ++j) {
          const double2 w = tw[p * j * s];
          v[u][j] = cmul(v[u][j], Cx{w.x, w.y});
        }
      }
      double* dst = D + l * L.ls + (q + s * R * p) * L.ps;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        dst[j * s * L.ps] = v[u][j].r;
        dst[j * s * L.ps + L.im] = v[u][j].i;
      }
    }
  }
  __syncthreads();
}

// A pass of any prime radix R >= 7, as R sums of R terms: a thread takes up to
// U groups of four outputs of one butterfly, whose inputs it reads once for
// all four (a butterfly of its own per thread would hold R values and as many
// constants in registers).  ceil(R / 4) * n / R * count <= U * nthr.
template <int U>
__device__ __forceinline__ void dht_pass_prime(double* D, const double2* tw, int n, int R, int s,
                                               const Lines& L, int tid, int nthr) {
  const int nb = n / R, m = nb / s, items = (R + 3) / 4 * nb * L.count;
  const float inv_l = 1.0f / L.count, inv_b = 1.0f / nb, inv_s = 1.0f / s;
  Cx v[U][4];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int it = tid + u * nthr;
#pragma unroll
    for (int c = 0; c < 4; ++c) v[u][c] = Cx{0.0, 0.0};
    if (it < items) {
      int l, t;
      const int rest = divide(it, L.count, inv_l, l);
      const int j0 = 4 * divide(rest, nb, inv_b, t);
      const double* src = D + l * L.ls + t * L.ps;
      int at[4] = {0, 0, 0, 0};
      for (int i = 0; i < R; ++i) {
        const Cx x{src[i * nb * L.ps], src[i * nb * L.ps + L.im]};
#pragma unroll
        for (int c = 0; c < 4; ++c) {
          const double2 w = tw[at[c] * nb];
          v[u][c] = cadd(v[u][c], cmul(x, Cx{w.x, w.y}));
          at[c] += j0 + c;                 // (i + 1) j mod R; j <= R + 2
          if (at[c] >= R) at[c] -= R;
          if (at[c] >= R) at[c] -= R;
        }
      }
    }
  }
  __syncthreads();
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int it = tid + u * nthr;
    if (it < items) {
      int l, t, q;
      const int rest = divide(it, L.count, inv_l, l);
      const int j0 = 4 * divide(rest, nb, inv_b, t);
      const int p = divide(t, s, inv_s, q);
      double* dst = D + l * L.ls + (q + s * R * p) * L.ps;
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        const int j = j0 + c;
        if (j >= R) continue;
        const double2 w = tw[p * j * s];
        const Cx y = m > 1 ? cmul(v[u][c], Cx{w.x, w.y}) : v[u][c];
        dst[j * s * L.ps] = y.r;
        dst[j * s * L.ps + L.im] = y.i;
      }
    }
  }
  __syncthreads();
}

// FFT of all lines (the caller has synchronised their values); EPT complex
// values per thread at most.  `tw` holds exp(-2 pi i k / n), k < n.  PRIME
// compiles in the pass of the primes from 7 on, whose registers would halve
// the waves in flight of the plans that have none.
template <int EPT, bool PRIME>
__device__ inline void fft_lines(double* D, const double2* tw, const DhtPlan& plan, const Lines& L,
                                 int tid, int nthr) {
  int s = 1, np = 0;
  unsigned long long code = plan.code;
#pragma unroll 1
  for (int k = 0; k < plan.count; ++k, code >>= 4) {
    int r = int(code & 15);
    switch (r) {
      case 2: dht_pass<2, (EPT + 1) / 2>(D, tw, plan.n, s, L, tid, nthr); break;
      case 3: dht_pass<3, (EPT + 2) / 3>(D, tw, plan.n, s, L, tid, nthr); break;
      case 4: dht_pass<4, (EPT + 3) / 4>(D, tw, plan.n, s, L, tid, nthr); break;
      case 5: dht_pass<5, (EPT + 4) / 5>(D, tw, plan.n, s, L, tid, nthr); break;
      case 8: dht_pass<8, (EPT + 7) / 8>(D, tw, plan.n, s, L, tid, nthr); break;
      default:
        if constexpr (PRIME) {
          r = np == 0 ? plan.prime[0] : np == 1 ? plan.prime[1] : plan.prime[2];
          ++np;
          dht_pass_prime<EPT / 4 + 1>(D, tw, plan.n, r, s, L, tid, nthr);
        }
    }
    s *= r;
  }
}

// True where every pass of the plan fits EPT values per thread.
inline bool fft_fits(const DhtPlan& plan, int lines, int ept, int nthr) {
  for (int k = 0, np = 0; k < plan.count; ++k) {
    const int code = int((plan.code >> (4 * k)) & 15);
    const bool own = code != PRIME_PASS;
    const int r = own ? code : plan.prime[np++];
    const long long u = own ? (ept + r - 1) / r : ept / 4 + 1;
    const long long items = (own ? 1 : (r + 3) / 4) * (long long)(plan.n / r) * lines;
    if (items > u * nthr) return false;
  }
  return true;
}

// The Hartley values of both lines at k and n - k from the FFT's Z.
struct HartleyPair {
  double a, an, b, bn;   // H_a[k], H_a[n - k], H_b[k], H_b[n - k]
};
__device__ __forceinline__ HartleyPair hartley(Cx z, Cx zn) {
  const double sr = z.r + zn.r, dr = z.r - zn.r, si = z.i + zn.i, di = z.i - zn.i;
  return {0.5 * (sr - di), 0.5 * (sr + di), 0.5 * (si + dr), 0.5 * (si - dr)};
}

// Separation in place: the lines become H_a (real parts) and H_b (imaginary).
__device__ inline void separate_lines(double* D, int n, const Lines& L, int tid, int nthr) {
  const int half = n / 2 + 1, items = half * L.count;
  const float inv_l = 1.0f / L.count;
  for (int it = tid; it < items; it += nthr) {
    int l;
    const int k = divide(it, L.count, inv_l, l);
    const int kn = k == 0 ? 0 : n - k;
    double* z = D + l * L.ls + k * L.ps;
    double* zn = D + l * L.ls + kn * L.ps;
    const HartleyPair h = hartley({z[0], z[L.im]}, {zn[0], zn[L.im]});
    z[0] = h.a;
    z[L.im] = h.b;
    zn[0] = h.an;
    zn[L.im] = h.bn;
  }
  __syncthreads();
}

// Multigrid cycles within which every tolerance that double precision can
// hold is met (a cycle takes a digit at the least).  A caller who allows fewer
// may mean the limit to bind, and it counts multigrid cycles: the direct
// solve, which needs one, is for those who allow this many.
constexpr int DIRECT_MIN_CYCLES = 20;

// The fields of one of several problems on the same grid, solved by the same
// launches (blockIdx.y picks the problem).
struct SpecItem {
  double* x;
  const double* f;
  const PoissonScalars* ps;
  double* partials;
  double* hat;
};

// A direct solver of one periodic grid: plans, tables and the work field.
struct Spectral {
  bool ok = false;
  int nx = 0, ny = 0, nz = 0;
  double h2 = 1.0;
  DhtPlan px, py, pz;
  const double2 *tx = nullptr, *ty = nullptr, *tz = nullptr;   // exp(-2 pi i k / n)
  const double *lx = nullptr, *ly = nullptr, *lz = nullptr;    // 2 cos(2 pi k / n) - 2
  double* hat = nullptr;
  // launch shapes of the passes (kernels_spectral.hip); plane_shape >= 0: x and
  // y in one pass over whole planes, else rows and columns in passes of their own
  int plane_shape = -1, row_shape = -1, col_shape = -1, z_shape = -1;
  // a plan of the pass has a prime factor from 7 on
  bool plane_prime = false, row_prime = false, col_prime = false, z_prime = false;
};

// Bytes of the work field and the tables (0: the grid has no plan).
size_t spectral_bytes(int nx, int ny, int nz);
size_t spectral_table_bytes(int nx, int ny, int nz);   // the tables alone
// Fills `s` for the grid in `mem` (256-byte aligned) and copies the tables
// there; s.ok stays false where the grid has no plan or a copy fails.  The
// work field comes first in `mem`; without it (own_field false) `mem` holds
// the tables alone and the fields come with each launch.
void spectral_setup(Spectral& s, char* mem, int nx, int ny, int nz, double h2,
                    bool own_field = true);
// Right-hand side into the work field, transformed along x and y.  With x
// (the current iterate) it is the residual f + shift - A x, whose norms (as
// launch_residual) go to `partials`; the number of blocks is returned.
// Without x it is f as it is.
// With `items` the same launches take `count` problems (residual and norms).
int launch_spectral_forward(const Spectral& s, const double* x, const double* f,
                            const PoissonScalars* ps, double* partials, hipStream_t st,
                            const SpecItem* items = nullptr, int count = 1);
int spectral_blocks(const Spectral& s);
// The rest: along z and back, then x += solution (add) or x = solution.
// With `items` for `count` problems: x += solution less the mean of the start
// (psum / n of the problem's scalars), which the solution leaves as it is.
void launch_spectral_solve(const Spectral& s, double* x, bool add, const PoissonScalars* ps,
                           hipStream_t st, const SpecItem* items = nullptr, int count = 1);

}  // namespace ek
