// Bead-spring chain coupled to the three species by friction (Sec. II.B)
// through the trilinear interpolation / spreading kernel (Sec. II.C): state,
// node table access and the per-step pieces, shared by the single-system
// kernels and the persistent ensemble kernel.
#pragma once

#include <climits>
#include <cmath>
#include <type_traits>

#include "ek_internal.h"
#include "md_table.h"
#include "philox.h"

namespace ek {

constexpr int BOX = 4;          // moment box edge (nodes floor(R0) - 1 .. floor(R0) + 2)
constexpr int BOX3 = BOX * BOX * BOX;

// Wall reach WR: the bead-wall WCA looks at the wall sites floor(R) - WR ..
// floor(R) + 1 + WR in each axis (an S^3 cube around the bead's cell), which
// holds every site closer than WR + 1 to the bead: WR = 1 for a cut-off
// 2^(1/6) sigma below 2, WR = 2 below 3.  Since the bead stays within one
// cell of its start over a step, the flag window of the step spans
// floor(R0) - 1 - WR .. floor(R0) + 2 + WR, W = 2 WR + 4 sites per axis.
template <int WR>
struct WallGeom {
  static constexpr int S = 2 * WR + 2;
  static constexpr int S3 = S * S * S;
  static constexpr int W = 2 * WR + 4;
  static constexpr int ITEMS = 64 * W;   // of bead_box_item: a wave per plane of the window
};
// The window's flags, a bit per site: plane wz (8 x 8 bits, site (wx, wy) at
// wx + 8 wy) of the fluid sites at word wz, of the wall sites at 8 + wz.
constexpr int FLAG_WORDS = 16;
constexpr int MOM = 15;         // x[3] (n^a / n), 1/n^a [3], j[3][3]

enum : int { ERR_BOX = 1, ERR_FLUID = 2, ERR_BOND = 4, ERR_TABLE = 8 };

struct BeadState {
  double* R;          // [maxb][3]
  double* V;          // [maxb][3]
  double* q;          // [maxb]
  int* origin;        // [maxb][3] floor(R0) - 1 of the current step
  double* mom;        // [maxb][BOX3][MOM]
  double* efield;     // [maxb][BOX3][3]
  unsigned long long* flags;  // [maxb][FLAG_WORDS] of the window of the wall reach
  int* err;           // error bits
  int* cross = nullptr;  // [maxb][3] plane crossings: first step, last step, net count
};

// Views of the bead state carved from a context's bead memory (host side).
BeadState bead_state_view(char* mem, int max_beads);

__device__ inline int wrap(int i, int n) {
  i %= n;
  return i < 0 ? i + n : i;
}

__device__ inline long long site_of(int x, int y, int z, const Dims& d) {
  return ((long long)wrap(z, d.nz) * d.ny + wrap(y, d.ny)) * d.nx + wrap(x, d.nx);
}

__device__ inline long long ld_i64(const long long* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ inline int ld_i32(const int* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Find or insert `site`; flags the site for the lattice kernels.
__device__ inline int table_insert(int* keys, uint32_t* mask, long long site, int* err, int bits) {
  const int slots = 1 << bits;
  int h = hash_slot(site, bits);
  for (int k = 0; k < slots; ++k) {
    const int prev = atomicCAS(&keys[h], -1, int(site));
    if (prev == -1) {
      atomicOr(&mask[site], MASK_BEAD);
      return h;
    }
    if (prev == int(site)) return h;
    h = (h + 1) & (slots - 1);
  }
  atomicOr(err, ERR_TABLE);
  return -1;
}

// Slot of `site` if present (reads that see the atomics of this launch).
__device__ inline int table_find(const int* keys, long long site, int bits) {
  const int slots = 1 << bits;
  int h = hash_slot(site, bits);
  for (int k = 0; k < slots; ++k) {
    const int key = ld_i32(&keys[h]);
    if (key == int(site)) return h;
    if (key < 0) return -1;
    h = (h + 1) & (slots - 1);
  }
  return -1;
}

// Empty table (once, when the context is created: the workspace arrives
// uninitialised).
struct MDParams {
  int n, n_sub;
  double M, k_fene, R0, eps, sigma, gamma;
  double Lx, Ly, Lz;
  // crossing record of the plane z = z_plane (and its periodic images) in
  // bs.cross; `step` is the number of completed steps once this one ends
  int track = 0;
  int step = 0;
  double z_plane = 0.0;
  // bonds: 0 FENE (k_fene, R0) with the WCA between all pairs; 1 harmonic
  // (k_bond, l_bond, Eq. polymermodel) with the WCA only for |i - j| > 1
  int bond = 0;
  double k_bond = 0.0, l_bond = 0.0;
  // thermal noise (philox.h): xi ~ N(0, xi_scale^2) per component and
  // substep, xi_scale = sqrt(2 gamma k_B T / h), from the counter
  // (bead, tstep, substep, 1); tstep = steps completed before this one
  int thermal = 0;
  uint32_t key0 = 0, key1 = 0, tstep = 0;
  double xi_scale = 0.0;
  // coupling kernel: 0 trilinear, 1 the occupation cube of side 2 half_sigma
  // (Eq. totalforcefluid) for the velocity at the bead and the friction
  int theta = 0;
  double half_sigma = 0.5;
  // insulating walls: the field at the bead with the trilinear weights
  // renormalised over the fluid corners (where its charge was deposited)
  int field_fluid = 0;
};

__device__ inline double min_image(double v, double L) { return v - L * rint(v / L); }

// WCA force on a pair at squared distance r2 (factor multiplying the separation).
__device__ inline double wca_coef(double r2, double eps, double sigma) {
  const double rc2 = 1.2599210498948732 * sigma * sigma;   // (2^(1/6) sigma)^2
  if (r2 >= rc2) return 0.0;
  const double s2 = sigma * sigma / r2;
  const double s6 = s2 * s2 * s2;
  return 24.0 * eps * (2.0 * s6 * s6 - s6) / r2;
}

// Nearest integer (ties to even, as llrint) of x.  For |x| < 2^51 the sum
// x + 1.5 * 2^52 has a unit in the last place of 1, so its low mantissa bits
// hold the rounded value as an offset from the bits of 1.5 * 2^52; larger
// values take llrint.
__device__ inline long long round_fixed(double x) {
  if (__builtin_expect(fabs(x) < 2251799813685248.0, 1)) {       // 2^51
    const double t = x + 6755399441055744.0;                        // 1.5 * 2^52
    return __double_as_longlong(t) - 0x4338000000000000ll;
  }
  return llrint(x);
}

// Nine values scaled by g and rounded by round_fixed, the test for values
// beyond its range made once for all of them.
__device__ inline void round_fixed9(const double (&x)[3][3], double g, long long (&v)[9]) {
  double y[9], top = 0.0;
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    y[k] = x[k / 3][k % 3] * g;
    v[k] = __double_as_longlong(y[k] + 6755399441055744.0) - 0x4338000000000000ll;
    top = fmax(top, fabs(y[k]));
  }
  if (__builtin_expect(!(top < 2251799813685248.0), 0)) {
#pragma unroll
    for (int k = 0; k < 9; ++k) v[k] = round_fixed(y[k]);
  }
}

// Node accumulators for the friction impulse: the context's global table, or
// a table in LDS (sites it has no room for stay in the global table) that is
// flushed to the global one once after the substeps.  Values are int64 fixed
// point, so the sums are exact whatever the order of the additions.
struct GlobalNodes {
  int* keys;
  long long* vals;
  uint32_t* mask;
  int* err;
  int bits;
  __device__ int slot(long long site) { return table_insert(keys, mask, site, err, bits); }
  __device__ void get(int h, long long (&v)[9]) const {
#pragma unroll
    for (int c = 0; c < 9; ++c) v[c] = ld_i64(&vals[(size_t)h * SLOT_VALUES + 1 + c]);
  }
  __device__ void add(int h, const long long (&v)[9]) {
#pragma unroll
    for (int c = 0; c < 9; ++c)
      atomicAdd((unsigned long long*)&vals[(size_t)h * SLOT_VALUES + 1 + c], (unsigned long long)v[c]);
  }
};

// LDS probes of an insertion before the site goes to the global table.
constexpr int LDS_PROBES = 32;

// The nine values of a global slot, 0 without one.
__device__ inline void gn_get(const GlobalNodes& gn, int h, long long (&v)[9]) {
#pragma unroll
  for (int c = 0; c < 9; ++c) v[c] = 0;
  if (h >= 0) gn.get(h, v);
}

// The LDS table has any number of slots (positions h = mulhi(mix(site), slots)
// and linear probing); a site whose probe path holds no free slot within
// LDS_PROBES probes is kept in the global table instead.  Every lane that
// looks up a site walks the same path over slots that, once taken, stay
// taken, so all of them reach the same decision.  Slot codes: h >= 0 the LDS
// slot, h <= -2 the global slot -2 - h, -1 none (the global table is full).
struct LdsNodes {
  int* keys;          // LDS [slots]
  long long* vals;    // LDS [slots][9]
  int slots;
  int* err;
  GlobalNodes global;
  __device__ int slot(long long site) {
    const unsigned long long mix = (unsigned long long)site * 0x9E3779B97F4A7C15ull;
    int h = int(((mix >> 32) * (unsigned long long)slots) >> 32);
    const int probes = slots < LDS_PROBES ? slots : LDS_PROBES;
    for (int k = 0; k < probes; ++k) {
      const int prev = atomicCAS(&keys[h], -1, int(site));
      if (prev == -1 || prev == int(site)) return h;
      h = h + 1 == slots ? 0 : h + 1;
    }
    const int g = global.slot(site);
    return g < 0 ? -1 : -2 - g;
  }
  // The nine values of slot code h (0 without a slot).  All LDS reads are
  // issued before any is used: deciding LDS or global per value took one LDS
  // round trip and a branch for each of the nine.
  __device__ void get(int h, long long (&v)[9]) const {
    const long long* p = vals + (h >= 0 ? h : 0) * 9;
#pragma unroll
    for (int c = 0; c < 9; ++c) v[c] = p[c];
    if (h < 0) {
#pragma unroll
      for (int c = 0; c < 9; ++c) v[c] = 0;
      if (h < -1) global.get(-2 - h, v);
    }
  }
  __device__ void add(int h, const long long (&v)[9]) {
    if (h >= 0) {
#pragma unroll
      for (int c = 0; c < 9; ++c)
        atomicAdd((unsigned long long*)&vals[h * 9 + c], (unsigned long long)v[c]);
    } else {
      global.add(-2 - h, v);
    }
  }
};

// One workgroup per chain, TPB threads per bead: the lanes of a bead split
// its 8 corners, its pair partners and its wall sites, and combine their
// parts with a butterfly over the TPB lanes (every lane ends with the same
// bits, so all lanes advance the bead identically).  The exchanges are DPP
// lane moves within a row of 16 lanes: xor 1 and xor 2 as quad permutations;
// after those every lane of a quad holds the quad's sum, so the last level
// takes the other quad's sum from the mirrored lane of the group of 8
// (lane l reads lane 7 - l).  A bead's lanes are active together.
template <int CTRL>
__device__ inline double dpp_move(double v) {
  // every lane has a source, so there is no old value to set up first (which
  // took as many instructions as the moves)
  const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), CTRL, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), CTRL, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

template <int TPB>
__device__ inline double group_sum(double v) {
  static_assert(TPB == 1 || TPB == 2 || TPB == 4 || TPB == 8, "lanes per bead");
  constexpr int XOR1 = 0xB1;          // quad_perm [1, 0, 3, 2]
  constexpr int XOR2 = 0x4E;          // quad_perm [2, 3, 0, 1]
  constexpr int HALF_MIRROR = 0x141;  // row_half_mirror (lane l reads lane 7 - l of its 8)
  if constexpr (TPB >= 2) v += dpp_move<XOR1>(v);
  if constexpr (TPB >= 4) v += dpp_move<XOR2>(v);
  if constexpr (TPB >= 8) v += dpp_move<HALF_MIRROR>(v);
  return v;
}

// ---------------------------------------------------------------------------
// Per-step pieces written for a team of threads (tid, nthreads): a whole
// grid of one-thread-per-item launches, or one workgroup.
// ---------------------------------------------------------------------------

// Drop a table's entries and their site flags.
__device__ inline void table_clear_items(int* keys, long long* vals, uint32_t* mask, long long n,
                                         int bits, int tid, int nthreads) {
  for (int h = tid; h < (1 << bits); h += nthreads) {
    const int key = keys[h];
    if (key >= 0 && key < n) {
      atomicAnd(&mask[key], ~MASK_BEAD);
      keys[h] = -1;
#pragma unroll
      for (int c = 0; c < SLOT_VALUES; ++c) vals[(size_t)h * SLOT_VALUES + c] = 0;
    }
  }
}

// Bead charges on the 8 corner nodes with the plain trilinear weights, or
// (fluid_only, insulating walls) with the weights renormalised over the
// fluid corners.
__device__ inline void deposit_items(const BeadState& bs, int n, int* keys, long long* vals,
                                     uint32_t* mask, const Dims& d, int bits, int tid,
                                     int nthreads, bool fluid_only = false) {
  for (int t = tid; t < 8 * n; t += nthreads) {
    const int i = t >> 3, k = t & 7;
    const double* R = bs.R + 3 * i;
    const double fx = floor(R[0]), fy = floor(R[1]), fz = floor(R[2]);
    const double dx = R[0] - fx, dy = R[1] - fy, dz = R[2] - fz;
    const int ox = k & 1, oy = (k >> 1) & 1, oz = (k >> 2) & 1;
    double w = (ox ? dx : 1.0 - dx) * (oy ? dy : 1.0 - dy) * (oz ? dz : 1.0 - dz);
    const long long site = site_of(int(fx) + ox, int(fy) + oy, int(fz) + oz, d);
    if (fluid_only) {
      if (mask[site] & MASK_SOLID) continue;
      double wsum = 0.0;
      for (int k2 = 0; k2 < 8; ++k2) {
        const int px = k2 & 1, py = (k2 >> 1) & 1, pz = (k2 >> 2) & 1;
        if (mask[site_of(int(fx) + px, int(fy) + py, int(fz) + pz, d)] & MASK_SOLID) continue;
        wsum += (px ? dx : 1.0 - dx) * (py ? dy : 1.0 - dy) * (pz ? dz : 1.0 - dz);
      }
      w /= wsum;
    }
    const int h = table_insert(keys, mask, site, bs.err, bits);
    if (h < 0) continue;
    atomicAdd((unsigned long long*)&vals[(size_t)h * SLOT_VALUES],
              (unsigned long long)llrint(bs.q[i] * w * FIX_CHARGE));
  }
}

// Fields of time t around bead i: the 64 items of wave t / 64 (whole waves
// call it) set one plane of the fluid / wall flags of the flag window (W
// planes for the wall reach WR), item t < BOX3 the moments and field of one
// node of the 4^3 box.  The box origin is written by item 0.
// With `defer` set, every box node is also flagged MASK_DEFER: the chain's
// friction can only reach nodes of the boxes, so the lattice update of all
// other sites need not wait for it.
// With `walls` (insulating walls) the field at a fluid node takes the ghost
// value psi + Sigma_f / eps for a solid face neighbour, and is 0 at a solid
// node (the beads then interpolate it over fluid corners only).
template <typename T, int WR = 1>
__device__ inline void bead_box_item(const BeadState& bs, int i, int t, const T* __restrict__ f,
                                     const uint32_t* mask,
                                     const double* __restrict__ psi, const LBParams& lp,
                                     const Dims& d, uint32_t* defer = nullptr,
                                     const double* face_q = nullptr, double inv_eps = 0.0) {
  const double* R = bs.R + 3 * i;
  const int bx = int(floor(R[0])) - 1, by = int(floor(R[1])) - 1, bz = int(floor(R[2])) - 1;
  if (t == 0) {
    bs.origin[3 * i] = bx;
    bs.origin[3 * i + 1] = by;
    bs.origin[3 * i + 2] = bz;
  }
  using G = WallGeom<WR>;
  if (t < G::ITEMS) {
    const int wx = t & 7, wy = (t >> 3) & 7, wz = t >> 6;
    const bool in = wx < G::W && wy < G::W;
    uint32_t m = MASK_SOLID;
    if (in) m = mask[site_of(bx - WR + wx, by - WR + wy, bz - WR + wz, d)];
    const unsigned long long fluid = __ballot(in && !(m & MASK_SOLID));
    const unsigned long long wall = __ballot(in && (m & MASK_WALL));
    if ((t & 63) == 0) {
      bs.flags[(size_t)i * FLAG_WORDS + wz] = fluid;
      bs.flags[(size_t)i * FLAG_WORDS + 8 + wz] = wall;
    }
  }
  if (t >= BOX3) return;
  const int cx = bx + t % BOX, cy = by + (t / BOX) % BOX, cz = bz + t / (BOX * BOX);
  // offsets of the node and its neighbours along each axis: three divisions
  // (the wraps) in all, where one per pulled site cost more than the pulls
  const int x = wrap(cx, d.nx), y = wrap(cy, d.ny), z = wrap(cz, d.nz);
  const long long nxy = (long long)d.nx * d.ny;
  const long long xo[3] = {x == 0 ? d.nx - 1 : x - 1, x, x == d.nx - 1 ? 0 : x + 1};
  const long long yo[3] = {(y == 0 ? d.ny - 1 : y - 1) * (long long)d.nx, y * (long long)d.nx,
                           (y == d.ny - 1 ? 0 : y + 1) * (long long)d.nx};
  const long long zo[3] = {(z == 0 ? d.nz - 1 : z - 1) * nxy, z * nxy, (z == d.nz - 1 ? 0 : z + 1) * nxy};
  const long long r = zo[1] + yo[1] + xo[1];
  if (defer) atomicOr(&defer[r], MASK_DEFER);
  const uint32_t m = mask[r];
  double* mo = bs.mom + ((size_t)i * BOX3 + t) * MOM;
  // all 57 pulls are issued before any sum (registers only, one store pass)
  double v[MOM];
#pragma unroll
  for (int c = 0; c < MOM; ++c) v[c] = 0.0;
  if (!(m & MASK_SOLID)) {
    T g[3][Q];
#pragma unroll
    for (int p = 0; p < Q; ++p) {
      const bool bounce = (m >> p) & 1u;
      const long long src = bounce ? r : zo[1 - CZ[p]] + yo[1 - CY[p]] + xo[1 - CX[p]];
      const int q = bounce ? OPP[p] : p;
#pragma unroll
      for (int s = 0; s < 3; ++s) g[s][p] = f[(size_t)(s * Q + q) * d.n + src];
    }
    double n[3];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      double dn = 0.0, jx = 0.0, jy = 0.0, jz = 0.0;
#pragma unroll
      for (int p = 0; p < Q; ++p) {
        const double gp = double(g[s][p]);
        dn += gp;
        jx += CX[p] * gp;
        jy += CY[p] * gp;
        jz += CZ[p] * gp;
      }
      n[s] = lp.nref[s] + dn;
      v[6 + 3 * s] = jx;
      v[7 + 3 * s] = jy;
      v[8 + 3 * s] = jz;
    }
    const double ntot = n[0] + n[1] + n[2];
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      v[3 + s] = 1.0 / n[s];
      v[s] = n[s] / ntot;
    }
  }
#pragma unroll
  for (int c = 0; c < MOM; ++c) mo[c] = v[c];
  double* e = bs.efield + ((size_t)i * BOX3 + t) * 3;
  if (face_q) {
    if (m & MASK_SOLID) {
      e[0] = e[1] = e[2] = 0.0;
      return;
    }
    const double pc = psi[r];
    // bit p of the link word: the neighbour r - c_p is solid (1/2: -x/+x,
    // 3/4: -y/+y, 5/6: -z/+z)
    auto side = [&](int bit, long long idx) {
      return ((m >> bit) & 1u) ? pc + face_q[idx] * inv_eps : psi[idx];
    };
    e[0] = -0.5 * (side(2, r - xo[1] + xo[2]) - side(1, r - xo[1] + xo[0])) + lp.eext[0];
    e[1] = -0.5 * (side(4, r - yo[1] + yo[2]) - side(3, r - yo[1] + yo[0])) + lp.eext[1];
    e[2] = -0.5 * (side(6, r - zo[1] + zo[2]) - side(5, r - zo[1] + zo[0])) + lp.eext[2];
    return;
  }
  e[0] = -0.5 * (psi[r - xo[1] + xo[2]] - psi[r - xo[1] + xo[0]]) + lp.eext[0];
  e[1] = -0.5 * (psi[r - yo[1] + yo[2]] - psi[r - yo[1] + yo[0]]) + lp.eext[1];
  e[2] = -0.5 * (psi[r - zo[1] + zo[2]] - psi[r - zo[1] + zo[0]]) + lp.eext[2];
}

// Pair partners kept per lane: lane l of bead i lists the beads j = l,
// l + TPB, ... within the WCA cut-off plus NB_SKIN at the last build, in
// increasing j, up to NBL of them (a template parameter).  The list is rebuilt
// when any bead has moved more than NB_SKIN / 2 since the build, so every
// pair inside the cut-off stays listed.  Chains of at most SMALL_CHAIN beads
// with eight lanes per bead have room for every candidate
// (NBL = SMALL_CHAIN / 8); longer chains keep up to NB_PER_LANE partners per
// lane and a lane that would list more switches the chain back to all pairs.
// A lane sums the same nonzero pair terms in the same order either way.
constexpr int NB_PER_LANE = 32;
constexpr double NB_SKIN = 0.6;
constexpr int SMALL_CHAIN = 64;

// LDS bytes of the pair lists.
__host__ __device__ inline size_t md_list_bytes(int threads, int nbl) {
  return (size_t)threads * nbl * sizeof(unsigned short);
}

// What bounds it: one workgroup on one compute unit, so a chain of 8 beads (a
// single wave) is a serial chain of some 500 vector instructions and three
// LDS round trips a substep, and one of 64 beads (two waves a SIMD) is bound
// by issue.  Hence no branch or wait per value where nine values are read or
// added together, lane moves without a value to replace, divisions off the
// chain, and reads issued before what they are needed for.  Measured for 8,
// 32, 64 and 100 beads: 1.75, 2.4, 3.2 and 4.2 us a substep (2.9, 3.1, 3.9 and
// 5.2 before), and 9 to 30 us for what comes before and after them (one
// substep of 100 beads with WR = 2: 48 us instead of 99).
//
// n_sub substeps of one chain by one workgroup (TPB lanes per bead; the
// threads beyond n * TPB only take part in the barriers).  smem: LDS for the
// bead positions, when LDS is set the node table of lds_slots slots (sites
// that find no room there go to the global table), and with NBL > 0 the pair
// lists (md_list_bytes; with NBL = 0 every lane walks all its candidate
// partners each substep: the persistent ensemble kernel, whose registers the
// lists would spill).  THERMAL = false compiles the bead noise out (the
// ensemble, which runs without thermal fluctuations).
template <bool LDS, int TPB, int NBL, int WR = 1, bool THERMAL = true>
__device__ inline void md_chain(const BeadState& bs, const MDParams& mp, int* gkeys,
                                long long* gvals, uint32_t* mask, const Dims& d, int gbits,
                                int lds_slots, unsigned char* smem) {
  using G = WallGeom<WR>;
  constexpr int CPL = 8 / TPB;                                 // corners per lane
  double* sR = (double*)smem;                                  // [3 * n]
  long long* lvals = (long long*)(smem + (((size_t)mp.n * 24 + 15) & ~size_t(15)));
  const int lslots = LDS ? lds_slots : 0;
  int* lkeys = (int*)(lvals + (size_t)lslots * 9);
  // pair lists: entry k of thread t at nbl[k * blockDim.x + t], after the
  // LDS node table
  constexpr bool NLIST = NBL > 0;
  unsigned short* nbl = (unsigned short*)(lkeys + lslots);
  __shared__ int s_rebuild, s_overflow, s_image;
  if (NLIST && threadIdx.x == 0) {
    // a single substep walks all pairs once, as the list's build would
    s_rebuild = mp.n_sub > 1;
    s_overflow = mp.n_sub > 1 ? 0 : 1;
    s_image = 0;
  }
  int nb_count = 0;
  double Rb[3] = {0, 0, 0};                 // position at the last list build

  const int i = threadIdx.x / TPB;          // bead
  const int lane = threadIdx.x % TPB;
  const bool live = i < mp.n;
  if (LDS) {
    for (int h = threadIdx.x; h < lslots; h += blockDim.x) lkeys[h] = -1;
    for (int h = threadIdx.x; h < lslots * 9; h += blockDim.x) lvals[h] = 0;
  }
  double R[3] = {0, 0, 0}, V[3] = {0, 0, 0}, q = 0.0;
  int org[3] = {0, 0, 0};
  if (live) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      R[c] = bs.R[3 * i + c];
      V[c] = bs.V[3 * i + c];
      org[c] = bs.origin[3 * i + c];
      if (lane == 0) sR[3 * i + c] = R[c];
    }
    q = bs.q[i];
  }
  const double z_start = R[2];   // for the plane crossing record
  __syncthreads();
  GlobalNodes gn{gkeys, gvals, mask, bs.err, gbits};
  LdsNodes ln{lkeys, lvals, lslots, bs.err, gn};

  const double h = 1.0 / mp.n_sub;
  const double hM = h / mp.M;
  const double L[3] = {mp.Lx, mp.Ly, mp.Lz};
  const double iL[3] = {1.0 / mp.Lx, 1.0 / mp.Ly, 1.0 / mp.Lz};
  const double rc2 = 1.2599210498948732 * mp.sigma * mp.sigma;   // (2^(1/6) sigma)^2
  const double s2w = mp.sigma * mp.sigma;
  const double iR02 = 1.0 / (mp.R0 * mp.R0);
  const double* mom = bs.mom + (size_t)(live ? i : 0) * BOX3 * MOM;
  const double* ef = bs.efield + (size_t)(live ? i : 0) * BOX3 * 3;
  const unsigned long long* fl = bs.flags + (size_t)(live ? i : 0) * FLAG_WORDS;
  int cell[3] = {0, 0, 0};
  int slot[CPL], bidx[CPL];
  double wfl[CPL];
  // With at most two corners per lane the node momenta of time t, which are
  // fixed for the whole step, and (up to four corners) the lane's wall-site
  // flags are kept in registers from the substep the bead enters its cell on;
  // with more corners per lane they are read each substep.
  constexpr bool CACHE = CPL <= 2;   // node momenta too
  constexpr bool CACHE_W = CPL <= 4; // wall flags
  // wall sites around the cell: the lanes share the S^2 columns of the cube;
  // a word of wall_bits holds the S sites of each of CPW columns
  constexpr int COLS = (G::S * G::S + TPB - 1) / TPB;   // columns per lane
  constexpr int CPW = 64 / G::S;
  constexpr int NWB = (COLS + CPW - 1) / CPW;
  double mo_c[CACHE ? CPL : 1][MOM];
  unsigned long long wall_bits[NWB];
#pragma unroll
  for (int b = 0; b < NWB; ++b) wall_bits[b] = 0;
  // this lane's share of q E(R(t)): the field is interpolated once, with the
  // plain weights at the position where the bead's charge was deposited for
  // this step's solve (the electrostatic forces on ions, walls and beads then
  // cancel exactly, and the bead never feels its own deposited charge)
  double qe[3] = {0.0, 0.0, 0.0};
  if (live) {   // the bead starts in the middle cell of its box
    const double dx = R[0] - floor(R[0]), dy = R[1] - floor(R[1]), dz = R[2] - floor(R[2]);
    double w[CPL], wsum = 0.0;
#pragma unroll
    for (int a = 0; a < CPL; ++a) {
      const int k8 = lane * CPL + a;
      const int ox = k8 & 1, oy = (k8 >> 1) & 1, oz = (k8 >> 2) & 1;
      w[a] = (ox ? dx : 1.0 - dx) * (oy ? dy : 1.0 - dy) * (oz ? dz : 1.0 - dz);
      if (mp.field_fluid) {
        w[a] *= (fl[1 + WR + oz] >> ((1 + WR + ox) + 8 * (1 + WR + oy))) & 1 ? 1.0 : 0.0;
        wsum += w[a];
      }
    }
    if (mp.field_fluid) {
      wsum = group_sum<TPB>(wsum);
#pragma unroll
      for (int a = 0; a < CPL; ++a) w[a] /= wsum > 0.0 ? wsum : 1.0;
    }
#pragma unroll
    for (int a = 0; a < CPL; ++a) {
      const int k8 = lane * CPL + a;
      const double* e =
          ef + 3 * ((1 + (k8 & 1)) + BOX * ((1 + ((k8 >> 1) & 1)) + BOX * (1 + ((k8 >> 2) & 1))));
#pragma unroll
      for (int c = 0; c < 3; ++c) qe[c] += q * w[a] * e[c];
    }
  }
  const int wall_lim = int(ceil(rc2));   // integer distances^2 below rc2 are below this
  // The bead in the cell at (fx, fy, fz), corner 0 at (lx, ly, lz) of its box:
  // the corners' slots and node momenta, and of the wall sites (site
  // floor(R) - WR + w at window index (lx + w)) those closer than the cut-off
  // to some point of the cell.  The reads do not depend on each other and so
  // overlap (a byte per site behind a test each had taken a round trip to
  // memory for every site: 99 us for one substep of 100 beads with WR = 2).
  auto enter = [&](int fx, int fy, int fz, int lx, int ly, int lz) {
#pragma unroll
    for (int a = 0; a < CPL; ++a) {
      const int k8 = lane * CPL + a;
      const int ox = k8 & 1, oy = (k8 >> 1) & 1, oz = (k8 >> 2) & 1;
      bidx[a] = (lx + ox) + BOX * ((ly + oy) + BOX * (lz + oz));
      wfl[a] = (fl[lz + oz + WR] >> ((lx + ox + WR) + 8 * (ly + oy + WR))) & 1 ? 1.0 : 0.0;
      if constexpr (CACHE) {
        const double* mo = mom + (size_t)bidx[a] * MOM;
#pragma unroll
        for (int c = 0; c < MOM; ++c) mo_c[CACHE ? a : 0][c] = mo[c];   // 0 at solid nodes
      }
    }
    if constexpr (CACHE_W) {
      unsigned long long plane[G::S];
#pragma unroll
      for (int k = 0; k < G::S; ++k) plane[k] = fl[8 + lz + k];
#pragma unroll
      for (int b = 0; b < NWB; ++b) wall_bits[b] = 0;
#pragma unroll 1
      for (int u = 0; u < COLS; ++u) {
        const int p = lane + u * TPB, wx = p % G::S, wy = p / G::S;
        const int gx = max(WR - wx, wx - WR - 1), gy = max(WR - wy, wy - WR - 1);   // to the cell's edge
        const int shift = ((lx + wx) + 8 * (ly + wy)) & 63, near = gx * gx + gy * gy - wall_lim;
        unsigned column = 0;
#pragma unroll
        for (int k = 0; k < G::S; ++k) {
          const int gz = k < WR ? WR - k : (k > WR + 1 ? k - WR - 1 : 0);
          // the flag, if near + gz^2 is negative
          column |= (unsigned(plane[k] >> shift) & (unsigned(near + gz * gz) >> 31)) << k;
        }
        if (p >= G::S * G::S) column = 0;
#pragma unroll
        for (int b = 0; b < NWB; ++b) {
          const int at = u - b * CPW;
          if (at >= 0 && at < CPW) wall_bits[b] |= (unsigned long long)column << (at * G::S);
        }
      }
    }
#pragma unroll
    for (int a = 0; a < CPL; ++a) {
      const int k8 = lane * CPL + a;
      const int ox = k8 & 1, oy = (k8 >> 1) & 1, oz = (k8 >> 2) & 1;
      slot[a] = -1;
      if (wfl[a] != 0.0) {
        const long long site = site_of(fx + ox, fy + oy, fz + oz, d);
        slot[a] = LDS ? ln.slot(site) : gn.slot(site);
      }
    }
  };
  if (live) {   // the start: the middle cell of the box
#pragma unroll
    for (int c = 0; c < 3; ++c) cell[c] = int(floor(R[c]));
    enter(cell[0], cell[1], cell[2], 1, 1, 1);
  }
  const double rl = 1.122462048309373 * mp.sigma + NB_SKIN;      // list radius
  const double rl2 = rl * rl, half_skin2 = 0.25 * NB_SKIN * NB_SKIN;
  // the lane's first partners (the bead itself past the end): their positions
  // are read at the substep's start, without a look at the list (eight lanes a
  // bead: with fewer the registers are not spared)
  constexpr int CH = 4;
  constexpr bool HEAD = NLIST && TPB == 8;
  int head[CH];
#pragma unroll
  for (int u = 0; u < CH; ++u) head[u] = live ? i : 0;
  for (int sub = 0; sub < mp.n_sub; ++sub) {
    if (NLIST && s_rebuild) {            // the same in every thread (set before the last barrier)
      if (live) {
        nb_count = 0;
        constexpr int AHEAD = 4;   // candidates whose positions are read together
        for (int j0 = lane; j0 < mp.n; j0 += AHEAD * TPB) {
          double P[AHEAD][3];
#pragma unroll
          for (int u = 0; u < AHEAD; ++u) {
            const int j = j0 + u * TPB < mp.n ? j0 + u * TPB : i;
#pragma unroll
            for (int c = 0; c < 3; ++c) P[u][c] = sR[3 * j + c];
          }
#pragma unroll
          for (int u = 0; u < AHEAD; ++u) {
            const int j = j0 + u * TPB;
            if (j >= mp.n || j == i) continue;
            double r2 = 0.0;
            bool image = false;   // of the pair, now or before the next build
#pragma unroll
            for (int c = 0; c < 3; ++c) {
              const double v = R[c] - P[u][c];
              const double dv = v - L[c] * rint(v * iL[c]);
              r2 += dv * dv;
              image = image || !(fabs(v) + NB_SKIN < 0.5 * L[c]);
            }
            const bool bonded = j == i - 1 || j == i + 1;
            if (image && (bonded || r2 < rl2)) s_image = 1;
            if (mp.bond == 1 && bonded) continue;
            if (r2 < rl2) {
              if (nb_count < NBL) nbl[nb_count * blockDim.x + threadIdx.x] = (unsigned short)j;
              ++nb_count;
            }
          }
        }
        if (nb_count > NBL) s_overflow = 1;
#pragma unroll
        for (int u = 0; u < CH; ++u)
          head[u] = HEAD && u < nb_count ? int(nbl[u * blockDim.x + threadIdx.x]) : i;
#pragma unroll
        for (int c = 0; c < 3; ++c) Rb[c] = R[c];
      }
      __syncthreads();
      if (threadIdx.x == 0) s_rebuild = 0;
    }
    double wt[CPL];
    double phi[3][3];
    double Rn[3];
#pragma unroll
    for (int a = 0; a < CPL; ++a) wt[a] = 0.0;
    if (live) {
      const int fx = int(floor(R[0])), fy = int(floor(R[1])), fz = int(floor(R[2]));
      const double dx = R[0] - fx, dy = R[1] - fy, dz = R[2] - fz;
      int lx = fx - org[0], ly = fy - org[1], lz = fz - org[2];   // corner 0 in the box
      if (fx != cell[0] || fy != cell[1] || fz != cell[2]) {
        // the bead entered another cell: new corners, their box entries and slots
        cell[0] = fx; cell[1] = fy; cell[2] = fz;
        if (lx < 0 || lx > BOX - 2 || ly < 0 || ly > BOX - 2 || lz < 0 || lz > BOX - 2) {
          if (lane == 0) atomicOr(bs.err, ERR_BOX);
          lx = min(max(lx, 0), BOX - 2);
          ly = min(max(ly, 0), BOX - 2);
          lz = min(max(lz, 0), BOX - 2);
        }
        enter(fx, fy, fz, lx, ly, lz);
      }
      // impulse of earlier substeps on this lane's corners, read before the
      // weights so that the reads overlap their arithmetic (one corner per
      // lane: with more the registers are not spared)
      constexpr bool PRE_K = CPL == 1;
      long long kpre[9];
      if constexpr (PRE_K) {
        if constexpr (LDS) ln.get(slot[0], kpre);
        else gn_get(gn, slot[0], kpre);
      }
      // and the first partners' positions
      double P0[HEAD ? CH : 1][3];
      if constexpr (HEAD) {
#pragma unroll
        for (int u = 0; u < CH; ++u)
#pragma unroll
          for (int c = 0; c < 3; ++c) P0[HEAD ? u : 0][c] = sR[3 * head[u] + c];
      }
      // The corners' plain trilinear weights over the fluid, or, with the
      // occupation cube, its node indicator per axis (offset 0: d < sigma/2,
      // offset 1: d >= 1 - sigma/2); both are renormalised over the fluid
      // corners.  The sums below take the weights as they are and are divided
      // by their sum afterwards, so the division does not stand before them.
      auto cube = [&](int ox, int oy, int oz) {
        const double hs = mp.half_sigma;
        return ((ox ? dx >= 1.0 - hs : dx < hs) && (oy ? dy >= 1.0 - hs : dy < hs) &&
                (oz ? dz >= 1.0 - hs : dz < hs)) ? 1.0 : 0.0;
      };
      double wsum = 0.0, wsum_c = 0.0;
#pragma unroll
      for (int a = 0; a < CPL; ++a) {
        const int k8 = lane * CPL + a;
        const int ox = k8 & 1, oy = (k8 >> 1) & 1, oz = (k8 >> 2) & 1;
        wt[a] = (ox ? dx : 1.0 - dx) * (oy ? dy : 1.0 - dy) * (oz ? dz : 1.0 - dz) * wfl[a];
        wsum += wt[a];
        if (mp.theta) {
          wt[a] = cube(ox, oy, oz) * wfl[a];
          wsum_c += wt[a];
        }
      }
      wsum = group_sum<TPB>(wsum);
      wsum_c = mp.theta ? group_sum<TPB>(wsum_c) : wsum;
      if (!(wsum_c > 0.0) || !(wsum > 0.0)) {
        if (lane == 0) atomicOr(bs.err, ERR_FLUID);
        wsum_c = wsum_c > 0.0 ? wsum_c : 1.0;
      }
      const double iws = 1.0 / wsum_c;
      // this lane's corners: velocities from the node momentum (populations of
      // time t plus the friction impulse of earlier substeps) and composition
      double acc[12];
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[c] = 0.0;
#pragma unroll
      for (int a = 0; a < CPL; ++a) {
        if (wt[a] != 0.0) {
          const double* mo = CACHE ? mo_c[CACHE ? a : 0] : mom + (size_t)bidx[a] * MOM;
          long long kv[9];
          if constexpr (PRE_K) {
#pragma unroll
            for (int k = 0; k < 9; ++k) kv[k] = kpre[k];
          } else {
            if constexpr (LDS) ln.get(slot[a], kv);
            else gn_get(gn, slot[a], kv);
          }
#pragma unroll
          for (int s = 0; s < 3; ++s) {
            acc[9 + s] += wt[a] * mo[s];
            const double wn = wt[a] * mo[3 + s];
#pragma unroll
            for (int c = 0; c < 3; ++c)
              acc[3 * s + c] += wn * (mo[6 + 3 * s + c] + double(kv[3 * s + c]) * (1.0 / FIX_FORCE));
          }
        }
      }
#pragma unroll
      for (int a = 0; a < CPL; ++a) wt[a] *= iws;
      // this lane's share of the conservative forces
      double F[3] = {0.0, 0.0, 0.0};
      // FENE bonds: the bond to i - 1 on lane 0 and the one to i + 1 on lane
      // 1 (both on lane 0 with one lane per bead); the bonded neighbour's
      // position is read up front with the partners' ones where the registers
      // allow (short chains with the lists)
      constexpr int NBOND = TPB >= 2 ? 1 : 2;        // bonds per bond lane
      const int bond0 = TPB >= 2 ? lane : 0;         // 0: bond to i - 1, 1: to i + 1
      const bool bond_lane = TPB >= 2 ? lane < 2 : true;
      constexpr bool PRE_B = LDS && NLIST;
      double PB[PRE_B ? NBOND : 1][3];
      if constexpr (PRE_B) {
#pragma unroll
        for (int k = 0; k < NBOND; ++k) {
          const int j = min(max(i + 2 * (bond0 + k) - 1, 0), mp.n - 1);
#pragma unroll
          for (int c = 0; c < 3; ++c) PB[PRE_B ? k : 0][c] = sR[3 * j + c];
        }
      }
      // IMAGE: nearest images (without it no pair of the list or bond has one)
      auto wca_at = [&](const double* P, auto IMAGE) {   // WCA with a partner at P
        double dv[3], r2 = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          const double v = R[c] - P[c];
          dv[c] = IMAGE ? v - L[c] * rint(v * iL[c]) : v;
          r2 += dv[c] * dv[c];
        }
        if (r2 < rc2) {
          const double ir2 = 1.0 / r2;
          const double s6 = s2w * ir2 * s2w * ir2 * s2w * ir2;
          const double coef = 24.0 * mp.eps * (2.0 * s6 * s6 - s6) * ir2;
#pragma unroll
          for (int c = 0; c < 3; ++c) F[c] += coef * dv[c];
        }
      };
      constexpr std::true_type images{};
      constexpr std::false_type no_images{};
      const bool image = !NLIST || __builtin_amdgcn_readfirstlane(s_image | s_overflow) != 0;
      if (NLIST && !s_overflow) {                    // WCA with the listed partners
        // four partners at a time: their indices, then their positions, are
        // read together (one LDS round trip each), the terms are added in
        // list order
        static_assert(NBL % CH == 0, "list chunks");
        auto listed = [&](auto IMAGE) {
          if constexpr (HEAD) {
#pragma unroll
            for (int u = 0; u < CH; ++u)
              if (u < nb_count) wca_at(P0[HEAD ? u : 0], IMAGE);
          }
          for (int k0 = HEAD ? CH : 0; k0 < nb_count; k0 += CH) {
            int jj[CH];
#pragma unroll
            for (int u = 0; u < CH; ++u)
              jj[u] = k0 + u < nb_count ? int(nbl[(k0 + u) * blockDim.x + threadIdx.x]) : i;
            double P[CH][3];
#pragma unroll
            for (int u = 0; u < CH; ++u)
#pragma unroll
              for (int c = 0; c < 3; ++c) P[u][c] = sR[3 * jj[u] + c];
#pragma unroll
            for (int u = 0; u < CH; ++u)
              if (k0 + u < nb_count) wca_at(P[u], IMAGE);
          }
        };
        if (image) listed(images);
        else listed(no_images);
      } else {
        constexpr int AHEAD = NLIST ? 4 : 1;         // WCA between all pairs
        for (int j0 = lane; j0 < mp.n; j0 += AHEAD * TPB) {
          double P[AHEAD][3];
#pragma unroll
          for (int u = 0; u < AHEAD; ++u) {
            const int j = j0 + u * TPB < mp.n ? j0 + u * TPB : i;
#pragma unroll
            for (int c = 0; c < 3; ++c) P[u][c] = sR[3 * j + c];
          }
#pragma unroll
          for (int u = 0; u < AHEAD; ++u) {
            const int j = j0 + u * TPB;
            if (j < mp.n && j != i && !(mp.bond == 1 && (j == i - 1 || j == i + 1)))
              wca_at(P[u], images);
          }
        }
      }
      // WCA against wall-site centres: site k of this lane is lane + k TPB of
      // the S^3 sites around the bead's cell
      auto wall_at = [&](int ax, int ay, int az) {
        const double dv[3] = {R[0] - ax, R[1] - ay, R[2] - az};
        const double r2 = dv[0] * dv[0] + dv[1] * dv[1] + dv[2] * dv[2];
        if (r2 < rc2) {
          const double ir2 = 1.0 / r2;
          const double s6 = s2w * ir2 * s2w * ir2 * s2w * ir2;
          const double coef = 24.0 * mp.eps * (2.0 * s6 * s6 - s6) * ir2;
#pragma unroll
          for (int c = 0; c < 3; ++c) F[c] += coef * dv[c];
        }
      };
      if constexpr (CACHE_W) {
        // only the wall sites among them, in increasing k
#pragma unroll
        for (int b = 0; b < NWB; ++b)
          for (unsigned long long mb = wall_bits[b]; mb; mb &= mb - 1) {
            const int k = __builtin_ctzll(mb), u = k / G::S;
            const int wz = k - u * G::S, p = lane + (b * CPW + u) * TPB;
            wall_at(fx - WR + p % G::S, fy - WR + p / G::S, fz - WR + wz);
          }
      } else {
        // lx, ly, lz as at the last entry of a cell
        const int bx = bidx[0] % BOX, by = (bidx[0] / BOX) % BOX, bz = bidx[0] / (BOX * BOX);
        const int cx = bx - (lane * CPL & 1), cy = by - ((lane * CPL >> 1) & 1), cz = bz - ((lane * CPL >> 2) & 1);
        for (int wz = 0; wz < G::S; ++wz) {
          const unsigned long long plane = fl[8 + cz + wz];
          if (plane == 0) continue;
          for (int p = lane; p < G::S * G::S; p += TPB) {
            const int wx = p % G::S, wy = p / G::S;
            if ((plane >> ((cx + wx) + 8 * (cy + wy))) & 1) wall_at(fx - WR + wx, fy - WR + wy, fz - WR + wz);
          }
        }
      }
      if (bond_lane) {
#pragma unroll
        for (int k = 0; k < NBOND; ++k) {            // FENE bonds
          const int j = i + 2 * (bond0 + k) - 1;
          if (j < 0 || j >= mp.n) continue;
          double dv[3], r2 = 0.0;
#pragma unroll
          for (int c = 0; c < 3; ++c) {
            const double v = (PRE_B ? PB[PRE_B ? k : 0][c] : sR[3 * j + c]) - R[c];
            dv[c] = image ? v - L[c] * rint(v * iL[c]) : v;
            r2 += dv[c] * dv[c];
          }
          double coef;
          if (mp.bond == 1) {   // harmonic: k (r - l) / r along the bond
            const double r = sqrt(r2);
            coef = r > 0.0 ? mp.k_bond * (r - mp.l_bond) / r : 0.0;
          } else {
            const double x2 = r2 * iR02;
            if (x2 >= 1.0) {
              atomicOr(bs.err, ERR_BOND);
              continue;
            }
            coef = mp.k_fene / (1.0 - x2);
          }
#pragma unroll
          for (int c = 0; c < 3; ++c) F[c] += coef * dv[c];
        }
      }
      // combine the lanes of this bead (the field enters only as q E, so each
      // lane adds its corners' share to its force first)
#pragma unroll
      for (int c = 0; c < 3; ++c) F[c] += qe[c];
#pragma unroll
      for (int c = 0; c < 12; ++c) acc[c] = group_sum<TPB>(acc[c]) * iws;
#pragma unroll
      for (int c = 0; c < 3; ++c) F[c] = group_sum<TPB>(F[c]);
      // friction of each species (with the thermal noise shared by the
      // species' number fractions) and the substep update
      double xi[3] = {0.0, 0.0, 0.0};
      if (THERMAL && mp.thermal) {
        const Philox4 w = philox4x32_10(uint32_t(i), mp.tstep, uint32_t(sub), 1u, mp.key0, mp.key1);
        double z[4];
        box_muller4<double>(w, z);
#pragma unroll
        for (int c = 0; c < 3; ++c) xi[c] = mp.xi_scale * z[c];
      }
      double ftot[3] = {F[0], F[1], F[2]};
#pragma unroll
      for (int s = 0; s < 3; ++s)
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          phi[s][c] = mp.gamma * acc[9 + s] * (acc[3 * s + c] - V[c]) + acc[9 + s] * xi[c];
          ftot[c] += phi[s][c];
        }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        V[c] += hM * ftot[c];
        Rn[c] = R[c] + h * V[c];
      }
    }
    __syncthreads();   // every bead has read positions and node momenta of this substep
    if (live) {
#pragma unroll
      for (int a = 0; a < CPL; ++a) {
        if (wt[a] == 0.0 || slot[a] == -1) continue;
        long long v[9];
        round_fixed9(phi, -h * wt[a] * FIX_FORCE, v);   // scaled to this corner's impulse
        if constexpr (LDS) ln.add(slot[a], v);
        else gn.add(slot[a], v);
      }
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        R[c] = Rn[c];
        if (lane == 0) sR[3 * i + c] = Rn[c];
      }
      if (NLIST) {   // moved more than half the skin since the build: rebuild next substep
        double dd = 0.0;
#pragma unroll
        for (int c = 0; c < 3; ++c) dd += (R[c] - Rb[c]) * (R[c] - Rb[c]);
        if (dd > half_skin2) s_rebuild = 1;
      }
    }
    // one workgroup advances the chain: the barrier's workgroup-scope ordering
    // (prior atomics completed) is enough for the table's atomic reads, which
    // go to the shared L2
    __syncthreads();
  }
  if (live && lane == 0) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      bs.R[3 * i + c] = R[c];
      bs.V[3 * i + c] = V[c];
    }
    if (mp.track && bs.cross) {   // the step moved the bead across an image of the plane
      const double k0 = floor((z_start - mp.z_plane) / mp.Lz);
      const double k1 = floor((R[2] - mp.z_plane) / mp.Lz);
      if (k0 != k1) {
        int* cr = bs.cross + 3 * i;
        if (cr[0] < 0) cr[0] = mp.step;
        cr[1] = mp.step;
        cr[2] += k1 > k0 ? 1 : -1;
      }
    }
  }
  if (LDS) {   // hand the accumulated impulses to the lattice kernels
    __syncthreads();
    // (four slots of a thread at a time: the first probe of each, which finds
    // most sites, is one round trip to the global table for all of them)
    constexpr int AHEAD = 4;
    for (int h0 = threadIdx.x; h0 < lslots; h0 += AHEAD * blockDim.x) {
      int key[AHEAD], prev[AHEAD];
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        const int hh = h0 + u * blockDim.x;
        key[u] = hh < lslots ? lkeys[hh] : -1;
      }
#pragma unroll
      for (int u = 0; u < AHEAD; ++u)
        prev[u] = key[u] < 0 ? 0 : ld_i32(&gkeys[hash_slot(key[u], gbits)]);
#pragma unroll
      for (int u = 0; u < AHEAD; ++u) {
        if (key[u] < 0) continue;
        const int g = prev[u] == key[u] ? hash_slot(key[u], gbits)
                                        : table_insert(gkeys, mask, key[u], bs.err, gbits);
        if (g < 0) continue;
        const long long* p = lvals + (size_t)(h0 + u * blockDim.x) * 9;
        long long v[9];
#pragma unroll
        for (int c = 0; c < 9; ++c) v[c] = p[c];
        gn.add(g, v);
      }
    }
  }
  __syncthreads();
}

}  // namespace ek
