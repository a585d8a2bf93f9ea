// Replica descriptors of the ensemble, shared by the persistent kernel
// (kernels_ensemble.hip) and the launched steps (kernels_replicas.hip).
#pragma once

#include "ek_internal.h"
#include "md_chain.h"
#include "spectral.h"

namespace ek {

constexpr int ENS_TABLE_BITS = 12;     // node table of a replica: 4096 slots
constexpr int ENS_MAX_BEADS = 64;      // node sums of a chain live in LDS
constexpr int ENS_MAX_GROUP = 4;

// ST_PAUSED (launched path, within a call): the step's first cycle of the
// Poisson solve did not meet the tolerance; the host takes it from there.
enum : int { ST_OK = 0, ST_NOCONV = 1, ST_UNSTABLE = 2, ST_TIMEOUT = 3, ST_PAUSED = 4 };

// Team barrier state and reduction partials of one replica (global memory,
// cleared by the host before every launch).  Partials are double-buffered by
// the parity of the reduction count, so a member that has summed reduction k
// can write reduction k + 1 while the others still read k.
struct TeamSync {
  int count;                  // barrier arrivals
  int abort;                  // set when a member waited beyond the spin limit
  int pad[14];
  double part[2][ENS_MAX_GROUP][8];
};

// Per-replica device pointers and parameters.
struct RepDev {
  void* f[2];                 // populations; f[cur] holds the current ones
  TeamSync* sync;
  uint32_t* mask;             // link words (own copy: the bead flag is per replica)
  double* psi;
  double* psi_old;            // psi(t-2) for the extrapolated start, or null
  int psi_hist;               // previous solutions held (0, 1 or 2)
  double* b;
  double* mg;                 // multigrid levels 1.. (x then f per level)
  int* keys;
  long long* vals;
  BeadState bs;
  MDParams mp;
  LBParams lp;
  int n_beads;
  int cur;
  int status;
  int steps;                  // steps completed
  int todo;                   // steps left of this call (launched path)
  int last_cycles;
  double last_res;
  double last_res0;
  double stats[6];            // species masses and fluid momentum of f(t)
  // wall-clock ticks spent by the team's first workgroup in the phases of
  // all steps so far: charge pass, Poisson solve, chain, collide-and-stream
  unsigned long long phase_ticks[4];
  unsigned long long phase_mark;   // clock at the start of the current phase
};

// The launched path: what its kernels need besides the descriptors.
struct RepBatch {
  RepDev* reps = nullptr;
  int n_rep = 0;
  Dims d{};
  const double* wall_q = nullptr;
  double inv_eps = 0.0, tol = 0.0;
  Spectral spec;
  SpecItem* items = nullptr;         // [n_rep] fields of the direct solve
  PoissonScalars* ps = nullptr;      // [n_rep]
  double* part = nullptr;            // [n_rep][part_stride] partial sums
  size_t part_stride = 0;
  int beads = 0;                     // longest chain
};

// Device bytes of the launched path beside the replicas' own (0: the box has
// no direct solver), and their carving.
size_t replicas_bytes(int nx, int ny, int nz, int n_rep);
void replicas_setup(RepBatch& b, char* mem, int nx, int ny, int nz, int n_rep);
// Before the steps of a call (and after the host has written descriptors).
hipError_t replicas_begin(const RepBatch& b, hipStream_t s);
// One step of every replica with status ST_OK and steps left.
hipError_t replicas_step(const RepBatch& b, hipStream_t s);
// One more cycle of the paused replicas' solves that miss the tolerance.
hipError_t replicas_cycle(const RepBatch& b, hipStream_t s);
// The rest of the paused replicas' step, which clears the pause.
hipError_t replicas_finish(const RepBatch& b, hipStream_t s);

}  // namespace ek
