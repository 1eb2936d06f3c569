// lbc_internal.h -- argument blocks and launchers shared by the host runtime
// (lbc_api.hip) and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <cmath>
#include <stdint.h>

#include "lbc.h"

namespace lbc {

// Lattice geometry passed to every kernel.
struct Geo {
  int nx, ny, nz;
  int wall;  // halfway bounce-back walls in y
  int wpr;   // 64-bit force-mask words per row
  long long N;
  long long ps;  // population stride: N rounded up to a multiple of 128 sites, so that
                 // every population array starts on a 256-byte boundary
};

// Whether the byte offsets inside a population array of this box need more
// than 32 bits.
inline bool big_box(const Geo& g, int storage) {
  return (unsigned long long)g.N * (storage == LB_F64 ? 8 : (storage == LB_F32 ? 4 : 2)) > 0xffffffffull;
}

// Whether a box takes the row-mapped launches: rows of whole 64-site mask words,
// whose byte offsets the lanes hold in 32 bits.  Others take the linear-site pass.
inline bool rows_fit(int nx, int storage_bytes) {
  return nx % 64 == 0 && (unsigned long long)nx * storage_bytes <= 0xffffffffull;
}

// floor(2^32 / d), the multiplier of div_rem (2^32 - 1 for d = 1).
inline uint32_t div_magic(int d) {
  return d <= 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (unsigned)d);
}

// Quotient and remainder of n / d for 32-bit n and d >= 1, with m =
// div_magic(d) from the host: n m / 2^32 lies in (n/d - 1, n/d], so its floor is
// the quotient or one less, and one correction step fixes it.
__host__ __device__ __forceinline__ uint32_t div_rem(uint32_t n, uint32_t d, uint32_t m, uint32_t& rem) {
  uint32_t q = (uint32_t)(((uint64_t)n * m) >> 32), r = n - q * d;
  if (r >= d) {
    q += 1;
    r -= d;
  }
  rem = r;
  return q;
}

// Bounds of the nearest image in a box of length L: floor(d/L + 1/2), rounded as
// written, is -1 for d < lo, 0 for lo <= d < hi and 1 from hi on (|d| < 3L/2); two
// compares for a division.  (A product with 1/L rounds otherwise: for a third of all
// L it takes another image one unit in the last place below half a box.)
inline void image_bounds(double L, double& lo, double& hi) {
  const auto image = [L](double d) { return std::floor(d / L + 0.5); };
  hi = 0.5 * L;
  while (image(hi) >= 1.0) hi = std::nextafter(hi, 0.0);
  while (image(hi) < 1.0) hi = std::nextafter(hi, L);
  lo = -0.5 * L;
  while (image(lo) >= 0.0) lo = std::nextafter(lo, -L);
  while (image(lo) < 0.0) lo = std::nextafter(lo, 0.0);
}

struct BondArgs {
  Geo g;
  const int32_t* perm;   // particles ordered by group
  const int32_t* loc;    // slot of each particle inside its group
  const int32_t* goff;   // group offsets into perm
  const int32_t* start;  // CSR of bond partners (global particle indices)
  const int32_t* nbr;
  double* pos;
  double* vel;
  const double* mass;
  double* fint;
  double k, r0;
  double lo[3], hi[3];  // image_bounds of nx, ny, nz
  int type;
};

// Population loads and stores of the lattice pass: kStream non-temporal stores
// (and loads, for the FP32 row-mapped pass without noise), kResident cached
// loads and stores, kKeepWritten non-temporal loads and cached stores.
enum CachePolicy { kStream = 0, kResident = 1, kKeepWritten = 2 };

constexpr int kMtsFields = 4;  // sub-step fields held before a fold (SubArgs)

// Fused lattice pass (stream, both pending half forces, collide).
struct LatArgs {
  Geo g;
  const void* fin;  // f* of the previous pass
  void* fout;       // f* of this pass
  void* FA;         // first-half coupling force of this step (vec4 per site)
  void* FB;         // second-half coupling force of the previous step
  uint64_t* mask;   // per-site flag: FA or FB nonzero
  void* G[kMtsFields];  // sub-step fields that join FA (step_mts_inside), ng of them
  int ng;
  double rho0;
  double Fx, Fy, Fz;  // body force times the number of pending halves (1 or 2)
  double omp, omm;    // 1 - lambda for even / odd non-conserved moments
  float scale, inv;   // 16-bit storage scale 2^p and its inverse (1 otherwise)
  double uin[3];      // storage reference velocity of fin (comoving frame; 0 otherwise)
  double uout[3];     // storage reference velocity of fout
  double cm[40];      // comoving reference terms of the pass (comoving_terms)
  float cmf[40];      // the same in FP32
  uint32_t mnx, mny;  // div_magic of nx and ny (linear-site pass)
  int clear_mask;     // clear the force mask after reading it (every kMaskKeep steps)
  int ib_copy;        // immersed boundary: FA becomes the pending FB (same spread)
  // fluctuating collision (noise != 0): S sqrt(mu lambda (2 - lambda)) for the
  // even / odd moments, generator key, step index
  int noise;
  double ap, am;
  uint32_t key0, key1, t0, t1;
  // general MRT (mrt != 0): rate of each moment group (bulk, shear, vector
  // ghosts, pseudo-vector ghosts, scalar ghost, tensor ghosts) and the noise
  // amplitude S sqrt(mu lambda (2 - lambda)) of each group
  int mrt;
  double lg[6], ag[6];
  CachePolicy cache;  // of the population loads and stores (set_cache_policy)
  int reverse;        // sweep from the last row to the first
  int occ_lds;  // dynamic LDS bytes reserved per workgroup (occupancy cap), 0: none
  // Intrinsic-force sub-steps run by extra workgroups of the same launch
  // (bond_groups > 0), each doing bond_nsub velocity-Verlet sub-steps of
  // bond_dt for one bond group.  Row-mapped pass: the workgroups of the first
  // z slab (blockIdx.z == 0) take group blockIdx.y * gridDim.x + blockIdx.x
  // and the lattice rows are at blockIdx.z - 1; linear-site pass: workgroup b
  // < bond_groups takes group b and the sites start at workgroup bond_groups.
  // They touch only particle state, the pass only fluid state.
  // Viscous stress output (non-null): sigma [6][N] in the compute precision,
  // (1 - lambda_+/2) sum_i (f_i - f^eq_i) c_i c_i of the pulled state, sp = 1 - lambda_+/2
  void* sigma;
  double sp;
  BondArgs bond;
  int bond_groups, bond_nsub;
  int bond_cap;  // particles per bond group at most (needs that many lanes and 24 B of LDS each)
  double bond_dt;
};

struct InitArgs {
  Geo g;
  void* f;
  const double* rho;
  const double* u;
  double rho0;
  float scale;
};

// Read access to the stored state for moments at a site.
struct SiteArgs {
  Geo g;
  const void* f;
  const void* FB;
  const uint64_t* mask;  // every nonzero vector of FB lies at a flagged site
  double rho0;
  double pfx, pfy, pfz;  // pending body force (0 before the first step, F_ext after)
  float inv;
  double uref[3];  // storage reference velocity of f (comoving frame; 0 otherwise)
};

struct PartArgs {
  SiteArgs s;
  void* FA;
  void* FB;  // writable alias of s.FB
  uint64_t* mask;
  int K;  // delta kernel points (2, 3, 4)
  long long n;
  double* pos;
  double* vel;
  const double* mass;
  double* fint;
  double* aux;  // IB predictor positions
  double gamma;
  double fext[3];   // body-force density the fluid feels over the coupling step; it
                    // enters the implicit force-coupling solve as +(beta/2) F_ext
  int coupling;
  int use_fint;     // F_int enters the coupling force and the kick (Alg. 3)
  int phys;         // interpolate the physical velocity (with pending FB)
  int target;       // spread into FA (0) or FB (1)
  int drift_before;  // first P^1/2 of Alg. 3 (when no intrinsic forces sit between)
  int drift_after;   // final P^1/2 of Alg. 3
  // random force of the force coupling (kT > 0): generator key, step index and
  // the index of this coupling step within the step
  double kT;
  uint32_t key0, key1, t0, t1;
  int jc;
  double hh;         // coupling step length: h/2 (half steps) or h/2n (coupled sub-steps)
  double hd;         // length of drift_before / drift_after
  int fa_rd;         // the interpolated momentum also takes (h/2) FA (earlier sub-steps)
  double sw;         // scale of the lattice force written: 1, or 2 hh for sub-steps
  const int* order;  // non-null: particles in the order to process them (spatial), else by index
  double* defer;     // non-null: store the lattice force per particle [n][3] here for a
                     // separate (deterministic) spread
  // Moment cache: the second coupling half stores, per particle and stencil
  // node, the moments it gathered; the next step's first half reads the same
  // populations (no lattice pass in between) and reuses them when the
  // particle's first stencil node is unchanged.
  double4* mcache;  // [n][L] (drho, j) of each node, before the pending force
  int4* mbase;      // [n] first stencil node (x, y, z) of the cached entries
  int cache_use;    // first half: cached entries are current
  int cache_fill;   // second half: store the gathered moments
};

// A coupled sub-step of the multiple time-step split with the coupling inside
// (Eq. multistep) as one launch.  The particle state is read from one buffer
// pair and written to the other, so that a particle takes its bond partners'
// midpoint positions from their start-of-sub-step state while they advance.
// The lattice force of a sub-step that later sub-steps of the same side read
// goes into a field of its own (gout), and the interpolation adds the target
// field and the fields of the earlier sub-steps (gin): a sub-step never sees
// its own spreads.  A fold launch moves those fields into the target field
// at the flagged sites.
constexpr int kSubPartners = 3;  // bond partners a sub-step holds in registers

struct SubArgs {
  const double* pin;
  const double* vin;
  double* pout;
  double* vout;
  const void* gin[kMtsFields];  // fields of the earlier sub-steps of this side
  int ngin;
  void* gout;    // null: spread into the target field
  int bonds;     // F_int from the bond partners at the midpoints
  const int4* pn;  // per particle: up to kSubPartners partners (x, y, z) and the
                   // partner count (w); more partners: the CSR list in b
  BondArgs b;
};

struct ShellArgs {
  Geo g;
  const double* pos;
  const double* tmpl;
  double* fint;
  double* rot;
  int M;
  double k;
};

// Binning of markers into 8^3 tiles (counting sort) for LDS-staged
// interpolation and spreading.
struct TileArgs {
  Geo g;
  int tx, ty, tz, ntiles;
  int* count;   // [ntiles]
  int* start;   // [ntiles + 1]
  int* cursor;  // [ntiles]
  int* occ;     // occupied tiles in increasing order
  int* nocc;    // [1]
  int* ptile;   // tile of every marker
  int* sorted;  // markers grouped by tile
  uint64_t* mask;
};

hipError_t launch_bin(const TileArgs& t, const double* pos, long long n, hipStream_t st);
// Interpolation from the velocity of the flagged sites; redo = false leaves
// the listed markers to launch_shell_redo_forces (a marker set of whole
// shells), which redoes them and then computes the tether forces.
hipError_t launch_flag_interp(int storage, int K, const SiteArgs& s, const uint64_t* mask,
                              void* U, uint32_t stamp, const double* at, double* pos, double* aux,
                              int mode, long long n, int* miss, bool all_miss, bool redo,
                              hipStream_t st);
hipError_t launch_shell_redo_forces(int storage, int K, const ShellArgs& sa, int nshell,
                                    const SiteArgs& s, const void* U, uint32_t stamp,
                                    const double* at, double* pos, double* aux, int mode,
                                    int* miss, hipStream_t st);
hipError_t launch_tile_spread(int storage, int K, const TileArgs& t, const double* at,
                              const double* F, void* field, long long n, hipStream_t st);

// One ensemble member as the batched kernels see it (device memory).  The
// fields cur, pend and steps_done are advanced on the device only.
struct EnsSlot {
  Geo g;  // wpr == 0: linear force mask
  uint32_t mnx, mny;  // div_magic of nx and ny for the site decomposition
  void* f[2];
  void* FA;
  void* FB;
  uint64_t* mask;
  double* pos;
  double* vel;
  const double* mass;
  long long np;
  double rho0, fx, fy, fz;
  double omp, omm, gamma;
  float scale, inv;
  int collision, coupling;
  int cur, pend;
  long long steps_done, steps_target;
  int live;
  int comoving;
  double uref[3];  // storage reference velocity of f[cur]
  double4* mcache;  // coupling moment cache (see PartArgs)
  int4* mbase;
  int mvalid;       // the cache holds the state of f[cur]
  double cm[40];    // comoving reference terms of the next pass (comoving_terms)
  float cmf[40];    // the same in FP32
  int det_on;       // deterministic spreading: lattice forces stored in aux, summed in det
  double* aux;      // [np][3]
  uint64_t* det;    // [N][3][2] fixed-point accumulator
};

struct EnsArgs {
  EnsSlot* slots;
  int nslots;
  const int2* litems;  // (slot, 256-site chunk)
  const int* nlitems;
  const int2* pitems;  // (slot, first particle of a 256-lane group block)
  const int* npitems;
};

// det: the deterministic spreading kernels run after each coupling half
// big: some box has populations of 4 GiB or more
hipError_t launch_ens_step(int storage, int K, const EnsArgs& e, int lat_grid, int part_grid,
                           int det, bool big, hipStream_t st);

// Workgroups of the row-mapped launches: one covers (part of) an x row.
inline dim3 lattice_block(const Geo& g) {
  int bx = ((g.nx + 63) / 64) * 64;
  if (bx > 256) bx = 256;
  return dim3(bx, 1, 1);
}
inline dim3 lattice_grid(const Geo& g, dim3 b) {
  return dim3((g.nx + b.x - 1) / b.x, g.ny, g.nz);
}

hipError_t launch_stream_collide(int storage, bool comoving, const LatArgs& a, hipStream_t st);
// The same for boxes on the linear-site pass (g.wpr == 0).
hipError_t launch_stream_collide_lin(int storage, bool comoving, const LatArgs& a,
                                     hipStream_t st);
hipError_t launch_init(int storage, const InitArgs& a, hipStream_t st);
hipError_t launch_moments(int storage, const SiteArgs& a, double* rho, double* u, hipStream_t st);
// gp, gm: factors of the even and odd non-equilibrium parts (1, 1: the
// physical populations; sqrt(1 - lambda+-): the collide-stream-collide state).
hipError_t launch_populations(int storage, const SiteArgs& a, double* out, double gp, double gm,
                              hipStream_t st);
// pref: factor of the traceless part; prefb: factor of the trace part
hipError_t launch_stress(int storage, const SiteArgs& a, double* out, double pref, double prefb,
                         hipStream_t st);
hipError_t launch_totals(int storage, const SiteArgs& a, double* partial, int nblk,
                         const double* vel, const double* mass, long long np, double* out,
                         hipStream_t st);
hipError_t launch_drift(const Geo& g, long long n, double* pos, const double* vel, double dt,
                        hipStream_t st);
hipError_t launch_wrap(const Geo& g, long long n, double* pos, hipStream_t st);
// Positions and velocities of n particles into d_pos and d_vel (either may be null).
hipError_t launch_copy_particles(long long n, const double* pos, const double* vel, double* d_pos,
                                 double* d_vel, hipStream_t st);
// Zeroes bytes (a multiple of 8) at p with a fill kernel.
hipError_t launch_zero(void* p, size_t bytes, hipStream_t st);
hipError_t launch_couple_half(int storage, const PartArgs& a, hipStream_t st);
// Whether np free particles of a box of N sites are processed in tile order
// (PartArgs::order).  A gather of one site takes whole 128-byte lines of 19
// populations, so particles in index order fetch a line for 8 useful bytes
// (20 000 at 128^3 FP32: 197 MB, 5.3 TB/s); in tile order particles that share
// lines come together.  It pays from about one row of stencil nodes per line of a
// population on (us per step, by index -> in order): 2-point, 128^3, 20 000
// particles, FP32 (1.2 rows per line) 113.5 -> 112.3; 3-point, 10 000 (1.4) 125.4
// -> 121.5; 4-point, 5 000 (1.2) 122.8 -> 119.4; 2-point, 10 000 (0.6) 93.2 ->
// 93.4, 200 x 150 x 130, 20 000 (0.7) 157.3 -> 158.7.
// Not with 16-bit storage, though it would pay most there (FP16, 2.4 rows per
// line, 76.1 -> 66.5).  By index the contributions of a site arrive in nearly the
// same order in every run; in tile order they arrive in another one, and where
// three or more meet, the last bit of their FP32 sum now and then moves a stored
// 16-bit population by a quantum (80 x 180 x 147 FP16, 13 694 particles, 10 steps:
// 36 of 36 pairs of runs, one in tile order and one by index, differ at single
// sites by 1.3e-3 of the stress's rms; 15 of 15 pairs by index agree to 6e-8).
inline bool order_pays(int storage_bytes, int K, long long np, long long N) {
  const double rows = (double)np * K * K, lines = (double)N * storage_bytes / 128.0;
  return storage_bytes >= 4 && np >= 4096 && rows >= lines;
}
// The second half a of one step and the first half b of the next by one
// workgroup of at most one wavefront per SIMD of a CU; with more particles the
// gathers and atomics of one CU take longer than the launch they save (64^3
// FP32, 2-point, us per step as two launches -> as one: 1 particle 20.1 -> 18.9,
// 32 particles 23.6 -> 22.6, 64 24.2 -> 27.6; 3-point, 16 particles 22.3 -> 23.1).
constexpr int kPairLanes = 256;
inline bool couple_pair_fits(long long n, int K) {
  return n * (K == 2 ? 8 : (K == 3 ? 32 : 64)) <= kPairLanes;
}
hipError_t launch_couple_pair(int storage, const PartArgs& a, const PartArgs& b, hipStream_t st);
// One coupled sub-step (SubArgs); and the fold: the nf fields u.gin moved
// into the target field of a (a.target) at the flagged sites and left zero.
hipError_t launch_mts_substep(int storage, const PartArgs& a, const SubArgs& u, hipStream_t st);
hipError_t launch_mts_fold(int storage, const PartArgs& a, const SubArgs& u, int nf,
                           hipStream_t st);
// Deterministic spreading: W F of every particle (positions X, lattice forces
// F [n][3]) into the 128-bit fixed-point accumulator acc [N][3][2], flagging
// the sites (and the closing drift if a.drift_after); then field += the sums
// at every flagged site and acc back to zero there.
hipError_t launch_spread_det(const PartArgs& a, const double* X, const double* F, uint64_t* acc,
                             hipStream_t st);
hipError_t launch_det_finalize(int storage, const Geo& g, const uint64_t* mask, uint64_t* acc,
                               void* field, hipStream_t st);
hipError_t launch_ib_predict(int storage, const PartArgs& a, hipStream_t st);
hipError_t launch_ib_advect(int storage, const PartArgs& a, int spread_fint, hipStream_t st);
hipError_t launch_bond_groups(const BondArgs& b, int ngroups, int gcap, int mode, int acc,
                              int nsub, double dt, hipStream_t st);
hipError_t launch_shell_forces(const ShellArgs& s, int nshell, hipStream_t st);

constexpr int kTotalsBlocks = 1024;

}  // namespace lbc
