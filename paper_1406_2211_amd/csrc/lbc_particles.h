// lbc_particles.h -- device code of the particle side: stencils, interpolation,
// spreading, the coupling update, the fixed-point sums of the deterministic
// mode and the bonded groups.
#pragma once

#include "lbc_device.h"
#include "lbc_internal.h"

namespace lbc {

// ======================================================================
// Particle side: interpolation I (Eq. IBM-interpolation), spreading I*
// (Eq. IBM-spreading), coupling forces (Eq. modified-force, Eq.
// modified-ebf), velocity kicks and position drifts (Alg. 2 and 3).
//
// Work mapping: an aligned group of L lanes (L = 8, 32, 64 for the 2-, 3- and
// 4-point kernels, L >= K^3) handles one particle, one lane per stencil site,
// so the site gathers and the spreading atomics of a particle are issued in
// parallel.  Weighted sums are reduced inside the group (fixed order), after
// which every lane holds the interpolated values and evaluates the FP64
// coupling update redundantly.  With few particles a launch is one chain of
// dependent loads and instructions, about one wavefront per SIMD, so the chain
// is kept short: DPP sums, closed-form weights (one square root per axis),
// one reciprocal per set of divisions (200 particles, 3-point kernel: first
// half 11 -> 7.4 us, second 11 -> 9.2; 1200 beads, coupled sub-step 8.7 -> 8.6;
// 20 000 particles, first half 15.5 -> 12.8).
// ======================================================================
struct SiteSlot {
  bool site;   // the node lies in the box (not beyond a wall)
  bool valid;  // ... and carries a nonzero weight
  double W;
  int x, y, z;  // wrapped node
  int j0[3];    // first stencil node, unwrapped
};

// Whether t of stencil_t is that of a position near its first node: at most 1, or
// 1/2 and the rounding of X + 1/2 for the 3-point kernel (whose square root exists
// up to 0.577).  One compare per axis, in every lane's chain: with two (t >= 0 as
// well, which only clamped positions miss) one particle at 32^3 took 1 % longer.
template <int K>
__device__ __forceinline__ bool in_reach(double t) {
  return fabs(t) <= (K == 3 ? 0.5625 : 1.0);
}

template <int K>
__device__ __forceinline__ SiteSlot slot_of(const Geo& g, const double X[3], int lane) {
  SiteSlot s{false, false, 0.0, 0, 0, 0, {0, 0, 0}};
  double t[3], q[3];
#pragma unroll
  for (int a = 0; a < 3; ++a) stencil_t<K, double>(X[a], s.j0[a], t[a], q[a]);
  if (lane >= K * K * K) return s;
  const int kx = lane % K, ky = (lane / K) % K, kz = lane / (K * K);
  int yy = s.j0[1] + ky;
  if (g.wall) {
    if (yy < 0 || yy >= g.ny) return s;  // beyond a wall: no weight
  } else {
    yy = wrap_near(yy, g.ny);
  }
  // A position that is no number, or so far off that safe_floor clamps it, has no
  // node within reach: no weight, so it neither reads nor forces the fluid (the
  // closed forms would give NaN, or weights that grow with the distance).  t = 1
  // is in reach: X - floor(X) rounds to it just below a node (a walled y of -1e-20),
  // and the closed forms then give the weights of that node.
  if (in_reach<K>(t[0]) && in_reach<K>(t[1]) && in_reach<K>(t[2]))
    s.W = node_weight<K, double>(kx, t[0], q[0]) * node_weight<K, double>(ky, t[1], q[1]) *
          node_weight<K, double>(kz, t[2], q[2]);
  s.site = true;
  s.valid = s.W != 0.0;
  s.x = wrap_near(s.j0[0] + kx, g.nx);
  s.y = yy;
  s.z = wrap_near(s.j0[2] + kz, g.nz);
  return s;
}

// Interpolated rho_p and u_p of particle p at X.  With a.cache_fill (second
// coupling half, post-stream moments without the pending force) every node in
// the box stores its gathered moments, also at zero weight, so that a later
// position with the same first node finds all of them; with a.cache_use and
// an unchanged first node the cached moments replace the gather, and the
// pending half force is added exactly as the gather would add it.  keep_base
// and keep_m receive what a fill stores.
template <int S, int K>
__device__ __forceinline__ void group_interp(const PartArgs& a, const double X[3], bool phys,
                                             int lane, double& rp, double up[3], long long p,
                                             const void* const* gin = nullptr, int ngin = 0,
                                             const int4* pre_base = nullptr,
                                             const double4* pre_m = nullptr,
                                             int4* keep_base = nullptr,
                                             double4* keep_m = nullptr) {
  constexpr int L = Lanes<K>::L;
  const SiteSlot sl = slot_of<K>(a.s.g, X, lane);
  const bool fill = a.cache_fill != 0 && !phys;
  bool hit = false;
  if (a.cache_use) {  // (pre_base, pre_m: the entries, loaded by the caller)
    const int4 b = pre_base ? *pre_base : a.mbase[p];
    hit = b.x == sl.j0[0] && b.y == sl.j0[1] && b.z == sl.j0[2];
  }
  double r = 0, ux = 0, uy = 0, uz = 0;
  if (sl.site && (sl.valid || fill)) {
    double drho, j[3];
    if (hit) {
      const double4 m = pre_m ? *pre_m : a.mcache[p * L + lane];
      drho = m.x;
      j[0] = m.y;
      j[1] = m.z;
      j[2] = m.w;
      if (phys) add_pending<S>(a.s, site_index(a.s.g, sl.x, sl.y, sl.z), j);
    } else {
      double fl[Q];
      site_phys<S>(a.s, sl.x, sl.y, sl.z, fl, drho, j, phys);
      if (fill) a.mcache[p * L + lane] = make_double4(drho, j[0], j[1], j[2]);
      if (keep_m) *keep_m = make_double4(drho, j[0], j[1], j[2]);
    }
    if (phys && a.fa_rd) add_field<S>(a.FA, site_index(a.s.g, sl.x, sl.y, sl.z), j);
    for (int f = 0; f < ngin; ++f) add_field<S>(gin[f], site_index(a.s.g, sl.x, sl.y, sl.z), j);
    if (sl.valid) {
      const double rr = a.s.rho0 + drho, w = sl.W / rr;
      r = sl.W * rr;
      ux = w * j[0];
      uy = w * j[1];
      uz = w * j[2];
    }
  }
  if (fill && lane == 0) a.mbase[p] = make_int4(sl.j0[0], sl.j0[1], sl.j0[2], 0);
  if (keep_base) *keep_base = make_int4(sl.j0[0], sl.j0[1], sl.j0[2], 0);
  rp = group_sum<L>(r);
  up[0] = group_sum<L>(ux);
  up[1] = group_sum<L>(uy);
  up[2] = group_sum<L>(uz);
}

// The mask word of the lane's stencil node at X, loaded ahead of the
// spreading so that its latency overlaps the gathers: bits are only set while
// a coupling kernel runs (the lattice pass clears them between kernels), so a
// bit seen set stays set, and one seen clear is set with an atomic.  A plain,
// cached load (see flag_site).
template <int K>
__device__ __forceinline__ uint64_t mask_preload(const PartArgs& a, const double X[3], int lane) {
  const SiteSlot sl = slot_of<K>(a.s.g, X, lane);
  if (!sl.valid) return ~0ull;
  uint64_t bit;
  return *mask_word(a.mask, a.s.g, sl.x, sl.y, sl.z, bit);
}

// Adds (c0, c1, c2) to the force vector of site sidx (kNoSite: nothing) for
// every lane of the wavefront, with the three components of a site issued by
// neighbouring lanes: the wavefront's contributions go through LDS and come
// back with lane 4q + k holding component k of site q, 16 sites per round.
// The spreading is bound by the number of requests its atomics make of L2: with
// each lane adding its three components in turn an instruction touched up to
// 64 lines for one word each and every line was visited three times; now an
// instruction touches 16 lines for three words each.  20 000 free particles at
// 128^3 (FP32, 2-point): first coupling half 26 -> 15.5 us, second 43 -> 37 us.
constexpr uint32_t kNoSite = 0xffffffffu;  // a box has at most 2^32 - 1 sites
template <typename E>
struct AddSlot {
  E c[3];
  uint32_t site;
};
template <typename E, int WAVES>
__device__ __forceinline__ void wave_add3(E* field, uint32_t sidx, E c0, E c1, E c2) {
  __shared__ AddSlot<E> slots[WAVES][64];  // WAVES: wavefronts of the workgroup at most
  AddSlot<E>* w = slots[threadIdx.x >> 6];
  const int l = (int)threadIdx.x & 63;
  w[l] = AddSlot<E>{{c0, c1, c2}, sidx};
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  const int k = l & 3;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const AddSlot<E>& q = w[16 * r + (l >> 2)];
    const uint32_t s = q.site;
    if (k < 3 && s != kNoSite) unsafeAtomicAdd(field + 4 * (size_t)s + k, q.c[k]);
  }
}

// Spread W F to the lane's stencil node; pre: the node's mask word from
// mask_preload at the same X (nullptr: load it here).
template <typename E, int K, int WAVES = 4>
__device__ __forceinline__ void group_spread(const PartArgs& a, const double X[3],
                                             const double F[3], void* field, int lane, bool live,
                                             const uint64_t* pre = nullptr) {
  const SiteSlot sl = slot_of<K>(a.s.g, X, lane);
  const bool on = live && sl.valid;
  const long long s = site_index(a.s.g, sl.x, sl.y, sl.z);
  wave_add3<E, WAVES>((E*)field, on ? (uint32_t)s : kNoSite, (E)(sl.W * F[0]), (E)(sl.W * F[1]),
               (E)(sl.W * F[2]));
  if (!on) return;
  uint64_t bit;
  uint64_t* mw = mask_word(a.mask, a.s.g, sl.x, sl.y, sl.z, bit);
  if (pre) {
    if (!(*pre & bit)) atomicOr((unsigned long long*)mw, bit);
  } else {
    flag_site(mw, bit);
  }
}

// Spreading of the 2-point kernel with the contributions of consecutive
// particles combined inside the wavefront before the atomics.  A wavefront
// holds 8 particles (8 lanes each, one per stencil node); consecutive
// particles of a chain sit about one spacing apart, so particle q + 1 shares
// on average three to four of its nodes with particle q.  From the last
// particle of the wavefront down to the second, each particle hands the
// (already combined) contribution of every node it shares with its
// predecessor to the predecessor's lane for that node, which adds it in FP64;
// only nodes that are not handed on issue the three float atomics.  The sum at
// a site is the same set of terms as with one atomic per contribution (the
// order of atomic additions is unspecified either way).
//
// Which lanes pair up follows from the particles' first nodes alone (read
// from lanes 8q into scalars): the predecessor's node k' is the successor's
// node k' - d, d the difference of their first nodes, and a pair counts when
// both lanes carry weight (a ballot).  Only the contributions themselves move
// between lanes, one shuffle round per particle.  next: the launch has a particle
// after this one; pre: the node's mask word from mask_preload.
template <typename E, int WAVES = 4>
__device__ __forceinline__ void group_spread_k2(const PartArgs& a, const double X[3],
                                                const double F[3], void* field, int lane,
                                                bool next, bool live_p, uint64_t pre) {
  const SiteSlot sl = slot_of<2>(a.s.g, X, lane);
  const bool on = live_p && sl.valid;
  const long long sidx = on ? site_index(a.s.g, sl.x, sl.y, sl.z) : -1;
  double c0 = on ? sl.W * F[0] : 0.0, c1 = on ? sl.W * F[1] : 0.0, c2 = on ? sl.W * F[2] : 0.0;
  const int wl = (int)(threadIdx.x & 63), qi = wl >> 3;
  const int kx = lane & 1, ky = (lane >> 1) & 1, kz = lane >> 2;
  const uint64_t live = __ballot(sidx >= 0);  // lanes that carry weight
  bool issue = sidx >= 0;
  int jx[8], jy[8], jz[8];  // first node of each particle of the wavefront
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    jx[q] = __builtin_amdgcn_readlane(sl.j0[0], 8 * q);
    jy[q] = __builtin_amdgcn_readlane(sl.j0[1], 8 * q);
    jz[q] = __builtin_amdgcn_readlane(sl.j0[2], 8 * q);
  }
#pragma unroll
  for (int i = 7; i >= 1; --i) {
    const int dx = jx[i] - jx[i - 1], dy = jy[i] - jy[i - 1], dz = jz[i] - jz[i - 1];
    // receiver (particle i - 1, node k'): its node k' - d of particle i
    const int sx = kx - dx, sy = ky - dy, sz = kz - dz;
    const bool rin = qi == i - 1 && next && sx >= 0 && sx <= 1 && sy >= 0 && sy <= 1 &&
                     sz >= 0 && sz <= 1;
    const int src = rin ? 8 * i + sx + 2 * sy + 4 * sz : wl;
    // donor (particle i, node k): the receiver's node k + d of particle i - 1
    const int tx = kx + dx, ty = ky + dy, tz = kz + dz;
    const bool din = qi == i && tx >= 0 && tx <= 1 && ty >= 0 && ty <= 1 && tz >= 0 && tz <= 1;
    const int dst = 8 * (i - 1) + tx + 2 * ty + 4 * tz;
    const double g0 = __shfl(c0, src, 64), g1 = __shfl(c1, src, 64), g2 = __shfl(c2, src, 64);
    if (rin && sidx >= 0 && ((live >> src) & 1)) {
      c0 += g0;
      c1 += g1;
      c2 += g2;
    }
    if (din && sidx >= 0 && ((live >> dst) & 1)) issue = false;  // handed on to particle i - 1
  }
  wave_add3<E, WAVES>((E*)field, issue ? (uint32_t)sidx : kNoSite, (E)c0, (E)c1, (E)c2);
  if (!issue) return;
  uint64_t bit;
  uint64_t* mw = mask_word(a.mask, a.s.g, sl.x, sl.y, sl.z, bit);
  if (!(pre & bit)) atomicOr((unsigned long long*)mw, bit);
}

__device__ __forceinline__ void wrap3(const Geo& g, double r[3]) {
  r[0] = wrap_pos(r[0], (double)g.nx);
  if (!g.wall) r[1] = wrap_pos(r[1], (double)g.ny);
  r[2] = wrap_pos(r[2], (double)g.nz);
}

// F^h over the coupling step a.hh from the interpolated rho_p, u_p, and the
// kick of v: the Crank-Nicolson solution of Eq. fc-vel (Eq. modified-force)
// for force coupling, Eq. modified-ebf for the modified EBF.
__device__ __forceinline__ void couple_update(const PartArgs& a, long long p, double m, double rp,
                                              const double up[3], const double Fi[3], double v[3],
                                              double Fh[3]) {
  const double hh = a.hh, al = a.gamma * hh / m, be = a.gamma * hh / rp;
  if (a.coupling == LB_COUPLE_FC) {
    const double rden = 1.0 / (1.0 + 0.5 * al + 0.5 * be);
    double zeta[4] = {0, 0, 0, 0};
    if (a.kT > 0.0) {
      // random force of Eq. viscous-coupling: variance 2 k_B T gamma / hh per
      // component, entering the implicit solution like the drag; deviates from
      // the Philox block (particle, step low, 2^16 + coupling step, step high)
      normals4<double>(philox(make_uint4((uint32_t)p, a.t0, 65536u + (uint32_t)a.jc, a.t1),
                              a.key0, a.key1), zeta);
      const double sig = sqrt(2.0 * a.kT * a.gamma / hh) * rden;
      for (int k = 0; k < 3; ++k) zeta[k] *= sig;
    }
    // Crank-Nicolson solution of Eq. fc-vel over hh (Eq. modified-force), the
    // fluid at the particle also accelerated by the body force: +(beta/2) F_ext
    const double hm = hh / m;
    for (int k = 0; k < 3; ++k) {
      Fh[k] = -(a.gamma * (v[k] - up[k]) + 0.5 * al * Fi[k] - 0.5 * be * a.fext[k]) * rden;
      if (a.kT > 0.0) Fh[k] += zeta[k];
      v[k] += hm * (Fh[k] + Fi[k]);
    }
  } else {
    const double rs = 1.0 / (al + be), as = al * rs, bm = hh / m * (be * rs);
    for (int k = 0; k < 3; ++k) {
      const double d = v[k] - up[k];
      Fh[k] = -a.gamma * rs * d - as * Fi[k];
      v[k] = v[k] - as * d + bm * Fi[k];
    }
  }
}

// ----------------------------------------------- deterministic spreading
// Spreading (Eq. IBM-spreading) as an exact sum: every contribution W F is
// converted to a 128-bit fixed-point number q 2^-96 (two's complement, words
// lo and hi) and added to the site's accumulator with 64-bit integer
// atomics.  Integer addition is associative, so the sum does not depend on
// the order in which the contributions arrive; a finalize pass then adds the
// converted sum to the force field.  Range: contributions below 2^20 in
// magnitude (larger or non-finite ones become a marker that reads back as
// NaN), resolution 2^-96.
constexpr int kFixShift = 96;

__device__ __forceinline__ void to_fixed(double c, uint64_t& lo, uint64_t& hi) {
  const double a = fabs(c);
  if (!(a < 1048576.0)) {  // non-finite or beyond any force of a stable run
    lo = 0ull;
    hi = 1ull << 56;
    return;
  }
  lo = hi = 0ull;
  if (a == 0.0) return;
  int e;
  const double m = frexp(a, &e);                     // a = m 2^e, m in [1/2, 1)
  const uint64_t mant = (uint64_t)ldexp(m, 53);      // exact 53-bit integer
  const int sh = e - 53 + kFixShift;                 // a 2^96 = mant 2^sh, sh < 64
  if (sh > 0) {
    lo = mant << sh;
    hi = mant >> (64 - sh);
  } else if (sh > -64) {
    lo = mant >> (-sh);  // truncation below the resolution
  }
  if (c < 0.0) {
    lo = ~lo + 1ull;
    hi = ~hi + (lo == 0ull ? 1ull : 0ull);
  }
}

__device__ __forceinline__ double from_fixed(uint64_t lo, uint64_t hi) {
  const bool neg = (int64_t)hi < 0;
  if (neg) {
    lo = ~lo + 1ull;
    hi = ~hi + (lo == 0ull ? 1ull : 0ull);
  }
  if (hi >= (1ull << 54)) return __builtin_nan("");  // the marker of a non-finite contribution
  const double v = ldexp((double)hi, 64 - kFixShift) + ldexp((double)lo, -kFixShift);
  return neg ? -v : v;
}

// q += (lo, hi) modulo 2^128: the carry out of the low word is known from the
// value the low atomic returns, so the result is exact whatever the order.
__device__ __forceinline__ void fixed_add(uint64_t* q, uint64_t lo, uint64_t hi) {
  const uint64_t old = (uint64_t)atomicAdd((unsigned long long*)q, (unsigned long long)lo);
  const uint64_t h = hi + (old + lo < old ? 1ull : 0ull);
  if (h) atomicAdd((unsigned long long*)(q + 1), (unsigned long long)h);
}

// field += the accumulated sum at site s if it is flagged, and the
// accumulator back to zero there (one lane per site: no two lanes touch a site).
template <typename E>
__device__ __forceinline__ void det_finalize_site(const Geo& g, const uint64_t* mask,
                                                  uint64_t* acc, E* field, long long s) {
  const int x = (int)(s % g.nx);
  const long long r = s / g.nx;
  const int y = (int)(r % g.ny), z = (int)(r / g.ny);
  uint64_t bit;
  const uint64_t w = *mask_word(const_cast<uint64_t*>(mask), g, x, y, z, bit);
  if (!(w & bit)) return;
  uint64_t* q = acc + 6 * s;
  for (int k = 0; k < 3; ++k) {
    const uint64_t lo = q[2 * k], hi = q[2 * k + 1];
    if (!(lo | hi)) continue;
    field[4 * s + k] += (E)from_fixed(lo, hi);
    q[2 * k] = 0ull;
    q[2 * k + 1] = 0ull;
  }
}

// ======================================================================
// Intrinsic forces.
// ======================================================================

// Bonded groups: block b owns the particles perm[goff[b] .. goff[b+1]), a
// union of whole bonded clusters, so every bond partner is in the block's
// LDS.  mode 0: F_int at the current positions (stored, or added with acc).
// mode 1: nsub velocity-Verlet sub-steps of length dt with F_int only
// (the [P F_int P]^n factor of the multiple time-step split, Sec. 6).
// mode 2: the positions drift by dt (r <- wrap(r + dt v)), then mode 0.
// Bond partners of one particle, held in registers across the sub-steps
// (up to kMaxBondsReg; a particle with more partners reads the CSR list).
constexpr int kMaxBondsReg = 6;

struct Partners {
  int n;
  long long p;
  int loc[kMaxBondsReg];
};

__device__ __forceinline__ void load_partners(const BondArgs& b, long long p, Partners& P) {
  const int e0 = b.start[p], e1 = b.start[p + 1];
  P.p = p;
  P.n = e1 - e0;
#pragma unroll
  for (int k = 0; k < kMaxBondsReg; ++k) P.loc[k] = (k < P.n) ? b.loc[b.nbr[e0 + k]] : 0;
}

// d - n floor(d/n + 1/2) for |d| < 3n/2 (positions are wrapped into [0, n]); a
// coupled sub-step of 1200 beads 8.6 us, with the product by 1/n 8.5.
__device__ __forceinline__ double nearest_image(double d, int n, double lo, double hi) {
  return d - (double)(d >= hi ? n : (d < lo ? -n : 0));
}

__device__ __forceinline__ void bond_pair(const BondArgs& b, const double r[3], const double* q,
                                          double F[3]) {
  double d[3];
  for (int k = 0; k < 3; ++k) d[k] = q[k] - r[k];
  d[0] = nearest_image(d[0], b.g.nx, b.lo[0], b.hi[0]);
  if (!b.g.wall) d[1] = nearest_image(d[1], b.g.ny, b.lo[1], b.hi[1]);
  d[2] = nearest_image(d[2], b.g.nz, b.lo[2], b.hi[2]);
  const double L = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
  double s;
  if (b.type == LB_FENE)  // infinite energy from L = r0 on: NaN, not the formula's sign flip
    s = L < b.r0 ? b.k / (1.0 - L * L / (b.r0 * b.r0)) : __builtin_nan("");
  else
    s = L > 0.0 ? b.k * (L - b.r0) / L : 0.0;
  for (int k = 0; k < 3; ++k) F[k] += s * d[k];
}

__device__ __forceinline__ void bond_force(const BondArgs& b, const Partners& P, const double r[3],
                                           const double* lds, double F[3]) {
  F[0] = F[1] = F[2] = 0;
  if (P.n <= kMaxBondsReg) {
#pragma unroll
    for (int k = 0; k < kMaxBondsReg; ++k)
      if (k < P.n) bond_pair(b, r, lds + 3 * P.loc[k], F);
  } else {
    for (int e = b.start[P.p]; e < b.start[P.p + 1]; ++e) bond_pair(b, r, lds + 3 * b.loc[b.nbr[e]], F);
  }
}

__device__ __forceinline__ void bond_group(const BondArgs& b, int grp, int mode, int acc, int nsub,
                                           double dt, double* lds) {
  const int g0 = b.goff[grp], cnt = b.goff[grp + 1] - g0;
  const int t = threadIdx.x;
  const bool on = t < cnt;
  const long long p = on ? b.perm[g0 + t] : 0;
  double r[3] = {0, 0, 0}, v[3] = {0, 0, 0}, m = 1.0;
  Partners P;
  P.n = 0;
  P.p = p;
  if (on) {
    for (int k = 0; k < 3; ++k) {
      r[k] = b.pos[3 * p + k];
      v[k] = b.vel ? b.vel[3 * p + k] : 0.0;
    }
    if (b.mass) m = b.mass[p];
    load_partners(b, p, P);
  }
  if (mode == 0 || mode == 2) {
    if (mode == 2 && on) {  // drift by dt first (as k_drift does), store the positions
      for (int k = 0; k < 3; ++k) r[k] = r[k] + dt * v[k];
      wrap3(b.g, r);
      for (int k = 0; k < 3; ++k) b.pos[3 * p + k] = r[k];
    }
    if (on)
      for (int k = 0; k < 3; ++k) lds[3 * t + k] = r[k];
    __syncthreads();
    if (on) {
      double F[3];
      bond_force(b, P, r, lds, F);
      for (int k = 0; k < 3; ++k) b.fint[3 * p + k] = acc ? b.fint[3 * p + k] + F[k] : F[k];
    }
    return;
  }
  const double dtm = dt / m;
  for (int s = 0; s < nsub; ++s) {
    if (on) {
      for (int k = 0; k < 3; ++k) r[k] += 0.5 * dt * v[k];
      wrap3(b.g, r);
    }
    __syncthreads();
    if (on)
      for (int k = 0; k < 3; ++k) lds[3 * t + k] = r[k];
    __syncthreads();
    if (on) {
      double F[3];
      bond_force(b, P, r, lds, F);
      for (int k = 0; k < 3; ++k) {
        v[k] += dtm * F[k];
        r[k] += 0.5 * dt * v[k];
      }
      wrap3(b.g, r);
    }
  }
  if (on)
    for (int k = 0; k < 3; ++k) {
      b.pos[3 * p + k] = r[k];
      b.vel[3 * p + k] = v[k];
    }
}

// Lane groups of n particles as 256-lane workgroups.
inline unsigned gblocks(long long n, int K) {
  const long long L = K == 2 ? 8 : (K == 3 ? 32 : 64);
  return (unsigned)((n * L + 255) / 256);
}

#define LBC_KERNEL_SWITCH(K, CALL)                        \
  switch (K) {                                            \
    case 2: { constexpr int KK = 2; CALL; } break;        \
    case 3: { constexpr int KK = 3; CALL; } break;        \
    default: { constexpr int KK = 4; CALL; } break;       \
  }

}  // namespace lbc
