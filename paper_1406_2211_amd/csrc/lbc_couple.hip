// lbc_couple.hip -- launches of the particle side: coupling halves, the
// deterministic spread, the gathering immersed boundary, bonded groups and the
// coupled sub-steps.
#include <algorithm>

#include "lbc_pass.h"
#include "lbc_particles.h"

namespace lbc {

// One coupling step for FC / modified EBF: interpolate rho_p, u_p at r,
// compute F^h over h' = a.hh (h/2 for the half steps of Alg. 3, h/2n for the
// sub-steps of Eq. multistep), kick v, optionally drift, and spread -F^h
// (scaled by a.sw) or store it for the deterministic spread.
template <int S, int K, int WAVES>
__device__ __forceinline__ void couple_spread(const PartArgs& a, const double r[3],
                                              const double Ff[3], int lane, bool next, bool live,
                                              uint64_t mpre) {
  using E = typename Store<S>::R;
  void* field = a.target ? a.FB : a.FA;
  if constexpr (K == 2)
    group_spread_k2<E, WAVES>(a, r, Ff, field, lane, next, live, mpre);
  else
    group_spread<E, K, WAVES>(a, r, Ff, field, lane, live, &mpre);
}

template <int S, int K>
__global__ __launch_bounds__(256) void k_couple_half(PartArgs a) {
  constexpr int L = Lanes<K>::L;
  // With a spatial order each of the 8 XCDs (which take the workgroups in turn)
  // gets a contiguous run of it, so that particles sharing lines of the
  // populations share an L2.
  const long long blk = a.order ? (long long)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3)
                                : (long long)blockIdx.x;
  const long long gid = blk * blockDim.x + threadIdx.x;
  const int lane = (int)(gid % L);
  if ((gid & ~63ll) / L >= a.n) return;  // whole wavefronts leave together
  // the lanes past the last particle follow it and write nothing (they serve
  // the wavefront's spreading)
  const bool live = gid / L < a.n;
  const long long slot = live ? gid / L : a.n - 1;
  const long long p = a.order ? a.order[slot] : slot;
  double r[3], v[3], Fi[3] = {0, 0, 0};
  for (int k = 0; k < 3; ++k) {
    r[k] = a.pos[3 * p + k];
    v[k] = a.vel[3 * p + k];
    if (a.use_fint) Fi[k] = a.fint[3 * p + k];
  }
  if (a.drift_before) {  // P^1/2: r <- wrap(r + (h/2) v), as k_drift does
    for (int k = 0; k < 3; ++k) r[k] += a.hd * v[k];
    wrap3(a.s.g, r);
  }
  const uint64_t mpre = a.defer ? ~0ull : mask_preload<K>(a, r, lane);
  const double m = a.mass[p];
  double rp, up[3];
  group_interp<S, K>(a, r, a.phys != 0, lane, rp, up, p);
  double Fh[3];
  couple_update(a, p, m, rp, up, Fi, v, Fh);
  const double Ff[3] = {-a.sw * Fh[0], -a.sw * Fh[1], -a.sw * Fh[2]};
  if (a.defer) {
    if (live && lane == 0)
      for (int k = 0; k < 3; ++k) a.defer[3 * p + k] = Ff[k];
  } else {
    couple_spread<S, K, 4>(a, r, Ff, lane, slot + 1 < a.n, live, mpre);
  }
  if (live && lane == 0) {
    if (a.drift_after) {
      for (int k = 0; k < 3; ++k) r[k] += a.hd * v[k];
      wrap3(a.s.g, r);
    }
    if (a.drift_after || a.drift_before)
      for (int k = 0; k < 3; ++k) a.pos[3 * p + k] = r[k];
    for (int k = 0; k < 3; ++k) a.vel[3 * p + k] = v[k];
  }
}

// The second coupling half of one step (a) and the first of the next (b) in one
// launch of one workgroup, for particle sets that fit it: both see the same
// populations, and the first half needs the forces that every particle spread
// in the second, so between them only the workgroup has to meet.  The state and
// the moments of the stencil nodes stay in registers.  Without intrinsic forces
// in either half.  One particle at 32^3 (FP64): 5.8 + 5.2 -> 9.5 us a step.
template <int S, int K>
__global__ __launch_bounds__(kPairLanes) void k_couple_pair(PartArgs a, PartArgs b) {
  constexpr int L = Lanes<K>::L, WAVES = kPairLanes / 64;
  const int lane = (int)threadIdx.x % L;
  const bool live = (int)threadIdx.x / L < a.n;
  const bool wave = (int)(threadIdx.x & ~63u) / L < a.n;  // the wavefront holds a particle
  const long long p = live ? threadIdx.x / L : a.n - 1;
  double r[3], v[3], rp, up[3], Fh[3];
  const double Fi[3] = {0, 0, 0};
  for (int k = 0; k < 3; ++k) {
    r[k] = a.pos[3 * p + k];
    v[k] = a.vel[3 * p + k];
  }
  const double m = a.mass[p];
  int4 base = make_int4(0, 0, 0, 0);
  double4 mom = make_double4(0, 0, 0, 0);
  if (wave) {
    const uint64_t mpre = mask_preload<K>(a, r, lane);
    group_interp<S, K>(a, r, false, lane, rp, up, p, nullptr, 0, nullptr, nullptr, &base, &mom);
    couple_update(a, p, m, rp, up, Fi, v, Fh);
    const double Ff[3] = {-Fh[0], -Fh[1], -Fh[2]};
    couple_spread<S, K, WAVES>(a, r, Ff, lane, p + 1 < a.n, live, mpre);
    if (a.drift_after) {
      for (int k = 0; k < 3; ++k) r[k] += a.hd * v[k];
      wrap3(a.s.g, r);
    }
    if (b.drift_before) {
      for (int k = 0; k < 3; ++k) r[k] += b.hd * v[k];
      wrap3(b.s.g, r);
    }
  }
  // the spread forces are performed and seen by every wavefront (the float
  // atomics go past the caches, so agent scope)
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
  if (!wave) return;
  const uint64_t mpre = mask_preload<K>(b, r, lane);
  group_interp<S, K>(b, r, true, lane, rp, up, p, nullptr, 0, &base, &mom);
  couple_update(b, p, m, rp, up, Fi, v, Fh);
  const double Ff[3] = {-Fh[0], -Fh[1], -Fh[2]};
  couple_spread<S, K, WAVES>(b, r, Ff, lane, p + 1 < a.n, live, mpre);
  if (live && lane == 0)
    for (int k = 0; k < 3; ++k) {
      if (a.drift_after || b.drift_before) b.pos[3 * p + k] = r[k];
      b.vel[3 * p + k] = v[k];
    }
}

// Adds W F of every particle (positions X, lattice forces F [n][3]) to the
// fixed-point accumulator acc [N][3][2] at its stencil nodes and flags them;
// then the closing drift of the coupling step when a.drift_after (X = a.pos).
template <int K>
__global__ __launch_bounds__(256) void k_spread_det(PartArgs a, const double* X, const double* F,
                                                    uint64_t* acc) {
  constexpr int L = Lanes<K>::L;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long p = gid / L;
  const int lane = (int)(gid % L);
  if (p >= a.n) return;  // whole groups leave together
  double r[3], f[3];
  for (int k = 0; k < 3; ++k) {
    r[k] = X[3 * p + k];
    f[k] = F[3 * p + k];
  }
  const SiteSlot sl = slot_of<K>(a.s.g, r, lane);
  if (sl.valid) {
    const long long s = site_index(a.s.g, sl.x, sl.y, sl.z);
    for (int k = 0; k < 3; ++k) {
      uint64_t lo, hi;
      to_fixed(sl.W * f[k], lo, hi);
      if (lo | hi) fixed_add(acc + 6 * s + 2 * k, lo, hi);
    }
    uint64_t bit;
    flag_site(mask_word(a.mask, a.s.g, sl.x, sl.y, sl.z, bit), bit);
  }
  if (lane == 0 && a.drift_after) {
    for (int k = 0; k < 3; ++k) r[k] += a.hd * a.vel[3 * p + k];
    wrap3(a.s.g, r);
    for (int k = 0; k < 3; ++k) a.pos[3 * p + k] = r[k];
  }
}

template <typename E>
__global__ __launch_bounds__(256) void k_det_finalize(Geo g, const uint64_t* mask, uint64_t* acc,
                                                      E* field) {
  const long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (s < g.N) det_finalize_site<E>(g, mask, acc, field, s);
}

// IB (Alg. 2): predictor X~ = X + (h/2) I[X] u(t)
template <int S, int K>
__global__ __launch_bounds__(256) void k_ib_predict(PartArgs a) {
  constexpr int L = Lanes<K>::L;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const long long p = gid / L;
  const int lane = (int)(gid % L);
  if (p >= a.n) return;
  double X[3] = {a.pos[3 * p], a.pos[3 * p + 1], a.pos[3 * p + 2]}, rp, up[3];
  group_interp<S, K>(a, X, true, lane, rp, up, p);
  if (lane == 0) {
    for (int k = 0; k < 3; ++k) X[k] += 0.5 * up[k];
    wrap3(a.s.g, X);
    for (int k = 0; k < 3; ++k) a.aux[3 * p + k] = X[k];
  }
}

// IB: X <- X + (h/2) I[X~] u with the current physical u; with spread_fint
// also spreads +F_int at X~ into the A field (first half force).
template <int S, int K>
__global__ __launch_bounds__(256) void k_ib_advect(PartArgs a, int spread_fint) {
  using E = typename Store<S>::R;
  constexpr int L = Lanes<K>::L;
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = (int)(gid % L);
  if ((gid & ~63ll) / L >= a.n) return;  // whole wavefronts leave together
  const bool live = gid / L < a.n;  // as in k_couple_half
  const long long p = live ? gid / L : a.n - 1;
  const double Xt[3] = {a.aux[3 * p], a.aux[3 * p + 1], a.aux[3 * p + 2]};
  double rp, up[3];
  group_interp<S, K>(a, Xt, true, lane, rp, up, p);
  if (live && lane == 0) {
    double X[3];
    for (int k = 0; k < 3; ++k) X[k] = a.pos[3 * p + k] + 0.5 * up[k];
    wrap3(a.s.g, X);
    for (int k = 0; k < 3; ++k) a.pos[3 * p + k] = X[k];
  }
  if (spread_fint) {
    const double F[3] = {a.fint[3 * p], a.fint[3 * p + 1], a.fint[3 * p + 2]};
    group_spread<E, K>(a, Xt, F, a.FA, lane, live);
  }
}

__global__ void k_bond_groups(BondArgs b, int mode, int acc, int nsub, double dt) {
  extern __shared__ double lds[];
  bond_group(b, blockIdx.x, mode, acc, nsub, dt, lds);
}

// One coupled sub-step of Eq. multistep in one launch (SubArgs): drift dt/2 to
// the midpoint, F_int there (each particle advances its bond partners itself,
// with the same arithmetic as their own drift), interpolation of the fluid
// that every earlier sub-step has forced, F^h and kick over dt, spread of the
// lattice force at the midpoint, drift dt/2.  Everything that depends only on
// the particle index (its state, partner list and cached moments) is loaded
// first, and the partners' state is loaded before the interpolation's gathers
// but used after them, so that the launch waits on about three memory round
// trips: state, gathers, spreading atomics.
template <int S, int K>
__global__ __launch_bounds__(256) void k_mts_substep(PartArgs a, SubArgs u) {
  using E = typename Store<S>::R;
  constexpr int L = Lanes<K>::L;
  constexpr int NP = kSubPartners;
  static_assert(NP == 3, "the packed partner entry holds three partners");
  const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int lane = (int)(gid % L);
  if ((gid & ~63ll) / L >= a.n) return;  // whole wavefronts leave together
  const bool live = gid / L < a.n;  // as in k_couple_half
  const long long p = live ? gid / L : a.n - 1;
  double pi[3], v[3];
  for (int k = 0; k < 3; ++k) {
    pi[k] = u.pin[3 * p + k];
    v[k] = u.vin[3 * p + k];
  }
  const int4 pn = u.bonds ? u.pn[p] : make_int4(0, 0, 0, 0);
  const double m = a.mass[p];
  int4 mb = make_int4(0, 0, 0, 0);
  double4 mc = make_double4(0, 0, 0, 0);
  if (a.cache_use) {
    mb = a.mbase[p];
    mc = a.mcache[p * L + lane];
  }
  double r[3];
  for (int k = 0; k < 3; ++k) r[k] = pi[k] + a.hd * v[k];
  wrap3(a.s.g, r);
  // the partners' start-of-sub-step state (pn.w <= NP: partners in pn.x..z)
  const int qs[3] = {pn.x, pn.y, pn.z};
  double pq[NP][3], vq[NP][3];
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const long long q = j < pn.w ? qs[j] : p;
    for (int k = 0; k < 3; ++k) {
      pq[j][k] = u.pin[3 * q + k];
      vq[j][k] = u.vin[3 * q + k];
    }
  }
  const uint64_t mpre = mask_preload<K>(a, r, lane);
  double rp, up[3];
  group_interp<S, K>(a, r, a.phys != 0, lane, rp, up, p, u.gin, u.ngin, &mb, &mc);
  double Fi[3] = {0, 0, 0};
  if (pn.w <= NP) {
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      if (j < pn.w) {
        double rq[3];
        for (int k = 0; k < 3; ++k) rq[k] = pq[j][k] + a.hd * vq[j][k];
        wrap3(a.s.g, rq);
        bond_pair(u.b, r, rq, Fi);
      }
    }
  } else {  // more partners than held in registers: the CSR list
    for (int e = u.b.start[p]; e < u.b.start[p + 1]; ++e) {
      const long long q = u.b.nbr[e];
      double rq[3];
      for (int k = 0; k < 3; ++k) rq[k] = u.pin[3 * q + k] + a.hd * u.vin[3 * q + k];
      wrap3(a.s.g, rq);
      bond_pair(u.b, r, rq, Fi);
    }
  }
  double Fh[3];
  couple_update(a, p, m, rp, up, Fi, v, Fh);
  const double Ff[3] = {-a.sw * Fh[0], -a.sw * Fh[1], -a.sw * Fh[2]};
  void* field = u.gout ? u.gout : (a.target ? a.FB : a.FA);
  if constexpr (K == 2)
    group_spread_k2<E>(a, r, Ff, field, lane, p + 1 < a.n, live, mpre);
  else
    group_spread<E, K>(a, r, Ff, field, lane, live, &mpre);
  if (live && lane == 0) {
    for (int k = 0; k < 3; ++k) r[k] += a.hd * v[k];
    wrap3(a.s.g, r);
    for (int k = 0; k < 3; ++k) {
      u.pout[3 * p + k] = r[k];
      u.vout[3 * p + k] = v[k];
    }
  }
}

// The sub-step fields into the target field at every flagged site (every
// nonzero entry of a field lies on a site its spread flagged), one lane per
// site: no two lanes share a site, so plain loads and stores suffice.  The
// fields are left zero.
//
// Mask words per wavefront: 32 (1200 beads at 128^3: 6.5 us with 64, which leaves
// half a wavefront per SIMD, 5.0 with 32, 16 or 8; 10^4 beads at 256^3: no difference).
constexpr int kFoldWords = 32;

template <int S>
__global__ __launch_bounds__(256) void k_mts_fold(Geo g, const uint64_t* __restrict__ mask,
                                                  long long nwords, SubArgs u, int nf, void* T) {
  using V4 = typename Store<S>::V4;
  for_flagged_sites<kFoldWords>(g, mask, nwords, [&](int x, int y, int z) {
    const long long s = site_index(g, x, y, z);
    V4 t = ((const V4*)T)[s];
    bool any = false;
    for (int f = 0; f < nf; ++f) {
      V4* G = (V4*)u.gin[f];
      const V4 w = G[s];
      if (w.x != 0 || w.y != 0 || w.z != 0) {
        t.x += w.x;
        t.y += w.y;
        t.z += w.z;
        G[s] = V4{0, 0, 0, 0};
        any = true;
      }
    }
    if (any) ((V4*)T)[s] = t;
  });
}

hipError_t launch_couple_half(int storage, const PartArgs& a, hipStream_t st) {
  if (a.n > 0) {
    unsigned nb = gblocks(a.n, a.K);
    if (a.order) nb = (nb + 7) / 8 * 8;
    LBC_KERNEL_SWITCH(a.K, LBC_STORAGE_SWITCH(storage, (k_couple_half<SS, KK><<<nb, 256, 0, st>>>(a))));
  }
  return hipGetLastError();
}

hipError_t launch_couple_pair(int storage, const PartArgs& a, const PartArgs& b, hipStream_t st) {
  if (a.n <= 0 || !couple_pair_fits(a.n, a.K)) return hipErrorInvalidValue;
  const unsigned lanes = (unsigned)(a.n * (a.K == 2 ? 8 : (a.K == 3 ? 32 : 64)) + 63) / 64 * 64;
  LBC_KERNEL_SWITCH(a.K, LBC_STORAGE_SWITCH(storage, (k_couple_pair<SS, KK><<<1, lanes, 0, st>>>(a, b))));
  return hipGetLastError();
}

hipError_t launch_mts_substep(int storage, const PartArgs& a, const SubArgs& u, hipStream_t st) {
  if (a.n > 0)
    LBC_KERNEL_SWITCH(a.K, LBC_STORAGE_SWITCH(storage, (k_mts_substep<SS, KK>
                                                        <<<gblocks(a.n, KK), 256, 0, st>>>(a, u))));
  return hipGetLastError();
}

hipError_t launch_mts_fold(int storage, const PartArgs& a, const SubArgs& u, int nf,
                           hipStream_t st) {
  if (nf <= 0) return hipSuccess;
  const Geo& g = a.s.g;
  const long long nwords = mask_nwords(g);
  void* T = a.target ? a.FB : a.FA;
  const long long per_wg = 4ll * kFoldWords;
  const unsigned gr = (unsigned)std::min<long long>((nwords + per_wg - 1) / per_wg, 16384ll);
  if (storage == LB_F64)
    k_mts_fold<LB_F64><<<gr, 256, 0, st>>>(g, a.mask, nwords, u, nf, T);
  else
    k_mts_fold<LB_F32><<<gr, 256, 0, st>>>(g, a.mask, nwords, u, nf, T);
  return hipGetLastError();
}

hipError_t launch_spread_det(const PartArgs& a, const double* X, const double* F, uint64_t* acc,
                             hipStream_t st) {
  if (a.n > 0)
    LBC_KERNEL_SWITCH(a.K, (k_spread_det<KK><<<gblocks(a.n, KK), 256, 0, st>>>(a, X, F, acc)));
  return hipGetLastError();
}

hipError_t launch_det_finalize(int storage, const Geo& g, const uint64_t* mask, uint64_t* acc,
                               void* field, hipStream_t st) {
  const unsigned nb = (unsigned)((g.N + 255) / 256);
  if (storage == LB_F64)
    k_det_finalize<double><<<nb, 256, 0, st>>>(g, mask, acc, (double*)field);
  else
    k_det_finalize<float><<<nb, 256, 0, st>>>(g, mask, acc, (float*)field);
  return hipGetLastError();
}

hipError_t launch_ib_predict(int storage, const PartArgs& a, hipStream_t st) {
  if (a.n > 0)
    LBC_KERNEL_SWITCH(a.K, LBC_STORAGE_SWITCH(storage, (k_ib_predict<SS, KK>
                                                        <<<gblocks(a.n, KK), 256, 0, st>>>(a))));
  return hipGetLastError();
}

hipError_t launch_ib_advect(int storage, const PartArgs& a, int spread_fint, hipStream_t st) {
  if (a.n > 0)
    LBC_KERNEL_SWITCH(a.K, LBC_STORAGE_SWITCH(storage, (k_ib_advect<SS, KK>
                                                        <<<gblocks(a.n, KK), 256, 0, st>>>(a, spread_fint))));
  return hipGetLastError();
}

hipError_t launch_bond_groups(const BondArgs& b, int ngroups, int gcap, int mode, int acc,
                              int nsub, double dt, hipStream_t st) {
  if (ngroups > 0)
    k_bond_groups<<<ngroups, gcap, (size_t)gcap * 3 * sizeof(double), st>>>(b, mode, acc, nsub, dt);
  return hipGetLastError();
}

}  // namespace lbc
