// lbc_pass.h -- device code of the fused lattice pass shared by its launches:
// the coupling forces of a site, the pass over linear site indices, and the
// choice of a pass variant.
#pragma once

#include <type_traits>

#include "lbc_device.h"
#include "lbc_internal.h"

namespace lbc {

// Coupling forces of one site for the fused pass, from the two force fields
// where the mask word flags the site, and with JOIN the ng sub-step fields that
// join FA; the fields are zeroed after the read, and the owning lane clears the
// word when the pass clears the mask.  FA's sum is complete before FB is added, as
// after a fold.  Not in the linear-site pass: the loop there makes the
// compiler contract another product of the equilibria, which rounds 16-bit
// populations otherwise, also where no field joins.
template <int S, bool JOIN>
__device__ __forceinline__ void take_forces(uint64_t word, uint64_t* mp, size_t site, uint32_t lane,
                                            void* FAp, void* FBp, void* const* G, int ng, bool clear,
                                            typename Store<S>::R& Fx, typename Store<S>::R& Fy,
                                            typename Store<S>::R& Fz) {
  using V4 = typename Store<S>::V4;
  if ((word >> lane) & 1ull) {
    V4* FA = (V4*)FAp;
    V4* FB = (V4*)FBp;
    V4 fa = FA[site];
    const V4 fb = FB[site];
    V4 zero;
    zero.x = zero.y = zero.z = zero.w = 0;
    for (int k = 0; JOIN && k < ng; ++k) {
      V4* Gk = (V4*)G[k];
      const V4 w = Gk[site];
      if (w.x != 0 || w.y != 0 || w.z != 0) {
        fa.x += w.x;
        fa.y += w.y;
        fa.z += w.z;
        Gk[site] = zero;
      }
    }
    Fx += fa.x + fb.x;
    Fy += fa.y + fb.y;
    Fz += fa.z + fb.z;
    FA[site] = zero;
    FB[site] = zero;
  }
  if (lane == 0 && clear) *mp = 0;
}

// Immersed boundary: the second half force of a step is the same spread of
// the same F_int as the first (Sec. 5.1), so the first-half field becomes the
// pending second half: FB <- FA, FA <- 0, and the owning lane rewrites the
// word to flag exactly the sites of the pending field (which the next pass
// must read).  Called by all lanes of a wavefront that owns the (nonzero)
// word.
template <int S>
__device__ __forceinline__ void take_forces_ib(uint64_t word, uint64_t* mp, size_t site,
                                               uint32_t lane, void* FAp, void* FBp,
                                               typename Store<S>::R& Fx, typename Store<S>::R& Fy,
                                               typename Store<S>::R& Fz) {
  using V4 = typename Store<S>::V4;
  bool live = false;
  if ((word >> lane) & 1ull) {
    V4* FA = (V4*)FAp;
    V4* FB = (V4*)FBp;
    const V4 fa = FA[site], fb = FB[site];
    Fx += fa.x + fb.x;
    Fy += fa.y + fb.y;
    Fz += fa.z + fb.z;
    V4 zero;
    zero.x = zero.y = zero.z = zero.w = 0;
    FA[site] = zero;
    FB[site] = fa;
    live = fa.x != 0 || fa.y != 0 || fa.z != 0;
  }
  const uint64_t keep = __ballot(live);
  if (lane == 0 && keep != word) *mp = keep;
}

// Fused pass over linear site indices: a wavefront covers 64 consecutive
// sites whatever the row length, and owns one word of a linear force mask
// (wpr == 0).  Used by the batched ensemble pass and by single boxes whose x
// extent is not a multiple of 64 (where row-aligned wavefronts would idle
// lanes).  Site coordinates come from a 32-bit quotient by nx and ny.
// V is a view of the pass parameters (kernel arguments or a slot record);
// its accessors read them where they are used, so the compiler can reload
// them from memory instead of holding every one in scalar registers.
struct LatView {
  const LatArgs& a;
  __device__ const Geo& g() const { return a.g; }
  __device__ uint32_t mnx() const { return a.mnx; }
  __device__ uint32_t mny() const { return a.mny; }
  __device__ const void* fin() const { return a.fin; }
  __device__ void* fout() const { return a.fout; }
  __device__ void* FA() const { return a.FA; }
  __device__ void* FB() const { return a.FB; }
  __device__ uint64_t* mask() const { return a.mask; }
  __device__ double F(int c) const { return c == 0 ? a.Fx : (c == 1 ? a.Fy : a.Fz); }
  __device__ double rho0() const { return a.rho0; }
  __device__ float scale() const { return a.scale; }
  __device__ float inv() const { return a.inv; }
  __device__ double omp() const { return a.omp; }
  __device__ double omm() const { return a.omm; }
  __device__ double uin(int c) const { return a.uin[c]; }
  __device__ const double* cm() const { return a.cm; }
  __device__ const float* cmf() const { return a.cmf; }
  __device__ bool ib_copy() const { return a.ib_copy != 0; }
  __device__ bool clear_mask() const { return a.clear_mask != 0; }
  __device__ void* sigma() const { return a.sigma; }
  __device__ double sp() const { return a.sp; }
  template <typename R>
  __device__ void noise(PassK<R>& k) const {
    k.ap = R(a.ap);
    k.am = R(a.am);
    k.k0 = a.key0;
    k.k1 = a.key1;
    k.t0 = a.t0;
    k.t1 = a.t1;
  }
  template <typename R>
  __device__ void mrt(PassK<R>& k) const {
    for (int c = 0; c < 6; ++c) {
      k.lg[c] = R(a.lg[c]);
      k.ag[c] = R(a.ag[c]);
    }
  }
};

struct SlotView {
  const EnsSlot& s;
  __device__ const Geo& g() const { return s.g; }
  __device__ uint32_t mnx() const { return s.mnx; }
  __device__ uint32_t mny() const { return s.mny; }
  __device__ const void* fin() const { return s.f[s.cur]; }
  __device__ void* fout() const { return s.f[1 - s.cur]; }
  __device__ void* FA() const { return s.FA; }
  __device__ void* FB() const { return s.FB; }
  __device__ uint64_t* mask() const { return s.mask; }
  __device__ double F(int c) const {
    return (1 + s.pend) * (c == 0 ? s.fx : (c == 1 ? s.fy : s.fz));
  }
  __device__ double rho0() const { return s.rho0; }
  __device__ float scale() const { return s.scale; }
  __device__ float inv() const { return s.inv; }
  __device__ double omp() const { return s.omp; }
  __device__ double omm() const { return s.omm; }
  __device__ double uin(int c) const { return s.uref[c]; }
  __device__ const double* cm() const { return s.cm; }
  __device__ const float* cmf() const { return s.cmf; }
  __device__ bool ib_copy() const { return false; }
  __device__ bool clear_mask() const { return s.steps_done % kMaskKeep == 0; }
  __device__ void* sigma() const { return nullptr; }
  __device__ double sp() const { return 0.0; }
  template <typename R>
  __device__ void noise(PassK<R>&) const {}  // ensemble members are deterministic
  template <typename R>
  __device__ void mrt(PassK<R>&) const {}  // ... and use the two-rate collision
};

template <int S, bool CM, bool WALL, class V, bool NS = false, bool MRT = false, bool SG = false,
          int CP = kStream, bool BIG = false>
__device__ __forceinline__ void linear_site(const V& v, uint32_t s) {
  using St = Store<S>;
  using T = typename St::T;
  using R = typename St::R;
  const Geo& g = v.g();
  if (s >= (uint32_t)g.N) return;
  const uint32_t nx = (uint32_t)g.nx, ny = (uint32_t)g.ny, nz = (uint32_t)g.nz;
  const size_t P = (size_t)g.ps;  // population stride
  uint32_t x, y;
  const uint32_t r = div_rem(s, nx, v.mnx(), x);
  const uint32_t z = div_rem(r, ny, v.mny(), y);
  uint64_t* mp = v.mask() + (s >> 6);
  const uint64_t word = *mp;
  R f[Q];
  // byte offsets inside a population array: 32 bits unless it is BIG (4 GiB or
  // more); the neighbours' as periodic steps from the site's own, which wrap
  // around in the offset type
  using Off = std::conditional_t<BIG, size_t, uint32_t>;
  const Off ob = (Off)s * (Off)sizeof(T);
  const Off bx = sizeof(T), by = (Off)nx * bx, bz = (Off)ny * by;
  const Off dx[3] = {x == 0 ? (Off)(nx - 1) * bx : (Off)0 - bx, 0,
                     x == nx - 1 ? (Off)0 - (Off)(nx - 1) * bx : bx};
  const Off dy[3] = {y == 0 ? (Off)(ny - 1) * by : (Off)0 - by, 0,
                     y == ny - 1 ? (Off)0 - (Off)(ny - 1) * by : by};
  const Off dz[3] = {z == 0 ? (Off)(nz - 1) * bz : (Off)0 - bz, 0,
                     z == nz - 1 ? (Off)0 - (Off)(nz - 1) * bz : bz};
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const Off off = ob + dx[1 - CX[i]] + dy[1 - CY[i]] + dz[1 - CZ[i]];
    gptr<const typename St::B> src;
    if (WALL && CY[i] != 0) {  // halfway bounce-back: opposite population, same site (per lane)
      const bool bb = y == (CY[i] == 1 ? 0 : ny - 1);
      src = at_bytes((gptr<const typename St::B>)(uint64_t)v.fin(),
                     (size_t)(bb ? OPP[i] : i) * P * sizeof(T) + (bb ? ob : off));
    } else {
      src = at_bytes(uniform_base<const typename St::B>(v.fin(), (size_t)i * P * sizeof(T)), off);
    }
    f[i] = ld_pop<S, CP == kKeepWritten>(src);
  }
  R Fx = R(v.F(0)), Fy = R(v.F(1)), Fz = R(v.F(2));
  if (word) {  // a 64-aligned group of 64 lanes owns this mask word
    if (v.ib_copy())
      take_forces_ib<S>(word, mp, s, s & 63, v.FA(), v.FB(), Fx, Fy, Fz);
    else
      take_forces<S, false>(word, mp, s, s & 63, v.FA(), v.FB(), nullptr, 0, v.clear_mask(), Fx, Fy, Fz);
  }
  PassK<R> k;
  k.rho0 = R(v.rho0());
  k.sc = R(v.scale());
  k.inv = R(v.inv());
  k.hp = R(0.5) * R(v.omp());
  k.hm = R(0.5) * R(v.omm());
  if (CM) {
    for (int c = 0; c < 3; ++c) k.ui[c] = R(v.uin(c));
  }
  k.cm = pick_terms<R>(v.cm(), v.cmf());
  if (NS) v.noise(k);
  if (MRT) {
    v.mrt(k);
    fused_site_mrt<S, NS, CP>(f, Fx, Fy, Fz, k, v.fout(), P, ob, s);
  } else {
    fused_site<S, CM, NS, SG, CP>(f, Fx, Fy, Fz, k, v.fout(), P, ob, s, (R*)v.sigma(),
                                  (size_t)g.N, R(v.sp()));
  }
}

#define LBC_STORAGE_SWITCH(S, CALL)                                 \
  switch (S) {                                                      \
    case LB_F64: { constexpr int SS = LB_F64; CALL; } break;        \
    case LB_F32: { constexpr int SS = LB_F32; CALL; } break;        \
    case LB_F16: { constexpr int SS = LB_F16; CALL; } break;        \
    default: { constexpr int SS = LB_BF16; CALL; } break;           \
  }

// The cache policies other than streaming exist for the passes that
// set_cache_policy gives them to.
template <bool CM, bool WALL, bool NS = false, bool MRT = false, bool SG = false, class Launch>
void select_cache(int storage, const LatArgs& a, const Launch& l) {
  if constexpr (!CM && !SG) {
    if (a.cache == kResident) {
      LBC_STORAGE_SWITCH(storage, (l.template go<SS, CM, WALL, NS, MRT, SG, kResident>()));
      return;
    }
    if constexpr (!NS) {
      if (a.cache == kKeepWritten) {
        if (storage == LB_F64)
          l.template go<LB_F64, CM, WALL, NS, MRT, SG, kKeepWritten>();
        else
          l.template go<LB_F32, CM, WALL, NS, MRT, SG, kKeepWritten>();
        return;
      }
    }
  }
  LBC_STORAGE_SWITCH(storage, (l.template go<SS, CM, WALL, NS, MRT, SG, kStream>()));
}

// BGK and the two-rate collision share one kernel (BGK: equal rates); the
// comoving storage frame is a compile-time switch so that the rest frame
// carries none of its arithmetic.  l.go<S, CM, WALL, NS, MRT, SG, CP>() launches
// a variant.
template <class Launch>
void select_pass(int storage, bool comoving, const LatArgs& a, const Launch& l) {
  if (a.mrt) {  // general MRT (not with the comoving frame), with or without noise
    if (a.noise) {
      if (a.g.wall) select_cache<false, true, true, true>(storage, a, l);
      else select_cache<false, false, true, true>(storage, a, l);
    } else {
      if (a.g.wall) select_cache<false, true, false, true>(storage, a, l);
      else select_cache<false, false, false, true>(storage, a, l);
    }
  } else if (a.noise) {  // fluctuating collision (the comoving frame is not combined with it)
    if (a.g.wall) select_cache<false, true, true>(storage, a, l);
    else select_cache<false, false, true>(storage, a, l);
  } else if (a.sigma) {  // the viscous stress of the state the pass starts from, written out
    if (comoving) {
      if (a.g.wall) select_cache<true, true, false, false, true>(storage, a, l);
      else select_cache<true, false, false, false, true>(storage, a, l);
    } else {
      if (a.g.wall) select_cache<false, true, false, false, true>(storage, a, l);
      else select_cache<false, false, false, false, true>(storage, a, l);
    }
  } else if (comoving) {
    if (a.g.wall) select_cache<true, true>(storage, a, l);
    else select_cache<true, false>(storage, a, l);
  } else {
    if (a.g.wall) select_cache<false, true>(storage, a, l);
    else select_cache<false, false>(storage, a, l);
  }
}

}  // namespace lbc
