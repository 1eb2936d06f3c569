// lbc_ensemble.hip -- the batched step of an ensemble of boxes.
#include "lbc_pass.h"
#include "lbc_particles.h"

namespace lbc {

// ======================================================================
// Batched ensemble step: many periodic boxes of different sizes advance
// together.  Every kernel is a persistent grid that strides over a flat work
// list: (slot, 256-site chunk) for the lattice, (slot, particle group) for
// the coupling halves.  A slot takes part while steps_done < steps_target;
// the per-slot state (ping-pong buffer, pending body-force half, step count)
// lives on the device, so a captured graph of steps stays valid while slots
// are admitted and retired.
// ======================================================================
__device__ __forceinline__ bool ens_active(const EnsSlot& s) {
  return s.live && s.steps_done < s.steps_target;
}

// The slot table is read-only during the lattice pass (only k_ens_advance
// writes it); with restrict-qualified arguments its fields are scalar loads.
template <int S, bool CM, bool BIG>
__device__ __forceinline__ void ens_lattice_item(const EnsSlot& sl, uint32_t chunk) {
  linear_site<S, CM, false, SlotView, false, false, false, kStream, BIG>(
      SlotView{sl}, chunk * 256u + threadIdx.x);
}

template <int S, bool BIG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(S == LB_F64 ? 4 : 8))) void k_ens_lattice(const EnsSlot* __restrict__ slots,
                                                     const int2* __restrict__ items,
                                                     const int* __restrict__ nitems) {
  const int n = *nitems;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const int2 w = items[it];
    const EnsSlot& sl = slots[w.x];
    if (!ens_active(sl)) continue;
    if (sl.comoving)
      ens_lattice_item<S, true, BIG>(sl, (uint32_t)w.y);
    else
      ens_lattice_item<S, false, BIG>(sl, (uint32_t)w.y);
  }
}

// half 0: P^1/2 then the first coupling half (physical u, spread into FA);
// half 1: the second coupling half (post-stream u, spread into FB), then P^1/2.
// The slot table and the work list are read-only here, as in k_ens_lattice.
template <int S, int K>
__global__ __launch_bounds__(256) void k_ens_couple(const EnsSlot* __restrict__ slots,
                                                    const int2* __restrict__ items,
                                                    const int* __restrict__ nitems, int half) {
  using E = typename Store<S>::R;
  constexpr int L = Lanes<K>::L;
  const int n = *nitems;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const int2 w = items[it];
    const EnsSlot& sl = slots[w.x];
    if (!ens_active(sl) || sl.coupling == LB_COUPLE_NONE) continue;
    const int lane = threadIdx.x % L;
    if ((long long)w.y + (threadIdx.x & ~63u) / L >= sl.np) continue;  // a whole wavefront
    const bool live = (long long)w.y + threadIdx.x / L < sl.np;  // as in k_couple_half
    const long long p = live ? (long long)w.y + threadIdx.x / L : sl.np - 1;
    PartArgs a;
    a.s.g = sl.g;
    a.s.f = half == 0 ? sl.f[sl.cur] : sl.f[1 - sl.cur];
    a.s.FB = sl.FB;
    a.s.mask = sl.mask;
    a.s.rho0 = sl.rho0;
    a.s.pfx = sl.pend * sl.fx;
    a.s.pfy = sl.pend * sl.fy;
    a.s.pfz = sl.pend * sl.fz;
    a.s.inv = sl.inv;
    for (int k = 0; k < 3; ++k) {  // reference of the buffer read (the new one in half 1)
      const double fk = k == 0 ? sl.fx : (k == 1 ? sl.fy : sl.fz);
      a.s.uref[k] = sl.comoving ? sl.uref[k] + (half == 1 ? fk / sl.rho0 : 0.0) : 0.0;
    }
    a.FA = sl.FA;
    a.FB = sl.FB;
    a.mask = sl.mask;
    a.K = K;
    a.mcache = sl.mcache;
    a.mbase = sl.mbase;
    a.cache_use = half == 0 ? sl.mvalid : 0;
    a.cache_fill = half == 1 ? 1 : 0;
    a.fa_rd = 0;
    const double hh = 0.5;
    double r[3], v[3];
    for (int k = 0; k < 3; ++k) {
      r[k] = sl.pos[3 * p + k];
      v[k] = sl.vel[3 * p + k];
    }
    if (half == 0) {
      for (int k = 0; k < 3; ++k) r[k] += hh * v[k];
      wrap3(sl.g, r);
    }
    const uint64_t mpre = mask_preload<K>(a, r, lane);
    const double m = sl.mass[p];
    double rp, up[3];
    group_interp<S, K>(a, r, half == 0, lane, rp, up, p);
    a.coupling = sl.coupling;
    a.gamma = sl.gamma;
    a.hh = hh;
    a.kT = 0.0;
    a.fext[0] = sl.fx;
    a.fext[1] = sl.fy;
    a.fext[2] = sl.fz;
    const double Fi[3] = {0, 0, 0};
    double Fh[3];
    couple_update(a, p, m, rp, up, Fi, v, Fh);
    const double Ff[3] = {-Fh[0], -Fh[1], -Fh[2]};
    if (sl.det_on) {  // stored; k_ens_spread_det spreads it (and drifts after half 1)
      if (live && lane == 0)
        for (int k = 0; k < 3; ++k) sl.aux[3 * p + k] = Ff[k];
    } else {
      group_spread<E, K>(a, r, Ff, half == 0 ? sl.FA : sl.FB, lane, live, &mpre);
    }
    if (live && lane == 0) {
      if (half == 1 && !sl.det_on) {
        for (int k = 0; k < 3; ++k) r[k] += hh * v[k];
        wrap3(sl.g, r);
      }
      for (int k = 0; k < 3; ++k) {
        sl.pos[3 * p + k] = r[k];
        sl.vel[3 * p + k] = v[k];
      }
    }
  }
}

// Deterministic spreading of the stored lattice forces of one coupling half
// of every deterministic slot (fixed-point accumulation, see k_spread_det),
// then the final P^1/2 after half 1.
template <int K>
__global__ __launch_bounds__(256) void k_ens_spread_det(EnsArgs e, int half) {
  constexpr int L = Lanes<K>::L;
  const int n = *e.npitems;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const int2 w = e.pitems[it];
    const EnsSlot& sl = e.slots[w.x];
    if (!ens_active(sl) || sl.coupling == LB_COUPLE_NONE || !sl.det_on) continue;
    const long long p = (long long)w.y + threadIdx.x / L;
    const int lane = threadIdx.x % L;
    if (p >= sl.np) continue;  // whole lane groups leave together
    double r[3], f[3];
    for (int k = 0; k < 3; ++k) {
      r[k] = sl.pos[3 * p + k];
      f[k] = sl.aux[3 * p + k];
    }
    const SiteSlot ss = slot_of<K>(sl.g, r, lane);
    if (ss.valid) {
      const long long s = site_index(sl.g, ss.x, ss.y, ss.z);
      for (int k = 0; k < 3; ++k) {
        uint64_t lo, hi;
        to_fixed(ss.W * f[k], lo, hi);
        if (lo | hi) fixed_add(sl.det + 6 * s + 2 * k, lo, hi);
      }
      uint64_t bit;
      flag_site(mask_word(sl.mask, sl.g, ss.x, ss.y, ss.z, bit), bit);
    }
    if (lane == 0 && half == 1) {
      for (int k = 0; k < 3; ++k) r[k] += 0.5 * sl.vel[3 * p + k];
      wrap3(sl.g, r);
      for (int k = 0; k < 3; ++k) sl.pos[3 * p + k] = r[k];
    }
  }
}

// The finalize of the deterministic spread for every deterministic slot, over
// the lattice work list (one lane per site).
template <int S>
__global__ __launch_bounds__(256) void k_ens_det_finalize(EnsArgs e, int half) {
  using E = typename Store<S>::R;
  const int n = *e.nlitems;
  for (int it = blockIdx.x; it < n; it += gridDim.x) {
    const int2 w = e.litems[it];
    const EnsSlot& sl = e.slots[w.x];
    if (!ens_active(sl) || sl.coupling == LB_COUPLE_NONE || !sl.det_on || sl.np == 0) continue;
    const long long s = (long long)w.y * 256 + threadIdx.x;
    if (s < sl.g.N) det_finalize_site<E>(sl.g, sl.mask, sl.det, (E*)(half ? sl.FB : sl.FA), s);
  }
}

__global__ void k_ens_advance(EnsArgs e) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= e.nslots) return;
  EnsSlot& sl = e.slots[i];
  if (!ens_active(sl)) return;
  sl.cur = 1 - sl.cur;
  sl.pend = 1;
  sl.steps_done += 1;
  if (sl.coupling != LB_COUPLE_NONE && sl.np > 0) sl.mvalid = 1;  // filled by the second half
  if (sl.comoving) {
    sl.uref[0] += sl.fx / sl.rho0;
    sl.uref[1] += sl.fy / sl.rho0;
    sl.uref[2] += sl.fz / sl.rho0;
    const double uo[3] = {sl.uref[0] + sl.fx / sl.rho0, sl.uref[1] + sl.fy / sl.rho0,
                          sl.uref[2] + sl.fz / sl.rho0};
    comoving_terms(sl.scale, sl.rho0, sl.uref, uo, sl.cm, sl.cmf);
  }
}

hipError_t launch_ens_step(int storage, int K, const EnsArgs& e, int lat_grid, int part_grid,
                           int det, bool big, hipStream_t st) {
  for (int half = 0; half < 2; ++half) {
    if (half == 1) {
      if (big)
        LBC_STORAGE_SWITCH(storage, (k_ens_lattice<SS, true><<<lat_grid, 256, 0, st>>>(
                                        e.slots, e.litems, e.nlitems)))
      else
        LBC_STORAGE_SWITCH(storage, (k_ens_lattice<SS, false><<<lat_grid, 256, 0, st>>>(
                                        e.slots, e.litems, e.nlitems)))
    }
    LBC_KERNEL_SWITCH(K, LBC_STORAGE_SWITCH(storage, (k_ens_couple<SS, KK><<<part_grid, 256, 0, st>>>(
                                e.slots, e.pitems, e.npitems, half))));
    if (det) {
      LBC_KERNEL_SWITCH(K, (k_ens_spread_det<KK><<<part_grid, 256, 0, st>>>(e, half)));
      LBC_STORAGE_SWITCH(storage, (k_ens_det_finalize<SS><<<lat_grid, 256, 0, st>>>(e, half)));
    }
  }
  k_ens_advance<<<(e.nslots + 63) / 64, 64, 0, st>>>(e);
  return hipGetLastError();
}

}  // namespace lbc
