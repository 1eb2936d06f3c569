// lbc_lattice.hip -- the fused lattice pass of the split-forcing lattice
// Boltzmann step (Schiller, arXiv:1406.2211) on row-mapped boxes.
//
// Lattice state between steps: post-collision populations f* (deviation from
// w rho0, structure of arrays [19][nz][ny][nx]), a pending second half force
// FB (per-site vector, nonzero only at sites flagged in a per-site bit mask)
// and a flag telling whether the body force's second half is pending.  The
// physical populations at a step boundary are S f* shifted by the equilibrium
// difference of that pending half force (Sec. 3.3: a midpoint half force is an
// exact equilibrium shift).
#include "lbc_particles.h"
#include "lbc_pass.h"

namespace lbc {

// ======================================================================
// Fused lattice pass: pull (streaming S, Sec. 3.1), moments, both pending
// half forces as one equilibrium shift (F^1/2 of the previous step and of
// this step, Sec. 3.3), collision C (Eq. collision-operator / Eq. mrt-coll),
// store.  One work-item per site; a 64-wide wavefront covers 64 consecutive
// x sites of one row, i.e. exactly one 64-bit word of the force mask.
// ======================================================================
//
// Addressing: a block covers (part of) one x row, so the y and z of the nine
// source rows are block-uniform and the row pointers of every population live in
// scalar registers; a work-item adds one of three 32-bit byte offsets (x - 1, x,
// x + 1), without vector address arithmetic.
// All 19 loads are issued before any arithmetic.  With y walls the
// bounce-back choice is also block-uniform (it depends on y only).

template <int S, bool CM, bool WALL, bool NS = false, bool MRT = false, bool SG = false,
          int CP = kStream>
__global__ __launch_bounds__(256) void k_stream_collide(LatArgs a) {
  using St = Store<S>;
  using T = typename St::T;
  using R = typename St::R;
  // Intrinsic-force sub-steps (workgroup-uniform branch).
  if (a.bond_groups > 0 && blockIdx.z == 0) {
    const int grp = (int)(blockIdx.y * gridDim.x + blockIdx.x);
    if (grp < a.bond_groups) {
      extern __shared__ double bond_lds[];
      bond_group(a.bond, grp, 1, 0, a.bond_nsub, a.bond_dt, bond_lds);
    }
    return;
  }
  const uint32_t nx = (uint32_t)a.g.nx, ny = (uint32_t)a.g.ny, nz = (uint32_t)a.g.nz;
  const uint32_t x = blockIdx.x * blockDim.x + threadIdx.x;
  uint32_t y = blockIdx.y, z = blockIdx.z - (a.bond_groups > 0 ? 1u : 0u);
  if (a.reverse) {
    y = ny - 1 - y;
    z = nz - 1 - z;
  }
  if (x >= nx) return;
  const uint32_t ys[3] = {y == 0 ? ny - 1 : y - 1, y, y == ny - 1 ? 0 : y + 1};
  const uint32_t zs[3] = {z == 0 ? nz - 1 : z - 1, z, z == nz - 1 ? 0 : z + 1};
  const uint32_t xs[3] = {x == 0 ? nx - 1 : x - 1, x, x == nx - 1 ? 0 : x + 1};
  const uint32_t own = (z * ny + y) * nx + x;
  const size_t N = (size_t)a.g.ps;  // population stride
  uint64_t* mp = a.mask + ((size_t)z * ny + y) * a.g.wpr + (x >> 6);
  const uint64_t word = *mp;
  R f[Q];
  const uint32_t xb[3] = {xs[0] * (uint32_t)sizeof(T), x * (uint32_t)sizeof(T),
                          xs[2] * (uint32_t)sizeof(T)};
  const size_t row0 = ((size_t)z * ny + y) * nx;
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    // source of population i: x - c_i
    size_t base = (size_t)i * N + ((size_t)zs[1 - CZ[i]] * ny + ys[1 - CY[i]]) * nx;
    uint32_t off = xb[1 - CX[i]];
    if (WALL && ((CY[i] == 1 && y == 0) || (CY[i] == -1 && y == ny - 1))) {
      base = (size_t)OPP[i] * N + row0;  // halfway bounce-back: opposite population, same site
      off = xb[1];
    }
    // non-temporal loads measured faster for the FP32 pass (256^3: 441 -> 432 us)
    // and slower for 16-bit storage and with thermal noise
    constexpr bool nt = CP == kKeepWritten || (CP == kStream && S == LB_F32 && !NS);
    f[i] = ld_pop<S, nt>(at_bytes(uniform_base<const typename St::B>(a.fin, base * sizeof(T)), off));
  }
  R Fx = R(a.Fx), Fy = R(a.Fy), Fz = R(a.Fz);
  if (word) {
    if (a.ib_copy)
      take_forces_ib<S>(word, mp, own, x & 63, a.FA, a.FB, Fx, Fy, Fz);
    else
      take_forces<S, true>(word, mp, own, x & 63, a.FA, a.FB, a.G, a.ng, a.clear_mask != 0, Fx, Fy, Fz);
  }
  PassK<R> k;
  k.rho0 = R(a.rho0);
  k.sc = R(a.scale);
  k.inv = R(a.inv);
  k.hp = R(0.5) * R(a.omp);
  k.hm = R(0.5) * R(a.omm);
  for (int c = 0; c < 3; ++c) k.ui[c] = R(a.uin[c]);
  k.cm = pick_terms<R>(a.cm, a.cmf);
  if (NS) {
    k.ap = R(a.ap);
    k.am = R(a.am);
    k.k0 = a.key0;
    k.k1 = a.key1;
    k.t0 = a.t0;
    k.t1 = a.t1;
  }
  if (MRT) {
    for (int c = 0; c < 6; ++c) {
      k.lg[c] = R(a.lg[c]);
      k.ag[c] = R(a.ag[c]);
    }
    fused_site_mrt<S, NS, CP>(f, Fx, Fy, Fz, k, (T*)a.fout + row0, N, xb[1], own);
  } else {
    fused_site<S, CM, NS, SG, CP>(f, Fx, Fy, Fz, k, (T*)a.fout + row0, N, xb[1], own, (R*)a.sigma,
                                  (size_t)a.g.N, R(a.sp));
  }
}

namespace {
struct RowLaunch {
  const LatArgs& a;
  dim3 grid, block;
  hipStream_t st;
  template <int S, bool CM, bool WALL, bool NS, bool MRT, bool SG, int CP>
  void go() const {
    k_stream_collide<S, CM, WALL, NS, MRT, SG, CP><<<grid, block, a.occ_lds, st>>>(a);
  }
};
}  // namespace

hipError_t launch_stream_collide(int storage, bool comoving, const LatArgs& a, hipStream_t st) {
  if (a.bond_groups > 0 && a.occ_lds < a.bond_cap * 3 * (int)sizeof(double))
    return hipErrorInvalidValue;
  if (a.g.wpr == 0) return launch_stream_collide_lin(storage, comoving, a, st);
  const dim3 b = lattice_block(a.g);
  dim3 gr = lattice_grid(a.g, b);
  if (a.bond_groups > 0) {  // one more z slab of workgroups in front runs the bond groups
    if ((unsigned)a.bond_groups > gr.x * gr.y || a.bond_cap > (int)b.x) return hipErrorInvalidValue;
    gr.z += 1;
  }
  select_pass(storage, comoving, a, RowLaunch{a, gr, b, st});
  return hipGetLastError();
}

}  // namespace lbc
