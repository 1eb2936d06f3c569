// lbc_sites.hip -- initialisation and read-out of the lattice state, totals,
// particle drifts and zero fills.
#include "lbc_pass.h"
#include "lbc_particles.h"

namespace lbc {

// ======================================================================
// Initialisation: physical state f = f^eq(rho, u).  Written as the pre-image
// under the pull gather (push of each population to the slot it will be
// pulled from), so that the first lattice pass sees exactly f^eq.
// ======================================================================
template <int S>
__global__ void k_init(InitArgs a) {
  using St = Store<S>;
  using T = typename St::T;
  using R = typename St::R;
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y, z = blockIdx.z;
  if (x >= a.g.nx) return;
  const long long s = site_index(a.g, x, y, z);
  const double rho = a.rho ? a.rho[s] : a.rho0;
  const double ux = a.u ? a.u[s] : 0.0, uy = a.u ? a.u[a.g.N + s] : 0.0,
               uz = a.u ? a.u[2 * a.g.N + s] : 0.0;
  const double usq = ux * ux + uy * uy + uz * uz;
  const double drho = rho - a.rho0;
  T* f = (T*)a.f;
  const int xs[3] = {x == 0 ? a.g.nx - 1 : x - 1, x, x == a.g.nx - 1 ? 0 : x + 1};
  const int ys[3] = {y == 0 ? a.g.ny - 1 : y - 1, y, y == a.g.ny - 1 ? 0 : y + 1};
  const int zs[3] = {z == 0 ? a.g.nz - 1 : z - 1, z, z == a.g.nz - 1 ? 0 : z + 1};
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const double v = feq_dev<double>(i, drho, rho, ux, uy, uz, usq);
    long long dst;  // x - c_i, or the opposite population of the same site beyond a wall
    if (CY[i] != 0 && a.g.wall && y == (CY[i] == 1 ? 0 : a.g.ny - 1))
      dst = (long long)OPP[i] * a.g.ps + s;
    else
      dst = (long long)i * a.g.ps + site_index(a.g, xs[1 - CX[i]], ys[1 - CY[i]], zs[1 - CZ[i]]);
    st_scaled<S>(f + dst, (R)v, (R)a.scale);
  }
}

template <int S>
__global__ void k_moments(SiteArgs a, double* rho, double* u) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y, z = blockIdx.z;
  if (x >= a.g.nx) return;
  double fl[Q], drho, j[3];
  const long long s = site_index(a.g, x, y, z);
  site_phys<S>(a, x, y, z, fl, drho, j, false);
  add_pending_flagged<S>(a, (uint32_t)s, j);
  const double r = a.rho0 + drho;
  if (rho) rho[s] = r;
  u[s] = j[0] / r;
  u[a.g.N + s] = j[1] / r;
  u[2 * a.g.N + s] = j[2] / r;
}

// Physical populations: the stored ones moved by the pending half force, an
// equilibrium shift f -> f + f^eq(rho, u_phys) - f^eq(rho, u).  With csc the
// non-equilibrium part f - f^eq(rho, u) is split into even and odd parts
// over opposite directions and scaled by gp, gm: the exact half collision of
// the two-rate operator (Sec. 3.2), which leaves rho and u unchanged.
template <int S>
__global__ void k_populations(SiteArgs a, double* out, double gp, double gm, int csc) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y, z = blockIdx.z;
  if (x >= a.g.nx) return;
  double fl[Q], drho, j[3], jb[3];
  const long long s = site_index(a.g, x, y, z);
  site_phys<S>(a, x, y, z, fl, drho, jb, false);
  for (int c = 0; c < 3; ++c) j[c] = jb[c];
  add_pending_flagged<S>(a, (uint32_t)s, j);
  const double r = a.rho0 + drho;
  const double ub[3] = {jb[0] / r, jb[1] / r, jb[2] / r}, up[3] = {j[0] / r, j[1] / r, j[2] / r};
  const double sb = ub[0] * ub[0] + ub[1] * ub[1] + ub[2] * ub[2];
  const double sp = up[0] * up[0] + up[1] * up[1] + up[2] * up[2];
  if (!csc) {
#pragma unroll
    for (int i = 0; i < Q; ++i)
      out[(long long)i * a.g.N + s] = fl[i] + feq_dev<double>(i, drho, r, up[0], up[1], up[2], sp) -
                                      feq_dev<double>(i, drho, r, ub[0], ub[1], ub[2], sb);
    return;
  }
  double ne[Q];
#pragma unroll
  for (int i = 0; i < Q; ++i) ne[i] = fl[i] - feq_dev<double>(i, drho, r, ub[0], ub[1], ub[2], sb);
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const double e = 0.5 * (ne[i] + ne[OPP[i]]), o = 0.5 * (ne[i] - ne[OPP[i]]);
    out[(long long)i * a.g.N + s] =
        feq_dev<double>(i, drho, r, up[0], up[1], up[2], sp) + gp * e + gm * o;
  }
}

// Local viscous stress pref * sum_i (f_i - f^eq_i(rho, u)) c_i c_i (order xx,
// yy, zz, xy, xz, yz).  The pending half force is an equilibrium shift and
// drops out, so the stored populations and their own velocity give it.
template <int S>
__global__ void k_stress(SiteArgs a, double* out, double pref, double prefb) {
  const int x = blockIdx.x * blockDim.x + threadIdx.x;
  const int y = blockIdx.y, z = blockIdx.z;
  if (x >= a.g.nx) return;
  double fl[Q], drho, j[3];
  site_phys<S>(a, x, y, z, fl, drho, j, false);
  const double r = a.rho0 + drho;
  const double u[3] = {j[0] / r, j[1] / r, j[2] / r};
  const double usq = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
  double p[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int i = 0; i < Q; ++i) {
    const double ne = fl[i] - feq_dev<double>(i, drho, r, u[0], u[1], u[2], usq);
    p[0] += ne * (CX[i] * CX[i]);
    p[1] += ne * (CY[i] * CY[i]);
    p[2] += ne * (CZ[i] * CZ[i]);
    p[3] += ne * (CX[i] * CY[i]);
    p[4] += ne * (CX[i] * CZ[i]);
    p[5] += ne * (CY[i] * CZ[i]);
  }
  const long long s = site_index(a.g, x, y, z);
  if (prefb != pref) {  // general MRT: the trace part relaxes at its own rate
    const double tr = (p[0] + p[1] + p[2]) / 3.0;
    for (int q = 0; q < 3; ++q) p[q] = pref * (p[q] - tr) + prefb * tr;
    for (int q = 3; q < 6; ++q) p[q] *= pref;
    for (int q = 0; q < 6; ++q) out[(long long)q * a.g.N + s] = p[q];
    return;
  }
#pragma unroll
  for (int q = 0; q < 6; ++q) out[(long long)q * a.g.N + s] = pref * p[q];
}

// Block reduction of 4 doubles in a fixed order (deterministic).
__device__ __forceinline__ void block_sum4(double v[4], double* lds /*[4*16]*/) {
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
#pragma unroll
  for (int k = 0; k < 4; ++k) v[k] = wave_sum(v[k]);
  if (lane == 0)
    for (int k = 0; k < 4; ++k) lds[4 * wv + k] = v[k];
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 0; k < 4; ++k) {
      double t = 0;
      for (int w = 0; w < nw; ++w) t += lds[4 * w + k];
      v[k] = t;
    }
  }
  __syncthreads();
}

template <int S>
__global__ __launch_bounds__(256) void k_totals_sites(SiteArgs a, double* partial) {
  __shared__ double lds[64];
  double v[4] = {0, 0, 0, 0};
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long s = (long long)blockIdx.x * blockDim.x + threadIdx.x; s < a.g.N; s += stride) {
    const uint32_t r = (uint32_t)s / (uint32_t)a.g.nx, z = r / (uint32_t)a.g.ny;
    const int x = (int)((uint32_t)s - r * (uint32_t)a.g.nx), y = (int)(r - z * (uint32_t)a.g.ny);
    double fl[Q], drho, j[3];
    site_phys<S>(a, x, y, (int)z, fl, drho, j, false);
    add_pending_flagged<S>(a, (uint32_t)s, j);
    v[0] += drho;
    v[1] += j[0];
    v[2] += j[1];
    v[3] += j[2];
  }
  block_sum4(v, lds);
  if (threadIdx.x == 0)
    for (int k = 0; k < 4; ++k) partial[4 * blockIdx.x + k] = v[k];
}

__global__ __launch_bounds__(256) void k_totals_final(const double* partial, int nblk,
                                                      const double* vel, const double* mass,
                                                      long long np, double* out) {
  __shared__ double lds[64];
  double v[4] = {0, 0, 0, 0};
  for (int b = threadIdx.x; b < nblk; b += blockDim.x)
    for (int k = 0; k < 4; ++k) v[k] += partial[4 * b + k];
  block_sum4(v, lds);
  if (threadIdx.x == 0)
    for (int k = 0; k < 4; ++k) out[k] = v[k];
  double p[4] = {0, 0, 0, 0};
  if (vel && mass)
    for (long long i = threadIdx.x; i < np; i += blockDim.x)
      for (int k = 0; k < 3; ++k) p[k] += mass[i] * vel[3 * i + k];
  block_sum4(p, lds);
  if (threadIdx.x == 0)
    for (int k = 0; k < 3; ++k) out[4 + k] = p[k];
}

// P^1/2: r <- r + (h/2) v, wrapped (first drift of Alg. 3).
__global__ void k_drift(Geo g, long long n, double* pos, const double* vel, double dt) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  double r[3];
  for (int k = 0; k < 3; ++k) r[k] = pos[3 * p + k] + dt * vel[3 * p + k];
  wrap3(g, r);
  for (int k = 0; k < 3; ++k) pos[3 * p + k] = r[k];
}

__global__ void k_wrap(Geo g, long long n, double* pos) {
  const long long p = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  if (p >= n) return;
  double r[3] = {pos[3 * p], pos[3 * p + 1], pos[3 * p + 2]};
  wrap3(g, r);
  for (int k = 0; k < 3; ++k) pos[3 * p + k] = r[k];
}

hipError_t launch_init(int storage, const InitArgs& a, hipStream_t st) {
  const dim3 b = lattice_block(a.g), gr = lattice_grid(a.g, b);
  LBC_STORAGE_SWITCH(storage, (k_init<SS><<<gr, b, 0, st>>>(a)));
  return hipGetLastError();
}

hipError_t launch_moments(int storage, const SiteArgs& a, double* rho, double* u, hipStream_t st) {
  const dim3 b = lattice_block(a.g), gr = lattice_grid(a.g, b);
  LBC_STORAGE_SWITCH(storage, (k_moments<SS><<<gr, b, 0, st>>>(a, rho, u)));
  return hipGetLastError();
}

hipError_t launch_populations(int storage, const SiteArgs& a, double* out, double gp, double gm,
                              hipStream_t st) {
  const dim3 b = lattice_block(a.g), gr = lattice_grid(a.g, b);
  const int csc = gp != 1.0 || gm != 1.0;
  LBC_STORAGE_SWITCH(storage, (k_populations<SS><<<gr, b, 0, st>>>(a, out, gp, gm, csc)));
  return hipGetLastError();
}

hipError_t launch_stress(int storage, const SiteArgs& a, double* out, double pref, double prefb,
                         hipStream_t st) {
  const dim3 b = lattice_block(a.g), gr = lattice_grid(a.g, b);
  LBC_STORAGE_SWITCH(storage, (k_stress<SS><<<gr, b, 0, st>>>(a, out, pref, prefb)));
  return hipGetLastError();
}

hipError_t launch_totals(int storage, const SiteArgs& a, double* partial, int nblk,
                         const double* vel, const double* mass, long long np, double* out,
                         hipStream_t st) {
  LBC_STORAGE_SWITCH(storage, (k_totals_sites<SS><<<nblk, 256, 0, st>>>(a, partial)));
  k_totals_final<<<1, 256, 0, st>>>(partial, nblk, vel, mass, np, out);
  return hipGetLastError();
}

static inline unsigned pblocks(long long n) { return (unsigned)((n + 127) / 128); }

hipError_t launch_drift(const Geo& g, long long n, double* pos, const double* vel, double dt,
                        hipStream_t st) {
  if (n > 0) k_drift<<<pblocks(n), 128, 0, st>>>(g, n, pos, vel, dt);
  return hipGetLastError();
}

hipError_t launch_wrap(const Geo& g, long long n, double* pos, hipStream_t st) {
  if (n > 0) k_wrap<<<pblocks(n), 128, 0, st>>>(g, n, pos);
  return hipGetLastError();
}

// Both particle arrays in one launch instead of two copies through the runtime
// (a 45 x 37 x 52 channel with 200 particles, stepped and read: 48.9 -> 47.2 us).
__global__ void k_copy_particles(long long m, const double* pos, const double* vel, double* d_pos,
                                 double* d_vel) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
    if (d_pos) d_pos[i] = pos[i];
    if (d_vel) d_vel[i] = vel[i];
  }
}

hipError_t launch_copy_particles(long long n, const double* pos, const double* vel, double* d_pos,
                                 double* d_vel, hipStream_t st) {
  if (n <= 0 || (!d_pos && !d_vel)) return hipSuccess;
  const long long blocks = (3 * n + 255) / 256 < 4096 ? (3 * n + 255) / 256 : 4096;
  k_copy_particles<<<(unsigned)blocks, 256, 0, st>>>(3 * n, pos, vel, d_pos, d_vel);
  return hipGetLastError();
}

// Zero fill of n 8-byte words (a kernel, so that a caller capturing the
// library's calls in a HIP graph records kernel nodes only).
__global__ void k_zero(unsigned long long* p, long long n) {
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0ull;
}

hipError_t launch_zero(void* p, size_t bytes, hipStream_t st) {
  const long long n = (long long)(bytes / 8);
  if (n <= 0) return hipSuccess;
  const long long blocks = (n + 255) / 256 < 4096 ? (n + 255) / 256 : 4096;
  k_zero<<<(unsigned)blocks, 256, 0, st>>>((unsigned long long*)p, n);
  return hipGetLastError();
}

}  // namespace lbc
