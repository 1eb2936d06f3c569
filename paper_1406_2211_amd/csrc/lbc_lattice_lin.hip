// lbc_lattice_lin.hip -- the fused lattice pass over linear site indices, for
// boxes whose x extent is not a multiple of 64.
#include "lbc_particles.h"
#include "lbc_pass.h"

namespace lbc {

template <int S, bool CM, bool WALL, bool NS, bool MRT, bool SG, int CP, bool BIG>
__global__ __launch_bounds__(256) void k_stream_collide_lin(LatArgs a) {
  uint32_t b = blockIdx.x;
  if (a.bond_groups > 0) {  // the first bond_groups workgroups run the intrinsic-force sub-steps
    if (b < (uint32_t)a.bond_groups) {
      extern __shared__ double bond_lds[];
      bond_group(a.bond, (int)b, 1, 0, a.bond_nsub, a.bond_dt, bond_lds);
      return;
    }
    b -= (uint32_t)a.bond_groups;
  }
  if (a.reverse) b = gridDim.x - (uint32_t)a.bond_groups - 1u - b;
  linear_site<S, CM, WALL, LatView, NS, MRT, SG, CP, BIG>(LatView{a}, b * 256u + threadIdx.x);
}

namespace {
struct LinLaunch {
  const LatArgs& a;
  unsigned blocks;
  bool big;
  hipStream_t st;
  template <int S, bool CM, bool WALL, bool NS, bool MRT, bool SG, int CP>
  void go() const {
    if constexpr (CP == kStream) {  // (a box with a cache policy is far smaller)
      if (big) {
        k_stream_collide_lin<S, CM, WALL, NS, MRT, SG, CP, true>
            <<<blocks, 256, a.occ_lds, st>>>(a);
        return;
      }
    }
    k_stream_collide_lin<S, CM, WALL, NS, MRT, SG, CP, false><<<blocks, 256, a.occ_lds, st>>>(a);
  }
};
}  // namespace

hipError_t launch_stream_collide_lin(int storage, bool comoving, const LatArgs& a,
                                     hipStream_t st) {
  // the bond groups run in bond_groups workgroups in front
  if (a.bond_groups > 0 && a.bond_cap > 256) return hipErrorInvalidValue;
  const unsigned nb = (unsigned)((a.g.N + 255) / 256) + (unsigned)a.bond_groups;
  select_pass(storage, comoving, a, LinLaunch{a, nb, big_box(a.g, storage), st});
  return hipGetLastError();
}

}  // namespace lbc
