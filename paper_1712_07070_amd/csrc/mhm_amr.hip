// The MHM step of an AMR level read from its own storage (hydro_amr_advance):
// a group's cells and its siblings' from the level's states through the
// lattice map, the cells where no sibling is from a padded block in which
// only those are filled (amr.hip: amr_fill_open).  The padded form wrote and
// read back every group's 22^3 block for each substep; here only the groups
// at a coarse-fine interface touch theirs.

#include "mhm_group.h"

namespace gh {

namespace {

// ff_all: face fluxes of every group (a level with a finer one), else only of
// groups with an open side (the flux registers read no others).
template <typename T, class Z>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void mhm_amr_kernel(
    const T* __restrict__ U, T* __restrict__ Uout, AmrLevelArgs F, const T* __restrict__ pad, int gh, AmrBc bc,
    Gas<T> gas, int first_order, int ws, int* __restrict__ n_bad, T* __restrict__ face_flux, int ff_all, int segs) {
  __shared__ Smem<T> sm;
  __shared__ int sib[27];
  __shared__ T stage[kFluxStage];
  const int64_t n = F.G * segs, per = (n + 7) / 8;
  const int64_t w = (blockIdx.x & 7) * per + (blockIdx.x >> 3);  // each XCD sweeps a contiguous range of groups
  if (w >= n) return;
  const int64_t g = w / segs;
  const int p0 = F.pos[3 * g], p1 = F.pos[3 * g + 1], p2 = F.pos[3 * g + 2];
  if (threadIdx.x < 27) sib[threadIdx.x] = amr_sibling(F, bc, p0, p1, p2, int(threadIdx.x));
  __syncthreads();
  const int P = 16 + 2 * gh;
  const AmrSource<T> src{U, pad + g * 5 * int64_t(P) * P * P, sib, __builtin_amdgcn_readfirstlane(sib[4]),
                         __builtin_amdgcn_readfirstlane(sib[13]), __builtin_amdgcn_readfirstlane(sib[22]), P, gh,
                         amr_outflow_faces(F, bc, p0, p1, p2)};
  const bool open_side = sib[4] < 0 || sib[22] < 0 || sib[10] < 0 || sib[16] < 0 || sib[12] < 0 || sib[14] < 0;
  T* ff = (ff_all || __builtin_amdgcn_readfirstlane(int(open_side))) ? face_flux + g * 9 * 5 * 256 : nullptr;
  Z zr;
  if constexpr (std::is_same<Z, ZPart>::value) {
    zr.lo = int(w % segs) * (16 / segs);
    zr.hi = zr.lo + 16 / segs;
  }
  const int bad = process_group<T, false>(src, Uout + g * 5 * 4096, gas, first_order, ws, sm, nullptr, 0.0,
                                          threadIdx.x, ff, nullptr, DefaultScheme(), zr, stage);
  if (n_bad != nullptr && bad != 0) atomicAdd(n_bad, bad);
}

}  // namespace

template <typename T>
hipError_t launch_mhm_amr(const T* U, T* U_out, const AmrLevelArgs& F, const T* pad, int ghost, const int bc[6],
                          const Gas<T>& gas, int first_order, int ws, int* n_bad, T* face_flux, int ff_all,
                          hipStream_t stream) {
  if (F.G == 0) return hipSuccess;
  const int segs = plm_segments<T>(F.G, false);
  const int64_t blocks = (F.G * segs + 7) / 8 * 8;
  if (blocks > (int64_t(1) << 31) - 1) return hipErrorInvalidValue;
  AmrBc b;
  for (int i = 0; i < 6; ++i) b.v[i] = bc[i];
  if (segs > 1)
    hipLaunchKernelGGL((mhm_amr_kernel<T, ZPart>), dim3(unsigned(blocks)), dim3(kThreads), 0, stream, U, U_out, F, pad,
                       ghost, b, gas, first_order, ws, n_bad, face_flux, ff_all, segs);
  else
    hipLaunchKernelGGL((mhm_amr_kernel<T, ZAll>), dim3(unsigned(blocks)), dim3(kThreads), 0, stream, U, U_out, F, pad,
                       ghost, b, gas, first_order, ws, n_bad, face_flux, ff_all, 1);
  return hipGetLastError();
}

template hipError_t launch_mhm_amr<double>(const double*, double*, const AmrLevelArgs&, const double*, int, const int*,
                                           const Gas<double>&, int, int, int*, double*, int, hipStream_t);
template hipError_t launch_mhm_amr<float>(const float*, float*, const AmrLevelArgs&, const float*, int, const int*,
                                          const Gas<float>&, int, int, int*, float*, int, hipStream_t);

}  // namespace gh
