// The MHM step of an AMR level read from its own storage (hydro_amr_advance):
// a group's cells and its siblings' from the level's states through the
// lattice map, the cells where no sibling is from scratch cells around the group
// of which only those are filled (amr.hip: amr_fill_open).  The padded form wrote and
// read back every group's 22^3 block for each substep; here only the groups
// at a coarse-fine interface touch theirs.

#include "mhm_group.h"

namespace gh {

namespace {

// Does a flux register read faces of plane k (at 8 k) of axis d of the group at
// p?  Those of a side that no sibling shares, and those with a patch of the
// finer level (N; N.map null: none) on one side only (here: the pair of patches
// i, of four).  One lane per pair: the look-ups are all in flight together
// while the siblings' are.  Writing every plane of every group of a level with a
// finer one took the coupled blast hierarchy 5.03 ms per coarse step, these 4.94
// (a march without the flux code 4.51).
__device__ __forceinline__ bool amr_flux_read(const AmrLevelArgs& F, const AmrLevelArgs& N, const AmrBc& bc, int p0,
                                              int p1, int p2, int d, int k, int i) {
  const int step = d == 0 ? 1 : d == 1 ? 3 : 9;
  bool read = false;
  if (k != 1) {
    const int p = (d == 0 ? p0 : d == 1 ? p1 : p2) + k - 1, n = F.n[d];
    const bool domain_end = (p < 0 && bc.v[2 * d] != 0) || (p >= n && bc.v[2 * d + 1] != 0);
    read = !domain_end && amr_sibling(F, bc, p0, p1, p2, 13 + (k - 1) * step) < 0;
  }
  if (N.map == nullptr) return read;
  const int a = i & 1, b = i >> 1;
  const int x = 2 * p0 + (d == 0 ? k : a), y = 2 * p1 + (d == 1 ? k : d == 0 ? a : b), z = 2 * p2 + (d == 2 ? k : b);
  const int below = amr_sibling(N, bc, x, y, z, 13 - step), above = amr_sibling(N, bc, x, y, z, 13);
  return read || (below < 0) != (above < 0);
}

template <typename T, class Z>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2))) void mhm_amr_kernel(
    const T* __restrict__ U, T* __restrict__ Uout, AmrLevelArgs F, const T* __restrict__ shell, AmrBc bc,
    Gas<T> gas, int first_order, int ws, int* __restrict__ n_bad, T* __restrict__ face_flux, AmrLevelArgs N, int segs) {
  __shared__ Smem<T> sm;
  __shared__ int sib[27];
  __shared__ unsigned planes;
  __shared__ T stage[kFluxStage];
  const int64_t n = F.G * segs, per = (n + 7) / 8;
  const int64_t w = (blockIdx.x & 7) * per + (blockIdx.x >> 3);  // each XCD sweeps a contiguous range of groups
  if (w >= n) return;
  const int64_t g = w / segs;
  const int p0 = F.pos[3 * g], p1 = F.pos[3 * g + 1], p2 = F.pos[3 * g + 2];
  if (threadIdx.x < 27) sib[threadIdx.x] = amr_sibling(F, bc, p0, p1, p2, int(threadIdx.x));
  if (threadIdx.x >= 64 && threadIdx.x < 128) {
    const int t = int(threadIdx.x) - 64;
    const unsigned long long b = __ballot(t < 36 && amr_flux_read(F, N, bc, p0, p1, p2, t / 12, (t / 4) % 3, t & 3));
    unsigned m = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) m |= ((b >> (4 * i)) & 15u) != 0 ? 1u << i : 0u;
    if (t == 0) planes = m;
  }
  __syncthreads();
  const AmrSource<T> src{U, shell + g * 5 * kShellCells, sib, __builtin_amdgcn_readfirstlane(sib[4]),
                         __builtin_amdgcn_readfirstlane(sib[13]), __builtin_amdgcn_readfirstlane(sib[22]),
                         amr_outflow_faces(F, bc, p0, p1, p2)};
  const unsigned ff_planes = __builtin_amdgcn_readfirstlane(planes);
  T* ff = ff_planes != 0 ? face_flux + g * 9 * 5 * 256 : nullptr;
  Z zr;
  if constexpr (std::is_same<Z, ZPart>::value) {
    zr.lo = int(w % segs) * (16 / segs);
    zr.hi = zr.lo + 16 / segs;
  }
  const int bad = process_group<T, false>(src, Uout + g * 5 * 4096, gas, first_order, ws, sm, nullptr, 0.0,
                                          threadIdx.x, ff, nullptr, DefaultScheme(), zr, stage, ff_planes);
  if (n_bad != nullptr && bad != 0) atomicAdd(n_bad, bad);
}

}  // namespace

template <typename T>
hipError_t launch_mhm_amr(const T* U, T* U_out, const AmrLevelArgs& F, const T* shell, const int bc[6],
                          const Gas<T>& gas, int first_order, int ws, int* n_bad, T* face_flux,
                          const AmrLevelArgs& N,
                          hipStream_t stream) {
  if (F.G == 0) return hipSuccess;
  const int segs = plm_segments<T>(F.G, false);
  const int64_t blocks = (F.G * segs + 7) / 8 * 8;
  if (blocks > (int64_t(1) << 31) - 1) return hipErrorInvalidValue;
  AmrBc b;
  for (int i = 0; i < 6; ++i) b.v[i] = bc[i];
  if (segs > 1)
    hipLaunchKernelGGL((mhm_amr_kernel<T, ZPart>), dim3(unsigned(blocks)), dim3(kThreads), 0, stream, U, U_out, F, shell,
                       b, gas, first_order, ws, n_bad, face_flux, N, segs);
  else
    hipLaunchKernelGGL((mhm_amr_kernel<T, ZAll>), dim3(unsigned(blocks)), dim3(kThreads), 0, stream, U, U_out, F, shell,
                       b, gas, first_order, ws, n_bad, face_flux, N, 1);
  return hipGetLastError();
}

template hipError_t launch_mhm_amr<double>(const double*, double*, const AmrLevelArgs&, const double*, const int*,
                                           const Gas<double>&, int, int, int*, double*,
                                           const AmrLevelArgs&, hipStream_t);
template hipError_t launch_mhm_amr<float>(const float*, float*, const AmrLevelArgs&, const float*, const int*,
                                          const Gas<float>&, int, int, int*, float*,
                                          const AmrLevelArgs&, hipStream_t);

}  // namespace gh
