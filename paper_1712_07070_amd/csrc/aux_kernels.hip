// Ghost-zone fill (Sec. 3.4, boundary conditions of Sec. 2.2) and the
// per-patch CFL time-step (Sec. 2.6 Eq. 2) of padded patch groups.

#include "mhm_group.h"

namespace gh {

namespace {

// ------------------------------------------------------------ ghost fill --
// The source index along each axis is mapped independently (wrap for periodic
// faces, clamp for outflow faces).
__device__ __forceinline__ int bc_map(int i, int n, int lo, int hi) {
  if (i < 0) return lo == 0 ? i + n : 0;
  if (i >= n) return hi == 0 ? i - n : n - 1;
  return i;
}

struct BC6 {
  int b[6];
};

// A pair of x-adjacent cells (P is even, so a pair never straddles a row),
// stored with one 2-element access where the destination is aligned to it.
template <typename T, bool kPair>
__device__ __forceinline__ void store_pair(T* d, T a, T b) {
  if constexpr (kPair) {
    typedef T V __attribute__((ext_vector_type(2)));
    *reinterpret_cast<V*>(d) = V{a, b};
  } else {
    d[0] = a;
    d[1] = b;
  }
}

// One workgroup per padded plane of a group, all five fields: a thread maps a
// pair of x-adjacent cells to its two source columns once and moves it for
// every field, 10 independent loads in flight.  Bound by HBM traffic (104 B
// written and at least 40 B read per cell, FP64 with 3 ghosts).  Each XCD
// sweeps a contiguous range of planes, whose shared rows then mostly hit its
// L2.  256^3 FP64, fill and the step that reads it (characteristic PLM, van
// Leer / PPM): 2.008 / 6.942 ms with a workgroup per (group, field, z),
// 8-byte accesses and round-robin planes, now 1.818 / 6.653 (the fill alone
// 0.834 -> 0.64).  Four planes per workgroup: 1.896 / 6.804; with stores past
// the caches the fill alone takes 0.556, but what it saves the step loses
// (1.820 / 6.704, and 3-4% on levels that fit the last-level cache).
template <typename T, bool kPair>
__global__ __launch_bounds__(256) void fill_ghosts_kernel(const T* __restrict__ level, T* __restrict__ U_pad,
                                                          int ngx, int ngy, int ngz, int gh, unsigned int planes,
                                                          bool blocked, BC6 bc) {
  const int P = 16 + 2 * gh, H = P / 2;
  const unsigned int per = (planes + 7u) / 8u;
  const unsigned int blk = blocked ? (blockIdx.x & 7u) * per + (blockIdx.x >> 3) : blockIdx.x;
  if (blk >= planes) return;
  const int z = int(blk % unsigned(P));
  const unsigned int g = blk / unsigned(P);
  const int gx = int(g % unsigned(ngx)), gy = int((g / unsigned(ngx)) % unsigned(ngy));
  const int gz = int(g / (unsigned(ngx) * unsigned(ngy)));
  const int Nx = ngx * 16, Ny = ngy * 16, Nz = ngz * 16;
  const int Z = bc_map(gz * 16 + z - gh, Nz, bc.b[4], bc.b[5]);
  const int64_t P3 = int64_t(P) * P * P;
  T* dst = U_pad + int64_t(g) * 5 * P3 + int64_t(z) * P * P;
  const T* src = level + (Z & 15) * 256;
  for (int i = threadIdx.x; i < P * H; i += blockDim.x) {
    const int x = 2 * (i % H), y = i / H;
    const int X0 = bc_map(gx * 16 + x - gh, Nx, bc.b[0], bc.b[1]);
    const int X1 = bc_map(gx * 16 + x + 1 - gh, Nx, bc.b[0], bc.b[1]);
    const int Y = bc_map(gy * 16 + y - gh, Ny, bc.b[2], bc.b[3]);
    const int64_t row = (int64_t(Z >> 4) * ngy + (Y >> 4)) * ngx;
    const T* s0 = src + (row + (X0 >> 4)) * (5 * 4096) + (Y & 15) * 16 + (X0 & 15);
    const T* s1 = src + (row + (X1 >> 4)) * (5 * 4096) + (Y & 15) * 16 + (X1 & 15);
    T a[5], b[5];
#pragma unroll
    for (int f = 0; f < 5; ++f) {
      a[f] = s0[f * 4096];
      b[f] = s1[f * 4096];
    }
#pragma unroll
    for (int f = 0; f < 5; ++f) store_pair<T, kPair>(dst + f * P3 + y * P + x, a[f], b[f]);
  }
}

// ------------------------------------------------------------------ CFL ---
// One workgroup of 16 waves per group: wave w takes patch column w & 3 (x, y
// halves) and planes 4 (w >> 2) .. + 3, a lane one (x, y) of the patch; the
// maximum signal speed |u|+|v|+|w|+3c is reduced over the wave by lane
// shuffles and over the two waves of a patch through LDS (a maximum is exact
// in any order).  cfl_signal_speed evaluates each cell in double for both
// state types with IEEE-rounded, uncontracted operations: four divisions and
// a square root per cell, a serial chain, so four cells per lane instead of
// 16 (8 groups FP64: 11.6 -> 6.6 us; 4096 groups without ghosts 119 -> 110).  The maximum keeps the running value
// unless a speed is strictly larger (a NaN speed from an unphysical cell
// never wins; the step counts such cells).
template <typename T>
__global__ __launch_bounds__(1024) void cfl_dt_kernel(const T* __restrict__ U_pad, int gh, double dx, double gamma,
                                                      double c_cfl, double* __restrict__ dt_patch,
                                                      unsigned long long* __restrict__ dt_min) {
  __shared__ double wave_max[16];
  const int P = 16 + 2 * gh;
  const int64_t P3 = int64_t(P) * P * P;
  const T* __restrict__ Ug = U_pad + int64_t(blockIdx.x) * 5 * P3;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, pxy = wave & 3;
  const int x = (pxy & 1) * 8 + (lane & 7), y = (pxy >> 1) * 8 + (lane >> 3), z0 = (wave >> 2) * 4;
  double m = 0.0;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int64_t o = (int64_t(z0 + j + gh) * P + (y + gh)) * P + (x + gh);
    const double s = cfl_signal_speed(double(Ug[o]), double(Ug[P3 + o]), double(Ug[2 * P3 + o]),
                                      double(Ug[3 * P3 + o]), double(Ug[4 * P3 + o]), gamma);
    if (s > m) m = s;
  }
  for (int k = 32; k > 0; k >>= 1) {
    const double s = __shfl_xor(m, k, 64);
    if (s > m) m = s;
  }
  if (lane == 0) wave_max[wave] = m;
  __syncthreads();
  // patch p = (pz*2 + py)*2 + px: waves 8 pz + (p & 3) and + 4
  if (threadIdx.x < 8) {
    const int p = threadIdx.x;
    const double a = wave_max[8 * (p >> 2) + (p & 3)], b = wave_max[8 * (p >> 2) + 4 + (p & 3)];
    const double dt = (c_cfl * dx) / (b > a ? b : a);
    dt_patch[int64_t(blockIdx.x) * 8 + p] = dt;
    if (dt_min != nullptr) atomicMin(dt_min, (unsigned long long)__double_as_longlong(dt));
  }
}

__global__ void set_inf_kernel(unsigned long long* p) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0x7ff0000000000000ull;
}

}  // namespace

template <typename T>
hipError_t launch_fill_ghosts(const T* level, T* U_pad, int ngx, int ngy, int ngz, int ghost, const int bc[6],
                              hipStream_t stream) {
  const int P = 16 + 2 * ghost;
  const int64_t planes = int64_t(ngx) * ngy * ngz * 5 * P;
  if (planes == 0) return hipSuccess;
  if (planes > (int64_t(1) << 31)) return hipErrorInvalidValue;
  BC6 b;
  for (int i = 0; i < 6; ++i) b.b[i] = bc[i];
  const unsigned n = unsigned(planes / 5);  // workgroups: padded planes of all five fields
  const dim3 grid((n + 7) / 8 * 8);
  // a contiguous range of planes per XCD, but round robin for FP64 blocks with
  // wide ghost zones of few groups, where eight distant write streams collide (us,
  // contiguous / round robin, and 8-byte stores per field before: 64 groups with
  // 16 ghosts 71.9 / 48.4, 61.7, with 12 39.7 / 28.4, 39.3; 128 with 14 111 / 92, 104;
  // but 256 with 16 281 / 309, 353; 96 with 11 53.6 / 55.4, 56.2; FP32 64 with 16
  // 34.8 / 34.6, 57.5)
  const bool blocked = sizeof(T) == 4 || ghost < 12 || int64_t(ngx) * ngy * ngz > 128;
  if (reinterpret_cast<uintptr_t>(U_pad) % (2 * sizeof(T)) == 0)
    hipLaunchKernelGGL((fill_ghosts_kernel<T, true>), grid, dim3(256), 0, stream, level, U_pad, ngx, ngy, ngz, ghost,
                       n, blocked, b);
  else
    hipLaunchKernelGGL((fill_ghosts_kernel<T, false>), grid, dim3(256), 0, stream, level, U_pad, ngx, ngy, ngz, ghost,
                       n, blocked, b);
  return hipGetLastError();
}

template <typename T>
hipError_t launch_cfl_dt(const T* U_pad, int64_t n_groups, int ghost, double dx, double gamma, double c_cfl,
                         double* dt_patch, double* dt_min, hipStream_t stream) {
  unsigned long long* m = reinterpret_cast<unsigned long long*>(dt_min);
  if (m != nullptr) {
    hipLaunchKernelGGL(set_inf_kernel, dim3(1), dim3(64), 0, stream, m);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (n_groups == 0) return hipSuccess;
  const int64_t chunk = int64_t(1) << 30;
  const int P = 16 + 2 * ghost;
  const int64_t P3 = int64_t(P) * P * P;
  for (int64_t g0 = 0; g0 < n_groups; g0 += chunk) {
    const int64_t n = n_groups - g0 < chunk ? n_groups - g0 : chunk;
    hipLaunchKernelGGL(cfl_dt_kernel<T>, dim3(unsigned(n)), dim3(1024), 0, stream, U_pad + g0 * 5 * P3, ghost, dx,
                       gamma, c_cfl, dt_patch + g0 * 8, m);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template hipError_t launch_fill_ghosts<double>(const double*, double*, int, int, int, int, const int*,
                                               hipStream_t);
template hipError_t launch_fill_ghosts<float>(const float*, float*, int, int, int, int, const int*, hipStream_t);
template hipError_t launch_cfl_dt<double>(const double*, int64_t, int, double, double, double, double*, double*,
                                          hipStream_t);
template hipError_t launch_cfl_dt<float>(const float*, int64_t, int, double, double, double, double*, double*,
                                         hipStream_t);

}  // namespace gh
