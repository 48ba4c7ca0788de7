// Arguments of the march of the other schemes (ext_march.h), and its launches.
#pragma once

#include "ext_device.h"
#include "kernels.h"

namespace gh {

enum MarchMode { kStep = 0, kPredict = 1, kCorrect = 2 };

constexpr int kMS = 18;                // state cells per axis: -1 .. 16
constexpr int kMS3 = kMS * kMS * kMS;  // cells of a flux-difference block

template <typename T>
struct MarchArgs {
  const T* U_pad;
  T* U_out;
  int gh;
  int segs;             // z segments per group (divides 16)
  Gas<T> gas;
  const double* dt_dev;
  double dx;
  ExtOpts o;
  T xi;
  int* n_bad;
  T* face_flux;         // optional [G][9][5][256] (NF = 5)
  T* dF;                // kPredict writes, kCorrect reads: [G][3][NF][18^3]
};

// One mode of the march over G groups (instantiated in march_step.hip,
// march_ctu_plm.hip, march_ctu_ppm.hip).
template <typename T, int NF, bool kPpm, int kMode>
hipError_t launch_march_mode(const MarchArgs<T>& args, int64_t G, hipStream_t stream);

}  // namespace gh
