// Host-side launchers of the fp32 build kernels for small calls (internal to the library). The arguments
// are those of the 64 x 64-tile kernels they stand in for; Mg, ssq and Z have the same layout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dv {

hipError_t launch_small_down(const float* E, const float* Dw, float* Z, int T, int d, int L, int r, int act,
                             hipStream_t s);
hipError_t launch_small_up(const float* E, const float* Z, const float* Uw, const float* gamma, float* Mg, float* ssq,
                           int T, int d, int r, int l0, int nl, hipStream_t s);
hipError_t launch_small_kv(const float* Mg, const float* ssq, const float* Wk, const float* Wv, float* Kv, float* Vv,
                           int B_, int Nv, int d, int Hkv, int hd, int l0, int nl, int np, float eps, hipStream_t s);

}  // namespace dv
