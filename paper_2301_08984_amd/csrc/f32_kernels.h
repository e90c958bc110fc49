// fp32 attention on the fp32 matrix instructions (f32_kernels.hip): which operators it serves, launchers.
// launch_generic_fwd / _dkdv send fp32 calls that f32_ok accepts here; the recompute launch does dQ too, the dK/dV
// launch the bias gradient, so there are no others.
#pragma once
#include "kparams.h"

namespace ssa {

// 16-byte loads of rows; the flat grid of f32_key_kernel has to fit
inline bool f32_ok(const KP& p) {
  if (p.plain || p.D > 64 || p.D % 4 || p.sb % 4 || p.ss % 4 || p.sh % 4) return false;
  if ((int64_t)((p.S + 15) / 16) * p.H * (p.B + 1) >= (1ll << 31)) return false;
  for (const void* t : {p.Q, p.K, p.V, p.G, p.dY, (const void*)p.Y, (const void*)p.dQ, (const void*)p.dK, (const void*)p.dV, (const void*)p.dG})
    if ((uintptr_t)t % 16) return false;
  return true;
}
hipError_t launch_f32_fwd(const KP& p, hipStream_t st);
hipError_t launch_f32_recompute_dq(const KP& p, hipStream_t st);
hipError_t launch_f32_dkdv_dbias(const KP& p, hipStream_t st);  // the bias gradient too, if it is wanted

}  // namespace ssa
