// fp32 attention on the fp32 matrix instructions (f32_kernels.hip): which operators it serves, launchers.
#pragma once
#include "kparams.h"

namespace ssa {

bool f32_ok(const KP& p);
hipError_t launch_f32_fwd(const KP& p, hipStream_t st);
hipError_t launch_f32_recompute_dq(const KP& p, hipStream_t st);
hipError_t launch_f32_dkdv_dbias(const KP& p, hipStream_t st);  // the bias gradient too, if it is wanted

}  // namespace ssa
