// Reverse-mode derivative of the 3D binary64 push: the kernels of
// gcb_push_backward_3d, organised as in 2D (gcb_adjoint.hip).
#define GCB_ARITH_NS arith_fast
#define GCB_FAST_ARITH 1
#include <hip/hip_runtime.h>

#include "gcb_adjoint_kernels.hpp"

namespace gcb {

hipError_t launch_adjoint3_batch(const AdjointLaunch& L, const PushConst3& pc,
                                 hipStream_t stream) {
    if (L.n == 0 || L.s_hi <= L.s_lo) return hipSuccess;
    return L.yee ? adj::launch_batch<3, true>(L, pc, stream)
                 : adj::launch_batch<3, false>(L, pc, stream);
}

}  // namespace gcb
