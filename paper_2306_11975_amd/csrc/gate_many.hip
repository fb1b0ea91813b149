// More than eight slices of the kernel in gate_kernel.h.
#include "gate_kernel.h"

namespace ozimmu {

hipError_t launch_gate_many(const GateArgs& g, int cls, int s, hipStream_t st) {
    switch (s) {
#define OZ_CASE(S_) case S_: return cls == 1 ? launch_gate<S_, 1>(g, st) : launch_gate<S_, 0>(g, st);
        OZ_CASE(9) OZ_CASE(10) OZ_CASE(11) OZ_CASE(12) OZ_CASE(13) OZ_CASE(14) OZ_CASE(15) OZ_CASE(16)
#undef OZ_CASE
    }
    return hipErrorInvalidValue;
}

}  // namespace ozimmu
