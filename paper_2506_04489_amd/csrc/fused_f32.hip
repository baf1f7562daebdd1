// fused_f32.hip - the FP32 instantiation of the three-launch solve.
#include "fused.hpp"

namespace psp {

#define PSP_FUSED(N) \
    template hipError_t fused_solve<float, N>(const Job &, const Job *, int, const void *, hipStream_t);
PSP_FUSED(8)
PSP_FUSED(12)
PSP_FUSED(16)
PSP_FUSED(24)
PSP_FUSED(32)
PSP_FUSED(36)
PSP_FUSED(48)
PSP_FUSED(64)
PSP_FUSED(72)
PSP_FUSED(96)
PSP_FUSED(108)
PSP_FUSED(128)
PSP_FUSED(144)
PSP_FUSED(192)
PSP_FUSED(256)
#undef PSP_FUSED

}  // namespace psp
