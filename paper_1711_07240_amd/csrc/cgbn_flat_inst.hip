// Explicit instantiations of the flat kernels, one translation unit per (element type, direction).  The build passes
// CGBN_INST_T (float or bf16_t), CGBN_INST_F32 (1 for float) and CGBN_INST_FWD (0/1).
#include "cgbn_flat.h"

namespace cgbn {
#if CGBN_INST_FWD
#define CGBN_X(LB_, S_, WAVES_)                                                        \
    template __global__ void flat_forward<CGBN_INST_T, LB_, S_, WAVES_, 0>(FlatArgs);  \
    template __global__ void flat_forward<CGBN_INST_T, LB_, S_, WAVES_, 1>(FlatArgs);  \
    template __global__ void flat_forward<CGBN_INST_T, LB_, S_, WAVES_, 2>(FlatArgs);
#else
#define CGBN_X(LB_, S_, WAVES_)                                                        \
    template __global__ void flat_backward<CGBN_INST_T, LB_, S_, WAVES_, 0>(FlatArgs); \
    template __global__ void flat_backward<CGBN_INST_T, LB_, S_, WAVES_, 1>(FlatArgs);
#endif
#define CGBN_X1(LB_, S_) CGBN_X(LB_, S_, 1)
#define CGBN_X4(LB_, S_) CGBN_X(LB_, S_, 4)
#define CGBN_X16(LB_, S_) CGBN_X(LB_, S_, 16)
CGBN_FLAT_ONE(CGBN_X1)
CGBN_FLAT_FOUR(CGBN_X4)
#if CGBN_INST_FWD
CGBN_FLAT_FOUR_FORWARD(CGBN_X4)
#endif
CGBN_FLAT_SIXTEEN(CGBN_X16)
#if !CGBN_INST_F32
CGBN_FLAT_BF16(CGBN_X1)
CGBN_FLAT_BF16(CGBN_X4)
CGBN_FLAT_BF16(CGBN_X16)
#endif
#undef CGBN_X
#undef CGBN_X1
#undef CGBN_X4
#undef CGBN_X16
}  // namespace cgbn
