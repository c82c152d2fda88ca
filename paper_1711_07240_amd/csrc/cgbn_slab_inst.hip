// Explicit instantiations of the column-slab kernels, one translation unit per element type and direction.  The build
// passes CGBN_INST_T (float or bf16_t) and CGBN_INST_FWD (0/1).
#include "cgbn_slab.h"

namespace cgbn {
#if CGBN_INST_FWD
#define CGBN_X(P_, SOLO_)                                                           \
    template __global__ void slab_forward<CGBN_INST_T, 0, P_, SOLO_>(SlabArgs);     \
    template __global__ void slab_forward<CGBN_INST_T, 1, P_, SOLO_>(SlabArgs);     \
    template __global__ void slab_forward<CGBN_INST_T, 2, P_, SOLO_>(SlabArgs);
CGBN_SLAB_FORWARD_P(CGBN_X)
#else
#define CGBN_X(P_, SOLO_)                                                           \
    template __global__ void slab_backward<CGBN_INST_T, 0, P_, SOLO_>(SlabArgs);    \
    template __global__ void slab_backward<CGBN_INST_T, 1, P_, SOLO_>(SlabArgs);
CGBN_SLAB_BACKWARD_P(CGBN_X)
#endif
#undef CGBN_X
}  // namespace cgbn
