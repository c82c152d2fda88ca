// Explicit instantiations of the column-slab kernels, one translation unit per element type and direction.  The build
// passes CGBN_INST_T (float or bf16_t), CGBN_INST_FWD (0/1) and CGBN_INST_DENSE (1: the DENSE variants alone, 0: the others).
#include "cgbn_slab.h"

namespace cgbn {
#if CGBN_INST_DENSE
#if CGBN_INST_FWD
template __global__ void slab_forward<CGBN_INST_T, 0, kSlabDenseForward, false, true>(SlabArgs);
template __global__ void slab_forward<CGBN_INST_T, 1, kSlabDenseForward, false, true>(SlabArgs);
#else
template __global__ void slab_backward<CGBN_INST_T, 0, kSlabDenseBackward, false, true>(SlabArgs);
template __global__ void slab_backward<CGBN_INST_T, 1, kSlabDenseBackward, false, true>(SlabArgs);
#endif
#elif CGBN_INST_FWD
#define CGBN_X(P_, SOLO_)                                                                  \
    template __global__ void slab_forward<CGBN_INST_T, 0, P_, SOLO_, false>(SlabArgs);     \
    template __global__ void slab_forward<CGBN_INST_T, 1, P_, SOLO_, false>(SlabArgs);     \
    template __global__ void slab_forward<CGBN_INST_T, 2, P_, SOLO_, false>(SlabArgs);
CGBN_SLAB_FORWARD_P(CGBN_X)
#define CGBN_Y(P_)                                                                         \
    template __global__ void slab_forward<CGBN_INST_T, 0, P_, true, false, 8>(SlabArgs);   \
    template __global__ void slab_forward<CGBN_INST_T, 1, P_, true, false, 8>(SlabArgs);   \
    template __global__ void slab_forward<CGBN_INST_T, 2, P_, true, false, 8>(SlabArgs);
CGBN_SLAB_NARROW_P(CGBN_Y)
#else
#define CGBN_X(P_, SOLO_)                                                                  \
    template __global__ void slab_backward<CGBN_INST_T, 0, P_, SOLO_, false>(SlabArgs);    \
    template __global__ void slab_backward<CGBN_INST_T, 1, P_, SOLO_, false>(SlabArgs);
CGBN_SLAB_BACKWARD_P(CGBN_X)
#define CGBN_Y(P_)                                                                         \
    template __global__ void slab_backward<CGBN_INST_T, 0, P_, true, false, 8>(SlabArgs);  \
    template __global__ void slab_backward<CGBN_INST_T, 1, P_, true, false, 8>(SlabArgs);
CGBN_SLAB_NARROW_P(CGBN_Y)
#endif
#undef CGBN_X
#undef CGBN_Y
}  // namespace cgbn
