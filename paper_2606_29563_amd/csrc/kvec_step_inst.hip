// One (dtype, head_dim) pair of the step kernel, for every group size; built
// once per pair with KVEC_INST_TT (BF16 or F32), KVEC_INST_D (64 or 128) and
// KVEC_INST_LONG (true: the variant for several key tiles per score work-group,
// BF16 only).
#include "kvec_step.h"

#if !defined(KVEC_INST_TT) || !defined(KVEC_INST_D) || !defined(KVEC_INST_LONG)
#error "define KVEC_INST_TT, KVEC_INST_D and KVEC_INST_LONG"
#endif

namespace kvec {
namespace step {

template <>
StepFn pick_g<KVEC_INST_TT, KVEC_INST_D, KVEC_INST_LONG>(int G) {
  switch (G) {
    case 1: return step_kernel<KVEC_INST_TT, KVEC_INST_D, 1, KVEC_INST_LONG>;
    case 2: return step_kernel<KVEC_INST_TT, KVEC_INST_D, 2, KVEC_INST_LONG>;
    case 3: return step_kernel<KVEC_INST_TT, KVEC_INST_D, 3, KVEC_INST_LONG>;
    case 4: return step_kernel<KVEC_INST_TT, KVEC_INST_D, 4, KVEC_INST_LONG>;
    case 5: return step_kernel<KVEC_INST_TT, KVEC_INST_D, 5, KVEC_INST_LONG>;
    case 6: return step_kernel<KVEC_INST_TT, KVEC_INST_D, 6, KVEC_INST_LONG>;
    case 7: return step_kernel<KVEC_INST_TT, KVEC_INST_D, 7, KVEC_INST_LONG>;
    default: return step_kernel<KVEC_INST_TT, KVEC_INST_D, 8, KVEC_INST_LONG>;
  }
}

}  // namespace step
}  // namespace kvec
