// The fused kernels of SDC_PREC_SPLIT_FP16.
#include "sdc_fused.h"

namespace sdc {

const void* fused_kernel_fp16(int sched, int radial, int paired, bool batch) {
    return pick_sched<SDC_PREC_SPLIT_FP16>(sched, radial, paired, batch);
}

}  // namespace sdc
