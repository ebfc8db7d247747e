// The fused kernels of SDC_PREC_FP32.
#include "sdc_fused.h"

namespace sdc {

const void* fused_kernel_fp32(int sched, int radial, int paired, bool batch) {
    return pick_sched<SDC_PREC_FP32>(sched, radial, paired, batch);
}

}  // namespace sdc
