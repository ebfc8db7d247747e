// The fused kernels of SDC_PREC_BF16X3.
#include "sdc_fused.h"

namespace sdc {

const void* fused_kernel_x3(int sched, int radial, int paired, bool batch) {
    return pick_sched<SDC_PREC_BF16X3>(sched, radial, paired, batch);
}

}  // namespace sdc
