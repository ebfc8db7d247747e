// The fused kernels of SDC_PREC_SPLIT_BF16.
#include "sdc_fused.h"

namespace sdc {

const void* fused_kernel_bf16(int sched, int radial, int paired, bool batch) {
    return pick_sched<SDC_PREC_SPLIT_BF16>(sched, radial, paired, batch);
}

}  // namespace sdc
