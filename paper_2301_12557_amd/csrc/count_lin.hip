// count_lin.hip -- the counting kernels with computed bins (uniform edges on every axis).
#include "count_kernel.h"

namespace fcfc {

CountKernel count_kernel_lin(int mode, int kind, int los, bool is_auto, bool w) {
    return count_kernel_pick<true>(mode, kind, los, is_auto, w);
}

}  // namespace fcfc
