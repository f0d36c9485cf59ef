// count_lut.hip -- the counting kernels with look-up tables.
#include "count_kernel.h"

namespace fcfc {

CountKernel count_kernel_lut(int mode, int kind, int los, bool is_auto, bool w) {
    return count_kernel_pick<false>(mode, kind, los, is_auto, w);
}

}  // namespace fcfc
