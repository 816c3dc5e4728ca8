// array_bf16.hip -- array-section reduction kernels for bf16 inputs.
#include "array_kernel.h"

namespace omprt {

ArrayLauncher array_launcher_bf16(int op, int loads, int u) {
    return array_launcher_impl<DT_BF16>(op, loads, u);
}

}  // namespace omprt
