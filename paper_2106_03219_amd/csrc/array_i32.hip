// array_i32.hip -- array-section reduction kernels for i32 inputs.
#include "array_kernel.h"

namespace omprt {

ArrayLauncher array_launcher_i32(int op, int loads, int u) {
    return array_launcher_impl<DT_I32>(op, loads, u);
}

}  // namespace omprt
