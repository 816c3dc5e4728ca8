// array_f32.hip -- array-section reduction kernels for f32 inputs.
#include "array_kernel.h"

namespace omprt {

ArrayLauncher array_launcher_f32(int op, int loads, int u) {
    return array_launcher_impl<DT_F32>(op, loads, u);
}

}  // namespace omprt
