// array_f64.hip -- array-section reduction kernels for f64 inputs.
#include "array_kernel.h"

namespace omprt {

ArrayLauncher array_launcher_f64(int op, int loads, int u) {
    return array_launcher_impl<DT_F64>(op, loads, u);
}

}  // namespace omprt
