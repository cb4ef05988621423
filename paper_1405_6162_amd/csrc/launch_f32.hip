// Kernels and launchers of FP32 storage.

#include "launch.h"

namespace lbl {
LB_LAUNCHERS(template, float)
}  // namespace lbl
