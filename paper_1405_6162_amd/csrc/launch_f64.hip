// Kernels and launchers of FP64 storage.

#include "launch.h"

namespace lbl {
LB_LAUNCHERS(template, double)
}  // namespace lbl
