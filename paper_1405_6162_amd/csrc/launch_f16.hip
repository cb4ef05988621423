// Kernels and launchers of binary16 storage.

#include "launch.h"

namespace lbl {
LB_LAUNCHERS(template, _Float16)
}  // namespace lbl
