// Rules by which the host launches the row kernels.  Plain host code: a test runs them without a GPU.
#pragma once

#include <stdint.h>

namespace difr {

// RowPace: the workgroup of a launch of `groups` from which on they share the issue slots by what they have left, where `resident` of
// them are held at once (0: not known, none does).
constexpr int pace_from(int64_t groups, int resident) { return (int)(groups - resident); }

}  // namespace difr
