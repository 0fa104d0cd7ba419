// How many blocks of a launch may wait for one another (GridBarrier): a pure function, compiled for
// the library and for the host check.
#pragma once

#include <algorithm>

namespace fsl {

// The blocks of such a launch have to come to run together, whatever else is running.  Kernels that
// do not wait end; others of this kind may hold part of the device each.  An eighth of what the
// device holds of the kernel's blocks (per_cu on each of its cus compute units: registers, LDS and
// threads together decide) leaves room for eight such launches at once; a process has four
// hardware queues.  At most want; 0 where that is no block: a launch per phase then.
constexpr int SYNC_SHARE = 8;
inline int sync_blocks(int want, int cus, int per_cu) {
    return (int)std::min((long long)std::max(want, 0), (long long)std::max(cus, 0) * std::max(per_cu, 0) / SYNC_SHARE);
}

}  // namespace fsl
