// See load_order.cpp.
#pragma once

#include <vector>

#include "graph.h"

namespace tn {

// Rearranges the keys (positions in the serial order) of the loads among themselves, such that kernels can run as early as
// the link allows.  seconds: a kernel vertex's estimated time.  Leaves the keys alone where more than a tenth
// of the loaded bytes waits for memory, where little is to be gained, and in programs too large to search.
void order_loads(const MemGraph& mg, const std::vector<double>& seconds, std::vector<int64_t>& key);

}  // namespace tn
