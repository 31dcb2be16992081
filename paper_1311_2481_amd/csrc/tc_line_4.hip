// The line kernels at 4 lanes per slot (see tc_line.hip).
#include "tc_line_dev.h"

namespace tc {
hipError_t run_line_4(tc_ctx* c, const LineArgs& x) { return run_rpl<4>(c, x); }
}  // namespace tc
