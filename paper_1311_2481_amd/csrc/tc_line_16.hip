// The line kernels at 16 lanes per slot (see tc_line.hip).
#include "tc_line_dev.h"

namespace tc {
hipError_t run_line_16(tc_ctx* c, const LineArgs& x) { return run_rpl<16>(c, x); }
}  // namespace tc
