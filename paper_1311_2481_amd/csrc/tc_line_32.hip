// The line kernels at 32 lanes per slot (see tc_line.hip).
#include "tc_line_dev.h"

namespace tc {
hipError_t run_line_32(tc_ctx* c, const LineArgs& x) { return run_rpl<32>(c, x); }
}  // namespace tc
