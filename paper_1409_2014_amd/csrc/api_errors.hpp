// Error reporting shared by the C-ABI sources: the message phi_last_error(NULL)
// returns for the calling thread.
#pragma once

#include <string>

#include "phi_solve.h"

namespace phi {

// Records msg as this thread's last error and returns st.
phi_status thread_error(phi_status st, const std::string& msg);


// phi_solve in the plain arithmetic of an FP32 plan: every node, one row per
// transform, the multiplier's quotient from its tables.  The same sums within FP32
// rounding; phi_ds_forward_plain says what it is for.  FP64 plans have one
// arithmetic.
phi_status solve_plain(phi_plan_t plan, const void* in, void* out, void* stream);

}  // namespace phi
