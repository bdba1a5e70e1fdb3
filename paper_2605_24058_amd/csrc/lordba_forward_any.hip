// The adapter forward branch on tensors that are aligned to their elements only, with any widths from 8 columns on: inference
// instantiations of the matrix-core kernel (ANY) for 1 to 4 envelopes.
#include "lordba_fwd_any.h"

lordba_status lordba_forward_any(const FwdArgs& a, hipStream_t stream) { return launch_any(a, stream); }
