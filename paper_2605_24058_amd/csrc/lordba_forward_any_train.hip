// The same as training runs it (t is kept).
#define LORDBA_FWD_TRAINING 1
#include "lordba_fwd_any.h"

lordba_status lordba_forward_any_train(const FwdArgs& a, hipStream_t stream) { return launch_any(a, stream); }
