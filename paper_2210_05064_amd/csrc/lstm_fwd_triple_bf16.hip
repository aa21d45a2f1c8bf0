// Three layers per launch, forward, bf16: see lstm_launch.h.
#include "lstm_launch_fwd.h"

namespace ver {
template bool launch_fwd_triple<MODE_BF16>(const FwdForm&, const TripleFwdArgs&, hipStream_t);
}  // namespace ver
