// Three layers per launch, forward, fp32: see lstm_launch.h.
#include "lstm_launch_fwd.h"

namespace ver {
template bool launch_fwd_triple<MODE_F32>(const FwdForm&, const TripleFwdArgs&, hipStream_t);
}  // namespace ver
