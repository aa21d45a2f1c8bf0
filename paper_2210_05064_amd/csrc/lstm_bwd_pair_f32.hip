// Two layers per launch, backward, fp32: see lstm_launch.h.
#include "lstm_launch_bwd.h"

namespace ver {
template bool launch_bwd_pair<MODE_F32>(const BwdForm&, const PipeBwdArgs&, bool, hipStream_t);
}  // namespace ver
