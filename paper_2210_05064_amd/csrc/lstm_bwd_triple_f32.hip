// Three layers per launch, backward, fp32: see lstm_launch.h.
#include "lstm_launch_bwd.h"

namespace ver {
template bool launch_bwd_triple<MODE_F32>(const BwdForm&, const TripleBwdArgs&, hipStream_t);
}  // namespace ver
