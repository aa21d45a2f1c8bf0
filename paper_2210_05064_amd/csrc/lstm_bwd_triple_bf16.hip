// Three layers per launch, backward, bf16: see lstm_launch.h.
#include "lstm_launch_bwd.h"

namespace ver {
template bool launch_bwd_triple<MODE_BF16>(const BwdForm&, const TripleBwdArgs&, hipStream_t);
}  // namespace ver
