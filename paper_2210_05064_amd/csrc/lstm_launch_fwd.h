// Forward launches, for the file of an arithmetic to instantiate.
#pragma once
#include "lstm_launch.h"

namespace ver {

#define VER_FWD_LAUNCH(KERNEL, TPW_, KS_, NBW_, ST_) do { if (!set_lds(KERNEL<MODE, TPW_, KS_, NBW_, ST_>, f.lds)) return false; \
        hipLaunchKernelGGL((KERNEL<MODE, TPW_, KS_, NBW_, ST_>), dim3(REC_GRID), dim3(REC_THREADS), f.lds, s, a); return true; } while (0)
#define VER_FWD_DISPATCH(KERNEL) do { \
        if constexpr (MODE == MODE_BF16) { \
            if (f.wide) { \
                if (!f.quarter && f.nb == 16) VER_FWD_LAUNCH(KERNEL, 2, 2, 16, true); \
                else VER_FWD_LAUNCH(KERNEL, 2, 2, 16, false); \
            } else { \
                if (!f.quarter && f.nb == 8) VER_FWD_LAUNCH(KERNEL, 1, 2, 8, true); \
                else if (!f.quarter) VER_FWD_LAUNCH(KERNEL, 1, 2, 8, false); \
                else if (f.nb == 4) VER_FWD_LAUNCH(KERNEL, 2, 4, 4, true); \
                else VER_FWD_LAUNCH(KERNEL, 2, 4, 4, false); \
            } \
        } else { \
            if (f.nb == 8) VER_FWD_LAUNCH(KERNEL, 2, 4, 8, true); \
            else VER_FWD_LAUNCH(KERNEL, 2, 4, 8, false); \
        } } while (0)

template <int MODE> bool launch_fwd_loop(const FwdForm& f, const RecFwdArgs& a, hipStream_t s) { VER_FWD_DISPATCH(lstm_rec_fwd_kernel); }
template <int MODE> bool launch_fwd_pair(const FwdForm& f, const PipeFwdArgs& a, bool planned, hipStream_t s) {
    if (planned) VER_FWD_DISPATCH(lstm_pipe_fwd_planned_kernel);
    else VER_FWD_DISPATCH(lstm_pipe_fwd_kernel);
}
template <int MODE> bool launch_fwd_triple(const FwdForm& f, const TripleFwdArgs& a, hipStream_t s) { VER_FWD_DISPATCH(lstm_triple_fwd_kernel); }
#undef VER_FWD_DISPATCH
#undef VER_FWD_LAUNCH

}  // namespace ver
