// Backward launches, for the file of an arithmetic to instantiate.
#pragma once
#include "lstm_launch.h"

namespace ver {

#define VER_BWD_LAUNCH(KERNEL, MT_, KS_, N_) do { if (!set_lds(KERNEL<MODE, MT_, KS_, N_>, f.lds)) return false; \
        hipLaunchKernelGGL((KERNEL<MODE, MT_, KS_, N_>), dim3(REC_GRID), dim3(REC_THREADS), f.lds, s, a); return true; } while (0)
#define VER_BWD_DISPATCH(KERNEL) do { \
        if constexpr (MODE == MODE_BF16) {   /* (fp32: hidden <= 512) */ \
            if (f.wide) { \
                if (f.ni == 32) VER_BWD_LAUNCH(KERNEL, 2, 4, 32); else VER_BWD_LAUNCH(KERNEL, 2, 4, 0); \
            } \
        } \
        if (f.ni == 16) VER_BWD_LAUNCH(KERNEL, 1, 8, 16); \
        else if (f.ni == 8) VER_BWD_LAUNCH(KERNEL, 1, 8, 8); \
        else if (f.ni == 4) VER_BWD_LAUNCH(KERNEL, 1, 8, 4); \
        else VER_BWD_LAUNCH(KERNEL, 1, 8, 0); } while (0)

template <int MODE> bool launch_bwd_loop(const BwdForm& f, const RecBwdArgs& a, hipStream_t s) { VER_BWD_DISPATCH(lstm_rec_bwd_kernel); }
template <int MODE> bool launch_bwd_pair(const BwdForm& f, const PipeBwdArgs& a, bool planned, hipStream_t s) {
    if (planned) VER_BWD_DISPATCH(lstm_pipe_bwd_planned_kernel);
    else VER_BWD_DISPATCH(lstm_pipe_bwd_kernel);
}
template <int MODE> bool launch_bwd_triple(const BwdForm& f, const TripleBwdArgs& a, hipStream_t s) { VER_BWD_DISPATCH(lstm_triple_bwd_kernel); }
#undef VER_BWD_DISPATCH
#undef VER_BWD_LAUNCH

}  // namespace ver
