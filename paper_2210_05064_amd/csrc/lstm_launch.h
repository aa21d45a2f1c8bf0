// Launches of the time-loop kernels.  They are compiled per direction and arithmetic in files of their own (lstm_fwd_*.hip,
// lstm_bwd_*.hip): together they took two minutes.
#pragma once
#include "lstm_pipe.h"

namespace ver {

template <typename K>
inline bool set_lds(K kernel, size_t bytes) {
    return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)bytes) == hipSuccess;
}

// What chooses the instantiation (run_fwd and run_bwd in lstm.hip say how).
struct FwdForm {
    bool wide, quarter;   // 8 instead of 4 row tiles per workgroup; a quarter instead of half of the contraction per wave
    int nb;               // operand blocks of that share
    size_t lds;
};
struct BwdForm {
    bool wide;            // 2 instead of 1 unit tiles per workgroup
    int ni;               // operand blocks of a wave's share
    size_t lds;
};
// One layer; two layers (planned: the kernels that ask the plan whether they run); three layers (always planned).
template <int MODE> bool launch_fwd_loop(const FwdForm& f, const RecFwdArgs& a, hipStream_t s);
template <int MODE> bool launch_fwd_pair(const FwdForm& f, const PipeFwdArgs& a, bool planned, hipStream_t s);
template <int MODE> bool launch_fwd_triple(const FwdForm& f, const TripleFwdArgs& a, hipStream_t s);
template <int MODE> bool launch_bwd_triple(const BwdForm& f, const TripleBwdArgs& a, hipStream_t s);
template <int MODE> bool launch_bwd_loop(const BwdForm& f, const RecBwdArgs& a, hipStream_t s);
template <int MODE> bool launch_bwd_pair(const BwdForm& f, const PipeBwdArgs& a, bool planned, hipStream_t s);

}  // namespace ver
