// Tile passes of subgraphs with the same number of qubit groups but other group
// sizes in one launch (batches of few tiles, see make_plan).
//
// They are a code object of their own. Beside sim.hip's kernels they made that
// object 0.19 MB larger (0.84 MB without), and its kernels, the same instructions,
// ran longer where it was then loaded: ten optimiser steps of 21 states of 20
// qubits 2.90 against 2.87 ms, a gradient of 24 qubits 461 against 460 us. (The
// same library loaded second in a process loses 1.2 to 1.6 % in the same way.)
#include "passes.h"

namespace pq {

// Groups of up to four and of more qubits in one launch: each workgroup walks the
// layouts of its own group, so a subgraph's results do not depend on the others.
__device__ inline bool few_qubits(const SubDesc* subs, const int2* work, const PassOps& ops)
{
    return subs[work[blockIdx.x].x].gsize[ops.group] <= 4;
}

template <int KIND>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(PQ_FWD_WAVES))) void k_fwd_mixed(
    uint8_t* ws, const SubDesc* subs, const int2* work, PassOps ops, Partials part)
{
    if (few_qubits(subs, work, ops)) fwd_pass_body<1, false, KIND, PREC_VALU>(ws, subs, work, ops, part);
    else fwd_pass_body<2, false, KIND, PREC_VALU>(ws, subs, work, ops, part);
}

template <int KIND, bool STORE_PSI>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(PQ_BWD_WAVES))) void k_bwd_mixed(
    uint8_t* ws, const SubDesc* subs, const int2* work, PassOps ops, Partials part)
{
    if (few_qubits(subs, work, ops)) bwd_pass_body<1, false, KIND, STORE_PSI>(ws, subs, work, ops, part);
    else bwd_pass_body<2, false, KIND, STORE_PSI>(ws, subs, work, ops, part);
}

#define PQ_LAUNCH_MIXED(...) hipLaunchKernelGGL((__VA_ARGS__), g, b, lds, s, ws, subs, work, ops, part)

hipError_t launch_fwd_mixed(uint8_t* ws, const SubDesc* subs, const int2* work, int nwork, PassOps ops, Partials part,
                            int lut_max, hipStream_t s)
{
    const size_t lds = pass_lds(lut_max);
    const dim3 g(nwork), b(THREADS);
    if (ops.epi_e) PQ_LAUNCH_MIXED(k_fwd_mixed<F_LAST>);
    else if (ops.ph >= 0) PQ_LAUNCH_MIXED(k_fwd_mixed<F_MID>);
    else PQ_LAUNCH_MIXED(k_fwd_mixed<F_SINGLE>);
    return hipGetLastError();
}

hipError_t launch_bwd_mixed(uint8_t* ws, const SubDesc* subs, const int2* work, int nwork, PassOps ops, Partials part,
                            int lut_max, hipStream_t s)
{
    const size_t lds = pass_lds(lut_max);
    const dim3 g(nwork), b(THREADS);
    if (ops.fused) PQ_LAUNCH_MIXED(k_bwd_mixed<B_FUSED, true>);
    else if (ops.ph >= 0 && ops.nopsi) PQ_LAUNCH_MIXED(k_bwd_mixed<B_MID, false>);
    else if (ops.ph >= 0) PQ_LAUNCH_MIXED(k_bwd_mixed<B_MID, true>);
    else if (ops.nopsi) PQ_LAUNCH_MIXED(k_bwd_mixed<B_SINGLE, false>);
    else PQ_LAUNCH_MIXED(k_bwd_mixed<B_SINGLE, true>);
    return hipGetLastError();
}

}  // namespace pq
