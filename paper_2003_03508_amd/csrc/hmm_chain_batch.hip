// Segment-chain kernels of a batch (hmm_chain.hpp): one kernel for every K.
// Compiled with MFMA results in ordinary VGPRs, as hmm_chain.hip.
#include "hmm_host.hpp"

namespace hmmh {

const void *chain_kernel_batch() { return reinterpret_cast<const void *>(&k_chain_batch); }

hipError_t launch_chain_finish(int n, hipStream_t st, const SetDesc *sets, const int *cls, int *words)
{
    hipLaunchKernelGGL(k_chain_finish, dim3((unsigned)n), dim3(256), 0, st, sets, cls, words);
    return hipGetLastError();
}

}  // namespace hmmh
