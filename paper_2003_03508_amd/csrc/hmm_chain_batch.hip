// Segment-chain kernels of a batch (hmm_chain.hpp): one kernel for every K.
// Compiled with MFMA results in ordinary VGPRs, as hmm_chain.hip.  Defined
// here and not in the header: a kernel in a header is compiled into every unit
// that includes it (0.8 MB each).
#include "hmm_host.hpp"

namespace hmm {

namespace {

// Batch (tremor model): workgroup blockIdx.x of any set, whatever its K, from
// the job table (ordered by decreasing cost).  One launch for all K, so that
// sets of different K fill the chip together; two pairs per workgroup.
template <int NSL>
__device__ __forceinline__ void chain_any(int nsl, const SetDesc &d, int64_t wg, int mode)
{
    if constexpr (NSL <= 20) {
        if (nsl == NSL) chain_body<(NSL + 3) / 4, NSL, false, 2, 1>(d, wg, mode);
        else chain_any<NSL + 1>(nsl, d, wg, mode);
    }
}

__global__ __launch_bounds__(256) void k_chain_batch(const SetDesc *__restrict__ sets,
                                                     const ChainJob *__restrict__ jobs, int mode)
{
    const ChainJob j = jobs[blockIdx.x];
    const SetDesc d = sets[j.set];
    chain_any<1>((d.K + 3) / 4, d, j.wg, mode);
}

// Batch, after the chains: workgroup s finishes ln L of set s where they
// served it, else raises the flag of the set's product class (words[2 c + 1];
// words[2 c] is the class's job counter), whose launches look at it first.
__global__ __launch_bounds__(256) void k_chain_finish(const SetDesc *__restrict__ sets,
                                                      const int *__restrict__ cls, int *__restrict__ words)
{
    __shared__ float smem[2 * 256];
    const SetDesc d = sets[blockIdx.x];
    if (d.chained()) chain_finish(d, smem);
    else if (threadIdx.x == 0) atomicOr(&words[2 * cls[blockIdx.x] + 1], 1);
}

}  // namespace

}  // namespace hmm

namespace hmmh {

const void *chain_kernel_batch() { return reinterpret_cast<const void *>(&k_chain_batch); }

hipError_t launch_chain_finish(int n, hipStream_t st, const SetDesc *sets, const int *cls, int *words)
{
    hipLaunchKernelGGL(k_chain_finish, dim3((unsigned)n), dim3(256), 0, st, sets, cls, words);
    return hipGetLastError();
}

}  // namespace hmmh
