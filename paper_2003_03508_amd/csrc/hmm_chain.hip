// Segment-chain kernels (hmm_chain.hpp), one instance per count of live
// contraction slots (K = 4 NSL - 3 .. 4 NSL) for the tremor model and for any
// emission kind.  Compiled with MFMA results in ordinary VGPRs: every step
// reads its accumulators with vector ALU code.
#include "hmm_host.hpp"

namespace hmmh {

namespace {

template <bool GEN, int NSL>
const void *pick(int nsl)
{
    if constexpr (NSL > 20) {
        return nullptr;
    } else {
        if (nsl == NSL) return reinterpret_cast<const void *>(&k_chain<(NSL + 3) / 4, NSL, GEN>);
        return pick<GEN, NSL + 1>(nsl);
    }
}

}  // namespace

const void *chain_kernel(int K, bool gen)
{
    const int nsl = (K + 3) / 4;
    return gen ? pick<true, 1>(nsl) : pick<false, 1>(nsl);
}

}  // namespace hmmh
