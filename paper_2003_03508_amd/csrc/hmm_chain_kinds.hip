// Segment-chain kernels (hmm_chain.hpp) of the other emission kinds, one instance
// per count of live contraction slots (K = 4 NSL - 3 .. 4 NSL) and workgroup
// shape.  Compiled with MFMA results in ordinary VGPRs: every step reads its
// accumulators with vector ALU code.
#include "hmm_host.hpp"

namespace hmmh {

namespace {

template <bool BIG, int NSL>
const void *pick(int nsl)
{
    if constexpr (NSL > 20) {
        return nullptr;
    } else {
        // as chain_shape
        constexpr int NP = (NSL <= 8 ? 1 : 2) * (BIG ? 2 : 1), NS = (NSL <= 8 && !BIG) ? 2 : 1;
        if (nsl == NSL) return reinterpret_cast<const void *>(&k_chain<(NSL + 3) / 4, NSL, true, NP, NS>);
        return pick<BIG, NSL + 1>(nsl);
    }
}

}  // namespace

// up to 16 states every sequence the chains serve takes the larger shape
static_assert(chain_min_T(16) >= chain_big_T(16) && chain_min_T(4) >= chain_big_T(4));

const void *chain_kernel_kinds(int nsl, bool big) { return big ? pick<true, 1>(nsl) : pick<false, 5>(nsl); }

}  // namespace hmmh
