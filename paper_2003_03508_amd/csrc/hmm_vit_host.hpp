// Plan and launch interface of the Viterbi segment chains (hmm_vit_chain.hip).
#pragma once

#include "hmm_host.hpp"
#include "hmm_vit_chain.hpp"

namespace hmmh {

struct VitChainPlan {
    const void *fn = nullptr;
    int64_t nb = 0;    // segments; 0: the max-plus product path alone
    int len = 0;       // longest segment
    int kr = 0;        // K rounded up to the compiled size
    int segs = 1;      // segments per workgroup (one wavefront)
    int fixed = 0;     // LDS of a segment without its backpointers
    int rows() const { return len + kVitAhead; }
    size_t lds() const { return (size_t)segs * (fixed + vit_psi_bytes(kr, rows())); }
};

VitChainPlan make_vit_chain_plan(int K, int64_t T, int64_t product_len);
hipError_t launch_vit_chain(const VitChainPlan &cp, VitChain v, hipStream_t st);

}  // namespace hmmh
