// Viterbi segment chains (hmm_vit_chain.hpp), one instance per K rounded up to
// a multiple of four, and their plan.
#include "hmm_vit_host.hpp"

#include <algorithm>
#include <cmath>

namespace hmmh {

namespace {

// Below this the product path's few segments end as soon (K = 3, T = 1000: 62
// against 63 us, T = 10,000: 85 against 65; K = 8, T = 100: 44 against 55; K =
// 25, T = 1000: 195 against 87).
constexpr int64_t kVitChainMinT = 1000;
constexpr int kVitSimds = 1024;   // 256 CUs of four

// K <= 32: an instance per K; above, per multiple of four.
template <int KK>
void pick(int kk, VitChainPlan *k)
{
    if constexpr (KK <= 80) {
        if (kk != KK) return pick<(KK < 32 ? KK + 1 : KK + 4)>(kk, k);
        constexpr int HW = KK <= 16 ? 16 : (KK <= 32 ? 32 : 64);
        k->fn = reinterpret_cast<const void *>(&k_vit_chain<KK, HW>);
        k->kr = vit_kr(KK);
        k->segs = 64 / HW;
        k->fixed = VitLds<vit_kr(KK), HW>::fixed;
    }
}

}  // namespace

VitChainPlan make_vit_chain_plan(int K, int64_t T, int64_t product_len)
{
    VitChainPlan cp;
    if (T < kVitChainMinT || K > 80) return cp;
    pick<1>(K <= 32 ? K : vit_kr(K), &cp);
    // A SIMD with o wavefronts takes about 0.17 + 0.2 o us for a step of each
    // (K = 25; warm-up steps, without backpointers, 0.6 of that), so with
    // o = T / (L segs 1024) the call is fastest near L = sqrt(146 o L).  Longer
    // than 256 (192) the backpointers leave too few wavefronts on a CU (K = 50,
    // T = 1e6: 735 us with 160, 750 with 224, 851 with 320).
    const double per_simd = (double)T / (double)(cp.segs * kVitSimds);
    const int64_t best = (int64_t)std::sqrt((0.6 * kVitWarm + kVitAhead) / 0.85 * per_simd);
    const int64_t L = std::min<int64_t>(K <= 32 ? 256 : 192, std::max<int64_t>(32, best));
    cp.nb = (T + L - 1) / L;
    cp.len = (int)((T + cp.nb - 1) / cp.nb);
    const int64_t fnb = (T + product_len - 1) / product_len;
    if (!grid_fits((cp.nb + cp.segs - 1) / cp.segs + (fnb + cp.segs - 1) / cp.segs, 64) ||
        !grid_fits((fnb + 3) / 4, 256))
        cp.nb = 0;
    return cp;
}

hipError_t launch_vit_chain(const VitChainPlan &cp, VitChain v, hipStream_t st)
{
    const int64_t flat = (v.fnb + cp.segs - 1) / cp.segs;
    v.cblocks = (int)((v.nb + cp.segs - 1) / cp.segs);
    for (int mode = 0; mode < (v.nb > 1 ? 2 : 1); ++mode) {
        void *args[] = {&v, &mode};
        const hipError_t e = hipLaunchKernel(cp.fn, dim3((unsigned)(v.cblocks + (mode == 0 ? flat : 0))), dim3(64),
                                             args, cp.lds(), st);
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)((v.fnb + 3) / 4));
    if (v.K > 32) hipLaunchKernelGGL(k_vit_path_score<true>, grid, dim3(256), 0, st, v);
    else hipLaunchKernelGGL(k_vit_path_score<false>, grid, dim3(256), 0, st, v);
    return hipGetLastError();
}

}  // namespace hmmh
