// Dispatch of the curve-ordered select by operand type and contraction length.
#include "knn_tree.h"

namespace kvb {

hipError_t launch_select_tree(int split, const void* Aq, const void* Bc, int n, int kpad, int kp, const float* ynorm2,
                              const unsigned* rmax, ErrModel em, uint64_t* lists, int cap, float* lb,
                              const CurveArgs& crv, unsigned long long* pairs, hipStream_t st)
{
    const int ks = kpad / mfma_kstep(split);
    const TreeCall c = {Aq, Bc, n, kp, ynorm2, rmax, em, lists, cap, lb, crv, pairs, st};
    const hipError_t e = split == 0 ? (ks <= 32 ? tree_f32(ks, c) : tree_f32_wide(ks, c))
                                    : (ks <= 10 ? tree_bf16(ks, c) : tree_bf16_wide(ks, c));
    if (e != hipSuccess || !tree_long(split, ks) || tree_wide_min(true, crv.layout.cnt[0]) >= TREACH) return e;
    // the query tiles handed over
    return launch_select_mfma(split, Aq, Bc, n, kpad, kp, ynorm2, rmax, em, lists, cap, lb, nullptr, 0, &crv, pairs, st);
}

}  // namespace kvb
