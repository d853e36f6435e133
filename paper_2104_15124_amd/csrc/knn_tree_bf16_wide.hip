// The curve-ordered select of BF16 operands beyond 10 K-steps.
#include "knn_tree.h"

namespace kvb {

hipError_t tree_bf16_wide(int ks, const TreeCall& c)
{
    switch (ks) {
    case 13: return launch_tree<TraitsBF16, 13>(c);
    case 16: return launch_tree<TraitsBF16, 16>(c);
    case 20: return launch_tree<TraitsBF16, 20>(c);
    case 25: return launch_tree<TraitsBF16, 25>(c);
    case 32: return launch_tree<TraitsBF16, 32>(c);
    default: return hipErrorNotSupported;
    }
}

}  // namespace kvb
