// The curve-ordered select of BF16 operands of up to 10 K-steps.
#include "knn_tree.h"

namespace kvb {

hipError_t tree_bf16(int ks, const TreeCall& c)
{
    switch (ks) {
    case 2: return launch_tree<TraitsBF16, 2>(c);
    case 3: return launch_tree<TraitsBF16, 3>(c);
    case 4: return launch_tree<TraitsBF16, 4>(c);
    case 5: return launch_tree<TraitsBF16, 5>(c);
    case 6: return launch_tree<TraitsBF16, 6>(c);
    case 7: return launch_tree<TraitsBF16, 7>(c);
    case 8: return launch_tree<TraitsBF16, 8>(c);
    case 10: return launch_tree<TraitsBF16, 10>(c);
    default: return hipErrorNotSupported;
    }
}

}  // namespace kvb
