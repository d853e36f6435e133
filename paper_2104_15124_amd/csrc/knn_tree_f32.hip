// The curve-ordered select of FP32 operands of up to 32 K-steps.
#include "knn_tree.h"

namespace kvb {

hipError_t tree_f32(int ks, const TreeCall& c)
{
    switch (ks) {
    case 2: return launch_tree<TraitsF32, 2>(c);
    case 4: return launch_tree<TraitsF32, 4>(c);
    case 6: return launch_tree<TraitsF32, 6>(c);
    case 8: return launch_tree<TraitsF32, 8>(c);
    case 10: return launch_tree<TraitsF32, 10>(c);
    case 12: return launch_tree<TraitsF32, 12>(c);
    case 16: return launch_tree<TraitsF32, 16>(c);
    case 24: return launch_tree<TraitsF32, 24>(c);
    case 32: return launch_tree<TraitsF32, 32>(c);
    default: return hipErrorNotSupported;
    }
}

}  // namespace kvb
