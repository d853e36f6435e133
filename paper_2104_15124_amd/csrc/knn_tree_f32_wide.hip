// The curve-ordered select of FP32 operands beyond 32 K-steps.
#include "knn_tree.h"

namespace kvb {

hipError_t tree_f32_wide(int ks, const TreeCall& c)
{
    switch (ks) {
    case 48: return launch_tree<TraitsF32, 48>(c);
    case 64: return launch_tree<TraitsF32, 64>(c);
    case 96: return launch_tree<TraitsF32, 96>(c);
    case 128: return launch_tree<TraitsF32, 128>(c);
    default: return hipErrorNotSupported;
    }
}

}  // namespace kvb
