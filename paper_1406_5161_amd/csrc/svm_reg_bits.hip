// svm_reg_bits.hip -- instances of the register-resident SMO loop for bitset rows.
#include "svm_regloop.h"

namespace svm {

template <typename KT>
static const void* pick(int W4, int R) {
    switch (W4) {
        case 1: return reg_pick_rows<true, KT, 1>(R);
        case 2: return reg_pick_rows<true, KT, 2>(R);
        case 3: return reg_pick_rows<true, KT, 3>(R);
        case 4: return reg_pick_rows<true, KT, 4>(R);
        case 6: return reg_pick_rows<true, KT, 6>(R);
        case 8: return reg_pick_rows<true, KT, 8>(R);
        default: return nullptr;
    }
}

const void* reg_fn_bits(bool fp64, int W4, int R) { return fp64 ? pick<double>(W4, R) : pick<float>(W4, R); }

}  // namespace svm
