// svm_reg_dense.hip -- instances of the register-resident SMO loop for dense rows.
#include "svm_regloop.h"

namespace svm {

template <typename KT>
static const void* pick(int W4, int R) {
    switch (W4) {
        case 1: return reg_pick_rows<false, KT, 1>(R);
        case 2: return reg_pick_rows<false, KT, 2>(R);
        case 3: return reg_pick_rows<false, KT, 3>(R);
        case 4: return reg_pick_rows<false, KT, 4>(R);
        case 5: return reg_pick_rows<false, KT, 5>(R);
        case 6: return reg_pick_rows<false, KT, 6>(R);
        case 7: return reg_pick_rows<false, KT, 7>(R);
        case 8: return reg_pick_rows<false, KT, 8>(R);
        case 12: return reg_pick_rows<false, KT, 12>(R);
        case 16: return reg_pick_rows<false, KT, 16>(R);
        case 24: return reg_pick_rows<false, KT, 24>(R);
        case 32: return reg_pick_rows<false, KT, 32>(R);
        default: return nullptr;
    }
}

const void* reg_fn_dense(bool fp64, int W4, int R) { return fp64 ? pick<double>(W4, R) : pick<float>(W4, R); }

}  // namespace svm
