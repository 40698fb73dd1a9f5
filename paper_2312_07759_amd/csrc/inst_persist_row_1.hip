// Instantiations of the persistent row <-> vector kernels for energy variant 1.
#include "dispatch.h"
#include "persist_lane.hpp"

namespace idkm {

template <int KB, int D>
static PersistFns pick(bool bwd) {
    return bwd ? PersistFns{persist_row_bwd<KB, D, 1>, persist_row_bwd_batch<KB, D, 1>, false, RT}
               : PersistFns{persist_row_fwd<KB, D, 1>, persist_row_fwd_batch<KB, D, 1>, false, RT};
}

// d = 8: the forward solve only (the backward's tables and partial sums do not fit the LDS beside the tiles).
template <int KB>
static PersistFns pick_forward_8() {
    return PersistFns{persist_row_fwd<KB, 8, 1>, persist_row_fwd_batch<KB, 8, 1>, false, RT};
}

// Offered for d in {1, 2, 8} and k <= 256.
PersistFns persist_row_kernel_1(int KB, int D, bool bwd) {
    if (D == 8 && !bwd) {
        switch (KB) {
            case 1: return pick_forward_8<1>();
            case 2: return pick_forward_8<2>();
            case 4: return pick_forward_8<4>();
            case 8: return pick_forward_8<8>();
            case 16: return pick_forward_8<16>();
        }
    }
    switch (KB * 16 + D) {
        case 1 * 16 + 1: return pick<1, 1>(bwd);
        case 2 * 16 + 1: return pick<2, 1>(bwd);
        case 4 * 16 + 1: return pick<4, 1>(bwd);
        case 8 * 16 + 1: return pick<8, 1>(bwd);
        case 16 * 16 + 1: return pick<16, 1>(bwd);
        case 1 * 16 + 2: return pick<1, 2>(bwd);
        case 2 * 16 + 2: return pick<2, 2>(bwd);
        case 4 * 16 + 2: return pick<4, 2>(bwd);
        case 8 * 16 + 2: return pick<8, 2>(bwd);
        case 16 * 16 + 2: return pick<16, 2>(bwd);
    }
    return PersistFns{};
}

}  // namespace idkm
