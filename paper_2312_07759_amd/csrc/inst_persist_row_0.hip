// Instantiations of the persistent row <-> vector kernels for energy variant 0.
#include "dispatch.h"
#include "persist_lane.hpp"

namespace idkm {

template <int KB, int D>
static PersistFns pick(bool bwd) {
    return bwd ? PersistFns{persist_row_bwd<KB, D, 0>, persist_row_bwd_batch<KB, D, 0>, false, RT}
               : PersistFns{persist_row_fwd<KB, D, 0>, persist_row_fwd_batch<KB, D, 0>, false, RT};
}

// Offered for d <= 2 and k <= 256.
PersistFns persist_row_kernel_0(int KB, int D, bool bwd) {
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
