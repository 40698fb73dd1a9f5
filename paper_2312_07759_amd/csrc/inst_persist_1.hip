// Instantiations of the persistent (one launch per solve) kernels, energy variant 1.
#include "dispatch.h"
#include "persist_small.hpp"

namespace idkm {

template <int K, int D>
static PersistFns pick(bool bwd) {
    if (!bwd) return PersistFns{persist_fwd<K, D, 1>, persist_fwd_batch<K, D, 1>};
    PersistFns f{persist_bwd<K, D, 1>, persist_bwd_batch<K, D, 1>};
    if constexpr (pair_shape(K, D, 1)) {
        f.pairs = persist_bwd<K, D, 1, false, true>;
        f.pairs_batch = persist_bwd_batch<K, D, 1, false, true>;
    }
    return f;
}

// Offered for every shape of the lane<->vector family: K (D+1) <= 80 sums per workgroup.
PersistFns persist_kernel_1(int K, int D, bool bwd) {
    switch (K * 16 + D) {
        case 2 * 16 + 1: return pick<2, 1>(bwd);
        case 4 * 16 + 1: return pick<4, 1>(bwd);
        case 8 * 16 + 1: return pick<8, 1>(bwd);
        case 16 * 16 + 1: return pick<16, 1>(bwd);
        case 2 * 16 + 2: return pick<2, 2>(bwd);
        case 4 * 16 + 2: return pick<4, 2>(bwd);
        case 8 * 16 + 2: return pick<8, 2>(bwd);
        case 2 * 16 + 4: return pick<2, 4>(bwd);
        case 4 * 16 + 4: return pick<4, 4>(bwd);
        case 16 * 16 + 2: return pick<16, 2>(bwd);
        case 8 * 16 + 4: return pick<8, 4>(bwd);
        case 16 * 16 + 4: return pick<16, 4>(bwd);
    }
    return PersistFns{};
}

}  // namespace idkm
