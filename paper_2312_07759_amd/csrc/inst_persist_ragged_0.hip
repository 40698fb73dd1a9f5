// Persistent kernels of the lane<->vector family for codebooks whose size is not a power of two, energy variant 0.
#include "dispatch.h"
#include "persist_small.hpp"

namespace idkm {

template <int K, int D>
static PersistFns pick(bool bwd) {
    if (!bwd) return PersistFns{persist_fwd<K, D, 0, true>, persist_fwd_batch<K, D, 0, true>};
    PersistFns f{persist_bwd<K, D, 0, true>, persist_bwd_batch<K, D, 0, true>};
    if constexpr (pair_shape(K, D, 0)) {
        f.pairs = persist_bwd<K, D, 0, true, true>;
        f.pairs_batch = persist_bwd_batch<K, D, 0, true, true>;
    }
    return f;
}

PersistFns persist_kernel_ragged_0(int K, int D, bool bwd) {
    switch (K * 16 + D) {
        case 4 * 16 + 1: return pick<4, 1>(bwd);
        case 8 * 16 + 1: return pick<8, 1>(bwd);
        case 16 * 16 + 1: return pick<16, 1>(bwd);
        case 4 * 16 + 2: return pick<4, 2>(bwd);
        case 8 * 16 + 2: return pick<8, 2>(bwd);
        case 16 * 16 + 2: return pick<16, 2>(bwd);
        case 4 * 16 + 4: return pick<4, 4>(bwd);
        case 8 * 16 + 4: return pick<8, 4>(bwd);
        case 16 * 16 + 4: return pick<16, 4>(bwd);
    }
    return PersistFns{};
}

}  // namespace idkm
