// Instantiations of the stream path's row <-> vector passes for energy variant 1.
#include "dispatch.h"
#include "row_k.hpp"

namespace idkm {

template <int KB, int D, bool SEVERAL>
static KernelFn pick(int pass) {
    switch (pass) {
        case PASS_FWD: return row_pass<KB, D, 1, PASS_FWD, SEVERAL>;
        case PASS_FIN: return row_pass<KB, D, 1, PASS_FIN, SEVERAL>;
        case PASS_B1: return row_pass<KB, D, 1, PASS_B1, SEVERAL>;
        case PASS_B2: return row_pass<KB, D, 1, PASS_B2, SEVERAL>;
        case PASS_B3: return row_pass<KB, D, 1, PASS_B3, SEVERAL>;
    }
    return nullptr;
}

template <int KB>
static KernelFn pick_d(int D, int pass, bool several) {
    switch (D) {
        case 1: return pick<KB, 1, true>(pass);
        case 2: return pick<KB, 2, true>(pass);
        case 8: return several ? pick<KB, 8, true>(pass) : pick<KB, 8, false>(pass);
    }
    return nullptr;
}

KernelFn row_kernel_1(int KB, int D, int pass, bool several) {
    switch (KB) {
        case 1: return pick_d<1>(D, pass, several);
        case 2: return pick_d<2>(D, pass, several);
        case 4: return pick_d<4>(D, pass, several);
        case 8: return pick_d<8>(D, pass, several);
        case 16: return pick_d<16>(D, pass, several);
    }
    return nullptr;
}

}  // namespace idkm
