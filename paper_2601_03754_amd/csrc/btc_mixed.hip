// Mixed-precision factorization level kernel, block sizes n <= 64.
#include "btc_node.h"

namespace btc {

// Padded tile of the mixed kernels: at least one 16 x 16 matrix-core tile.
int padded_block_mixed(int n) {
    const int np = padded_block(n);
    return (np != 0 && np < 16) ? 16 : np;
}

hipError_t launch_factor_mixed(const Launch<FactorDesc>& p, int np, bool bf16, int64_t items, hipStream_t st) {
    return bf16 ? node::launch_factor_node<2>(p, np, items, st) : node::launch_factor_node<1>(p, np, items, st);
}

}  // namespace btc
