// FP64 factorization level kernel on matrix cores, block sizes n <= 64.
#include "btc_node.h"

namespace btc {

hipError_t launch_factor_mfma(const Launch<FactorDesc>& p, int np, int64_t items, hipStream_t st) {
    return node::launch_factor_node<0>(p, np, items, st);
}

}  // namespace btc
