// Instantiation of the traversal kernel with matrix-core tiles for 8 computed
// dimensions (plain form).
#include "search_valu.hpp"

namespace knnx {
hipError_t launch_search_mt_d8(const SearchArgs &a, int K, int grid, hipStream_t s) {
    return launch_search_valu_mt<8>(a, K, grid, s);
}
}  // namespace knnx
