// Instantiation of the two-leaves-per-wave sweep for stride 32.
#include "search_pair.hpp"

namespace knnx {

hipError_t launch_search_pair_dp32(const SearchArgs &a, int kk, hipStream_t s) {
    return launch_search_pair<32>(a, kk, pair_grid(a.q_n_leaves, a.split != 0), s);
}

}  // namespace knnx
