// Instantiations of the one-query-per-wave kernel.
#include "search_few.hpp"

namespace knnx {

hipError_t launch_search_few_d(const SearchArgs &a, int d, int64_t n_q, hipStream_t s) {
    switch (d <= 4 ? d : pad_dim(d)) {
        case 1: return launch_search_few<1>(a, n_q, s);
        case 2: return launch_search_few<2>(a, n_q, s);
        case 3: return launch_search_few<3>(a, n_q, s);
        case 4: return launch_search_few<4>(a, n_q, s);
        case 8: return launch_search_few<8>(a, n_q, s);
        case 16: return launch_search_few<16>(a, n_q, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace knnx
