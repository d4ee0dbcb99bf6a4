// Banded LU with a pivot wavefront (getrf_split.hpp), any number of update
// wavefronts, instantiated for kl + 1 = 17..24 (one file per range keeps
// compiles parallel).
#include "getrf_split.hpp"

namespace bandlu {

WinKernel split_kernel_h17_24(int H) {
    static constexpr auto table = SplitRange<17, 24, 1, 0>::make(std::make_integer_sequence<int, 24 - 17 + 1>{});
    return (H >= 17 && H <= 24) ? table[H - 17] : nullptr;
}

}  // namespace bandlu
