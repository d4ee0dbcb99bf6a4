// Banded LU with a pivot wavefront (getrf_split.hpp), any number of update
// wavefronts, instantiated for kl + 1 = 2..16 (one file per range keeps
// compiles parallel).
#include "getrf_split.hpp"

namespace bandlu {

WinKernel split_kernel_h2_16(int H) {
    static constexpr auto table = SplitRange<2, 16, 1, 0>::make(std::make_integer_sequence<int, 16 - 2 + 1>{});
    return (H >= 2 && H <= 16) ? table[H - 2] : nullptr;
}

}  // namespace bandlu
