// Banded LU with a pivot wavefront (getrf_split.hpp), one update wavefront
// (windows of at most 64 columns), instantiated for kl + 1 = 2..16.
#include "getrf_split.hpp"

namespace bandlu {

WinKernel split_one_h2_16(int H) {
    static constexpr auto table = SplitRange<2, 16, 1, 1>::make(std::make_integer_sequence<int, 16 - 2 + 1>{});
    return (H >= 2 && H <= 16) ? table[H - 2] : nullptr;
}

}  // namespace bandlu
