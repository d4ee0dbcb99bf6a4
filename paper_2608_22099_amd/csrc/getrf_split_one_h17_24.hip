// Banded LU with a pivot wavefront (getrf_split.hpp), one update wavefront
// (windows of at most 64 columns), instantiated for kl + 1 = 17..24.
#include "getrf_split.hpp"

namespace bandlu {

WinKernel split_one_h17_24(int H) {
    static constexpr auto table = SplitRange<17, 24, 1, 1>::make(std::make_integer_sequence<int, 24 - 17 + 1>{});
    return (H >= 17 && H <= 24) ? table[H - 17] : nullptr;
}

}  // namespace bandlu
