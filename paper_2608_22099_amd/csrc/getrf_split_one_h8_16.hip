// Banded LU with a pivot wavefront (getrf_split.hpp), one update wavefront
// (windows of at most 64 columns), instantiated for kl + 1 = 8..16.
#include "getrf_split.hpp"

namespace bandlu {

WinKernel split_one_h8_16(int H) {
    static constexpr auto table = SplitRange<8, 16, 1, 1>::make(std::make_integer_sequence<int, 16 - 8 + 1>{});
    return (H >= 8 && H <= 16) ? table[H - 8] : nullptr;
}

}  // namespace bandlu
