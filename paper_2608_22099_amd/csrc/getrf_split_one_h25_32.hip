// Banded LU with a pivot wavefront (getrf_split.hpp), one update wavefront
// (windows of at most 64 columns), instantiated for kl + 1 = 25..32.
#include "getrf_split.hpp"

namespace bandlu {

WinKernel split_one_h25_32(int H) {
    static constexpr auto table = SplitRange<25, 32, 1, 1>::make(std::make_integer_sequence<int, 32 - 25 + 1>{});
    return (H >= 25 && H <= 32) ? table[H - 25] : nullptr;
}

}  // namespace bandlu
