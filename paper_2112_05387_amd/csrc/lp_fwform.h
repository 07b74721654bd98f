// Which form of the narrow filter-gradient kernel (lp_fwgrad.hip) takes a layer.  One rule for the kernel's dispatch, for the
// LDS the launcher asks for and for the host's own test.
#pragma once
#include <type_traits>
#ifdef __HIPCC__
#define LP_FW_HD __host__ __device__ inline
#else
#define LP_FW_HD inline
#endif

namespace lp {

// f(micro-tiles of filter columns, image-facing), both as types.  A layer that does not face the image has a micro-tile for each
// of its R * R taps: the body writes exactly that many columns.
template <class F> LP_FW_HD void fwgrad_form(int Cin, int R, F f) {
    if (Cin < 16) f(std::integral_constant<int, 2>(), std::true_type());
    else if (R == 3) f(std::integral_constant<int, 9>(), std::false_type());
    else f(std::integral_constant<int, 1>(), std::false_type());
}

}  // namespace lp
