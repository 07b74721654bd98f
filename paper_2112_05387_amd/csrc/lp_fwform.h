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

// f(micro-tiles of filter columns, image-facing, 16 -> 16 channels), all three as types.  A layer that does not face the image has a
// micro-tile for each of its R * R taps: the body writes exactly that many columns.  3x3 filters of 16 to 16 channels in fp32 are told
// apart: a body that knows its widths is the faster one (steps of two blocks on 8 x 8 images, 4 samples: 61.2 -> 59.0 us; of
// ResNet-20, 128 samples in one module: 816 -> 809).
template <int ESZ, class F> LP_FW_HD void fwgrad_form(int Cin, int Cout, int R, F f) {
    typedef std::integral_constant<int, 9> nine;
    typedef std::integral_constant<int, 1> one;
    if (Cin < 16) f(std::integral_constant<int, 2>(), std::true_type(), std::false_type());
    else if (R != 3) f(one(), std::false_type(), std::false_type());
    else if (ESZ == 4 && Cin == 16 && Cout == 16) f(nine(), std::false_type(), std::true_type());
    else f(nine(), std::false_type(), std::false_type());
}

}  // namespace lp
