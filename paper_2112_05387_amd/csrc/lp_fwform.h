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

// fp32 blocks whose operands lie in LDS as three bf16 parts: all but 16 x 16 channels, whose sums over the most pixels would lose
// precision by it, and image-facing layers
LP_FW_HD constexpr bool fwgrad_split(int Cin, int Cout, int esz) { return esz == 4 && Cin >= 16 && (Cin > 16 || Cout > 16); }

// f(micro-tiles of filter columns, image-facing, operands in three bf16 parts), all three as types.  A layer that does not face the image
// has a micro-tile for each of its R * R taps: the body writes exactly that many columns.
template <int ESZ, class F> LP_FW_HD void fwgrad_form(int Cin, int Cout, int R, F f) {
    typedef std::integral_constant<bool, ESZ == 4> fp32;
    typedef std::integral_constant<int, 9> nine;
    typedef std::integral_constant<int, 1> one;
    if (Cin < 16) f(std::integral_constant<int, 2>(), std::true_type(), std::false_type());
    else if (fwgrad_split(Cin, Cout, ESZ)) {
        if (R == 3) f(nine(), std::false_type(), fp32());
        else f(one(), std::false_type(), fp32());
    } else {
        if (R == 3) f(nine(), std::false_type(), std::false_type());
        else f(one(), std::false_type(), std::false_type());
    }
}

}  // namespace lp
