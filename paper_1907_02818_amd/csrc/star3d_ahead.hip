// Launches of the march of ahead3d.hpp for the free-weight star, both directions.
#include "ahead3d.hpp"

namespace sadj {

template <StarOp OP, class T> static hipError_t launch_T(AheadShape shape, int radius, const AheadArgs &a, unsigned pad, hipStream_t stream)
{
    switch (radius) {
    case 1: return launch_ahead<OP, T, 1, 0>(shape, a, pad, stream);
    case 2: return launch_ahead<OP, T, 2, 0>(shape, a, pad, stream);
    case 3: return launch_ahead<OP, T, 3, 0>(shape, a, pad, stream);
    default: return launch_ahead<OP, T, 4, 0>(shape, a, pad, stream);
    }
}

hipError_t launch_star3d_ahead(int adjoint, int is_f64, int radius, const AheadArgs &a, AheadShape shape, unsigned pad, hipStream_t stream)
{
    if (adjoint)
        return is_f64 ? launch_T<StarOp::StarAdjoint, double>(shape, radius, a, pad, stream)
                      : launch_T<StarOp::StarAdjoint, float>(shape, radius, a, pad, stream);
    return is_f64 ? launch_T<StarOp::StarPrimal, double>(shape, radius, a, pad, stream)
                  : launch_T<StarOp::StarPrimal, float>(shape, radius, a, pad, stream);
}

}  // namespace sadj
