// Launches of the march of ahead3d.hpp for the 3-D wave primal.
#include "ahead3d.hpp"

namespace sadj {

template <class T> static hipError_t launch_T(AheadShape shape, int radius, const AheadArgs &a, unsigned pad, hipStream_t stream)
{
    switch (radius) {
    case 1: return launch_ahead<StarOp::WavePrimal, T, 1, 0>(shape, a, pad, stream);
    case 2: return launch_ahead<StarOp::WavePrimal, T, 2, 0>(shape, a, pad, stream);
    case 3: return launch_ahead<StarOp::WavePrimal, T, 3, 0>(shape, a, pad, stream);
    default: return launch_ahead<StarOp::WavePrimal, T, 4, 0>(shape, a, pad, stream);
    }
}

hipError_t launch_primal_wave3d_ahead(int is_f64, int radius, const AheadArgs &a, AheadShape shape, unsigned pad, hipStream_t stream)
{
    return is_f64 ? launch_T<double>(shape, radius, a, pad, stream) : launch_T<float>(shape, radius, a, pad, stream);
}

}  // namespace sadj
