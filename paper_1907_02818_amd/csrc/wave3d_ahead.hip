// Launches of the march of ahead3d.hpp for the 3-D wave adjoint.
#include "ahead3d.hpp"

namespace sadj {

template <class T, int R, int UPREV> static hipError_t launch_uprev(AheadShape shape, const AheadArgs &a, unsigned pad, hipStream_t stream)
{
    return launch_ahead<StarOp::WaveAdjoint, T, R, UPREV>(shape, a, pad, stream);
}

template <class T, int R> static hipError_t launch_R(AheadShape shape, const AheadArgs &a, unsigned pad, hipStream_t stream)
{
    if (a.m.in2) return a.m.out1 ? launch_uprev<T, R, 4>(shape, a, pad, stream) : launch_uprev<T, R, 3>(shape, a, pad, stream);
    if (!a.m.out1) return launch_uprev<T, R, 0>(shape, a, pad, stream);
    return a.m.out1_assign ? launch_uprev<T, R, 2>(shape, a, pad, stream) : launch_uprev<T, R, 1>(shape, a, pad, stream);
}

template <class T> static hipError_t launch_T(AheadShape shape, int radius, const AheadArgs &a, unsigned pad, hipStream_t stream)
{
    switch (radius) {
    case 1: return launch_R<T, 1>(shape, a, pad, stream);
    case 2: return launch_R<T, 2>(shape, a, pad, stream);
    case 3: return launch_R<T, 3>(shape, a, pad, stream);
    default: return launch_R<T, 4>(shape, a, pad, stream);
    }
}

hipError_t launch_adjoint_wave3d_ahead(int is_f64, int radius, const AheadArgs &a, AheadShape shape, unsigned pad, hipStream_t stream)
{
    return is_f64 ? launch_T<double>(shape, radius, a, pad, stream) : launch_T<float>(shape, radius, a, pad, stream);
}

}  // namespace sadj
