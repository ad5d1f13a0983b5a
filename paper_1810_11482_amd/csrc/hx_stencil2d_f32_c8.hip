// The 2D band kernel for float cells, eight columns per lane.
#include "hx_stencil2d.hpp"

namespace hx {

hipError_t launch_stencil2d_f32_c8(const Band2D* b, int n, const Geom2D& g, hipStream_t st) {
    switch (g.steps) {
    case 1: return launch_cd<float, 8, 1>(b, n, g, st);
    case 2: return launch_cd<float, 8, 2>(b, n, g, st);
    case 3: return launch_cd<float, 8, 3>(b, n, g, st);
    case 4: return launch_cd<float, 8, 4>(b, n, g, st);
    case 5: return launch_cd<float, 8, 5>(b, n, g, st);
    case 6: return launch_cd<float, 8, 6>(b, n, g, st);
    case 7: return launch_cd<float, 8, 7>(b, n, g, st);
    case 8: return launch_cd<float, 8, 8>(b, n, g, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace hx
