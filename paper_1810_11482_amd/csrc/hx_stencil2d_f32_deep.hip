// The 2D band kernel for float cells, four columns per lane, 10, 12 and 16 fused steps.
#include "hx_stencil2d.hpp"

namespace hx {

hipError_t launch_stencil2d_f32_deep(const Band2D* b, int n, const Geom2D& g, hipStream_t st) {
    switch (g.steps) {
    case 10: return launch_cd<float, 4, 10>(b, n, g, st);
    case 12: return launch_cd<float, 4, 12>(b, n, g, st);
    case 16: return launch_cd<float, 4, 16>(b, n, g, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace hx
