// Launch of the 2D band kernel: the instantiations live in hx_stencil2d_*.hip.
#include <hip/hip_runtime_api.h>

#include "hx_internal.h"

namespace hx {

hipError_t launch_stencil2d_f32(const Band2D* b, int n, const Geom2D& g, hipStream_t st);
hipError_t launch_stencil2d_f32_deep(const Band2D* b, int n, const Geom2D& g, hipStream_t st);
hipError_t launch_stencil2d_f32_c8(const Band2D* b, int n, const Geom2D& g, hipStream_t st);
hipError_t launch_stencil2d_f64(const Band2D* b, int n, const Geom2D& g, hipStream_t st);

bool stencil2d_supported(int dtype, int cpl, int steps) {
    const bool small = steps >= 1 && steps <= 8;
    const bool deep = steps == 10 || steps == 12 || steps == 16;
    if (dtype == 0 && cpl == 4) return small || deep;
    if (dtype == 0 && cpl == 8) return small;
    return dtype == 1 && cpl == 4 && small;
}

hipError_t launch_stencil2d_bands(int dtype, const Band2D* b, int n, const Geom2D& g,
                                  hipStream_t stream) {
    if (!stencil2d_supported(dtype, g.cpl, g.steps) || n < 1 || n > kMaxBands)
        return hipErrorInvalidValue;
    for (int k = 1; k < n; ++k)
        if (b[k].nx != b[0].nx) return hipErrorInvalidValue;
    if (dtype != 0) return launch_stencil2d_f64(b, n, g, stream);
    if (g.cpl == 8) return launch_stencil2d_f32_c8(b, n, g, stream);
    return g.steps > 8 ? launch_stencil2d_f32_deep(b, n, g, stream)
                       : launch_stencil2d_f32(b, n, g, stream);
}

hipError_t launch_stencil2d(int dtype, const Band2D& b, const Geom2D& g, hipStream_t stream) {
    return launch_stencil2d_bands(dtype, &b, 1, g, stream);
}

}  // namespace hx
