// The 2D band kernel for float cells, four columns per lane, 10, 12 and 16 fused steps.
#include "hx_stencil2d.hpp"

namespace hx {

// Ten levels: whether the waves follow one another on a SIMD (three run there at
// once) or all run from the start, where the short fill is the faster one
// (hx_stencil2d.hpp; ragged rows always take that).
static bool many_waves(const Band2D* b, int n, const Geom2D& g) {
    const int64_t strips = (b[0].nx + 255 - 2 * g.halo) / (256 - 2 * g.halo);
    int64_t waves = 0;
    for (int k = 0; k < n; ++k) waves += strips * ((b[k].ny + g.rows - 1) / g.rows);
    return waves > 3 * 1024;
}

hipError_t launch_stencil2d_f32_deep(const Band2D* b, int n, const Geom2D& g, hipStream_t st) {
    switch (g.steps) {
    case 10: return many_waves(b, n, g) ? launch_cd<float, 4, 10, true>(b, n, g, st)
                                        : launch_cd<float, 4, 10>(b, n, g, st);
    case 12: return launch_cd<float, 4, 12>(b, n, g, st);
    case 16: return launch_cd<float, 4, 16>(b, n, g, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace hx
