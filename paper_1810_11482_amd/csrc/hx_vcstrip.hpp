// Which cells a lane of a fused variable-coefficient pass holds, and which of
// them it stores.  A wave holds a strip of 64 lanes x 4 columns; the strips
// overlap by one lane on each side, and lanes 1 .. 62 store.  The accumulator
// of the reverse sweep is updated in place, so every cell of a row has exactly
// one storing lane.  (No HIP header: the host checks the mapping, too.)
#pragma once

#include <stdint.h>

namespace hx {

constexpr int kVcCols = 4;  // columns per lane
constexpr int kVcStripCols = 62 * kVcCols;  // columns a strip stores

constexpr int64_t vc_strips(int64_t nx) { return (nx + kVcStripCols - 1) / kVcStripCols; }

// The lane's first column (negative, or nx and more: outside the domain).
constexpr int64_t vc_lane_column(int64_t strip, int lane) {
    return strip * kVcStripCols + (int64_t)(lane - 1) * kVcCols;
}

// The lane at column xl stores those of its cells that lie inside [0, nx).
// Lane 63 holds cells of the next strip's lane 1 also where a row ends among
// them; only lane 1 stores those.
constexpr bool vc_lane_stores(int lane, int64_t xl, int64_t nx) {
    return lane >= 1 && lane <= 62 && xl < nx;
}

}  // namespace hx
