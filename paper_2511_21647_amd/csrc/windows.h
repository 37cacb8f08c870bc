// What the kernels' buffer descriptors cover, as plain functions of the sizes, so that
// the host can check them without a GPU (tests/test_descriptor_windows.py).
//
// A descriptor holds a 32-bit length, and a load outside it returns zero.  That rests on
// the vector offset alone: a load's scalar offset is not part of the bounds check that
// the compiler documents, so a row or frame is never excluded by one.
#pragma once

#include <stddef.h>

namespace ulm {

constexpr int kMotFrames = 32;     // motion estimation: frames per work-group (the MFMA's M)
constexpr int kMotRows = 16;       // slice rows per work-group
constexpr int kMotStage = 128;     // pixels staged in LDS per step

struct Window {
    size_t at;      // its first value
    int bytes;      // its length
};

// The band of `rows` rows from z0 on of frame f of slice s: none of a frame past the last.
// One band's bytes are bounded by the reference band that LDS holds, whatever the slice's.
constexpr Window mot_window(int s, int F, int f, int nz, int nu, int z0, int rows) {
    const size_t frame = (size_t)nz * nu;
    if (f >= F) return {(size_t)s * F * frame, 0};
    return {((size_t)s * F + f) * frame + (size_t)z0 * nu, rows * nu * 8};
}

// Network training: the columns [first, first + n) of a row of W pixels that a strip of 32
// from column sx on reads with `halo` columns on either side.
constexpr int kStripCols = 32;

struct Columns {
    int first, n;
};

constexpr Columns strip_columns(int W, int sx, int halo) {
    const int first = sx > halo ? sx - halo : 0, end = sx + kStripCols + halo;
    return {first, (end < W ? end : W) - first};
}

}  // namespace ulm
