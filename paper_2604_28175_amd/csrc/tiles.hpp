// Where a workgroup's tile lies and which pixel a row of it is, without dividing: the launcher has prepared the divisors (kernels.hpp).
#pragma once
#include "kernels.hpp"

namespace strait {

// Hardware workgroup id b of nb runs on XCD b mod 8; each XCD gets a contiguous range.
__device__ __forceinline__ int xcd_range(int nb, int b) {
    const int per = nb >> 3, rem = nb & 7, xcd = b & 7, idx = b >> 3;
    return xcd * per + (xcd < rem ? xcd : rem) + idx;
}
__device__ __forceinline__ void place_tile(const TileOrder& o, int tile, int& tm, int& tn) {
    const int g = divide(tile, o.by_group), r = tile - g * o.group;
    const bool whole = g < o.full;
    const Divisor by{whole ? o.by_cw.mul : o.by_last.mul, whole ? o.by_cw.shift : o.by_last.shift};
    tm = divide(r, by);
    tn = g * o.cw + (r - tm * (whole ? o.cw : o.last));
}
// Bit r S + s: whether tap (r, s) of a window with its top left corner at (h, w) lies inside the image.
__device__ __forceinline__ unsigned taps_inside(const ConvParams& p, int h, int w) {
    unsigned columns = 0, mask = 0;
    for (int s = 0; s < p.S; ++s) columns |= (unsigned)(w + s) < (unsigned)p.W ? 1u << s : 0u;
    for (int r = 0; r < p.R; ++r) mask |= (unsigned)(h + r) < (unsigned)p.H ? columns << (r * p.S) : 0u;
    return mask;
}
// Image, row and column of slot v of a bordered numbering (the 3x3 kernels that hold a patch): an image is by_image's H + 1 rows of by_row's `pitch` slots.
__device__ __forceinline__ void bordered_place(const ConvParams& p, int v, int pitch, int& img, int& y, int& x) {
    img = divide(v, p.by_image);
    const int rem = v - img * (p.H + 1) * pitch;
    y = divide(rem, p.by_row);
    x = rem - y * pitch;
}

}  // namespace strait
