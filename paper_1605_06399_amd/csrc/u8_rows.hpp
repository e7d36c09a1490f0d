// Addresses of the unsigned char walk: which bytes of the image a strip of 256 columns reads.  Plain constexpr
// arithmetic of the host and the device, so that a host test can enumerate every read against the image's extent.
#pragma once
#include <cstddef>

namespace icl {

constexpr int U8_COLS = 256;    // output columns of a strip
constexpr int U8_LEFT = 8;      // a strip at column xs reads columns xs - 8 .. xs + 263
constexpr int U8_RIGHT = 264;

// first of the 16 columns that lane n + 16 g reads
constexpr int u8_col(int xs, int n, int g) { return xs - U8_LEFT + 16 * n + 16 * (g & 1); }

// every column the strip reads lies in the rows
constexpr bool u8_inside(int xs, int W) { return xs >= U8_LEFT && xs + U8_RIGHT <= W; }

// The first row whose columns must not be read straight, for every strip: the last strip's read ends at byte xs + 264
// of its row, the image at byte W of its last row, so that as many rows must follow as the difference takes.  H - 1 in
// most images, H - 16 where W = 16 (a strip's reads reach over several rows shorter than they are).
constexpr int u8_tail(int W, int H, unsigned sp) {
    const int over = (W - 1) / U8_COLS * U8_COLS + U8_RIGHT - W;   // 8 at least
    return H - (int)(((unsigned)over + sp - 1) / sp);
}

// The row pair (q, q + 1) is read from clamped columns.  The others are read straight, into the padding or the neighbour
// rows on both sides: a row lies before the first (16 bytes or more, for the 8 on the left) and enough after the second.
constexpr bool u8_guarded(int q, int tail) { return q <= 0 || q + 1 >= tail; }

// The row that stands for row q, and a lane's offset from its first byte: `second` is the row pitch for lanes of row
// q + 1 and 0 for those of row q, cb the lane's column c clamped to 0 .. W - 16.
constexpr int u8_row(int q, int H) {
    const int at = q > 0 ? q : 0, last = H - 1;   // a minimum and a maximum
    return at < last ? at : last;
}
constexpr ptrdiff_t u8_lane(int q, int H, int tail, unsigned second, int c, int cb) {
    return (ptrdiff_t)(q >= 0 && q + 1 < H ? second : 0u) + c + (-(int)u8_guarded(q, tail) & (cb - c));
}

}  // namespace icl
