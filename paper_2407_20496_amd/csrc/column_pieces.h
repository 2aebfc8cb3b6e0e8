// Which 16-byte pieces of a row of X the kernels with 16-column blocks load.
//
// X is readable up to column 8 ceil(N / 8) - 1 of every row, the last row included, and no further: the leading dimension
// may be wider than that while the last row ends there (the last columns of a wider matrix).  So a piece is loaded only if
// it begins inside N.  Host code can include this header: the bounds are checked there.
#pragma once

namespace hinm {

// The piece that begins at column `first` holds at least one of the N columns (first a multiple of 8).
constexpr bool piece_inside(int first, int N) { return first < N; }

// Offset of a lane's half (0 or 1) of the 16-column block at n0 < N; the second half, where it holds none of the N
// columns, repeats the first: what it feeds is never stored.
constexpr int half_offset(int n0, int half, int N) { return piece_inside(n0 + 8 * half, N) ? 8 * half : 0; }

}  // namespace hinm
