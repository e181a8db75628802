// Where the lanes of a wavefront put the columns of a row that they hold side by side (no HIP).
#pragma once

namespace als {

// Columns of a row of d that a lane holds: two adjacent ones, one where d < 128.
constexpr int columns_per_lane(int d) { return d >= 128 ? 2 : 1; }
// Whether `lane` holds any: with d = 32 the upper half of the wavefront does not.
constexpr bool holds_columns(int d, int lane) { return lane * columns_per_lane(d) < d; }
// Copies of several rows in LDS: floats from one to the next (16-byte reads of eight rows meet in different groups of banks), and
// the place of the columns of row n that `lane` holds.  Only lanes that hold columns may store: what the others would write belongs to
// row n + 1, and no order is defined between the stores of different lanes.
constexpr int row_copy_stride(int d) { return d + 4; }
constexpr int row_copy_place(int d, int n, int lane) { return n * row_copy_stride(d) + lane * columns_per_lane(d); }

}  // namespace als
