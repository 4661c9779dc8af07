// Sizes shared by the host driver and the device code.
#pragma once

namespace lsdd {

// Doubles per tridiagonal row of the inverse-iteration scratch: 64 solving
// lanes x (u0, u1, u2, iterate), interleaved by lane.
constexpr int INVIT_SLOTS = 4 * 64;
// The same for the blocked path: 64 lanes x (reciprocal pivots, two superdiagonals, iterate,
// multipliers), and the row-exchange bits (64 words per 8 rows).
constexpr int INVIT_BLK_SLOTS = 5 * 64 + 4;

}  // namespace lsdd
