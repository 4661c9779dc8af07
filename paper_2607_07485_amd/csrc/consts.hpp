// Sizes shared by the host driver and the device code.
#pragma once

#include <cstdint>

namespace lsdd {

// Doubles per tridiagonal row of the inverse-iteration scratch: 64 solving lanes x
// (reciprocal pivots, two superdiagonals, iterate, multipliers), and the row-exchange bits
// (64 words per 8 rows).
constexpr int INVIT_SLOTS = 5 * 64 + 4;
// Doubles of scratch one workgroup of the inverse iteration needs for n rows: the slots, the
// exchange bits of a last partial block, and 64 x 64 dots.
constexpr int64_t invit_ws(int64_t n) { return INVIT_SLOTS * n + 64 + 64 * 64; }

}  // namespace lsdd
