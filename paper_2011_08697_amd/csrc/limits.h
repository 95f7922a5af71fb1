// limits.h -- bounds that the host decides before it launches (plain C++, compiled by the CPU tests too).
#pragma once

namespace ftk {

// Hits that the 32-bit hit indices hold.
constexpr long long kMaxHits = 0xFFFFFFFELL;

// True when the offsets of one more 2D step fit the 32-bit hit indices whatever the step holds (12 faces a vertex), given
// `total` <= kMaxHits hits before it.  Only then may kernels read the step's offsets before the host has read its total.
constexpr bool step_fits(long long total, long long vertices) { return vertices <= (kMaxHits - total) / 12; }

}  // namespace ftk
