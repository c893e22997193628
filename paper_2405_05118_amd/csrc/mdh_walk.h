// Bounds of the custom reduce's walk over the records of B, in plain C++: 32-bit positions up to 2^31 - 1, so an
// end is never formed by adding to a position that may stand near the last one.
#pragma once

namespace mdh {

constexpr int kRun = 512;  // records of B between two checks of their values

// the run of records that begins at `done` (done < b1) ends before this one
constexpr int run_end(int done, int b1) { return b1 - done > kRun ? done + kRun : b1; }

// A run is walked in blocks of four: the position after the last block may lie up to three past b1, so a walk is
// taken only up to this many records.
constexpr long long kMaxWalked = 0x7ffffff0;

}  // namespace mdh
