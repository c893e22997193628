// Bounds of the custom reduce's walk over the records of B, in plain C++: 32-bit positions up to 2^31 - 1, so an
// end is never formed by adding to a position that may stand near the last one.
#pragma once

namespace mdh {

// Records of B between two checks of their values: what a value outside costs is the run it stands in, evaluated again.
// The first run is shorter, for values that are outside everywhere (hashes).  us, runs of 512 / these (integer loop from
// the start): 2^13 x 2^15 records of 4 fields, all outside 174 / 121 (124), one in 2000 outside 118 / 101 (123); 2^14 x
// 2^17 of 16 fields, all outside 4430 / 3050 (2760), one in 2000 2820 / 2410 (2740); none outside: equal within 1 %, runs
// of 64 up to 1 % more.
constexpr int kFirstRun = 32, kRun = 128;

// the run of records of [b0, b1) that begins at `done` (done < b1) ends before this one
constexpr int run_end(int done, int b0, int b1) {
  const int run = done == b0 ? kFirstRun : kRun;
  return b1 - done > run ? done + run : b1;
}

// A run is walked in blocks of four: the position after the last block may lie up to three past b1, so a walk is
// taken only up to this many records.
constexpr long long kMaxWalked = 0x7ffffff0;

}  // namespace mdh
