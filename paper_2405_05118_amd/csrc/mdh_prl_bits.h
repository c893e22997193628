// Custom reduce on bit maps (mdh_custom_reduce_bits.hip): when it is taken, its grid and its memory, in plain C++.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define MDH_PRL_BOTH __host__ __device__
#else
#define MDH_PRL_BOTH
#endif

namespace mdh {

constexpr int kPrlChunk = 128;     // records of B in the maps at a time: a map is the 16 bytes of one LDS read
constexpr int kPrlMaps = 1 << 16;  // bytes of the maps of all fields: two workgroups of 16 wavefronts per compute unit
constexpr int kPrlQueue = 80;      // pairs a wavefront puts off: 64, and one step's
constexpr int kPrlPartBits = 20;   // records of B in a part: a queued pair is 32 bits

// Slots of the fields: 2^bits(f) of them from first(f) on, 4 to 10 bits, together at most 4096.
struct PrlSlots {
  unsigned long long packed;  // four bits a field
  MDH_PRL_BOTH int bits(int f) const { return (int)(packed >> (4 * f)) & 15; }
  MDH_PRL_BOTH unsigned first(int f) const {
    unsigned at = 0;
    for (int i = 0; i < f; ++i) at += 1u << bits(i);
    return at;
  }
};

// As many as the bits in use (`used`, the values seen ORed) ask for; the largest give way if that is too much.
template <int NF>
MDH_PRL_BOTH inline PrlSlots prl_slots(const unsigned (&used)[NF], int nF) {
  int width[NF];
  for (int f = 0; f < NF; ++f) {
    width[f] = 4;
    while (width[f] < 10 && used[f] >> width[f]) ++width[f];
  }
  for (int most = 10;; --most) {
    unsigned all = 0;
    PrlSlots s{0};
    for (int f = 0; f < NF; ++f) {
      const int w = width[f] < most ? width[f] : most;
      if (f < nF) all += 1u << w, s.packed |= (unsigned long long)w << (4 * f);
    }
    if (all <= kPrlMaps / 16) return s;
  }
}

constexpr int kSearch = 64;  // workgroups that look for weights
struct PrlBitsHead {
  int32_t stop;  // 1: the loop over fields has to do it
  int32_t pad;
  unsigned long long bits;  // PrlSlots
  struct {
    unsigned long long q;  // four bits a field
    float cost;
    int32_t pad;
  } found[kSearch];
};

// The head lies at the end of the workspace, in the last of the S parts' results, which the loop over fields (S - 1 parts)
// leaves alone.  After a call its first word tells which of the two the result is from.
inline PrlBitsHead* prl_bits_head(void* ws, int64_t nA, int S) {
  return (PrlBitsHead*)(((uintptr_t)((int32_t*)ws + 2 * (int64_t)S * nA) - sizeof(PrlBitsHead)) & ~(uintptr_t)7);
}

// maps, records of the chunk, the largest scores of 32 sums, the flag, 16 queues, t of the records of A
constexpr int64_t prl_bits_lds_bytes(int nF, int sets) {
  return kPrlMaps + 4ll * kPrlChunk * nF + 4 * 32 + 16 + 16 * 4 * kPrlQueue + 1024ll * sets;
}

// a workgroup owns `sets` x 1024 records of A and walks `chunks` chunks of B
struct PrlBitsGrid {
  int groups, parts, sets, chunks;
};

// Two workgroups a compute unit.  A chunk costs a set of 1024 records of A 4.8, and once more for bringing it into the maps
// 1 (thousand cycles); the first chunk of a part, which finds most of its best records, counts as two more.
inline PrlBitsGrid prl_bits_grid(int64_t nA, int64_t nB, int nF) {
  const int64_t all = (nA + 1023) / 1024, c = (nB + kPrlChunk - 1) / kPrlChunk, most = (1 << kPrlPartBits) / kPrlChunk;
  PrlBitsGrid best{};
  double least = -1;
  for (int sets = 1; sets <= (nF <= 12 ? 4 : 2); ++sets) {
    const int64_t groups = (all + sets - 1) / sets;
    int64_t parts = groups < 512 ? 512 / groups : 1;
    if (parts > c) parts = c;
    if (parts < (c + most - 1) / most) parts = (c + most - 1) / most;
    const int64_t chunks = (c + parts - 1) / parts;
    parts = (c + chunks - 1) / chunks;
    const double t = (double)((groups * parts + 511) / 512) * (chunks + 2) * (4.8 * sets + 1.0);
    if (least < 0 || t < least) {
      least = t;
      best = PrlBitsGrid{(int)groups, (int)parts, sets, (int)chunks};
    }
  }
  return best;
}

// Keys and slots have to fit the workspace of S parts less one.  S is the loop's split, which a caller's workspace has been
// sized for: it falls with more records of A and with fewer of B, and so the maps are not taken from 2^20 records of A on (two
// parts: 2^20 x 2^15 of 8 fields 13.5 ms with the loop, 2^19 x 2^16, four parts, 13.4 / 2.05), for more than 8 fields from 2^19
// (of 10 17.5 ms); nor below 4096 records of B, 8192 for more than 8 fields, where there are 2^15 records of A or more.
// The rest is what the launches and the search for weights take (us, the loop over fields / the maps: 2^12 x 2^14 records of
// 8 fields 63 / 51, 2^13 x 2^14 91 / 60; 2^11 x 2^18 of 12, with a search over 4096 patterns, 525 / 168; 2^11 x 2^15 89 / 100
// when the line was drawn).  Below 1024 records of A most lanes would have none.
inline bool prl_bits_applies(int S, int64_t nA, int64_t nB, int nF) {
  return nF <= 16 && 8 + 4 * ((nF + 1) / 2) <= 8 * (S - 1) && nA >= 1024 &&
         (double)nA * (double)nB * nF >= (nF <= 10 ? 536870912.0 : 2147483648.0);
}

}  // namespace mdh
