// f64_slabs.hpp -- which k a workgroup of the binary64 tiles reads, and how much
// of B that addresses.  Plain C++ (no HIP), so that a host program can walk it.
#pragma once

namespace mm {
namespace f64 {

constexpr int BK = 16;  // k per slab

// The slabs of one wave group.  The grid of slabs ends exactly at K, so only the
// first of all slabs can be partial (it begins before k = 0 then).  With kg = 2
// the second group starts at slab ceil(all / 2); an odd slab count leaves it one
// slab short, and a single slab leaves it none.
struct Slabs {
  int turns;  // slabs of the first group: both groups take that many steps
  int own;    // slabs of this group
  int base;   // first k of its slab 0
  constexpr Slabs(int K, int kg, int group) : turns(0), own(0), base(0) {
    const int all = (K + BK - 1) / BK;
    turns = (all + kg - 1) / kg;
    own = group ? all - turns : turns;
    base = K - all * BK + group * turns * BK;
  }
  // First k of slab s.  Loads past the last slab are clamped to it (never
  // multiplied), so that every step issues the same instructions; the result is
  // negative where the group owns no slab or its only one is partial.
  constexpr int k(int s) const { return base + (s < own ? s : own - 1) * BK; }
};

// Binary64 elements of B, from its row max(k0, 0), that the unmasked load of the
// slab at k0 may address (cols columns, row stride ldb): a whole slab, which lies
// in [0, K), or nothing where it would begin before k = 0 (a mask: the compiler
// makes a branch of a conditional here).
constexpr long long slab_extent(int k0, long long ldb, int cols) {
  return ((BK - 1) * ldb + cols) & ~((long long)k0 >> 63);
}

}  // namespace f64
}  // namespace mm
