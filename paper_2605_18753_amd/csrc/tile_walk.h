// How s2_attend_kernel walks a workgroup's list of tiles, as far as it is arithmetic.  Plain C++: the CPU tests compile it too.
#pragma once

namespace dash {

// Chunks of the list before a part, chunks of the part, and the last of its iterations (one more than tiles)
struct ListPart { int first, chunks, last_it; };

// The part of group grp (0 or 1) of two that walk the halves of a list of n chunks: both go through as many iterations as the longer half takes,
// whose barriers they share.  Of a single chunk the second half is empty.
constexpr ListPart list_half(int n, int grp, int sub_log) {
  const int per = (n + 1) >> 1;
  return {grp * per, grp == 0 ? per : n - per, per << sub_log};
}

// Index, within its part of n_it tiles, of the entry that iteration i >= 0 looks at: behind the last that one again, -1 where the part has
// none (what lies at its place in the list was never written).
constexpr int walk_index(int i, int n_it) { return i < n_it ? i : n_it - 1; }

}  // namespace dash
