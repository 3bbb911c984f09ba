// inplace.h -- which word (row, slot) of the single population buffer holds
// what when a level streams in place.  Even phase: row i of a cell holds the
// population i its next update takes.  Odd phase (after an even step): row
// opp(i) of a cell holds its own post-collision population i, and the next
// update pulls through the link sources s_i: another cell's slot, the cell's
// own slot c (a fine ghost or boundary cell without a source keeps the
// population), or a negative value (a wall returns population opp(i)).
//
// A kept population has a word of its own, row i of c.  In row opp(i) the
// cell c + xi_i, which pulls population i from there too, overwrites it in
// the odd step with its push, and nothing orders that before c's own read.
// Row i is free: it would hold population opp(i) for the cell c - xi_i, and
// that cell does not exist.  So in the odd step no word is read by a cell
// other than the one that writes it, and none has two writers.
#pragma once

#include <cstdint>

namespace lbm {

struct Word {
  int row;
  int32_t slot;
};

// odd phase: the word population i is pulled from (s: the source of link i)
constexpr Word odd_pull(int i, int opp, int32_t s, int32_t c) {
  return s >= 0 && s != c ? Word{opp, s} : Word{i, c};
}

// both phases: the cell keeps population i in row i of c
constexpr bool keeps(int32_t s, int32_t c) { return s == c; }

// where else population i goes, with t the source of link opp(i); nowhere if
// the cell keeps population opp(i): its word is that row, and there is no
// cell to take population i
constexpr Word even_store(int opp, int32_t t, int32_t c) { return t != c ? Word{opp, c} : Word{-1, c}; }
constexpr Word odd_store(int i, int opp, int32_t t, int32_t c) {
  return t == c ? Word{-1, c} : t >= 0 ? Word{i, t} : Word{opp, c};
}

}  // namespace lbm
