// Orderings of sparse matrices found on the host (no arithmetic of the method).
#pragma once
#include <stdint.h>

#include <vector>

namespace fsi {

// A banded order of the n rows and columns of a sparse matrix.
struct BandOrder {
  std::vector<int> colpos, rowpos;   // position of each column and row
  std::vector<int> hi, cend;         // per panel of `nb` columns: rows that reach it, end of their columns
  int window = 0;                    // most rows that wait for a pivot at a time
  // as many rows reach the columns of each panel and those before as there are
  // such columns; without it the pattern is singular (the other rows outnumber
  // the columns left to them) and a panel may begin with no row waiting
  bool full = true;
};
// The columns go by the difference of their distances (in the graph of the
// pattern and its transpose) from the two ends of a longest level structure,
// the rows by their first column; of the two directions the one with the
// smaller window.  rowptr, colind: the pattern, columns in [0, n).
BandOrder band_order(int n, const std::vector<int64_t> &rowptr, const std::vector<int> &colind, int nb);

}  // namespace fsi
