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

// Estimated time (us) of the inverse of n unknowns by the banded elimination
// in this order (panels of 16 columns) and by the Gauss-Jordan chain.  The
// elimination runs in one workgroup: a panel takes its pivot steps, which grow
// with the waiting rows, and the update of those rows' entries in its columns'
// reach at the rate of one compute unit (16 bytes each, 50 GB/s).  The chain
// has the whole device for its updates and a serial step per 16 columns (8
// above 1,536 unknowns).  Constants fitted to 55 operators of 60 to 3,426
// unknowns and 52 to 456 waiting rows (dense, random banded, the coarsest
// operators of 8x4 to 24x8 and 8x2x2 to 16x2x2 meshes), within 11 % and 8 %
// of the times measured; the faster one is chosen but for ties.  Measured
// (elimination, chain): 16x4 0.98, 2.6 ms; 24x6 3.6, 11.0; 24x8 7.1, 21.1;
// 8x8 (273 rows) 2.9, 2.7; 8x2x4 (412) 12.0, 9.1; 384 dense 0.94, 0.68.
double band_time(const BandOrder &b, int n);
double chain_time(int n);

}  // namespace fsi
