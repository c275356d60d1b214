// Host arithmetic of the selection's launch, apart from HIP so that a CPU test can compile it.
#pragma once

namespace da {

// Rows of `g` scores of which `columns` >= g, starting at the row's first, are read: how many of the `rows` rows, from the
// first on, may read all of them without leaving the array (all but the last few; all of them with readable slack behind it).
inline long long rows_that_read_on(long long rows, long long g, long long columns, bool slack) {
  const long long spill = columns - g;                // read past the end of a row
  const long long last = spill > 0 && !slack ? (spill + g - 1) / g : 0;
  return rows > last ? rows - last : 0;
}

}  // namespace da
