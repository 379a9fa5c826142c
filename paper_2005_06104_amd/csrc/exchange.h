// Who publishes and who waits in a column of the tridiagonal reduction
// (eigh.hip).  In column k the owners of rows publish entries of x under tag
// k + 1 into one of two alternating buffers, and every workgroup reads what it
// needs of them.  A buffer is written again two columns later, by workgroups
// that have read all they wait for in column k + 1; none of them may be so far
// ahead that another has yet to read column k.  So every workgroup waits in
// every column for an entry of every other, also of those whose rows are all
// finished (they read on, for their rows of Q): the last G rows lie on
// different workgroups (row r on workgroup r % G), and their owners publish in
// every column.
#pragma once

#ifdef __HIPCC__
#define TDX_HD __host__ __device__
#else
#define TDX_HD
#endif

namespace tdx {

// the owner of row r publishes an entry of x in column k (zero for a finished row)
TDX_HD inline bool publishes(int r, int k, int n, int G) { return r >= k + 1 || r >= n - G; }
// every workgroup waits in column k for the entries from here to n - 1
TDX_HD inline int first_awaited(int k, int n, int G) { return k + 1 < n - G ? k + 1 : n - G; }

}  // namespace tdx
