// Offsets of state rows as the kernels form them, in plain C++ so that the host
// can check them too.
#pragma once

namespace sem {

// Byte offset of a row in a field for loads and stores through a buffer
// descriptor: NOWHERE, and everything from there on, is past the range of
// every state array that the 32-bit offsets reach (below 2 GiB), so that the
// hardware drops the access.  The row of a unique node g >= 0 starts at
// g * ldz doubles; a hanging point -(hh + 1) has no row of its own, and its
// entry stays past the range at every level of a row (hh < 2^27: a mesh has
// fewer of them than nodes, and 2 GiB hold five fields of 3.4 million rows).
constexpr unsigned NOWHERE = 0x80000000u;
constexpr unsigned row_offset(int g, int ldz) {
    return g >= 0 ? unsigned(g) * unsigned(ldz) * 8u : NOWHERE + 8u * unsigned(-(g + 1));
}
constexpr int row_hanging(unsigned row) { return int((row - NOWHERE) / 8u); }

// First level of the two that a 16-byte access of levels k and k + 1 covers
// (k < nzn): where k is the last level, the pair below, so that the row's padding
// is not read (nzn >= 2).
constexpr int level_pair(int k, int nzn) { return k + 1 < nzn ? k : k - 1; }

}  // namespace sem
