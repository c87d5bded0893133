// cic_path.h -- which of its two paths a deposit takes (host only, no HIP).
#pragma once
#include <cstdint>

namespace mgg {

// Whether np particles on n^3 cells are deposited faster binned by tiles than
// with global atomics.  In ns, the direct path costs 11000 + 2.8 to 4.4e-3 a cell
// (cleared, read, written) + 0.25 a particle in grid order and 0.35 in none; the
// binned path 21000 (five dependent launches) + 1.7e-3 a cell + 0.02 to 0.06 a
// particle + 5 (grid order) or 12 (none) for each particle that a tile of 16^3
// cells holds on average, since the tiles run in parallel.  The order is not
// known.  On sides of whole tiles the binned path runs unless the direct one is
// faster in grid order too, on others it has to be faster in no order as well.
// Binned / direct, us, in grid order and in none: 64^3 cells 25 / 17 and 31 / 19
// at 32^3 particles, 52 / 69 and 87 / 97 at 64^3; 32^3 cells (8 tiles) 63 / 20 and
// 103 / 29 at 40^3; 512^3 cells 217 / 594 at 10^3; 200^3 cells 46 / 42 and 51 / 43
// at 32^3, 61 / 352 and 174 / 395 at 102^3.  The differences below are fitted to
// 258 such pairs from 32^3 to 512^3 cells and 10^3 to 128^3 particles: 1.1% above
// the faster path on average.
inline bool cic_prefers_binned(int n, int64_t np) {
  const double m = double(n) * n * n, p = double(np), per_tile = p / (m / 4096.0);
  if (n % 16 == 0) return 0.22 * p - 5.0 * per_tile + 1.0e-3 * m > 1.0e4;
  return 0.24 * p - 10.0 * per_tile + 0.5e-3 * m > 1.75e4;
}

// Whether a deposit takes the binned path, given the faster path (want_binned)
// and the buffers that earlier deposits on the context have left.  The binned
// path's buffers (16 bytes a particle) may be too small for this deposit, the
// direct path's (8 bytes a cell) are all or none.  A deposit of no more
// particles than an earlier one must find what it needs: it may run under
// stream capture, where nothing can be allocated, and a context that has been
// warmed up takes no more memory.  So the binned path also runs where the
// direct one would be faster but has no buffer; and a larger deposit under
// capture runs on the direct path if only that has one.
inline bool cic_takes_binned(bool want_binned, bool have_binned, bool have_direct, bool capturing) {
  if (want_binned) return have_binned || !(capturing && have_direct);
  return have_binned && !have_direct;
}

// Whether a deposit that runs binned also makes the direct path's buffer: on
// sides of no multiple of 16, where a captured deposit of any number of
// particles has to run after the first one.
inline bool cic_makes_both(int n) { return n % 16 != 0; }

}  // namespace mgg
