// cic_path.h -- which of its two paths a deposit takes (host only, no HIP).
#pragma once
#include <cstdint>

namespace mgg {

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
