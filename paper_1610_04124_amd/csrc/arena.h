// arena.h -- table space handed out to the columns of one launch from a
// workspace that may be too small for all of them.
#pragma once

namespace stx::persist {

constexpr unsigned int kNoPlace = ~0u;

// Place of need units of a workspace of room units, or kNoPlace.  add(n) adds n
// to the number handed out and returns it as it was (atomic).  A request that
// finds no room has raised the number past it, so every later one finds none
// either: full, the caller's own, says so and keeps it from raising the number
// again.  With 2^10 callers and 2^17 units a request it stays below room + 2^27.
// (Raised by every request, it wrapped after 65,000 columns of 1024 rows and 256
// bins, and places in use were handed out again.  Looking at the number before
// raising it costs a column another trip to memory: 1024x437 at half pixels 72.7 ->
// 74.3 us.)
template <class Add>
#ifdef __HIP__
__device__
#endif
inline unsigned int arena_take(unsigned int room, unsigned int need, bool full, Add&& add) {
    if (full) return kNoPlace;
    const unsigned int at = add(need);
    return at < room && need <= room - at ? at : kNoPlace;
}

}  // namespace stx::persist
