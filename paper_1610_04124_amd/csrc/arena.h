// arena.h -- table space handed out to the columns of one launch from a
// workspace that may be too small for all of them.
#pragma once

namespace stx::persist {

constexpr unsigned int kNoPlace = ~0u;

// Place of need units of a workspace of room units, or kNoPlace.  load() reads
// the number handed out, add(n) adds n to it and returns it as it was (both
// atomic).  A request that finds the workspace used up leaves the number as it
// is: each concurrent caller can raise it past room once, so with 2^10 callers
// and 2^17 units a request it stays below room + 2^27.  (Raised by every request,
// it wrapped after 65,000 columns of 1024 rows and 256 bins, and places in use
// were handed out again.)
template <class Load, class Add>
#ifdef __HIP__
__device__
#endif
inline unsigned int arena_take(unsigned int room, unsigned int need, Load&& load, Add&& add) {
    if (load() >= room) return kNoPlace;
    const unsigned int at = add(need);
    return at < room && need <= room - at ? at : kNoPlace;
}

}  // namespace stx::persist
