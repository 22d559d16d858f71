// arena_take over `columns` requests by 1024 workgroups in turn, each of which
// keeps the place it was given: the number of places that overlap one in use.
#include <cstdio>
#include <cstdlib>

#include "arena.h"

int main(int argc, char** argv) {
    if (argc != 4) return 2;
    const unsigned int room = (unsigned)strtoul(argv[1], nullptr, 10);
    const unsigned int need = (unsigned)strtoul(argv[2], nullptr, 10);
    const long columns = atol(argv[3]);
    static unsigned int own[1024];
    static bool full[1024];
    for (unsigned int& o : own) o = stx::persist::kNoPlace;
    unsigned int used = 0;
    long given = 0, bad = 0;
    for (long c = 0; c < columns; ++c) {
        unsigned int& mine = own[c % 1024];
        if (mine != stx::persist::kNoPlace) continue;
        const unsigned int at = stx::persist::arena_take(
            room, need, full[c % 1024],
            [&](unsigned int n) { const unsigned int was = used; used += n; return was; });
        full[c % 1024] = at == stx::persist::kNoPlace;
        if (full[c % 1024]) continue;
        ++given;
        bad += at > room || need > room - at;
        for (const unsigned int o : own)
            bad += o != stx::persist::kNoPlace && at < o + need && o < at + need;
        mine = at;
    }
    std::printf("%ld %ld\n", given, bad);
    return 0;
}
