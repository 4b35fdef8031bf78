// claim_step over a memory in which, before a chosen access of the claiming
// workgroup, the host publishes a system of four units and other workgroups
// claim some of them.  argv: access number, units claimed.  Prints the result
// and whether the launch was closed with a system partly claimed.
#include <cstdio>
#include <cstdlib>

#include "ring_claim.hpp"

struct Memory {
    uint64_t h = 8;
    uint32_t t = 8;  // two systems of four units, all claimed
    int at, claims, access = 0;
    uint64_t closed_at = UINT64_MAX;
    void step() {
        if (access++ != at) return;
        t += 4;
        h += (uint64_t)claims;
    }
    uint64_t head() { step(); return h; }
    uint32_t tail() { step(); return t; }
    uint32_t unit(uint32_t i) { step(); return 7u | (i & 3u) << 16; }
    bool stop() { step(); return false; }
    bool cas(uint64_t from, uint64_t to) {
        step();
        if (h != from) return false;
        if (to & cb::kRingClosed) closed_at = from;
        h = to;
        return true;
    }
};

int main(int argc, char** argv) {
    if (argc != 5) return 2;
    Memory m;
    m.at = atoi(argv[1]);
    m.claims = atoi(argv[2]);
    const int r = cb::claim_step(m, atoi(argv[3]) != 0, atoi(argv[4]) != 0);
    const bool split = m.closed_at != UINT64_MAX && (m.closed_at & 3) != 0;
    std::printf("%d %d\n", r, split ? 1 : 0);
    return 0;
}
