// The budget of the stored BiCGStab basis ends a solve at the same iteration whether or not unused buffers of an
// earlier solve were taken ahead.  Arguments: FP64 iterations, budget (in FP32 vectors), unused FP64 buffers and
// iterations ahead; prints the iterations that the budget holds, the vectors counted and the buffers allocated.
#include <cstdio>
#include <cstdlib>

#include "basis_slots.h"

using namespace sgn;

int main(int argc, char **argv)
{
    if (argc != 5) return 2;
    const int fp64 = std::atoi(argv[1]), poll = 4, ahead = std::atoi(argv[4]), maxiter = 1000;
    const size_t b32 = 8, b64 = 16;
    BsSlotPools pools;
    pools.budget = std::atof(argv[2]) * (double)b32;
    std::map<size_t, size_t> size{{b64, (size_t)std::atoi(argv[3])}, {b32, 0}};
    int allocated = 0;
    auto take = [&](size_t bytes) -> void * {
        size_t &next = pools.next[bytes];
        if (next == size[bytes]) ++size[bytes], ++allocated;
        ++next;
        return nullptr;
    };
    BsSlotTables t;
    int k = 0;
    for (; k < maxiter; k += poll) {
        const size_t bytes = k < fp64 ? b64 : b32;
        if (!t.need(k + poll, bytes, pools, take)) break;
        if ((int)t.r.size() < k + poll + 2 || (int)t.s.size() < k + poll + 1) return 3;
        if (ahead)
            t.ahead(std::min<size_t>(maxiter + poll, (size_t)k + poll + ahead), bytes, size[bytes], pools, take);
        if (t.r.size() > (size_t)maxiter + poll + 2 || t.s.size() > (size_t)maxiter + poll + 1) return 4;
    }
    if (pools.used > pools.budget) return 5;
    std::printf("%d %g %d\n", k, pools.used / b32, allocated);
    return 0;
}
