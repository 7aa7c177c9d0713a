// Slots of the stored basis of multishift BiCGStab: buffers handed out from per-size pools, and the byte budget
// that ends a solve.  Host only.
#pragma once

#include <algorithm>
#include <cstddef>
#include <map>
#include <vector>

namespace sgn {

// Stored-basis slots handed out from the context's per-size pools; shared by the problems of a
// lockstep batch (each takes the next unused buffers) together with one byte budget.
struct BsSlotPools {
    std::map<size_t, size_t> next;  // next unused buffer of each per-size pool
    double budget = 0.0, used = 0.0;
};

// The r- and s-slots of one problem.  A slot counts against the budget once an iteration needs it, with the size
// that the iteration's vector has; slots taken ahead are unused buffers of the pool and count nothing until then,
// so the budget ends a solve at the same iteration whatever the pool holds.
class BsSlotTables {
  public:
    std::vector<void *> r, s;

    // r-slots 0 .. upto + 1 and s-slots 0 .. upto, vectors of `bytes` from here on; take(bytes) gives a buffer.
    // False if the budget does not hold them.
    template <typename Take>
    bool need(int upto, size_t bytes, BsSlotPools &pools, Take take)
    {
        return grow(r, r_needed_, (size_t)upto + 2, bytes, pools, take) &&
               grow(s, s_needed_, (size_t)upto + 1, bytes, pools, take);
    }

    // further pairs of slots up to r-slot last + 1 and s-slot last, as far as the pool of `pool` buffers has unused ones
    template <typename Take>
    void ahead(size_t last, size_t bytes, size_t pool, BsSlotPools &pools, Take take)
    {
        while (r.size() < last + 2 && s.size() < last + 1 && pools.next[bytes] + 2 <= pool) {
            r.push_back(take(bytes));
            s.push_back(take(bytes));
        }
    }

  private:
    size_t r_needed_ = 0, s_needed_ = 0;

    template <typename Take>
    static bool grow(std::vector<void *> &slots, size_t &needed, size_t count, size_t bytes, BsSlotPools &pools, Take take)
    {
        for (; needed < count; ++needed) {
            if (pools.used + (double)bytes > pools.budget) return false;
            if (slots.size() == needed) slots.push_back(take(bytes));
            pools.used += (double)bytes;
        }
        return true;
    }
};

}  // namespace sgn
