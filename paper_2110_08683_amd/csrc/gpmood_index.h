// Index arithmetic of the 2D cascade's lists, free of overflow up to the largest grid
// (32768 x 32768: 2^30 cells).
#ifndef GPMOOD_INDEX_H
#define GPMOOD_INDEX_H

namespace gpm {

// Groups of `per` items that hold n items.
constexpr unsigned groups_of(unsigned n, unsigned per) { return n / per + (n % per != 0u ? 1u : 0u); }

// Four lanes an item: the item of thread t in round r of rounds of `threads` threads.
// Counted in items, not in lanes: the lanes of 2^29 items no longer fit 31 bits.
constexpr unsigned quad_item(unsigned r, unsigned threads, unsigned t) { return r * (threads / 4u) + t / 4u; }

}  // namespace gpm

#endif
