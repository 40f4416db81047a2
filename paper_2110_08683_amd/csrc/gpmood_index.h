// Index arithmetic of the 2D cascade's lists, free of overflow up to the largest grid
// (32768 x 32768: 2^30 cells).
#ifndef GPMOOD_INDEX_H
#define GPMOOD_INDEX_H

namespace gpm {

// Faces of an nx x ny grid, x faces and then y faces: on 32768 x 32768 they no longer fit 31
// bits, so a list holds face ids as unsigned numbers.
constexpr unsigned faces_of(int nx, int ny) { return (unsigned)(nx + 1) * (unsigned)ny + (unsigned)nx * (unsigned)(ny + 1); }

// Groups of `per` items that hold n items (n + per below 2^32: any list of faces or cells).
constexpr unsigned groups_of(unsigned n, unsigned per) { return (n + (per - 1u)) / per; }

// Four lanes an item: the item of thread t in round r of rounds of `threads` threads.
// Counted in items, not in lanes: the lanes of 2^29 items no longer fit 31 bits.
constexpr unsigned quad_item(unsigned r, unsigned threads, unsigned t) { return r * (threads / 4u) + t / 4u; }

}  // namespace gpm

#endif
