// Host build of the small calls' closed-form split (paper_2607_12696_amd/csrc/split.hpp) for the CPU tests.
#include "split.hpp"

using namespace ecospec::split;

extern "C" {
// first[0..G], and per item the first and last workgroup that hold its units; returns the units per item.
unsigned small_split_table(unsigned items, unsigned rounds, unsigned bytes, unsigned G, unsigned *first, unsigned *w0,
                           unsigned *w1)
{
    const SmallSplit s = small_split(items, rounds, bytes, G, [G](unsigned x) { return x / G; });
    for (unsigned w = 0; w <= G; ++w) first[w] = s.first(w, G);
    for (unsigned i = 0; i < items; ++i) {
        w0[i] = s.owner(i * s.per_item, G);
        w1[i] = s.owner(i * s.per_item + s.per_item - 1, G);
    }
    return s.per_item;
}
unsigned small_piece_slot(unsigned f, unsigned ib) { return small_piece(f, ib); }
}
