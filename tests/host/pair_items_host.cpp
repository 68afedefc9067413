// Host build of the pair products' work items and partial places
// (paper_2511_09798_amd/csrc/pair_items.hpp), for CPU tests.
#include "../../paper_2511_09798_amd/csrc/pair_items.hpp"

using namespace mqh;

// out: nb_int, nb, blk, F, Lb, nsr, nitems, kSymMaxF, kSymMaxLb; the first `room` items (4 each)
// and super-rows' first items are copied.  Returns the blocks of column partials.
extern "C" int64_t pair_layout(int64_t n, int64_t n_int, int fp64, int32_t* out, int32_t* it, int32_t* first,
                               int64_t room) {
    SymLayout L;
    std::vector<PairItem> items;
    std::vector<int32_t> fi;
    sym_tables(n, n_int, fp64 != 0, L, items, fi);
    const int32_t v[9] = {L.nb_int, L.nb, L.blk, L.F, L.Lb, L.nsr, L.nitems, kSymMaxF, kSymMaxLb};
    std::copy(v, v + 9, out);
    for (size_t i = 0; i < items.size() && (int64_t)i < room; ++i) {
        const int32_t q[4] = {items[i].x, items[i].y, items[i].z, items[i].w};
        std::copy(q, q + 4, it + 4 * i);
    }
    for (size_t i = 0; i < fi.size() && (int64_t)i < room; ++i) first[i] = fi[i];
    return sym_col_blocks(L);
}
extern "C" int64_t pair_col_base(int beta, int F) { return sym_col_base(beta, F); }
