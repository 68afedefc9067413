// pair_items.hpp -- the work items of the matrix-free single products and the
// places of their partial sums.  Usable on the host and on the device.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <vector>

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define MQH_HD __host__ __device__
#else
#define MQH_HD
#endif

namespace mqh {

#ifdef __HIPCC__
using PairItem = int4;
#else
struct PairItem {
    int x, y, z, w;
};
#endif

// The matrix-free single products over unordered node pairs (each pair's t and
// rsqrt once, feeding y_i and y_j): nodes in the sorted order cut into
// blocks of blk per class (interior blocks 0 .. nb_int-1, boundary
// blocks nb_int .. nb-1).  Work item (k, s): fixed blocks [kF, kF + F) (a
// super-row) against loop blocks [kF + s Lb, kF + (s+1) Lb) (a segment),
// only pairs of blocks b <= c (b == c: the block's own square, row sums
// only).  Each item writes F x blk row partials and the column partials of its
// loop blocks (for each block one from every super-row up to its own); a
// node's output adds the row partials of its super-row's items and its block's
// column partials.
constexpr int kSymMaxF = 8;    // fixed blocks per super-row (at most)
constexpr int kSymMaxLb = 14;  // loop blocks per segment (at most; the LDS of four workgroups per CU)
struct SymLayout {
    int64_t n, n_int;
    int32_t nb_int, nb;         // blocks of blk nodes per class, all blocks
    int32_t blk, pad;           // 128 (FP32 form), 64 or 128 (FP64 form)
    int32_t F, Lb;              // fixed blocks per super-row (a power of two), loop blocks per segment
    int32_t nsr, nitems;        // super-rows, work items
    const PairItem* items;      // (super-row, segment, place in the partials, 0) in launch order (largest first)
    const int32_t* item_first;  // nsr + 1 entries: first item of each super-row
};

MQH_HD inline int sym_shift(int F) { return __builtin_ctz((unsigned)F); }

// Place of block beta's column partials in ColP (in blocks): one from each
// super-row k <= beta / F, in order of k, block after block.
MQH_HD inline int64_t sym_col_base(int beta, int F) {
    const int64_t k = beta >> sym_shift(F);
    return (int64_t)F * (k * (k + 1) / 2) + (beta - k * F) * (k + 1);
}

// Blocks of column partials of a pair product: one per block and super-row up
// to its own.
inline int64_t sym_col_blocks(const SymLayout& L) {
    const int64_t k = L.nb / L.F;  // whole super-rows before the last, partial one
    return (int64_t)L.F * (k * (k + 1) / 2) + (L.nb - k * L.F) * (k + 1);
}

// Work items of the pair products (SymLayout): blocks of blk sorted nodes per
// class; super-rows of F fixed blocks and segments of Lb loop blocks; first[k]
// indexes the items in (super-row, segment) order, the list itself is in
// launch order.  A larger item writes fewer partials and sets up fewer fixed
// blocks; too few items leave a round of resident workgroups nearly empty.
// FP32 form: the largest shape with 1200 items (its FP32 sums follow the shape).
// FP64 form (768 workgroups of 128-node blocks resident): the largest shape with
// 3000 items; below that 1 x 2 blocks of 128 nodes, and with fewer of those
// than CUs blocks of 64.  Whole products, us: 20 000 nodes 174 with (1, 4), 178
// (2, 4), 230 (4, 8), 462 (8, 14); 70 000 nodes 1645 (4, 8), 1659 (1, 4), 1769
// (8, 14); 1 800 nodes 32 with blocks of 64, 37 with 128.
inline void sym_tables(int64_t n, int64_t n_int, bool fp64, SymLayout& L, std::vector<PairItem>& items,
                       std::vector<int32_t>& first) {
    struct Shape {
        int blk, F, Lb, want;
    };
    static const Shape shapes32[] = {{128, 8, 14, 1200}, {128, 4, 8, 1200}, {128, 2, 4, 1200}, {128, 1, 2, 0}};
    static const Shape shapes64[] = {{128, 8, 14, 3000}, {128, 4, 8, 3000}, {128, 2, 8, 3000}, {128, 2, 4, 3000},
                                     {128, 1, 4, 3000},  {128, 1, 2, 256},  {64, 1, 2, 0}};
    for (const Shape* sh = fp64 ? shapes64 : shapes32;; ++sh) {
        L = SymLayout{};
        L.n = n;
        L.n_int = n_int;
        L.blk = sh->blk;
        L.F = sh->F;
        L.Lb = sh->Lb;
        L.nb_int = (int32_t)((n_int + L.blk - 1) / L.blk);
        L.nb = L.nb_int + (int32_t)((n - n_int + L.blk - 1) / L.blk);
        items.clear();
        first.clear();
        L.nsr = (L.nb + L.F - 1) / L.F;
        for (int k = 0; k < L.nsr; ++k) {
            first.push_back((int32_t)items.size());
            const int nseg = (L.nb - k * L.F + L.Lb - 1) / L.Lb;
            for (int sg = 0; sg < nseg; ++sg) items.push_back(PairItem{k, sg, (int32_t)items.size(), 0});
        }
        first.push_back((int32_t)items.size());
        L.nitems = (int32_t)items.size();
        if (L.nitems >= sh->want) break;
    }
    // launch order: items by their number of block pairs, largest first
    // (stable), so the last workgroups to start are the short ones
    auto pairs = [&](const PairItem& it) {
        const int b0 = it.x * L.F, b1 = std::min(b0 + L.F, L.nb);
        const int c0 = b0 + it.y * L.Lb, c1 = std::min(c0 + L.Lb, L.nb);
        int64_t cnt = 0;
        for (int b = b0; b < b1; ++b) cnt += std::max(0, c1 - std::max(c0, b));
        return cnt;
    };
    std::stable_sort(items.begin(), items.end(), [&](const PairItem& a, const PairItem& b) { return pairs(a) > pairs(b); });
}

}  // namespace mqh
