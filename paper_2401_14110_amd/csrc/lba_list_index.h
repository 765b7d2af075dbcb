// lba_list_index.h -- layout of a row tile of the packed FP16 carriers in LDS (lba_rows.h) and the order in which a list of non-zero
// codes is read.  Plain C++: tests/sanitize_pieces.cpp walks lists of every length over a model of a row.
#ifndef LBA_LIST_INDEX_H_
#define LBA_LIST_INDEX_H_

#include "lba_piece_index.h"

namespace lba {

// Geometry of one workgroup tile: each of the four waves takes RW rows (8, 12 or 16) and all BN = 8 TN columns.  A row set is 8
// rows of 8 lanes, TN columns per lane; 12 rows are one such set and one of 4 rows of 16 lanes, TN / 2 columns per lane.
// LDS: two stages of B as words (n, n + 1) of one k, [k][n / 2]; one stage of A, every row written and read by its own wave:
// its words (k, k + 1), or the list of its non-zero codes (value in the low half, byte offset of the code's row of B in the high).
template <int RW, int TN>
struct RowTile {
    static constexpr int BM = 4 * RW, BN = 8 * TN, SETS = RW / 8;
    static constexpr bool HALF = RW % 8 != 0;
    static constexpr int U = TN >= 8 ? 4 : 8;                  // list entries taken at a time
    static constexpr int BROW = BN / 2, B_WORDS = HBK * BROW;
    static constexpr int PAD = 2 * U;                          // a list is read on for that many words (walk_list), which are zero
    static constexpr int PITCH = HBK + PAD + (U == 8 ? 4 : 0);     // words per row of A
    static constexpr int A_WORDS = BM * PITCH, WORDS = 2 * B_WORDS + A_WORDS;
};

// The words behind a row's 64 codes, zeroed once by the wave that owns the row: store(word of the row) for lane l of the four of a row.
// Nothing writes them later (a tile's words and a list end before them), so a list of all 64 codes goes on into entries of value 0
// whose row of B is the stage's first.
template <class T, class Store>
LBA_HOST_DEVICE void pad_row(int l, Store store) {
#pragma unroll
    for (int j = 0; j < T::PAD / 4; ++j) store(HBK + l * (T::PAD / 4) + j);
}

// The rounds of a list of n entries (a multiple of U): one at entry i takes entries i .. i + U - 1, asks for the rows of B of the next U and
// reads the U after those, so the first U entries past n serve as addresses and the next U are read.  Two entry registers change
// places: first and second are the rounds by which holds the entries taken.
template <int U, class First, class Second>
LBA_HOST_DEVICE void walk_list(int n, First first, Second second) {
#pragma unroll 1
    for (int i = 0; i < n; i += 2 * U) {
        first(i);
        if (i + U >= n) break;
        second(i + U);
    }
}

}  // namespace lba
#endif
