// The exchange of words between the workgroups that hold a factor's rows (eig_chip.h): who publishes for a column, whose words are
// waited for, what is emptied afterwards.  Plain functions of row and column numbers: the kernel runs on them, and so does a model of
// the exchange on the CPU that takes its steps in any order.
//
// In column t every workgroup with unfinished rows (r0 + nr > t) publishes a word for each of its rows in slot t mod 4, waits for the
// others' words, and then empties its own words of column t - 1.  It may do that only if nobody still looks for them.  The
// words of column t say so for every workgroup that publishes in column t; but a workgroup whose last row was t - 1
// has gathered column t - 1 and has no row left to publish for.  So it publishes one word more, for its last row, as its
// receipt for column t - 1, and the words that are waited for begin with row t - 1.
//  - Whoever has gathered column t knows that all who gathered column t - 1 are through with it.
//  - A slot is used again after four columns.  Its words of rows from t + 3 on, which column t + 4 waits for, were emptied by their
//    writers after column t + 1, before they published for column t + 2 (the writer waits for its stores in between).
//    Words of finished rows stay as they are and are not looked at again.
#pragma once

constexpr int CHIP_RING = 4;      // columns whose words are in flight

struct ChipRing {
    static constexpr int slot(int t) { return t & (CHIP_RING - 1); }
    // a workgroup with rows r0 .. r0 + nr - 1, in column t
    static constexpr bool leaves(int r0, int nr, int t) { return r0 + nr <= t; }               // no unfinished row: not part of the column any more
    static constexpr int receipt(int r0, int nr, int t) { return r0 + nr == t ? t - 1 : -1; }   // row of its last word, as it leaves (-1: none)
    static constexpr int first(int t) { return t > 0 ? t - 1 : 0; }                            // first row whose word is waited for
    static constexpr int emptied(int t) { return t - 1; }                                      // column whose own words are emptied after the gather (-1: none)
};
