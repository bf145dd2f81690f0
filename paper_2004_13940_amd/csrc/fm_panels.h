// How the rows of a matrix are cut into the panels of the column side.  Standard library alone.
#pragma once

#include <cstdint>

constexpr int FM_XCDS = 8;  // L2 domains; workgroup b runs on XCD b % 8
// Panel b goes to XCD b % FM_XCDS, so there are as many to each: with 25 to 47 of them, as halving a power of two left, the
// longest of the eight lists had up to 1.17 times the mean number of rows.  At least three to an XCD: fewer and
// taller ones make longer items, and with that fewer partial sums; what they bring is gone once a panel is far beyond an L2 (4
// MB) or the XCDs' work gets uneven.  Epochs in us with 2 / 3 / 4 / 6 panels to an XCD, and 24 to 47 by halving: text-like rows, K = 16
// 7e4 73.9 / 78.6 / 81.8 / 86.9, 85.8, 2e5 171 / 176 / 184 / 196, 181, K = 64 2e5 343 / 369 / 388 / 415, 375; hashed 7e4, K = 64 340
// / 344 / 353 / 366, 363, 4e5 2180 / 2202 / 2225 / 2272, 2213; click-style, K = 16 1e5 99.4 / 100.2 / 102 / 104, 100.3, 4.5e5 383 /
// 345 / 339 / 338, 345, 7.8e5 568 / 560 / 556 / 558, 558; K = 32 6e5 550 / 548 / 630 / 636, 558.
constexpr int FM_XCD_PANELS = 3;

// Rows per panel: at most `limit`, FM_XCD_PANELS panels or more to every XCD, as many to each.
inline int64_t fm_panel_rows(int64_t N, int64_t limit)
{
    int64_t each = (N + FM_XCDS * limit - 1) / (FM_XCDS * limit);
    if (each < FM_XCD_PANELS) each = FM_XCD_PANELS;
    const int64_t rows = (N + FM_XCDS * each - 1) / (FM_XCDS * each);
    return rows > 0 ? rows : 1;
}
