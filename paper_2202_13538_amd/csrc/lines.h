// Where outputs lie in the lines of the caches (128 bytes), for kernels that write whole lines past them.
#pragma once

#include <stdint.h>

namespace surel {

// Joined rows of more bytes go past the caches, from rounds that lie like the output's lines.  What fits the
// 256 MB memory-side cache is written faster there, whatever the lines.  Fill in us, through / past the
// caches: 10,000 pairs of M = 60, m = 3 (54 MB) 18 / 21; 60,000 of M = 30, m = 2 (86 MB) 67 / 74;
// 18,772 triples of M = 66, m = 3 (180 MB) 77 / 87; 20,000 pairs of M = 100, m = 4 (270 MB) 80 / 88;
// 35,000 of them (470 MB) 156 / 143; 500,000 of M = 30, m = 3 (900 MB) 623 / 501.
constexpr int64_t kPastBytes = 5 << 26;

// Whether the codes of a table's rows go past the caches when walks + RPE-IDs renumber them.  Where half of the
// 256 MB memory-side cache holds them, they stay there for the join, in us with its time, past / through the
// caches: 5.4 M rows and 20,000 pairs 229 / 229, 14.6 M and 200,000 pairs 672 / 660, 18 M and 20,000 433 / 430,
// 27 M and 20,000 583 / 578.
constexpr bool codes_go_past(int64_t n_rows) { return n_rows > (int64_t)1 << 25; }

// The join's filling launch puts a row at the place inside kRowsAlign rows that it has in the output's
// lines: 32 ids are a line, 32 vectors one or more.  (64 took as long, 16 and 1 % more.)
constexpr int kRowsAlign = 32;

// The place of an output's row 0.  An output may be a part of a larger one: of two that start the same
// number of rows behind a line it is that number.  Where ids and vectors cannot both lie in lines, the
// vectors do, which are most of the bytes.  Fill in us, placed by the number of the row / by the address:
// 262,144 pairs of M = 100, m = 4 with ids and vectors one row behind a line 1,199 / 1,097, 16 rows
// 1,138 / 1,095, ids at a line and vectors three rows behind one 1,160 / 1,141; 100,000 triples of m = 3
// seven rows behind 500 / 486, vectors alone three rows 503 / 475.
inline int join_first_place(const void* out_ids, const void* out_cnt, int row_bytes) {
    const uintptr_t vectors = (uintptr_t)out_cnt;
    const int place = (int)(((uintptr_t)out_ids >> 2) & (kRowsAlign - 1));
    for (int t = 0; t < kRowsAlign; ++t) {
        const int p = (place + t) & (kRowsAlign - 1);
        if (((vectors - (uintptr_t)(p * row_bytes)) & 127u) == 0) return p;
    }
    return place;
}

}  // namespace surel
