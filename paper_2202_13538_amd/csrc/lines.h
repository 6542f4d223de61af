// Where outputs lie in the lines of the caches (128 bytes), for kernels that write whole lines past them.
#pragma once

#include <stdint.h>

namespace surel {

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
