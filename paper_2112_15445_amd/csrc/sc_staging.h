// Host-side arithmetic of the staging of the matrix-core kernels, worked out once per launch shape.  Plain C++.
#pragma once

#include <algorithm>
#include <cstdint>

namespace sc {

// The least number of input rows that a row tile stages, of those that stage any (0: none does).  Tile t of `tiles` stages the rows
// [t step - pad, t step - pad + Hs) that lie inside [0, H).  Their number is a concave function of t, so that its least
// positive value is that of the first or of the last tile that reaches the input.
inline int64_t least_staged_rows(int64_t H, int64_t Hs, int64_t step, int64_t pad, int64_t tiles)
{
    const int64_t first = pad >= Hs ? (pad - Hs) / step + 1 : 0, last = std::min(tiles - 1, (H - 1 + pad) / step);
    auto rows = [&](int64_t t) {
        const int64_t row0 = t * step - pad;
        return std::min(Hs, H - row0) - std::max<int64_t>(0, -row0);
    };
    return first > last ? 0 : std::min(rows(first), rows(last));
}

// Log2 of the columns per staging load, at most `widest` and at most the shortest run that a tile stages (loads may have any
// alignment): the least estimated time of a chunk, rounds of `threads` blocks times a block's instructions, `block` for its
// loads and addresses and `column` for each column.  `rows` runs of `run` elements for each of `groups` (channel group, sample) pairs.
inline int load_columns(int widest, int block, int column, int64_t groups, int64_t threads, int64_t rows, int64_t run, int64_t minrun)
{
    int64_t best = 0;
    int lepv = 0;
    for (int l = widest; l >= 0; --l) {
        const int64_t e = 1ll << l;
        if (e > 1 && e > minrun) continue;
        const int64_t blocks = groups * rows * ((run + e - 1) / e);
        const int64_t cost = ((blocks + threads - 1) / threads) * (block + e * column);
        if (best == 0 || cost < best) { best = cost; lepv = l; }
    }
    return lepv;
}

}  // namespace sc
