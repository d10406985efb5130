// The key rows of a matrix-core distance workgroup and the fused select's
// sample, as plain arithmetic: kernels, launchers and host tests share it.
#pragma once

#include <stdint.h>

namespace knnlm {

struct RowRange {
    int64_t first, end;  // rows [first, end) of a set; none when end <= first
};

// The rows of a workgroup on `tile` of a set of N keys: the tile (fm 0), the
// sample piece at its start (fm 1), or what lies past that piece (fm 2; every
// sample_every-th tile has one, which may be the whole tile).
constexpr RowRange mfma_rows(int fm, int64_t tile, int64_t rows_per_tile, int64_t sample_rows, int64_t sample_every,
                             int64_t N) {
    const int64_t start = tile * rows_per_tile;
    const int64_t end = start + (fm == 1 ? sample_rows : rows_per_tile);
    const int64_t first = fm == 2 && tile % sample_every == 0 ? start + sample_rows : start;
    return RowRange{first, end < N ? end : N};
}

// The row, counted from the range's first, that a load of row `row` reads:
// those past the end read the last.  nrows >= 1.
constexpr uint32_t mfma_load_row(uint32_t row, uint32_t nrows) { return row < nrows ? row : nrows - 1u; }

// The fused select's sample: the first `rows` rows of every `every`-th tile,
// about 1/64 of the keys (1/64 keeps about 2,300 candidates per query for
// r = 1024 against about 1,900 at 1/32, both well inside the lists, and halves
// the sample pass and the threshold kernel's reads), in pieces small enough
// that the sample launch fills the chip: an eighth of a tile, in whole passes
// of 256 rows.  rows_per_tile >= 256.
struct FusedSample {
    int rows, every;
};

constexpr FusedSample fused_sample(int rows_per_tile) {
    const int eighth = rows_per_tile / 8 / 256 * 256;
    const int rows = eighth > 256 ? eighth : 256;
    const int every = 64 * rows / rows_per_tile;
    return FusedSample{rows, every > 1 ? every : 1};
}

}  // namespace knnlm
