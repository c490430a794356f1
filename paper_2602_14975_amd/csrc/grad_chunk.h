// Rows per partial sum of the weight adjoints.
#pragma once
#include <cstdint>

namespace nnp {

// The outputs are small (at most a few 64 x 64 tiles), so the chunks of rows
// are what fills the chip.  24,576 frames' rows: 96 chunks; with 2,048 rows, 12
// to 36 blocks per product took 53 us each and the column sums 100 us.  The
// chunks are a launch's y or z dimension, which ends at 65,535 blocks: past
// 16,776,960 rows they grow instead of their number.
constexpr int64_t kMaxChunks = 65535;
constexpr int grad_chunk(int64_t rows) {
    int c = 256;
    while ((rows + c - 1) / c > kMaxChunks) c *= 2;
    return c;
}

}  // namespace nnp
