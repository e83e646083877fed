// How many strided rows of a Dense layer one launch may take (host arithmetic only).
#pragma once
#include <stdint.h>

namespace ivit {

// The tallest tile of the kernel for any shape (gemm_st.hip) that is taken without a look at the row stride; its tiles of 192 and 256 rows are
// taken only where their own offsets fit (linear_st_one_round, big_tiles).
constexpr int64_t kTileRows = 128;

// That kernel addresses the rows of a tile by 32-bit byte offsets from the tile's first one; they are kept below kTileBytes =
// 2^31, where it does not matter whether anything on the way takes them as signed.  kTileBytes is also the size in its buffer
// descriptors: a row may end there, at its last byte.
constexpr uint32_t kTileBytes = 0x80000000u;

// The number of rows, from 1 up, that a launch can take for a row stride of ldx >= K bytes; where tiles of full height fit there
// is no limit.
constexpr int64_t linear_rows_per_launch(int64_t ldx, int64_t K) {
    const int64_t reach = ((int64_t)kTileBytes - K) / ldx + 1;
    return reach >= kTileRows ? INT64_MAX : reach;
}

}  // namespace ivit
