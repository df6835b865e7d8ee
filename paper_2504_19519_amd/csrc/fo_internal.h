// Internal declarations shared by the planner, the kernels' launchers and the
// runtime glue of libfo. Not part of the public ABI (see include/fo.h).
#pragma once

#include <stdint.h>

#include <string>
#include <vector>

#include "fo.h"

#if defined(__HIPCC__)
#define FO_HD __host__ __device__
#else
#define FO_HD
#endif

namespace fo {

// Tile computed by the workgroup at dispatch position p (fo_order in fo.h).
// The GEMM kernel evaluates this on the device for its blockIdx, the planner
// on the host for the reorder map, so both always agree. In 32 bits: the caller
// sees to 1 <= group_m <= max(tiles_m, 1) and num_xcds <= max(tiles, 1) (a plan
// holds them so; block_band for a grid of blocks).
FO_HD inline int32_t tile_of_position(int32_t p, int32_t tiles_m, int32_t tiles_n,
                                      int32_t order, int32_t group_m, int32_t num_xcds) {
    if (order == FO_ORDER_ROWMAJOR) return p;
    const int32_t tiles = tiles_m * tiles_n;
    int32_t q = p;
    if (order == FO_ORDER_XCD) {
        const int32_t per = (tiles + num_xcds - 1) / num_xcds;
        int32_t full = tiles % num_xcds;
        if (full == 0) full = num_xcds;
        const int32_t x = p % num_xcds;
        const int32_t l = p / num_xcds;
        q = x < full ? x * per + l : full * per + (x - full) * (per - 1) + l;
    }
    const int32_t band_tiles = group_m * tiles_n;
    const int32_t band = q / band_tiles;
    const int32_t first = band * group_m;
    const int32_t rows = (tiles_m - first) < group_m ? (tiles_m - first) : group_m;
    const int32_t r = q - band * band_tiles;
    const int32_t tm = first + r % rows;
    const int32_t tn = r / rows;
    return tm * tiles_n + tn;
}

// Band height, in blocks of block_m rows, of a launch whose workgroups compute
// blocks and not the plan's tiles: the rows of the plan's band, rounded up, and
// no taller than the grid of blocks_m block rows.
inline int32_t block_band(int32_t group_m, int32_t tile_m, int32_t block_m, int32_t blocks_m) {
    const int64_t band = ((int64_t)group_m * tile_m + block_m - 1) / block_m;
    return band < blocks_m ? (int32_t)band : blocks_m < 1 ? 1 : blocks_m;
}

inline int dtype_bytes(int32_t) { return 2; }

// Set the calling thread's last error and return `st`.
fo_status fail(fo_status st, const std::string& msg);
void clear_error();

// Poll timeout in microseconds (runtime.hip).
int64_t poll_timeout_us();

}  // namespace fo

// Word offsets of the tables inside the device image (all int32, each
// section starts on a 16-byte boundary).
struct fo_dev_layout {
    int64_t tile_to_slot = 0;   // [tiles]
    int64_t slot_group = 0;     // [tiles]
    int64_t group_first = 0;    // [P+1]
    int64_t dest_perm = -1;     // [R]          SUBTILE
    int64_t row_bucket = -1;    // [M]          SUBTOKEN
    int64_t row_rank = -1;      // [M]          SUBTOKEN
    int64_t pool_base = -1;     // [(tiles+1)B] SUBTOKEN
    int64_t pool_off = -1;      // [B+1]        SUBTOKEN
    int64_t words = 0;
};

struct fo_plan {
    int64_t M = 0, N = 0, K = 0;
    int32_t dtype = 0, tile_m = 0, tile_n = 0, order = 0, group_m = 1, num_xcds = 1;
    int32_t num_cus = 0, wg_per_cu = 1, reserved_cus = 0, pattern = 0, num_dest = 0;
    int32_t unit = FO_UNIT_WAVES;
    int32_t tiles_m = 0, tiles_n = 0, tiles = 0, W = 0, T = 0, P = 0;
    double predicted_us = 0.0;
    int64_t dest_elems = 0;
    std::vector<int32_t> sizes;         // [P] in `unit`
    std::vector<int32_t> order_tbl;     // [tiles] position -> tile
    std::vector<int32_t> tile_to_slot;  // [tiles]
    std::vector<int32_t> slot_group;    // [tiles]
    std::vector<int32_t> group_first;   // [P+1]
    std::vector<int32_t> targets;       // [P]
    std::vector<int32_t> dest_perm;     // [R]
    std::vector<int32_t> row_bucket;    // [M]
    std::vector<int32_t> row_rank;      // [M]
    std::vector<int32_t> pool_base;     // [(tiles+1)*B]
    std::vector<int32_t> pool_off;      // [B+1]
    std::vector<int64_t> segs;          // [nseg*5]
    fo_dev_layout layout;
    std::vector<int32_t> image;         // device image (layout.words)
};

namespace fo {

// Whether the groups of an overlapped run are consumed together, after the
// GEMM. On one device a consumer beside the GEMM takes from the GEMM about what
// it saves behind it, and every group costs a wait kernel and a launch, while
// consumed together the groups share one pass with the post-reorder. Measured
// (us per run, a launch per group / together):
//   256x256x256     4 groups  49 / 19     4096x7168x2048  2 groups  146 / 128
//   1216x2880x1984  4 groups  60 / 32     8192x4096x4096  2 groups  253 / 248
//   4096x4096x4096  2 groups 168 / 136    8192x8192x1024  3 groups  290 / 207
//   16384x8192x2048 4 groups 611 / 591    8192x8192x3584  3 groups  456 / 447
//   16384x4096x3584 4 groups 442 / 445    32768x4096x3584 4 groups  869 / 878
//   8192x8192x7168  4 groups 747 / 763
// A launch per group pays once the GEMM (at the 5.5 TFLOP/s that a compute unit
// reaches) lasts 300 us and three times as long as the consumer alone (at 5.1
// TB/s): below that the groups after the first still run when the GEMM ends. (Two
// of the table's shapes have the same estimates and differ the other way,
// 8192x8192x3584 by 2 % and 16384x4096x3584 by 1 %; no line in the sizes parts
// them.)
// Consumed together, one wait (limit_us) holds the consumer stream for all of the
// GEMM, where a launch per group waits for a group at a time. A caller's limit that
// was set for the groups must not expire on that: it has to exceed the estimate a
// hundredfold, and 10 ms, which a device shared with other work does not use up.
inline bool consumed_together(const fo_plan& p, bool sum, int64_t limit_us) {
    const double gemm_us = 2.0 * (double)p.M * (double)p.N * (double)p.K / ((p.W > 1 ? p.W : 1) * 5.5e6);
    const double consume_us = 2.0 * (double)p.M * (double)p.N * (sum ? 3 : 2) / 5.1e6;
    return (gemm_us < 300.0 || gemm_us < 3.0 * consume_us) && (double)limit_us >= 100.0 * gemm_us && limit_us >= 10000;
}

// Whether an unsignalled GEMM of plans with 256 x tile_n tiles computes 128x128
// blocks instead of whole tiles: where the tiles' last wave is emptier than the
// blocks' or one tile per compute unit covers its barriers less than a pair of
// blocks (bf16, us per launch, K 4096 / 1024, tiles -> blocks):
//   256x128  0.5 W  52 -> 32 / 18 -> 12    0.75 W  55 -> 48 / 19 -> 17
//            W      60 -> 57 / 20 -> 18    1.25 W 107 -> 85 / 34 -> 28
//            2 W   121 -> 119 / 37 -> 34   (8 W, K 3584: 430 us in tiles, 480 by
//            the rate of 4 W in blocks: the clock is power-limited there and the
//            larger tile reads less per flop)
//   256x256  0.25 W 72 -> 33 / 25 -> 13    0.5 W   74 -> 57 / 26 -> 19
//            0.75 W 82 -> 90 / 28 -> 29    W      101 -> 119 / 32 -> 34
//            1.25 W 168 -> 158 / 52 -> 45  1.5 W  178 -> 182 / 55 -> 51
//            1.75 W 190 -> 214 / 57 -> 59
// Where blocks may not run in pairs (compute units reserved), they take a round of
// single blocks for W of them, 0.6 of a round of 256x128 tiles and 0.4 of one of
// 256x256 (W = 240, fp16, K 4096 / 1024, tiles -> blocks):
//   256x128  0.5 W   53 -> 34 / 18.0 -> 12.8  0.53 W 51.9 -> 52.8 / K 256 9.5 -> 11.7
//            W       62 -> 65 / 20.4 -> 22.2  1.25 W 106 -> 89 / 33.8 -> 29.6
//            1.5 W  109 -> 96 / 34.5 -> 31.9  2 W      - / 38.3 -> 41.0
//   256x256  0.25 W  72 -> 34 / 24.9 -> 12.6  0.5 W   75 -> 65 / 25.9 -> 22.6
//            1.04 W 161 -> 145 / -            1.25 W 163 -> 156 / -
//            1.33 W   - / 51.2 -> 54.2
inline bool takes_parts(int tile_n, int64_t tiles, int64_t W, int64_t K, bool share_cus) {
    if (!share_cus) {
        const int64_t rounds = (tiles + W - 1) / W, block_rounds = (tiles * (tile_n / 64) + W - 1) / W;
        return tile_n == 128 ? tiles <= 2 * W && 4 * block_rounds < 7 * rounds : block_rounds < 3 * rounds;
    }
    if (tile_n == 128) return tiles <= 2 * W;
    return 2 * tiles <= W || (tiles > W && (4 * tiles <= 5 * W || (K <= 1024 && 2 * tiles <= 3 * W)));
}

}  // namespace fo
