// Sides of the lines in sc_rules.h that measurements have settled, for 256 compute units and for others.
#include "sc_rules.h"

using namespace sc;
constexpr int64_t tiles(int64_t rows) { return (rows + 63) / 64; }

// 110 k rows of three sweeps and 100 k of one: runs; 53 k: eighths
static_assert(map_in_runs(tiles(110545), 3, 256) && map_in_runs(tiles(100000), 3, 256) && !map_in_runs(tiles(53373), 3, 256), "K = 3");
static_assert(map_in_runs(tiles(64000), 5, 256) && !map_in_runs(tiles(53373), 5, 256), "K = 5");
// the first tile past the line, and the line goes with the compute units
static_assert(!map_in_runs(1536, 3, 256) && map_in_runs(1537, 3, 256) && !map_in_runs(896, 5, 256) && map_in_runs(897, 5, 256), "first tile");
static_assert(map_in_runs(385, 3, 64) && !map_in_runs(384, 3, 64) && !map_in_runs(1537, 3, 304), "per compute unit");

// bytes of the offset table of a layer with K == stride
constexpr int64_t table(int64_t rows, int K) { return tiles(rows) * K * K * K * 256; }
constexpr bool is_short(int64_t rows, int K) { return short_strided_build(rows, K, K, table(rows, K)); }
static_assert(is_short(1, 7) && is_short(200000, 2) && is_short(150000, 3) && is_short(49000, 4) && is_short(16000, 5) && is_short(3000, 7), "short");
static_assert(!is_short(33000, 5) && !is_short(17000, 6) && !is_short(12000, 7) && !is_short(262145, 2) && !is_short(155329, 3), "general");
static_assert(!short_strided_build(1000, 3, 2, 1), "one candidate per input only");

// 32 -> 64: 7 tiles per compute unit where strided cells overlap, however exactly the caller knows the rows; 13 elsewhere, K == stride = 3 too
static_assert(general_32_to_64(tiles(115000), true, 256) == false && general_32_to_64(tiles(114000), true, 256), "stride 2");
static_assert(general_32_to_64(tiles(150000), false, 256) && !general_32_to_64(tiles(213100), false, 256), "the others");
// 128 -> 128: the rounds of a layer that is not strided count, a strided one's are not known
static_assert(general_128_to_128(3, tiles(400000), false, 256) && !general_128_to_128(3, tiles(400000), true, 256), "part-filled rounds");
static_assert(!general_128_to_128(3, tiles(500000), false, 256) && !general_128_to_128(2, tiles(400000), false, 256), "full rounds, K = 2");
static_assert(general_128_to_128(3, tiles(436864), false, 256) && !general_128_to_128(3, tiles(436865), false, 256), "fourth round five sixths full");
static_assert(!general_128_to_128(3, 8192, false, 256) && general_128_to_128(3, 8193, false, 256) && general_128_to_128(3, 8533, false, 256) &&
              !general_128_to_128(3, 8534, false, 256) && !general_128_to_128(3, 10241, false, 256), "a fifth round begun, a sixth");
static_assert(general_128_to_128(3, 20 * 256, true, 256) && general_128_to_128(2, 20 * 256, true, 256), "up to 20 tiles per compute unit");

// longer steps up to three workgroups per compute unit, one for 64 output channels: 32 -> 64 on 40 k rows too
static_assert(few_workgroups(tiles(40000), 4, 256) && few_workgroups(768, 4, 256) && !few_workgroups(769, 4, 256), "64 output channels");
static_assert(few_workgroups(384, 8, 256) && !few_workgroups(385, 8, 256) && few_workgroups(768, 1, 256), "128 and 16 output channels");

// SC_N_MAX rows, fp32, 240 and 256 output channels: 8 blocks of 512 threads a tile, two rows of the grid, none left out; one row up to 2^22 workgroups
constexpr int64_t most = tiles(67108864) * 8;
static_assert(!grid_fits(most, 512) && grid_fits(grid_columns(most), 512) && grid_columns(most) * grid_rows(most) >= most && grid_rows(most) == 2, "largest launch");
constexpr int64_t past = (int64_t)1 << 22;
static_assert(grid_columns(past) == past && grid_rows(past) == 1 && grid_rows(past + 32) == 2 && grid_fits(grid_columns(past + 32), 512), "second row");
static_assert(grid_columns(32) == 32 && grid_rows(32) == 1, "small launch");

// 16-bit weights beyond 12 MiB, more than 2 1/4 tiles per compute unit, beyond 6, more than 3 1/4: blocks of output channels apart
constexpr int64_t k7 = 343 * 128 * 256 * 2, k5 = 125 * 128 * 256 * 2, k3 = 27 * 256 * 256 * 2;
static_assert(first_tiles_apart(k5, 2, false, 256) == 833 && first_tiles_apart(k5, 2, true, 64) == 209 && first_tiles_apart(k5 / 2, 2, true, 256) == INT64_MAX, "K = 5");
static_assert(first_tiles_apart(k7, 2, false, 256) == 577 && first_tiles_apart(2 * k5, 2, false, 256) == 577 && first_tiles_apart(k3, 2, true, 256) == INT64_MAX, "K = 7, 3");
static_assert(first_tiles_apart(k7, 1, true, 256) == 577 && first_tiles_apart(k5, 1, true, 256) == 833 && first_tiles_apart(k7, 1, false, 256) == INT64_MAX, "one block");

// fp32, 16 output channels: four workgroups per CU are a round fewer than three, by more than half a workgroup per CU
static_assert(!fewer_rounds_of_four(1, 256) && !fewer_rounds_of_four(896, 256) && fewer_rounds_of_four(897, 256) && fewer_rounds_of_four(1024, 256) &&
              !fewer_rounds_of_four(1025, 256) && fewer_rounds_of_four(1665, 256) && fewer_rounds_of_four(225, 64), "rounds");

// tiles with many offsets first: from two workgroups per compute unit on, from 1 1/4 where no more than two fit, up to 12 tiles per compute unit
static_assert(!dense_tiles_first(512, 512, false, 256) && dense_tiles_first(513, 513, false, 256) && dense_tiles_first(129, 516, false, 256), "two workgroups");
static_assert(!dense_tiles_first(80, 320, true, 256) && dense_tiles_first(81, 324, true, 256), "two at a time");
static_assert(dense_tiles_first(3072, 3072, false, 256) && !dense_tiles_first(3073, 6146, false, 256) && dense_tiles_first(768, 768, false, 64), "12 tiles");
static_assert(density_wanted(65, 256) && !density_wanted(64, 256) && density_wanted(3072, 256) && !density_wanted(3073, 256), "of the maps, where a layer may ask");
static_assert(!dense_tiles_first(64, 1024, false, 256), "what the map does not hold is not asked for");

// two sets of wavefronts up to two workgroups per compute unit, with 32 input channels 1 1/4; not for 16 output channels, nor for 256 input channels
static_assert(two_sets(512, 27, 4, 64, false, 256) && !two_sets(513, 27, 4, 64, false, 256) && two_sets(256, 8, 8, 128, false, 256) && !two_sets(257, 8, 8, 128, false, 256), "two");
static_assert(two_sets(320, 27, 4, 32, false, 256) && !two_sets(321, 27, 4, 32, false, 256) && two_sets(512, 27, 2, 128, false, 256) && two_sets(128, 27, 4, 64, false, 64), "1 1/4");
static_assert(two_sets(512, 125, 2, 32, false, 256) && !two_sets(513, 125, 2, 32, false, 256) && two_sets(512, 64, 4, 32, false, 256) && !two_sets(257, 343, 8, 64, false, 256), "K > 3: two");
static_assert(!two_sets(1, 27, 1, 64, false, 256) && !two_sets(1, 27, 4, 256, false, 256) && !two_sets(1, 125, 1, 32, false, 256) && !two_sets(1, 125, 4, 256, false, 256), "one set");
// strided with K >= 2 stride: 1 1/4, whatever the channels
static_assert(two_sets(320, 125, 4, 64, true, 256) && !two_sets(321, 125, 4, 64, true, 256) && two_sets(160, 8, 8, 128, true, 256) && !two_sets(161, 8, 8, 128, true, 256), "many rows");
static_assert(two_sets(320, 27, 4, 32, true, 256) && !two_sets(321, 27, 4, 32, true, 256) && two_sets(80, 64, 4, 64, true, 64), "many rows, 32 input channels");

// 256 input channels, one output block per wavefront: 1 3/4 pairs of blocks per compute unit, inverse maps 1 1/2, K == stride and K > 3 2
static_assert(one_block_of_256(448, 27, SUBMANIFOLD, 256) && !one_block_of_256(449, 27, SUBMANIFOLD, 256) && one_block_of_256(448, 27, OVERLAPPING, 256) &&
              !one_block_of_256(449, 27, OVERLAPPING, 256), "submanifold, overlapping");
static_assert(one_block_of_256(384, 8, INVERSE, 256) && !one_block_of_256(385, 27, INVERSE, 256) && one_block_of_256(96, 8, INVERSE, 64), "inverse maps");
static_assert(one_block_of_256(512, 27, CELLS, 256) && !one_block_of_256(513, 27, CELLS, 256) && one_block_of_256(512, 8, CELLS, 256), "K == stride");
static_assert(one_block_of_256(512, 125, SUBMANIFOLD, 256) && !one_block_of_256(513, 125, OVERLAPPING, 256) && one_block_of_256(512, 64, INVERSE, 256), "K > 3");

// the resident kernels' shares: a division rounded up, up to the most that a workgroup takes
constexpr bool shares_are_quotients() {
    const int teams[] = {1, 8, 31, 32, 38};
    for (int most = 2; most <= 4; most += 2)
        for (int team : teams)
            for (int left = 1; left <= 6 * team; ++left) {
                const int quotient = (left + team - 1) / team;
                if (tiles_per_workgroup(left, team, most) != (quotient < most ? quotient : most)) return false;
            }
    return true;
}
static_assert(shares_are_quotients(), "tiles per workgroup");
