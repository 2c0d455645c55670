// Lines between kernels that give the same result, as functions of sizes alone: a host compiler can read them, so a test
// holds them without a GPU.  Tiles are 64 rows, `cus` the compute units of the device.
#pragma once

#include <stdint.h>

namespace sc {

// Submanifold maps, K = 3 and 5: tiles to the XCDs in runs instead of contiguous eighths, of which the one nearest the sensor, whose
// rows find more, ends last.  K = 3 beyond 6 tiles per CU, K = 5 beyond 3.5 (us of the whole 32 -> 32 layer, eighths / runs, 256 CUs.  K = 3:
// sweeps 53 k 23.3 / 23.8, 80 k 32.0 / 31.9, 98 k 36.3 / 35.8, 110 k 38.6 / 38.2, 147 k 47.7 / 47.1, 170 k 53.6 / 52.6; indoor 64 k 26.0 / 26.2, 100 k 38.0 /
// 38.1, 200 k 61.9 / 62.1; random cells in random order 110 k 45.7 / 46.7, 147 k 63.5 / 63.7, 200 k 86.0 / 85.9.  K = 5: sweeps 30 k 42.6 / 43.3, 53 k
// 58.2 / 58.6, 57 k 63.3 / 61.2, 64 k 68.6 / 65.2, 100 k 106.6 / 95.3; indoor 57 k 59.0 / 58.6, 100 k 90.3 / 90.3; random 70 k 109 / 110).
constexpr bool map_in_runs(int64_t tiles, int K, int64_t cus) { return 2 * tiles > (K == 5 ? 7 : 12) * cus; }

// Strided builds with K == stride that are three launches instead of four or five: every input's cell flags as it is claimed, and the offset table is
// cleared beside the cell table, before the number of its rows is known.  Every workgroup of the last launch counts all the flags for itself:
// SHORT_WORDS words of 64 inputs.  What is cleared for nothing grows with the table and the launch saved does not, so up to 16 MiB of
// table; 8 from K = 5 on, where fewer of the rows exist (us of the whole 32 -> 32 layer, sweep and indoor rows, short / general build: K = 2
// 53 k 18.6 / 21.2 and 17.6 / 20.2, 200 k 27.3 / 29.2 and 23.9 / 25.9; K = 3 53 k 25.4 / 26.8 and 25.0 / 26.6, 155 k 33.5 / 34.5 and 31.2 / 32.2; K = 4 20 k 32.5 /
// 34.1 and 33.7 / 35.4, 49 k 36.8 / 37.1 and 37.3 / 37.5, 65 k (16 MiB) 37.9 / 38.1 and 38.2 / 38.0; K = 5 5 k 39.9 / 41.8 and 46.4 / 48.5, 16 k (8 MiB) 44.6 /
// 45.5 and 49.4 / 50.4, 21 k 45.6 / 45.6 and 51.7 / 50.7, 33 k 48.9 / 48.7 and 53.3 / 51.7; K = 6 5 k 53.0 / 54.4 and 67.3 / 69.2, 9.7 k (8 MiB) 57.5 / 57.8 and
// 70.9 / 70.3, 17 k 61.7 / 60.1 and 74.3 / 71.9; K = 7 3 k 66.1 / 66.5 and 95.9 / 96.6, 6 k (8 MiB) 71.7 / 70.5 and 101.3 / 101.9, 12 k 78.5 / 77.1 and 103.7 / 103.6).
constexpr int SHORT_WORDS = 4096;                      // 262,144 inputs
constexpr bool short_strided_build(int64_t n, int K, int stride, int64_t table_bytes) {
    return K == stride && n <= 64 * SHORT_WORDS && table_bytes <= (K <= 4 ? 16 << 20 : 8 << 20);
}

}  // namespace sc
