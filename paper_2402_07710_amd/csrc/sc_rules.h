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

}  // namespace sc
