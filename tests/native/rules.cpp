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
