// Lines between kernels that give the same result (two_sets: the same up to the order of a row's sums), as functions of sizes alone: a host compiler can read them, so a test
// holds them without a GPU.  Tiles are 64 rows, `cus` the compute units of the device.
#pragma once

#include <stdint.h>

namespace sc {

// Kinds of layers, as far as lines differ between them: submanifold, over an inverse map, strided with K == stride and with K != stride (an input in several cells).
enum LayerKind { SUBMANIFOLD, INVERSE, CELLS, OVERLAPPING };

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

// 32 -> 64, K = 3, 16 bit: general kernel or streaming kernel (false).  The streaming kernel walks all offsets, four tiles in step, which is the
// longer chain of few tiles and the cheaper one of many dense ones.  `likely` tiles; `overlapping`: strided with K != stride, whose rows
// have few neighbours each but most offsets.  Up to 13 tiles per CU, overlapping 7 (us of the whole layer, general / streaming, sweep
// and indoor rows.  Submanifold: 53 k 27.6 / 28.5 and 27.3 / 27.9, 115 k 43.2 / 43.1 and 45.2 / 44.2, 150 k 52.5 / 55.7 and 54.6 / 57.5, 213 k 75.6 / 78.7 and 76.4 /
// 78.1, 262 k 96.2 / 96.1 and 96.4 / 92.1.  K == stride = 3, a cell's rows in one place: 53 k 26.5 / 29.8 and 26.3 / 29.2, 150 k 34.2 / 35.2 and 31.6 / 34.0, 213 k
// 39.0 / 39.1 and 34.7 / 36.9, 400 k 57.3 / 53.7 and 45.5 / 44.7.  Stride 2: 53 k 38.5 / 40.8 and 34.9 / 37.0, 85 k 53.9 / 51.9 and 45.9 / 46.6, 115 k 61.6 / 62.7 and
// 51.0 / 50.5, 150 k 76.0 / 73.1 and 63.6 / 65.8, 180 k 87.6 / 86.6 and 71.8 / 69.7, 262 k 123 / 114 and 93.3 / 84.2; the convolution where the caller knows the rows, indoor:
// 53 k 16.1 / 15.1, 69 k 18.6 / 21.0, 83 k 24.2 / 21.7, 121 k 28.0 / 22.4).
constexpr bool general_32_to_64(int64_t likely, bool overlapping, int64_t cus) { return likely <= (overlapping ? 7 : 13) * cus; }

// 128 -> 128, K = 2 and 3, 16 bit: general kernel or streaming kernel (false).  A workgroup of the streaming kernel is eight tiles and takes ~75 us
// however few there are; full, it moves the weights once for them.  General up to 20 tiles per CU (us of the convolution, general / streaming:
// 4 k voxels 17 / 71, 53 k 43 / 75, 262 k 127 / 157; denser sets 265 k 209 / 251, 320 k 259 / 276, 500 k 404 / 347, 10^6 854 / 714; K = 2 on 150 k 25 / 32, 900 k
// 110 / 82).  Beyond, the streaming kernel takes about 86 us a round of eight tiles per CU, full or not, and the general one up to 0.05 us a tile, so
// K = 3 layers whose rounds are less than five sixths full stay with it where the rows are known to the caller: 24 to 26 2/3 and 32 to 33 1/3
// tiles per CU, from six rounds on none.  On sweeps, whose rows find fewer neighbours, it is ahead at every size; on dense sets there only, and how dense a
// set is is not known here.  us of whole layers, general / streaming, sweep and indoor rows, and how full the rounds are: 330 k 0.84 233 / 286 and 314 / 322,
// 394 k 0.75 267 / 359 and 353 / 390, 421 k 0.80 284 / 366 and 376 / 400, 440 k 0.84 296 / 372 and 394 / 406, 460 k 0.88 314 / 376 and 421 / 410, 500 k 0.95 327 / 391 and
// 458 / 419, 530 k 0.81 354 / 466 and 501 / 508, 560 k 0.85 376 / 460 and 528 / 515, 600 k 0.92 399 / 468 and 569 / 527, 660 k 0.84 438 / 537 and 621 / 611, 790 k
// 0.86 512 / 621 and 750 / 710, 10^6 0.95 651 / 738 and 945 / 825.  Fused: 262 k 157 / 195 and 206 / 192, 330 k 199 / 282 and 260 / 277, 394 k 244 / 376 and 312 / 371,
// 440 k 275 / 388 and 361 / 384, 500 k 303 / 391 and 415 / 392, 530 k 322 / 477 and 452 / 484, 600 k 367 / 484 and 519 / 496, 10^6 614 / 775 and 884 / 795.  Convolution of
// inverse maps, K = 3: 394 k 162 / 236 and 235 / 248, 419 k 147 / 227 and 217 / 237, 437 k 149 / 228 and 220 / 237, 545 k 183 / 279 and 255 / 296.  Of strided
// layers only the inputs are known, and the rows decide how full the rounds are: stride 2 on 400 k sweeps 396 / 386, indoor 270 / 267, stride 3 132 / 111 and
// 109.4 / 110.9.
constexpr bool general_128_to_128(int K, int64_t likely, bool strided, int64_t cus) {
    const int64_t round = 8 * cus;
    return likely <= 20 * cus || (K == 3 && !strided && 6 * likely < 5 * ((likely + round - 1) / round * round));
}

// The general kernel, K <= 3, up to three workgroups per CU: steps of four offsets of 32-channel rows and of two of 64-channel ones, the shorter walk; 39 KB of LDS,
// four workgroups a CU.  A workgroup's walk is bound by the instructions of its steps there (list, loop and barrier once for more offsets), beyond
// by the loads, and steps of two and one (23 KB, six workgroups a CU; groups without a neighbour left out) are worth more.
// us of whole layers, four and two offsets: 32 -> 64 sweeps 30 k / 38 k / 46 k / 53 k / 70 k 21.0 / 23.0 / 24.1 / 28.1 / 33.8 and 22.0 / 23.6 / 24.4 / 27.5 / 32.0,
// indoor 21.1 / 23.7 / 25.0 / 28.8 / 34.4 and 21.6 / 23.5 / 24.6 / 27.4 / 31.7; K = 3, stride 2, sweeps 30.6 / 33.4 / 36.2 / 40.4 / 49.2 and 31.5 / 33.9 / 36.2 / 38.7 /
// 48.4, indoor 28.4 / 31.1 / 32.8 / 34.1 / 40.8 and 30.1 / 32.5 / 34.0 / 35.4 / 41.9; fused sweeps 17.1 / 19.9 / 20.3 / 23.0 / 26.9 and 18.2 / 20.2 / 20.8 / 23.1 / 25.8;
// 32 -> 128 sweeps 14 k / 20 k / 28 k 18.2 / 20.6 / 24.0 and 19.0 / 20.6 / 23.1, indoor 19.1 / 21.8 / 25.3 and 19.1 / 21.2 / 24.2.
// Two offsets and one: 64 -> 64 sweeps 36 k / 46 k / 55 k / 60 k 26.2 / 28.0 / 32.6 / 34.3 and 27.9 / 29.7 / 33.2 / 34.9, indoor 27.4 / 29.3 / 34.7 / 35.6 and 27.5 / 29.1 / 33.4 /
// 34.7; K = 3, stride 2, sweeps 36.3 / 40.3 / 46.0 / 49.0 and 37.5 / 40.5 / 44.6 / 46.9, indoor 33.7 / 35.5 / 37.3 / 38.0 and 36.9 / 39.0 / 40.2 / 40.9; 64 -> 128 sweeps
// 18 k / 26 k / 30 k 23.0 / 26.7 / 28.2 and 25.5 / 27.2 / 28.3, indoor 25.4 / 30.1 / 31.2 and 25.4 / 28.9 / 30.5.
constexpr bool few_workgroups(int64_t likely, int CB, int64_t cus) { return likely * ((CB + 3) / 4) <= 3 * cus; }

// The general kernel, 16 bit, up to 128 input channels: two sets of four wavefronts walk alternate offsets of the tile and add up their sums in the end.  The other
// 16-bit kernels, and this one beyond the line, add the offsets up in increasing order, so a row's last bits differ between the sides; `tiles` are
// those of the rows the map was built from (strided layers: the inputs), which a caller's capacity does not move.  Up to
// two workgroups per CU (32 input channels, K <= 3, 1 1/4) a layer takes as long as the workgroup of a dense tile walks its offsets, one wavefront per SIMD, and of 27
// offsets each set walks 14; beyond, the CUs have enough wavefronts and the sums are traded for nothing.  us of whole layers, one set / two, sweeps: 64 -> 64 500 15.5 /
// 14.5, 2 k 18.0 / 16.0, 10 k 19.9 / 18.9, 14 k 20.8 / 20.2, 25 k 23.1 / 22.4, 30 k 23.8 / 22.9, 42 k 26.5 / 26.1, 53 k 32.4 / 32.0, 80 k 38.1 / 41.2; indoor 3 k 18.6 / 16.7, 10 k 19.2 / 17.5, 30 k 23.9 / 23.2, 40 k 28.4 /
// 29.1; stride 2 2 k 26.1 / 23.9, 20 k 30.1 / 29.3; 64 -> 128 5 k 19.3 / 17.6, 20 k 23.6 / 23.1, 40 k 30.3 / 34.3; 128 -> 128 500 18.9 / 17.3, 2 k 23.1 / 20.3, 8 k 27.6 / 24.4, 14 k 29.6 / 25.8, 20 k 31.1 /
// 31.6, 26 k 32.4 / 35.3; indoor 5 k 26.4 / 23.8, 15 k 29.6 / 30.2; 128 -> 256 1 k 22.4 / 20.0, 8 k 29.1 / 25.3, 12 k 30.4 / 32.9; 128 -> 32 30 k 29.3 / 26.4; 32 -> 64 1 k 15.3 / 14.6, 10 k 16.5 / 16.1, 14 k 17.5 / 17.0, 20 k 18.7 /
// 18.7, 53 k 26.8 / 30.4.  256 input channels, whose offsets take 64 KB through the L1 of a CU, as fast as that goes, are the same with two sets (1 k 27.8 / 28.0, 14 k 49.1 / 50.8).
// K > 3, whose walks are longer: two workgroups per CU, sweeps gain up to four and dense sets lose from one and a half (32 input channels) or two on (one set / two,
// K = 5, sweeps: 32 -> 32 2 k 24.2 / 22.2, 6 k 34.2 / 29.1, 20 k 40.3 / 36.3, 35 k 46.8 / 43.0, 46 k 49.7 / 49.7, 53 k 56.1 / 57.9; 32 -> 64 2 k 27.2 / 23.8, 20 k 41.7 / 37.6, 53 k 58.1 / 60.0; 64 -> 64 2 k
// 34.0 / 29.1, 12 k 50.9 / 41.5, 35 k 62.6 / 53.4, 53 k 73.0 / 66.7, 75 k 87.3 / 89.8; 128 -> 128 2 k 51.8 / 42.0, 12 k 78.8 / 64.1, 25 k 87.3 / 75.6, 53 k 118.5 / 128.4; 64 -> 32 30 k 59.7 / 48.3;
// indoor 32 -> 32 5 k 30.5 / 26.8, 20 k 36.8 / 35.8, 30 k 38.8 / 40.0, 36 k 46.1 / 49.8; 64 -> 64 5 k 42.5 / 35.3, 30 k 52.2 / 51.7, 40 k 65.2 / 71.0; 128 -> 128 15 k 70.9 / 71.7, 20 k 87.6 / 94.9; random
// cells 64 -> 64 5 k 36.5 / 32.0, 20 k 53.4 / 48.1; K = 7 64 -> 64 10 k 118 / 94.5, 30 k 138 / 113).
// `many_rows`: strided with K >= 2 stride, where an input is in eight cells and more, and even on surfaces more rows than inputs come: 1 1/4 too (us of the convolution, one
// set / two, sweep, indoor and random rows: K = 4, stride 2, 64 -> 64 8 k 20.3 / 16.0, 22.1 / 17.2 and 27.2 / 30.1, 16 k 21.1 / 16.5, 22.2 / 17.3 and 45.7 / 51.4, 24 k 22.1 / 20.9,
// 22.3 / 17.4 and 62.7 / 71.4, 32 k 28.6 / 28.5, 25.2 / 25.6 and 79.4 / 93.1; K = 5, stride 2, 32 -> 64 8 k 23.4 / 17.6, 24.2 / 18.3 and 38.9 / 42.4, 16 k 24.1 / 18.1, 24.4 / 18.7 and 62.9 / 78.6, 21 k
// 24.4 / 19.5, 26.2 / 26.5 and 80 / 101, 24 k 24.6 / 22.8, 26.8 / 26.8 and 90.7 / 115.6, 32 k 33.6 / 33.8, 27.3 / 33.0 and 117 / 154; K = 7, 64 -> 64 16 k 102 / 74, 118 / 107 and 232 / 271, 30 k 117 / 101, 156 / 175 and 506 / 591).  Random cells, which have up to eight times the rows, lose below the line as well; how many rows
// there are is not known here.  The other overlapping strides keep two: K = 3, stride 2, 64 -> 64 16 k 11.7 / 9.4, 11.8 / 9.5 and 16.8 / 16.5, 32 k 13.5 / 13.3, 11.8 / 9.5 and 28.0 / 26.6, 64 -> 128 16 k
// 12.9 / 11.3, 11.9 / 9.6 and 27.7 / 26.4, 128 -> 128 8 k 17.3 / 14.1, 19.0 / 15.2 and 24.0 / 27.2, 16 k 19.3 / 17.6, 19.1 / 15.3 and 40.4 / 44.0; K = 5, stride 3, 64 -> 64 16 k 31.8 / 24.8, 39.7 / 30.1
// and 33.9 / 38.6, 32 k 32.7 / 25.2, 39.8 / 30.2 and 59.4 / 59.7.
constexpr bool two_sets(int64_t tiles, int K3, int CB, int C_in, bool many_rows, int64_t cus) {
    return CB > 1 && C_in <= 128 && tiles * ((CB + 3) / 4) * 4 <= ((C_in == 32 && K3 <= 27) || many_rows ? 5 : 8) * cus;
}

// The general kernel, 16 bit, 256 input channels, whose step is the longest: one or two output blocks per wavefront.  `pairs` are tiles times pairs of blocks of 64
// channels.  Two halve how often a tile's rows are gathered and leave CUs idle where there are few.  us of the convolution, one / two blocks, sweep, indoor and random rows (256 CUs: 1 pair per CU is 128
// tiles of 256 -> 256 and 256 of 256 -> 128).
// Submanifold layers, K = 3, 1 3/4 pairs per CU: sweeps gain up to there and, from 1 5/8 on, less than the others lose; how dense a set is is not known here (means of five sets): 256 -> 256 12.4 k 30.9 / 38.9, 56.1 / 48.1 and 26.6 / 24.1, 13 k
// 32.7 / 39.0, 58.4 / 49.6 and 27.5 / 24.4, 14 k 36.2 / 39.5, 59.4 / 51.0 and 27.7 / 24.1, 16 k 41.5 / 41.7, 66.4 / 56.8 and 29.2 / 24.4; 256 -> 128 24 k 33.7 / 41.1, 55.8 / 52.1 and 26.6 / 24.2, 26 k 38.2 / 41.2, 58.5 / 51.1 and
// 27.3 / 24.3, 31 k 43.7 / 42.8, 65.6 / 57.7 and 28.7 / 24.9.  K > 3 2 (whole layers, 229 tiles 138 / 161 and 203 / 187, 255 tiles 149 / 178 and 216 / 190).
// Inverse maps, 1 1/2: K = 2 256 -> 256 9 k 16.9 / 17.8, 21.1 / 20.5 and 21.2 / 20.9, 12.4 k 18.4 / 18.3, 22.8 / 20.6 and 22.7 / 20.2, 16 k 20.2 / 18.3, 24.9 / 20.6 and 24.9 / 20.4; K = 3 12.4 k 30.8 / 31.3, 47.1 / 42.8 and 46.0 / 42.0, 16 k
// 35.2 / 31.9, 52.1 / 43.6 and 49.9 / 42.9; 256 -> 128 K = 2 18 k 15.5 / 16.8, 19.9 / 19.6 and 19.9 / 19.8, 24 k 18.4 / 17.5, 20.8 / 20.3 and 21.0 / 20.2.
// Strided layers with K == stride, whose rows are fewer than the inputs that are counted, 2 (beyond not tried): K = 2 256 -> 256 12 k 9.7 / 12.7, 10.5 / 14.3 and 21.4 / 21.0, 16 k 11.7 / 12.9, 12.8 / 14.4 and
// 25.1 / 21.9; K = 3 12 k 19.4 / 27.8, 26.5 / 39.5 and 46.3 / 44.3, 16 k 20.7 / 29.4, 26.7 / 39.8 and 52.5 / 45.7; 256 -> 128 K = 2 24 k 11.3 / 13.0, 10.4 / 14.4 and 21.5 / 21.0, K = 3 31 k 20.8 / 29.9, 26.5 / 39.5 and 51.4 / 46.2.
// Overlapping ones, 1 3/4: K = 3, stride 2, 256 -> 256 9 k 30.2 / 36.4, 31.5 / 39.1 and 91.5 / 82.0, 12 k 41.5 / 38.8, 34.3 / 39.3 and 116 / 103, 14 k 47.3 / 43.8, 37.5 / 39.5 and 136 / 119, 16 k 52.4 / 46.3,
// 38.9 / 39.8 and 150 / 124; 256 -> 128 24 k 48.4 / 47.3, 33.1 / 38.9 and 116 / 103, 31 k 57.0 / 52.1, 36.5 / 39.3 and 148 / 123.
constexpr bool one_block_of_256(int64_t pairs, int K3, LayerKind kind, int64_t cus) {
    return 4 * pairs <= (K3 > 27 || kind == CELLS ? 8 : kind == INVERSE ? 6 : 7) * cus;
}

// The general kernel, 16 bit: a tile's blocks of output channels one after the other on an XCD, whose L2 then holds the tile's rows for the second,
// or all tiles' first blocks before any second one: the tile count from which it is the latter.  Where the weights are larger than an
// L2 (4 MiB), workgroups of one block at a time share half the weights of a few offsets.  Of the tiles that are there, with two output blocks per wavefront:
// beyond 12 MiB from 2 1/4 per CU on, beyond 6 MiB from 3 1/4 (us of the convolution, one after the other / apart, sweep and indoor rows, 256 CUs.  K = 5,
// 64 -> 256, 3.9 MiB: 100 k 151 / 154 and 234 / 237; 128 -> 256, 7.8 MiB: 40 k
// 150 / 165 and 197 / 207, 55 k 196 / 200 and 254 / 252, 70 k 251 / 236 and 320 / 322, 100 k 317 / 291 and 489 / 471, 200 k 567 / 505 and 1004 / 912; 256 -> 256, 15.6 MiB:
// 100 k 775 / 658 and 1145 / 1089, 200 k 1549 / 1181 and 2480 / 2136; stride 2 80 k 1419 / 1145 and 1151 / 1072.  K = 7, 64 -> 256, 10.7 MiB: 40 k 169 / 199 and
// 202 / 214, 55 k 232 / 232 and 262 / 262, 100 k 363 / 333 and 521 / 517; 128 -> 256, 21 MiB: 100 k 902 / 802 and 1361 / 1301.  K = 4, stride 2, 256 -> 256, 8 MiB:
// 2.8 tiles per CU 364 / 373, 3.2 429 / 426, 6.4 490 / 459, 15.4 1130 / 1045.  Apart over one after the other, map and convolution, mean of five sweeps, of five
// indoor sets, and random cells, whose groups of rows fetch weights for few neighbours: K = 5, 256 -> 256, 1.2 tiles per CU 1.06, 1.05, 0.90, 1.6 1.04, 1.01, 0.83, 2.1
// 1.04, 1.01, 0.78, 2.4 0.97, 1.02, 0.78, 2.9 0.91, 1.03, 0.75; K = 7 1.2 1.13, 1.06, 0.86, 2.1 1.01, 0.99, 0.77, 2.9 0.96, 0.99, 0.80; K = 7, 128 -> 256, 2.1
// 1.13, 0.99, 0.79, 2.4 1.01, 1.00, 0.83).  With one output block per wavefront, which is for few tiles to expect, only where a strided layer has many more rows than
// inputs (256 -> 256 on random cells K = 6, stride 3, 3.8 tiles per CU 1257 / 650, 6.1 to 7 with K = 4, stride 2, 8 MiB 611 / 509; sweeps K = 6 2.7 604 / 493): in the others
// apart is slower (K = 7, 128 -> 128 56 k 265 / 287, 256 -> 128 1.2 to 1.8 tiles per CU 1.04 to 1.19 of one after the other).  In fp32, whose multiplies take
// the time, apart is slower at every size: K = 5, 256 -> 256 50 k 2317 / 2700.
constexpr int64_t first_tiles_apart(int64_t weight_bytes, int blocks_per_wavefront, bool strided, int64_t cus) {
    if (weight_bytes <= 6 << 20 || (blocks_per_wavefront == 1 && !strided)) return INT64_MAX;
    return (weight_bytes > 12 << 20 ? 9 : 13) * cus / 4 + 1;
}

// The general kernel, fp32, 16 output channels, K >= 4: the list of offsets in registers instead of behind the buffers in LDS, which are a quarter of it.  A step takes
// longer, but four workgroups are on a CU at a time instead of three; so where that is a round fewer, and not for less than half a workgroup per CU (us of map and
// convolution, before there was a list / in LDS / in registers.  3.3 workgroups per CU, K = 5 and 7, sweeps 69 / 64 / 67 and 149 / 139 / 143.  3.8: 16 -> 16, K = 5, indoor
// 76 / 85 / 75, K = 7, indoor 184 / 196 / 177, random 242 / 259 / 237, sweep 165 / 160 / 157, K = 5, stride 2, indoor 159 / 172 / 157; 32 -> 16, K = 5, sweep 79 / 75 / 75, random 90 /
// 95 / 88, K = 7, stride 3, sweep 215 / 203 / 209.  7.9: K = 5, indoor 138 / 141 / 134, sweep 125 / 120 / 120, K = 4, stride 2, sweep 153 / 156 / 150; K = stride = 4, inverse, 14:
// indoor 119 / 117 / 110; slower on surfaces with stride 3, K = 7, indoor 62 k rows 216 in LDS, 225 in registers).  K <= 3 and 16-channel blocks of wider layers: within 2 %, some
// sets 5 % to 8 % slower.
constexpr bool fewer_rounds_of_four(int64_t workgroups, int64_t cus) {
    return (workgroups + 4 * cus - 1) / (4 * cus) < (workgroups - cus / 2 + 3 * cus - 1) / (3 * cus);
}

// Maps that such a layer may follow hold how many offsets their tiles take part in.  (A tile has up to 16 workgroups: fp32, 256 output channels.)
constexpr bool density_wanted(int64_t tiles, int64_t cus) { return 4 * tiles > cus && tiles <= 12 * cus; }
// The general kernel on submanifold maps: the tiles with many offsets first (xcd_dense_first).  A workgroup of a tile with 27 offsets runs three
// times as long as one with 9, which is what most tiles of a sweep have, and the dispatcher deals workgroups to the CUs in turn: in the order of the rows,
// 110 k rows 64 -> 64, a CU gets 48 to 159 offsets (93 on average) and the last dense tile starts when most others are done.  Finding the tile is a round trip,
// about 0.6 us a workgroup, in front of all others.  From two workgroups per CU on (1 1/4 where LDS holds no more than two at a time), up to
// 12 tiles per CU; beyond, sweeps gain less than sets without sparse tiles lose, and how dense a set is is not known here.  Sets whose tiles are all alike
// pay for the look-up and gain nothing: up to 4 % of a layer, 1 % to 11 % of the convolution.  us of whole layers, in the order of the rows / dense first, sweep, indoor and random rows (means of three
// sets): 64 -> 64 36 k 26.7 / 25.8 and 28.4 / 29.0, 53 k 32.5 / 31.7, 33.9 / 34.8 and 33.9 / 34.3, 70 k 37.8 / 36.3 and 39.8 / 40.8, 100 k 45.3 / 42.1 and 51.9 / 52.3, 150 k 60.9 / 58.9 and 67.2 / 68.4, 190 k 72.5 / 70.2 and
// 82.6 / 83.4; 32 -> 64 36 k 22.3 / 21.8 and 23.4 / 23.8, 53 k 27.4 / 26.6, 28.0 / 28.8 and 30.7 / 31.6, 150 k 52.1 / 50.8 and 54.1 / 55.6; 64 -> 128 20 k 23.9 / 23.0, 25.7 / 26.4 and 22.7 / 23.1, 53 k 39.8 / 37.4, 46.9 / 48.1 and
// 39.4 / 40.2; 128 -> 128 20 k 31.8 / 30.4, 35.8 / 36.5 and 26.9 / 27.2, 53 k 54.2 / 48.0, 68.1 / 69.4 and 46.3 / 47.4, 100 k 85.3 / 73.5 and 102.6 / 104.3, 150 k 110.7 / 106.1 and 144.2 / 145.8; 128 -> 256 53 k 75.9 / 64.4 and
// 98.9 / 100.6; 256 -> 256 6 k 36.4 / 35.1 and 40.3 / 40.4, 8 k 42.0 / 36.9 and 43.0 / 42.9, 14 k 60.2 / 48.9, 67.1 / 69.7 and 38.6 / 40.3, 53 k 121.7 / 104.3 and 177.5 / 182.4; fp32 64 -> 64 12 k 34.3 / 32.2 and 39.4 / 40.0, 53 k
// 86.8 / 73.7 and 121.8 / 122.4, 110 k 154.2 / 144.3 and 226.7 / 227.7; K = 5 32 -> 32 40 k 46.2 / 46.6 and 48.1 / 49.4, 53 k 56.9 / 56.0 and 56.9 / 56.5, 100 k 87.9 / 81.7 and 88.4 / 88.1, 64 -> 64 53 k 72.3 / 71.6 and 79.7 / 77.8, 100 k
// 113.3 / 98.2 and 127.2 / 125.2.  Below the line, one set of rows: 64 -> 64 14 k 20.7 / 21.3, 30 k 24.1 / 24.2, 256 -> 256 4 k 32.9 / 33.8; above it 262 k 113 / 111.5 and, indoor, 400 k 178 / 180.
constexpr bool dense_tiles_first(int64_t tiles, int64_t workgroups, bool two_at_a_time, int64_t cus) {
    return 4 * workgroups > (two_at_a_time ? 5 : 8) * cus && density_wanted(tiles, cus);
}

// The resident kernels: tiles that a workgroup of a round takes when `left` (at least one) are left for `team` workgroups: as few as give all their share, `most` at most.  A
// division, in front of everything a workgroup does, cost 0.15 us (us of the convolution, K = 2, packed weights, with it and without: 32 -> 32 sweeps 80 k / 110 k 4.44 / 4.70 and 4.23 / 4.52, indoor
// 200 k 5.15 and 4.99, random cells 100 k 5.85 and 5.60; 32 -> 64 30 k / 110 k / 200 k 4.02 / 6.81 / 9.20 and 3.89 / 6.65 / 8.95).
constexpr int tiles_per_workgroup(int left, int team, int most) {
    int each = 1;
    for (int t = 1; t < most; ++t) each += left > t * team ? 1 : 0;
    return each;
}

// Workgroups of the general kernel, tiles times blocks of output channels: a launch takes fewer than 2^32 threads along x, which 2^20
// tiles (SC_N_MAX rows) of 8 blocks and 512 threads are not.  Past GRID_COLUMNS they go on in the next row of the grid, workgroup by workgroup.
constexpr int64_t GRID_COLUMNS = 1 << 22;
constexpr bool grid_fits(int64_t columns, int64_t threads) { return columns * threads < (int64_t)1 << 32; }
constexpr int64_t grid_columns(int64_t groups) { return groups < GRID_COLUMNS ? groups : GRID_COLUMNS; }
constexpr int64_t grid_rows(int64_t groups) { return (groups + GRID_COLUMNS - 1) / GRID_COLUMNS; }

}  // namespace sc
