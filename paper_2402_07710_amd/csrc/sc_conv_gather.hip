// The general convolution kernel: 16-bit layers of 32, 64, 128 and 256 input channels without a kernel of their own in sc_conv.hip,
// or on this kernel's side of the line to that one (sc_rules.h, conv_16bit), and fp32 layers with enough work for it.
#include "sc_conv.h"
#include "sc_rules.h"

namespace sc {

// A row of zeros that stands in for "no neighbour": 512 bytes, up to 256 16-bit channels.
static __device__ __align__(512) uint4 g_zero_row[32];

// where a tile's table entries come from: the map's lines as they are needed, look-ups, the map's lines copied to LDS first, the one line
// of a pointwise layer, or the map's lines as they are needed by a list of offsets in registers
enum { FROM_MAP, FROM_TABLE, FROM_LINES, FROM_LINE, FROM_MAP_BY_REGISTERS };
constexpr int LIST_PAD = 12;                            // places of the list past the last offset: three steps of four, the longest

// One workgroup of NW wavefronts per 64-row tile and block of output channels.  The sum over (offset,
// input channel) is walked in steps of SL slices of 64 bytes of a row (32 16-bit or 16 fp32 channels):
// four slices per step (one offset of 256 bytes, 2 of 128, 4 of 64, a part of a longer one; eight
// for 16-bit rows of 512 bytes), only the offsets at which the tile has a neighbour.
//  * The rows of the next step are gathered straight into the other half of a double LDS buffer
//    while this step multiplies, with eight (four in 64-byte rows) consecutive lanes on one row: whole
//    lines, a quarter of the address cycles of a gather in operand order.  The 16-byte pieces of a row
//    are placed XOR-ed with the row number, so the operand reads (16 rows x one piece) use all banks.
//  * 16-bit weights of the next step go from the packed tiles in global memory (whole lines, the same
//    for all tiles: cache hits) to a second set of registers.  A wavefront owns CT 16-channel output
//    blocks, so no two wavefronts of a tile load the same weights unless the layer has fewer than 64
//    output channels (then they split the rows: WR).
//  * fp32 weights are used as they lie in memory, so an operand is 4-byte reads of four rows: loaded
//    straight to registers they cost as many address cycles as the gathers save (104 us at the size
//    below); they go through LDS instead.  An fp32 multiply takes eight times as long per byte, so the
//    wavefronts (eight) split rows as well as channels.
//  * The steps are read from a list of the tile's offsets that is made once, in LDS: walking the mask words in every step was
//    a third of a step's instructions, and scalar ones issue once per four cycles for all wavefronts of a SIMD (us of whole layers, before
//    and with the list: K = 5 32 -> 32 4 k / 53 k voxels 37.6 / 65.5 -> 31.1 / 58.8, K = 5 64 -> 64 20 k 64.6 -> 56.0, 64 -> 64 4 k / 110 k
//    23.8 / 52.8 -> 22.5 / 51.6, 128 -> 256 5 k 28.8 -> 27.1, fp32 64 -> 64 8 k / 53 k 33.2 / 91.5 -> 31.1 / 88.2, 256 -> 256 14 k 62.6 -> 62.0; 32 -> 64
//    80 k the same).
//  * FROM_LINES (K = 2 and 3, 16 bit): the tile's lines of the map are copied to LDS at the start, beside the
//    masks' round trip.  Read from the map step by step, 32 bytes at a time, they were a third of the loads that the address unit
//    serves at 17 cycles each, and the first gathers waited for them (us of whole layers, before -> with: 64 -> 64 110 k / 262 k / 10^6 voxels
//    51.4 / 117.3 / 457 -> 50.6 / 114.4 / 429, 128 -> 128 20 k / 53 k / 262 k 32.6 / 56.4 / 205.6 -> 31.5 / 54.5 / 201, 256 -> 256 14 k 58.9 -> 56.9, 32 -> 64
//    40 k 24.6 -> 23.7).  7 KB of LDS: fp32 would lose a workgroup per CU to them.
//  * One wait for everything and one barrier per step.  What a step costs is issuing its loads (17
//    cycles of the CU's address unit per instruction) plus its multiplies; the waits are short.
//  * What hides the latency of a step is other workgroups: OCC wavefronts per SIMD (64 -> 64, 262 k voxels:
//    65 us with 2, 51.5 with 4, 50 with 6).  That also decides the step length, 16 KB of LDS for 64 channels.
//  * HV = 2 (two_sets): few workgroups leave most of a CU idle, and two sets of NW wavefronts walk alternate steps of the list, each with its own
//    buffers.  In the end a set hands the sums of half of its groups to the other through LDS.
// A group without a neighbour at an offset is not multiplied by its weights (a weight that is not finite stays out
// of its sums).  SKIP: nor is it gathered and read (64 channels: 62 -> 50 us at that size).  32-channel rows in steps of four
// offsets (few workgroups, or K > 3; steps of two skip) are too short for that: such groups read the row of zeros, and the places of the last step that have no offset are fetched
// like the others (of offset 0, rows of zeros); the operands of an offset are read together, then the
// multiplies tested (whole layers K = 5 32 -> 32 on 2 k / 53 k voxels and 32 -> 64 on 110 k: 30.0 / 63.4 / 116 us; with SKIP
// 31.0 / 64.5 / 121, with zeroed weights instead of the test 30.3 / 64.2 / 120, all of a step's operands first 29.4 / 63.2 / 120).
// FROM_TABLE (fused layers): there is no kernel map; the four (two sets: eight) wavefronts look up every fourth (eighth) of the 27 offsets of the tile's rows in the
// dense location table and leave entries and votes in LDS (7 KB).  Whole fused layers on 2 k / 53 k / 262 k voxels, against
// the kernels that gave a wavefront 64 rows: 64 -> 64 21.2 / 33.6 / 95 -> 17.6 / 30.0 / 81 us, 64 -> 128 38.9 / 46.6 / 124 ->
// 17.8 / 40.0 / 108, 128 -> 128 88.7 / 93.9 / 193 -> 22.4 / 55.3 / 160.
// Measured, before (one wavefront per 16 rows, rows and weights loaded at their use) -> now: 14 k
// voxels 256 -> 256 f16 480-555 -> 44 us; 53 k voxels K = 5 32 -> 32 bf16 116 -> 38 us; 53 k voxels 64 -> 64
// fp32 118 -> 72 us.  Against the kernels that shared W[k] in LDS or gave a wavefront 64 rows: 64 -> 64 2 k /
// 20 k / 110 k / 262 k voxels 14.8 / 15.8 / 29.4 / 58.2 -> 10.7 / 14.1 / 28.6 / 50.3 us; 64 -> 128 4 k / 110 k 27.4 /
// 47.1 -> 11.7 / 40.7; 128 -> 128 4 k / 53 k / 262 k 70.8 / 75.5 / 157 -> 16.8 / 43 / 127.5.
template <int DT, int KS, int NW, int WR, int CT, int SL, int SKIP, int OCC, int SRC, int HV>
__global__ void __launch_bounds__(64 * NW * HV, OCC)
k_conv_gather(const void* feat, const void* wp, void* __restrict__ out, int out_f32, const MapSource ms, int K3, int mw, int CB,
              int blocks_y, int64_t tiles_apart, const int64_t* __restrict__ n_out_ptr, int64_t n_out_cap) {
    constexpr bool FUSED = SRC == FROM_TABLE, HELD = FUSED || SRC == FROM_LINES, POINT = SRC == FROM_LINE, REGS = SRC == FROM_MAP_BY_REGISTERS;      // HELD: the tile's entries are in LDS
    static_assert(!HELD || (DT != SC_F32 && NW == 4), "a quarter of the 27 offsets per wavefront");
    static_assert(HV == 1 || (HV == 2 && DT != SC_F32 && !POINT && !REGS), "two sets of wavefronts: 16 bit, a list of offsets in LDS");
    const uint32_t* __restrict__ gmask = ms.gmask;
    const int32_t* __restrict__ nbr = ms.nbr;
    constexpr bool F32 = DT == SC_F32;
    constexpr int KP = KS < SL ? KS : SL, PARTS = KS / KP;     // slices of an offset taken in one step, steps per offset
    constexpr int OPS = SL / KP;                       // offsets per step
    // the two steps after the last are read too: up to 3 OPS - 1 places past the last offset, which have to be zeros
    static_assert(!REGS || WAVE % OPS == 0, "a step's places are in one register");
    static_assert(3 * OPS <= LIST_PAD, "the list's zeros reach as far as the steps read");
    constexpr int PAD = LIST_PAD * HV;
    constexpr int CH = KP == 1 ? 1 : KP / 2;           // chunks per offset and step: 64 rows x 128 (64) bytes
    constexpr int CHB = KS == 1 ? 4096 : 8192;         // bytes per chunk
    constexpr int NI = KS == 1 || NW == 8 ? 1 : 2;     // gather instructions per wavefront and chunk
    constexpr int STEP_BYTES = SL * 4096;
    constexpr int WC = NW / WR, RG = 4 / WR;           // wavefronts across channels, 16-row groups per wavefront
    static_assert(SL % KP == 0 && KS % KP == 0, "a step is whole offsets, or an offset whole steps");
    constexpr int NC = 16 * WC * CT;                   // output channels of the workgroup
    constexpr int W_BYTES = F32 ? SL * 16 * NC * 4 : 0;        // fp32 weights of a step, in LDS behind the rows
    // rows[HV][2][STEP_BYTES] | weights[2][W_BYTES] | list[K3 + PAD], but POINT and REGS | HELD: entries[28 or 32][64], masks[4 HV][4]
    extern __shared__ __align__(16) char smem_all[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wv = HV == 1 ? wave : wave % NW, set = HV == 1 ? 0 : wave / NW;
    char* const smem = smem_all + set * (2 * STEP_BYTES);
    const int r = lane & 15, qq = lane >> 4;
    const int wr = wv / WC;
    const int64_t n_out = FUSED ? n_out_cap : output_rows(n_out_ptr, n_out_cap);
    // a tile's blocks of output channels follow each other on its XCD; from tiles_apart tiles on block after block takes all tiles (not where
    // the lines are held: K <= 3, whose weights are never that large)
    const int64_t tiles = (n_out + TILE - 1) / TILE;
    const bool apart = !F32 && SRC == FROM_MAP && tiles >= tiles_apart;
    const unsigned turn = (blockIdx.y * (unsigned)GRID_COLUMNS + blockIdx.x) / NUM_XCD;
    const unsigned divisor = apart ? xcd_run_grid(tiles) / NUM_XCD : (unsigned)blocks_y;
    const unsigned quotient = turn / divisor, rest = turn - quotient * divisor;
    const int by = (int)(apart ? quotient : rest);
    const unsigned place = (apart ? rest : quotient) * NUM_XCD + blockIdx.x % NUM_XCD;
    const int64_t tile = SRC != FROM_TABLE && !POINT && ms.density != nullptr ? xcd_dense_first(place, tiles, ms.density, K3) : xcd_run_of(place, tiles);
    if (tile < 0 || by >= blocks_y) return;            // the whole workgroup
    const int cb0 = by * (WC * CT) + (wv % WC) * CT;

    // The offsets the tile takes part in, in increasing order, as a list in LDS: number and 4-bit pattern of groups, zeros past
    // the last.  Every wavefront makes it for itself (lane = offset), all with the same contents.
    // A pointwise layer has one entry, `only`, and no list: making one of one entry in LDS and reading it there was a round trip
    // before the first gather and one before the second (us of map and convolution, before there was a list / with it / now: fp32 32 -> 64 200 k rows 32.8 / 34.2 /
    // 26.7, 300 k 46.6 / 48.5 / 37.5, 64 -> 128 90 k 34.0 / 34.9 / 30.3, 128 -> 128 200 k 96.1 / 91.6 / 86.1; 16 bit 32 -> 32 200 k 18.2 / 11.6 / 9.6, 256 -> 256 90 k
    // 38.7 / 35.1 / 32.8).
    // REGS: it is made in the half of the rows' buffer that is filled second and then lies in the lanes of PLACES registers: behind both buffers it takes
    // the 16-channel workgroups of fp32, whose buffers are a quarter of the LDS, from four per CU to three (fewer_rounds_of_four).
    constexpr int WAVES = NW * HV, LINES = (27 + WAVES - 1) / WAVES;       // HELD: lines of the map a wavefront copies or looks up
    constexpr int PLACES = REGS ? 6 : 1;               // 64 offsets each: K^3 <= 343 and what is read past them
    uint32_t places[PLACES] = {};
    uint32_t* list = reinterpret_cast<uint32_t*>(smem_all + (REGS ? STEP_BYTES + 128 : HV * 2 * STEP_BYTES + 2 * W_BYTES));
    int32_t* found = reinterpret_cast<int32_t*>(list + (28 + PAD));
    uint32_t only = 0u;
    int listed = 0;
    auto add_to_list = [&](int k, uint32_t pat) __attribute__((always_inline)) {
        const uint64_t in = __ballot(pat != 0u);
        if (pat != 0u) list[listed + __popcll(in & ((1ull << lane) - 1ull))] = (uint32_t)k << 4 | pat;
        listed += __popcll(in);
    };
    if constexpr (POINT) {
#pragma unroll
        for (int g = 0; g < 4; ++g) only |= (gmask[tile * 4 + g] & 1u) << g;       // submanifold: the map has masks
        only = __builtin_amdgcn_readfirstlane(only);
    } else if constexpr (FUSED) {
        // lane = row; each wavefront looks up every fourth offset (two sets: every eighth), its part of the masks is a vote
        uint32_t* votes = reinterpret_cast<uint32_t*>(found + LINES * WAVES * TILE);
        int32_t part[LINES];
        grid_neighbours_part<3, WAVES>(ms, tile * TILE + lane, n_out, wave, part);
        uint32_t vg[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int u = 0; u < LINES; ++u) {
            found[(wave + WAVES * u) * TILE + lane] = part[u];
            const uint64_t vote = __ballot(part[u] >= 0);
#pragma unroll
            for (int g = 0; g < 4; ++g) vg[g] |= (((vote >> (16 * g)) & 0xffffull) != 0ull ? 1u : 0u) << (wave + WAVES * u);
        }
        if (lane == 0) *reinterpret_cast<uint4*>(votes + 4 * wave) = make_uint4(vg[0], vg[1], vg[2], vg[3]);
        __syncthreads();
        uint32_t pat = 0u;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            uint32_t any = 0u;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) any |= votes[4 * w + g];
            pat |= ((any >> (lane & 31)) & 1u) << g;
        }
        add_to_list(lane, lane < 27 ? pat : 0u);
    } else {
        int32_t part[LINES];
        if constexpr (HELD) {
#pragma unroll
            for (int u = 0; u < LINES; ++u) part[u] = wave + WAVES * u < K3 ? nbr[(tile * K3 + wave + WAVES * u) * TILE + lane] : -1;
        }
        auto hold = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < LINES; ++u) found[(wave + WAVES * u) * TILE + lane] = part[u];
        };
        if (gmask != nullptr) {
            for (int k = lane; k - lane < K3; k += WAVE) {
                uint32_t pat = 0u;
                if (k < K3) {
#pragma unroll
                    for (int g = 0; g < 4; ++g) pat |= ((gmask[tile * (4 * mw) + g * mw + (k >> 5)] >> (k & 31)) & 1u) << g;
                }
                add_to_list(k, pat);
            }
            if constexpr (HELD) {
                hold();
                __syncthreads();
            }
        } else {
            // a map without masks (K^3 <= 32): its lines are voted on, every NWth by a wavefront, and the patterns traded through
            // LDS, in the half of the rows' buffer that is filled second
            uint32_t* patterns = reinterpret_cast<uint32_t*>(smem_all + STEP_BYTES);
            if constexpr (HELD) hold();
#pragma unroll
            for (int u = 0; u < 32 / WAVES; ++u) {
                const int k = wave + WAVES * u;
                if (k < K3) {
                    const uint32_t pat = line_pattern(HELD && u < LINES ? part[u] : nbr[(tile * K3 + k) * TILE + lane]);
                    if (lane == 0) patterns[k] = pat;
                }
            }
            __syncthreads();
            add_to_list(lane, lane < K3 ? patterns[lane] : 0u);
        }
    }
    if constexpr (REGS) {
#pragma unroll
        for (int j = 0; j < PLACES; ++j)
            if (j * WAVE < listed) places[j] = j * WAVE + lane < listed ? list[j * WAVE + lane] : 0u;
    } else if (!POINT && lane < PAD) {
        list[listed + lane] = 0u;
    }
    const uint32_t* next = list + set * OPS;
    uint32_t fetched[OPS];                             // the list's entries of the next step, read a step before they are needed
    int part = 0, at = 0;
    auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int o = 0; o < OPS; ++o) fetched[o] = next[o];
    };
    if constexpr (!POINT && !REGS) fetch();
    // numbers (times PARTS, plus the part; -1: none) and patterns of the next step's offsets
    auto next_step = [&](int (&k)[OPS], uint32_t (&p)[OPS]) __attribute__((always_inline)) {
#pragma unroll
        for (int o = 0; o < OPS; ++o) {
            const uint32_t e = POINT  ? (o == 0 && part < PARTS ? only : 0u)
                               : REGS ? __builtin_amdgcn_readlane(places[0], at + o)
                                      : __builtin_amdgcn_readfirstlane(fetched[o]);
            p[o] = e & 15u;
            k[o] = e != 0u ? (int)(e >> 4) * PARTS + part : -1;
        }
        if constexpr (POINT) {
            ++part;
        } else {
            if (PARTS == 1 || ++part == PARTS) {
                part = 0;
                next += HV * OPS;
                if (REGS && (at += OPS) == WAVE) {
                    at = 0;
#pragma unroll
                    for (int j = 0; j < PLACES; ++j) places[j] = j + 1 < PLACES ? places[j + 1] : 0u;
                }
            }
            if constexpr (!REGS) fetch();
        }
    };

    // gathers: this wavefront fetches group gw (of eight wavefronts, two share a group: each takes every other
    // offset, or half of the rows); its lane's row inside the group and 16-byte piece
    const int gw = NW == 4 ? wv : KS == 1 ? wv & 3 : wv >> 1, half = NW == 4 ? 0 : KS == 1 ? wv >> 2 : wv & 1;
    int grow[NI], gpiece;
    if constexpr (KS == 1) {
        const int logical = (lane & 7) ^ (lane >> 3);  // line = two 64-byte rows, slots XOR-ed with the line number
        grow[0] = (lane >> 3) * 2 + (logical >> 2);
        gpiece = logical & 3;
    } else {
#pragma unroll
        for (int i = 0; i < NI; ++i) grow[i] = (NW == 8 ? half : i) * 8 + (lane >> 3);
        gpiece = (lane & 7) ^ (lane >> 3);
    }
    const int32_t* line = HELD ? nullptr : nbr + tile * (int64_t)K3 * TILE + gw * 16;
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const char* fbase = reinterpret_cast<const char*>(feat) + gpiece * 16;
    const char* zbase = reinterpret_cast<const char*>(g_zero_row) + gpiece * 16;

    int k1[OPS], k2[OPS];                              // offsets of the next step and the one after
    uint32_t p0[OPS], p1[OPS], p2[OPS];
    int32_t ev[OPS][NI];                               // table entries of the next step's gathers
    auto entries = [&](const int (&k)[OPS]) {
#pragma unroll
        for (int o = 0; o < OPS; ++o)
#pragma unroll
            for (int i = 0; i < NI; ++i)
                if (!SKIP || k[o] >= 0) {
                    const int32_t* at = (HELD ? found + gw * 16 : line) + (k[o] >= 0 ? k[o] / PARTS : 0) * TILE;
                    ev[o][i] = at[(uint32_t)grow[i]];
                }
    };
    auto gather = [&](const int (&k)[OPS], const uint32_t (&p)[OPS], int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int o = 0; o < OPS; ++o) {
            if ((!SKIP || ((p[o] >> gw) & 1u) != 0u) && (NW == 4 || KS > 1 || (o & 1) == half)) {
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const char* src = (SKIP || k[o] >= 0) && ev[o][i] >= 0 ? fbase + (int64_t)ev[o][i] * (KS * 64) + k[o] % PARTS * (KP * 64) : zbase;
#pragma unroll
                    for (int c = 0; c < CH; ++c)
                        load_to_lds(src + c * 128, __builtin_amdgcn_readfirstlane(lds_base + buf * STEP_BYTES + (o * CH + c) * CHB +
                                                                                  gw * (CHB / 4) + (NW == 8 && KS > 1 ? half : i) * 1024));
                }
            }
        }
    };
    // 16-bit weights: operand tiles, straight into the registers of the next step
    auto weights = [&](u32x4 (&a)[SL][CT], const int (&k)[OPS]) {
#pragma unroll
        for (int o = 0; o < OPS; ++o)
            if (!SKIP || k[o] >= 0) {
                const char* w = reinterpret_cast<const char*>(wp) + (uint32_t)(k[o] >= 0 ? k[o] : 0) * (uint32_t)(CB * KP * 1024);
#pragma unroll
                for (int ks = 0; ks < KP; ++ks)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        const int cb = cb0 + ct < CB ? cb0 + ct : CB - 1;      // past the last block: not stored
                        a[o * KP + ks][ct] = *reinterpret_cast<const u32x4*>(w + (KS == 1 ? cb : ((ks >> 1) * CB + cb) * 2 + (ks & 1)) * 1024 + (uint32_t)lane * 16u);
                    }
            }
    };
    // fp32 weights: rows of W[k] as they lie in memory, into LDS.  Of a slice's 16 input channels
    // 4 q + j (q the operand's lane quarter, j the multiply) goes to row 4 j + q, and its 16-channel blocks are
    // XOR-ed with q as far as the row is long, so that the four quarters of an operand read use different banks.
    auto swizzle = [&](int q) -> int { return NC == 16 ? 0 : NC == 32 ? q >> 1 : q; };
    auto weights_lds = [&](const int (&k)[OPS], int buf) __attribute__((always_inline)) {
        constexpr int PS = WC * CT;                    // instructions per slice
        const int prow = lane / (NC / 4), piece = lane % (NC / 4);
#pragma unroll
        for (int i = 0; i < (SL * PS + NW - 1) / NW; ++i) {
            const int t = i * NW + wv, sl = t / PS, row = t % PS * (16 / PS) + prow;
            const int q = row & 3, j = row >> 2;
            int kk = k[0];                             // of offset sl / KP: a chain of selects, the array stays in registers
#pragma unroll
            for (int o = 1; o < OPS; ++o) kk = sl >= o * KP ? k[o] : kk;
            if (t < SL * PS && kk >= 0) {
                int col = by * NC + ((piece ^ (swizzle(q) << 2)) << 2);
                if (col > CB * 16 - 4) col = CB * 16 - 4;      // past the last block: not stored
                const float* src = reinterpret_cast<const float*>(wp) + ((int64_t)kk * (KP * 16) + sl % KP * 16 + 4 * q + j) * (CB * 16) + col;
                load_to_lds(src, __builtin_amdgcn_readfirstlane(lds_base + 2 * STEP_BYTES + buf * W_BYTES + t * 1024));
            }
        }
    };
    f32x4 acc[RG][CT];
#pragma unroll
    for (int g = 0; g < RG; ++g)
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[g][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    // byte of operand piece (row r of a group, 16-byte piece 4 j + qq) inside the group's part of a chunk
    auto operand = [&](int j) -> int {
        return KS == 1 ? (r >> 1) * 128 + (((((r & 1) << 2) + qq) ^ (r >> 1)) << 4) : r * 128 + (((j * 4 + qq) ^ (r & 7)) << 4);
    };
    const int op0 = operand(0), op1 = operand(1);
    auto compute = [&](const u32x4 (&a)[SL][CT], const uint32_t (&p)[OPS], int buf) {
        if constexpr (!F32 && (KP == 1 || KP == 8)) {
            // Operands are read a batch of groups ahead of its multiplies, also of a group without a neighbour: its products are
            // left out.  Batches are all groups of an offset (32 channels) or one (256).  (us of whole layers, before -> now: 256 -> 256 500 / 2 k /
            // 5 k / 14 k voxels 25.9 / 33.6 / 37.8 / 62.3 -> 24.0 / 30.9 / 34.2 / 59.6; K = 5 32 -> 32 the same.  64 and 128
            // channels, whose batches are short next to the latency, lose the registers: convolution of 110 k 64 -> 64 30.5 -> 32.3.)
            constexpr int GB = KP == 1 ? RG : 1, NB = RG / GB, BATCHES = OPS * NB;
            uint4 b[2][GB][KP];
            auto read = [&](uint4 (&b)[GB][KP], int i) __attribute__((always_inline)) {
#pragma unroll
                for (int g = 0; g < GB; ++g) {
                    const char* rows = smem + buf * STEP_BYTES + i / NB * CH * CHB + (wr * RG + i % NB * GB + g) * (CHB / 4);
#pragma unroll
                    for (int ks = 0; ks < KP; ++ks) b[g][ks] = *reinterpret_cast<const uint4*>(rows + (ks >> 1) * CHB + ((ks & 1) ? op1 : op0));
                }
            };
            read(b[0], 0);
#pragma unroll
            for (int i = 0; i < BATCHES; ++i) {
                if (i + 1 < BATCHES) read(b[(i + 1) & 1], i + 1);
                __builtin_amdgcn_sched_barrier(0);     // read here, not under the tests
#pragma unroll
                for (int gb = 0; gb < GB; ++gb) {
                    const int o = i / NB, g = i % NB * GB + gb;
                    if (((p[o] >> (wr * RG + g)) & 1u) == 0u) continue;
#pragma unroll
                    for (int ks = 0; ks < KP; ++ks)
#pragma unroll
                        for (int ct = 0; ct < CT; ++ct)
                            acc[g][ct] = mfma16x16x32<DT>(__builtin_bit_cast(uint4, a[o * KP + ks][ct]), b[i & 1][gb][ks], acc[g][ct]);
                }
            }
            return;
        }
#pragma unroll
        for (int o = 0; o < OPS; ++o) {
            if (p[o] == 0u) continue;
            f32x4 af[F32 ? KP : 1][CT];
            if constexpr (F32) {
#pragma unroll
                for (int ks = 0; ks < KP; ++ks)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        const int block = ((wv % WC) * CT + ct) ^ swizzle(qq);
                        const float* w = reinterpret_cast<const float*>(smem + 2 * STEP_BYTES + buf * W_BYTES) + (o * KP + ks) * (16 * NC) +
                                         qq * NC + block * 16 + r;
#pragma unroll
                        for (int j = 0; j < 4; ++j) af[ks][ct][j] = w[j * (4 * NC)];
                    }
            }
            uint4 b[RG][KP];
            auto operands = [&](int g) __attribute__((always_inline)) {
                const char* rows = smem + buf * STEP_BYTES + o * CH * CHB + (wr * RG + g) * (CHB / 4);
#pragma unroll
                for (int ks = 0; ks < KP; ++ks) b[g][ks] = *reinterpret_cast<const uint4*>(rows + (ks >> 1) * CHB + ((ks & 1) ? op1 : op0));
            };
            // two short groups (64 input channels) are read together, also one without a neighbour: its products are left
            // out (4 k voxels 64 -> 64 11.3 -> 10.3 us; all four: 10.2, but 110 k 30.9 -> 31.5 and 10^6 324 -> 332)
            constexpr int GB = KP == 2 && RG > 1 && CT == 1 ? 2 : 1;
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                if (GB > 1 && g % GB == 0) {
#pragma unroll
                    for (int i = g; i < g + GB; ++i) operands(i);
                    __builtin_amdgcn_sched_barrier(0);         // read here, not under the tests below
                }
                if (((p[o] >> (wr * RG + g)) & 1u) == 0u) continue;
                if (GB == 1) operands(g);
#pragma unroll
                for (int ks = 0; ks < KP; ++ks) {
                    if constexpr (F32) {
                        // component j of both operands: input channel 16 ks + 4 qq + j at position qq of multiply j
                        const f32x4 fb = __builtin_bit_cast(f32x4, b[g][ks]);
#pragma unroll
                        for (int j = 0; j < 4; ++j)
#pragma unroll
                            for (int ct = 0; ct < CT; ++ct)
                                acc[g][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(af[ks][ct][j], fb[j], acc[g][ct], 0, 0, 0);
                    } else {
#pragma unroll
                        for (int ct = 0; ct < CT; ++ct)
                            acc[g][ct] = mfma16x16x32<DT>(__builtin_bit_cast(uint4, a[o * KP + ks][ct]), b[g][ks], acc[g][ct]);
                    }
                }
            }
        }
    };
    // everything requested has arrived (said in a form the compiler's own wait-count pass sees), and so it has for all four wavefronts
    auto step_end = [&]() {
        __builtin_amdgcn_s_waitcnt(0x0070);            // vmcnt(0) lgkmcnt(0)
        asm volatile("s_barrier" ::: "memory");
    };

    u32x4 a0[SL][CT], a1[SL][CT];
    next_step(k1, p1);
    entries(k1);
    next_step(k2, p2);
    gather(k1, p1, 0);
    if constexpr (F32) weights_lds(k1, 0);
    else weights(a0, k1);
    entries(k2);
    step_end();
    // one step: request the next one's rows and weights and the entries of the one after, multiply
    auto step = [&](const u32x4 (&a)[SL][CT], u32x4 (&a_next)[SL][CT], int buf) {
#pragma unroll
        for (int o = 0; o < OPS; ++o) {
            p0[o] = p1[o];
            k1[o] = k2[o];
            p1[o] = p2[o];
        }
        next_step(k2, p2);
        gather(k1, p1, buf ^ 1);
        if constexpr (F32) weights_lds(k1, buf ^ 1);
        else weights(a_next, k1);
        entries(k2);
        __builtin_amdgcn_sched_barrier(0);             // requested here, not next to their use
        compute(a, p0, buf);
        step_end();
    };
    if constexpr (HV == 1) {
#pragma unroll 1
        while (p1[0] != 0u) {
            step(a0, a1, 0);
            if (p1[0] == 0u) break;
            step(a1, a0, 1);
        }
    } else {
        // as many steps for both sets; then each gives the other its sums of two groups and stores the other two
#pragma unroll 1
        for (int left = (listed + HV * OPS - 1) / (HV * OPS) * PARTS; left > 0; --left) {
            step(a0, a1, 0);
            if (--left <= 0) break;
            step(a1, a0, 1);
        }
        constexpr int G = RG / 2;
        f32x4* sums = reinterpret_cast<f32x4*>(smem_all) + (size_t)wave * (G * CT * 64) + lane;
        const f32x4* theirs = reinterpret_cast<const f32x4*>(smem_all) + (size_t)(wave ^ NW) * (G * CT * 64) + lane;
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) sums[(g * CT + ct) * 64] = set == 0 ? acc[G + g][ct] : acc[g][ct];
        lds_barrier();
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                const f32x4 other = theirs[(g * CT + ct) * 64];
                acc[g][ct] = set == 0 ? acc[g][ct] + other : other + acc[G + g][ct];
            }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const int64_t row = tile * TILE + (wr * RG + set * G + g) * 16 + r;
            if (row < n_out) {
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    if (cb0 + ct < CB) store_acc<DT>(out, out_f32, row, CB * 16, (cb0 + ct) * 16 + qq * 4, acc[g][ct]);
            }
        }
        return;
    }
#pragma unroll
    for (int g = 0; g < RG; ++g) {
        const int64_t row = tile * TILE + (wr * RG + g) * 16 + r;
        if (row < n_out) {
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                if (cb0 + ct < CB) store_acc<DT>(out, out_f32, row, CB * 16, (cb0 + ct) * 16 + qq * 4, acc[g][ct]);
        }
    }
}

template <int DT, int KS, int SL, int SKIP, int NW, int WR, int CT, int OCC, int SRC, int HV = 1>
static int launch_gather_as(int K3, int mw, int CB, int64_t tiles, int cus, hipStream_t s, const void* feat, const void* wp, void* out,
                            int out_f32, const MapSource& ms, const int64_t* n_out_ptr, int64_t n_out_cap) {
    constexpr bool held = SRC == FROM_TABLE || SRC == FROM_LINES;
    constexpr size_t entries = held ? (HV == 1 ? 28 : 32) * TILE * 4 + 64 * HV : 0;
    constexpr size_t fixed = HV * 2 * SL * 4096 + (DT == SC_F32 ? 2 * SL * 1024 * (NW / WR * CT) : 0) + entries;
    static_assert(fixed <= 65536 + entries, "loads into LDS land in the first 64 KB");
    constexpr auto list_bytes = [](int K3) { return SRC == FROM_LINE || SRC == FROM_MAP_BY_REGISTERS ? (size_t)0 : (size_t)((held ? 28 : K3) + LIST_PAD * HV + 3) / 4 * 16; };     // entries lie behind a list of 28
    const size_t lds = fixed + list_bytes(K3);
    if constexpr (fixed + list_bytes(343) > 65536) {
        static bool allowed[MAX_DEVICES] = {};
        if (int rc = allow_lds((const void*)k_conv_gather<DT, KS, NW, WR, CT, SL, SKIP, OCC, SRC, HV>, fixed + list_bytes(343), allowed)) return rc;
    }
    const unsigned blocks_y = (unsigned)((CB + NW / WR * CT - 1) / (NW / WR * CT));
    static_assert(grid_fits(GRID_COLUMNS, 64 * NW * HV) && GRID_COLUMNS % NUM_XCD == 0, "a row of the grid is whole turns of the XCDs");
    const int64_t groups = (int64_t)xcd_run_grid(tiles) * blocks_y;
    MapSource source = ms;
    if (!dense_tiles_first(tiles, tiles * blocks_y, 3 * fixed > 160 * 1024, cus)) source.density = nullptr;
    SC_LAUNCH(DT == SC_F32 ? KID_CONV_F32 : KID_CONV_MFMA, (k_conv_gather<DT, KS, NW, WR, CT, SL, SKIP, OCC, SRC, HV>),
              dim3((unsigned)grid_columns(groups), (unsigned)grid_rows(groups)), dim3(64 * NW * HV), lds, s, feat, wp, out, out_f32, source, K3, mw, CB,
              (int)blocks_y, first_tiles_apart((int64_t)K3 * CB * KS * 1024, CT, n_out_ptr != nullptr, cus), n_out_ptr, n_out_cap);
    return SC_OK;
}

// O1, O2: wavefronts per SIMD with one and with two output blocks per wavefront
template <int DT, int KS, int SL, int SKIP, int O1, int O2, int SRC = FROM_MAP>
static int launch_gather_ks(int K3, int mw, int CB, int64_t tiles, int64_t likely, LayerKind kind, int cus, hipStream_t s, const void* feat, const void* wp,
                            void* out, int out_f32, const MapSource& ms, const int64_t* n_out_ptr, int64_t n_out_cap) {
#define SC_GATHER(NW, WR, CT, OCC) \
    return launch_gather_as<DT, KS, SL, SKIP, NW, WR, CT, OCC, SRC>(K3, mw, CB, tiles, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap)
    if constexpr (DT == SC_F32) {
        // 32 output channels per workgroup: gathering a tile's rows once more costs less than a workgroup of 64 channels
        // that others wait for (a tile near the sensor is 27 offsets x 2,048 cycles of multiplies per SIMD; us with
        // 64 and with 32: 64 -> 64 at 4 k / 53 k / 80 k voxels 28.8 / 82 / 105 and 20.3 / 72 / 99.5, 128 -> 128 at 4 k / 53 k
        // 56 / 245 and 39 / 235).  16 where the CUs' last round is shorter then, up to four rounds of 32 (64 -> 64 at 4 k /
        // 8 k / 12 k 18.0 / 25.5 / 27.6 us against 20.3 / 23.6 / 34.3 with 32).
        const int64_t w = likely * CB;
        const bool narrow = w <= 8 * (int64_t)cus && (w + cus - 1) / cus < 2 * ((w + 2 * cus - 1) / (2 * cus));
        if constexpr (SRC == FROM_MAP) {
            if (CB == 1 && K3 >= 64 && fewer_rounds_of_four(w, cus))
                return launch_gather_as<DT, KS, SL, SKIP, 4, 4, 1, 3, FROM_MAP_BY_REGISTERS>(K3, mw, CB, tiles, cus, s, feat, wp, out, out_f32, ms,
                                                                                             n_out_ptr, n_out_cap);
        }
        if (CB == 1 || narrow) SC_GATHER(4, 4, 1, 3);
        SC_GATHER(8, 4, 1, 4);
    } else {
        if constexpr (SRC != FROM_TABLE) {
            if (CB == 1) SC_GATHER(4, 4, 1, O1);
            if constexpr (KS > 1 || SRC != FROM_LINES)        // K = 2 and 3, 32 -> 32 are the resident kernel's
                if (CB == 2) SC_GATHER(4, 2, 1, O1);
        }
        // two output blocks per wavefront halve how often a tile's rows are gathered; one, where that leaves CUs
        // idle or, up to 128 channels either way, with few wavefronts (us with one and with two blocks: 256 -> 128 at
        // 219 tiles 29.0, 34.2; 256 -> 256 49.1, 44.1; 64 -> 256 at 157 tiles 17.6, 19.3, at 250 22.9, 20.9; 128 -> 128 at
        // 625 tiles 36.0, 38.2, at 4,088 132, 127.5; 64 -> 128 at 469 tiles 20.2, 21.4, at 834 26.9, 26.7; 256 input channels: one_block_of_256)
        const int64_t pairs = likely * ((CB + 7) / 8);
        if (CB <= 4 || (CB <= 8 && KS <= 4 ? likely <= 4 * (int64_t)cus
                        : KS == 8          ? one_block_of_256(pairs, K3, kind, cus)
                                           : 2 * pairs < 3 * (int64_t)cus))
            SC_GATHER(4, 1, 1, O1);
        SC_GATHER(4, 1, 2, O2);
    }
#undef SC_GATHER
}

// Two sets of wavefronts (two_sets), one output block per wavefront.
template <int DT, int KS, int SL, int SKIP, int O1, int SRC>
static int launch_gather_sets(int K3, int mw, int CB, int64_t tiles, int cus, hipStream_t s, const void* feat, const void* wp, void* out, int out_f32,
                              const MapSource& ms, const int64_t* n_out_ptr, int64_t n_out_cap) {
    if constexpr (SRC == FROM_MAP || (SRC == FROM_LINES && KS > 1)) {
        if (CB == 2) return launch_gather_as<DT, KS, SL, SKIP, 4, 2, 1, O1, SRC, 2>(K3, mw, CB, tiles, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap);
    }
    return launch_gather_as<DT, KS, SL, SKIP, 4, 1, 1, O1, SRC, 2>(K3, mw, CB, tiles, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap);
}

int launch_gather(int dtype_in, int K3, int mw, int C_in, int C_out, int64_t tiles, int64_t likely, LayerKind kind, bool sets, int cus, hipStream_t s, const void* feat,
                  const void* wp, void* out, int out_f32, const MapSource& ms, const int64_t* n_out_ptr, int64_t n_out_cap) {
    const int CB = C_out / 16;
    // Slices per step, skipping, wavefronts per SIMD.  256 channels: a whole offset.  128: an offset (half of one,
    // with more workgroups: 128 -> 64 at 53 k voxels 36.7 us instead of 28.8).  64: an offset; two for K = 5 and 7, whose
    // tiles walk many more offsets (K = 3 -> 64 at 262 k voxels 50.3 us with one, 56.5 with two; K = 5 -> 64 at 53 k 55.1
    // and 50.7).  32: four (K = 5 -> 32 at 53 k: 30.4 us; two 32.1, eight with half the workgroups 36).
#define SC_GATHER_SETS(KS, SL, SKIP, O1, SRC)                                                                                                      \
    return dtype_in == SC_F16                                                                                                     \
               ? launch_gather_sets<SC_F16, KS, SL, SKIP, O1, SRC>(K3, mw, CB, tiles, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap)    \
               : launch_gather_sets<SC_BF16, KS, SL, SKIP, O1, SRC>(K3, mw, CB, tiles, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap)
#define SC_GATHER_KS(KS, SL, SKIP, O1, O2, SRC)                                                                                      \
    return dtype_in == SC_F16                                                                                                     \
               ? launch_gather_ks<SC_F16, KS, SL, SKIP, O1, O2, SRC>(K3, mw, CB, tiles, likely, kind, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap)    \
               : launch_gather_ks<SC_BF16, KS, SL, SKIP, O1, O2, SRC>(K3, mw, CB, tiles, likely, kind, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap)
    if (dtype_in == SC_F32) {
#define SC_GATHER_F32(KS)                                                                                                              \
    return K3 == 1 ? launch_gather_ks<SC_F32, KS, 4, 1, 4, 4, FROM_LINE>(K3, mw, CB, tiles, likely, kind, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap) \
                   : launch_gather_ks<SC_F32, KS, 4, 1, 4, 4>(K3, mw, CB, tiles, likely, kind, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap)
        switch (C_in) {
            case 16: SC_GATHER_F32(1);
            case 32: SC_GATHER_F32(2);
            case 64: SC_GATHER_F32(4);
            case 128: SC_GATHER_F32(8);
            case 256: SC_GATHER_F32(16);
        }
#undef SC_GATHER_F32
        return SC_EINVAL;
    }
    // K = 1: one offset, so the shortest steps, and the one line is read as it is needed
    if (K3 == 1) {
        switch (C_in) {
            case 32: SC_GATHER_KS(1, 2, 1, 5, 4, FROM_LINE);
            case 64: SC_GATHER_KS(2, 2, 1, 6, 5, FROM_LINE);
            case 128: SC_GATHER_KS(4, 4, 1, 4, 3, FROM_LINE);
            case 256: SC_GATHER_KS(8, 8, 1, 2, 2, FROM_LINE);
        }
        return SC_EINVAL;
    }
    const bool few = few_workgroups(likely, CB, cus);
    if (sets) {
        if (K3 <= 27) {
            switch (C_in) {
                case 32: SC_GATHER_SETS(1, 2, 1, 4, FROM_LINES);
                case 64: SC_GATHER_SETS(2, 2, 1, 6, FROM_LINES);
                case 128: SC_GATHER_SETS(4, 4, 1, 4, FROM_LINES);
            }
        }
        switch (C_in) {
            case 32: SC_GATHER_SETS(1, 4, 0, 2, FROM_MAP);
            case 64: SC_GATHER_SETS(2, 4, 1, 4, FROM_MAP);
            case 128: SC_GATHER_SETS(4, 4, 1, 4, FROM_MAP);
        }
    }
    if (K3 <= 27) {
        switch (C_in) {
            case 32:
                if (few) SC_GATHER_KS(1, 4, 0, 2, 2, FROM_LINES);
                SC_GATHER_KS(1, 2, 1, 5, 4, FROM_LINES);
            case 64:
                if (few) SC_GATHER_KS(2, 4, 1, 4, 4, FROM_LINES);
                SC_GATHER_KS(2, 2, 1, 6, 5, FROM_LINES);
            case 128: SC_GATHER_KS(4, 4, 1, 4, 3, FROM_LINES);
            case 256: SC_GATHER_KS(8, 8, 1, 2, 2, FROM_LINES);
        }
    }
    switch (C_in) {
        case 32: SC_GATHER_KS(1, 4, 0, 2, 2, FROM_MAP);
        case 64: SC_GATHER_KS(2, 4, 1, 5, 4, FROM_MAP);
        case 128: SC_GATHER_KS(4, 4, 1, 4, 3, FROM_MAP);
        case 256: SC_GATHER_KS(8, 8, 1, 2, 2, FROM_MAP);
    }
#undef SC_GATHER_KS
#undef SC_GATHER_SETS
    return SC_EINVAL;
}

// 3x3x3 layers that look their neighbours up in the dense table themselves: 32, 64 and 128 channels, at least 64 out.
int launch_gather_fused(int dtype_in, int C_in, int C_out, int64_t tiles, bool sets, int cus, hipStream_t s, const void* feat, const void* wp,
                        void* out, int out_f32, const MapSource& ms, int64_t n) {
    const int CB = C_out / 16;
    if (CB < 4) return SC_EINVAL;
#define SC_GATHER_FUSED(KS, SL, SKIP, O1, O2)                                                                                                    \
    return dtype_in == SC_F16                                                                                                                \
               ? launch_gather_ks<SC_F16, KS, SL, SKIP, O1, O2, FROM_TABLE>(27, 1, CB, tiles, tiles, SUBMANIFOLD, cus, s, feat, wp, out, out_f32, ms, nullptr, n)    \
               : launch_gather_ks<SC_BF16, KS, SL, SKIP, O1, O2, FROM_TABLE>(27, 1, CB, tiles, tiles, SUBMANIFOLD, cus, s, feat, wp, out, out_f32, ms, nullptr, n)
#define SC_GATHER_FUSED_SETS(KS, SL, SKIP, O1)                                                                                                    \
    return dtype_in == SC_F16 ? launch_gather_sets<SC_F16, KS, SL, SKIP, O1, FROM_TABLE>(27, 1, CB, tiles, cus, s, feat, wp, out, out_f32, ms, nullptr, n)    \
                              : launch_gather_sets<SC_BF16, KS, SL, SKIP, O1, FROM_TABLE>(27, 1, CB, tiles, cus, s, feat, wp, out, out_f32, ms, nullptr, n)
    if (sets) {
        if (C_in == 32) SC_GATHER_FUSED_SETS(1, 2, 1, 4);
        if (C_in == 64) SC_GATHER_FUSED_SETS(2, 2, 1, 6);
        if (C_in == 128) SC_GATHER_FUSED_SETS(4, 4, 1, 4);
    }
#undef SC_GATHER_FUSED_SETS
    const bool few = few_workgroups(tiles, CB, cus);
    if (C_in == 32 && few) SC_GATHER_FUSED(1, 4, 0, 2, 2);
    if (C_in == 32) SC_GATHER_FUSED(1, 2, 1, 5, 4);
    if (C_in == 64 && few) SC_GATHER_FUSED(2, 4, 1, 4, 4);
    if (C_in == 64) SC_GATHER_FUSED(2, 2, 1, 6, 5);
    if (C_in == 128) SC_GATHER_FUSED(4, 4, 1, 4, 3);
#undef SC_GATHER_FUSED
    return SC_EINVAL;
}

}  // namespace sc
