// Compute step: out[o] = sum_k sum_{(i,o) in M_k} in[i] . W[k]   (paper Algorithm 2).
//
// The paper's kernel gives one thread one (output row, output channel) and walks K^3 x C_in
// scalar FMAs with one output channel's weights cached in shared memory, so every gathered
// feature row is re-read C_out times.  Here a wavefront owns 16 consecutive output rows (a
// quarter of a kernel-map tile).  For every offset k at which that group has a neighbour (one
// bit test) it gathers the 16 input rows straight into MFMA operand registers, 16 bytes per
// lane, zero where a row has no neighbour, and multiplies them by W[k] on the matrix cores
// (v_mfma_f32_16x16x32, fp32 accumulation).  Because an output row keeps its place in the group
// for every offset, the accumulators stay in registers for the whole layer: no atomics, no
// scatter, one conversion and one store per output row.  Groups without a neighbour at k are
// skipped; on surface-like voxel sets this issues about 1.8x the MACs that exist.
// A layer of ~10^5 voxels is a few microseconds of matrix work, so what decides its time is how
// many loads are in flight: the kernels below issue the offset-table reads of all K^3 offsets,
// then all feature gathers, before the first multiply.
#include "sc_conv.h"
#include "sc_rules.h"

namespace sc {

__global__ void __launch_bounds__(256)
k_weight_pack(const uint16_t* __restrict__ w, uint4* __restrict__ wp, int K3, int C_in, int C_out) {
    const int KS = C_in / 32, CB = C_out / 16;
    const int64_t total = (int64_t)K3 * CB * KS * 64;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total) return;
    const int lane = (int)(t & 63);
    int64_t rest = t >> 6;
    const int ks = (int)(rest % KS); rest /= KS;
    const int cb = (int)(rest % CB);
    const int k = (int)(rest / CB);
    const int co = cb * 16 + (lane & 15);
    const int ci0 = ks * 32 + 8 * (lane >> 4);
    const uint16_t* src = w + ((int64_t)k * C_in + ci0) * C_out + co;
    uint32_t v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        v[j] = (uint32_t)src[(int64_t)(2 * j) * C_out] | ((uint32_t)src[(int64_t)(2 * j + 1) * C_out] << 16);
    wp[((int64_t)k * CB * KS + wtile(KS, CB, cb, ks)) * 64 + lane] = make_uint4(v[0], v[1], v[2], v[3]);
}

// ---- small layers: all of W resident in LDS ----------------------------------------------------
// One wavefront per 16 output rows, up to NT tiles (4*NT wavefronts) per workgroup at a time.  The workgroup
// copies the weights of all K3 offsets into LDS once, raw ones re-laid out as MFMA operand tiles on
// the way, so no separate packing pass is needed; meanwhile every wavefront has its K3 offset-table lines and then all its feature
// gathers in flight.  KS = C_in/32, CB = C_out/16.
// Packed weights go straight to LDS, requested before the lines and waited for with them.  Through registers they were a loop of round
// trips between the lines and the gathers (us of whole layers on sweeps 2 k / 10 k / 30 k / 53 k, before and now: 13.2 / 14.4 / 18.4 / 23.3 and 12.8 / 14.0 /
// 17.3 / 23.2; two layers and the strided one 10 k / 53 k 40.0 / 51.5 and 37.5 / 50.4).
// Which tiles a workgroup takes is decided here, by the rows there are (of a coarse map they are known on the device only): a round is a workgroup per
// compute unit with at most NT tiles each, and as few as give all of them their share.  A workgroup per two tiles, however many there were, came to
// two for some CUs and one for the others, and to a copy of the weights for every two tiles.  With the loop (resident_loop) the weights are copied once per CU.  us, before and
// now, sweeps: up-sampling by the transposed map 64 -> 32 53 k / 110 k / 260 k 9.2 / 14.9 / 26.4 and 8.5 / 11.6 / 17.6, 64 -> 64 12.2 / 19.8 / 34.7 and 11.4 / 15.4 /
// 24.3; from the strided map 128 -> 64 20 k / 80 k / 110 k / 260 k 9.8 / 19.2 / 20.3 / 36.7 and 9.0 / 14.2 / 17.1 / 24.9, 64 -> 64 8.0 / 12.6 / 13.5 / 22.3 and 6.9 / 11.1 /
// 13.9 / 20.5, 64 -> 32 5.3 / 7.1 / 7.8 / 12.7 and 4.8 / 6.5 / 8.1 / 12.6; layers K = 2, 64 -> 64 20 k / 53 k / 120 k 20.3 / 23.4 / 27.4 and 17.9 / 21.0 / 26.3.
// FUSED: there is no kernel map; the K^3 neighbours of a row are looked up in the dense location
// table right here (one index computation and one 8-byte load each, all in flight together), and
// the group's mask is a vote over what was found.  n_out_cap is then the number of rows.
// UP: the inverse (up-sampling) layer of a K == stride layer, straight from that layer's own map
// (Section III-E: the same pairs with input and output swapped).  The wavefront's 16 rows are
// coarse rows, read in place; entry k of a row's table column names the fine row that receives
// row . W[k].  Every fine row has exactly one parent, so results are stored, not accumulated, and
// nothing needs to be transposed first.
// Round after round in one workgroup, or every workgroup one: the loop pays from 32 KB of weights on (K = 2 32 -> 32, 16 KB, 200 k inputs 27.8 us with it, 26.9
// without), and with 27 gathers in flight its registers are too many (sweep 53 k 37 with it, 23.3 without).
constexpr bool resident_loop(int K3, int KS, int CB, int UP) { return (K3 < 27 || UP) && K3 * KS * CB >= 32; }
template <int DT, int K3, int KS, int CB, int NT, int FUSED, int UP = 0, int WPACKED = 0>
__global__ void __launch_bounds__(256 * NT)
k_conv_rows16(const uint16_t* __restrict__ feat, const uint4* __restrict__ wraw, void* __restrict__ out, int out_f32,
              const MapSource ms, int team, const int64_t* __restrict__ n_out_ptr, int64_t n_out_cap) {
    static_assert(K3 <= 32, "one mask word per group");
    static_assert(!FUSED || K3 == 27, "fused look-ups: 3x3x3 layers");
    static_assert(!(FUSED && UP), "one or the other");
    const uint32_t* __restrict__ gmask = ms.gmask;
    const int32_t* __restrict__ nbr = ms.nbr;
    constexpr int C_in = KS * 32, C_out = CB * 16;
    constexpr bool LOOP = resident_loop(K3, KS, CB, UP);
    extern __shared__ __align__(16) uint4 w_lds[];                   // [K3][CB][KS][64]
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = wv & 3;
    SC_MARK(0);
    const int64_t n_out = FUSED ? n_out_cap : output_rows(n_out_ptr, n_out_cap);
    // an XCD's workgroups share a contiguous eighth of the tiles, so that neighbours meet in its L2
    const int tiles = (int)((n_out + TILE - 1) / TILE), eighth = (tiles + NUM_XCD - 1) / NUM_XCD;
    const int first = (int)(blockIdx.x % NUM_XCD) * eighth, share = tiles - first < eighth ? tiles - first : eighth;
    const int turn = (int)(blockIdx.x / NUM_XCD);
    int done = 0, each = share > 0 ? tiles_per_workgroup(share, team, NT) : 0;
    if (turn * each >= share) return;                  // no tile: the whole workgroup, before any barrier

    // packed weights land in LDS beside everything up to the gathers, which wait for the lines behind them
    static_assert(!WPACKED || (!FUSED && K3 * CB * KS <= 64), "loads into LDS land in its first 64 KB, which the weights have to themselves");
    if constexpr (WPACKED) {
        const uint32_t base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)w_lds;
#pragma unroll
        for (int i = 0; i < (K3 * CB * KS + 4 * NT - 1) / (4 * NT); ++i) {
            const int t = wv + i * 4 * NT;
            if (t < K3 * CB * KS) load_to_lds(wraw + t * 64 + (threadIdx.x & 63), base + t * 1024);
        }
    }
    // raw weights -> LDS as operand tiles (every thread helps, also wavefronts without rows): a thread reads four output
    // channels of 8 input channels (8-byte loads) and writes four lanes' 16 bytes.  With a thread per lane, 2-byte loads, they were
    // four times as many loads of 17 cycles each (us: up-sampling from the strided map 64 -> 32 53 k 6.1 -> 5.4, 64 -> 64 200 k 22.8 ->
    // 20.8, 128 -> 64 53 k 12.8 -> 11.4; layers K = 2 64 -> 64 200 k 40.7 -> 38.6, fused 32 -> 32 53 k 15.1 -> 14.8)
    constexpr int ITEMS = K3 * CB * KS * 16, PASSES = WPACKED ? 1 : (ITEMS + 256 * NT - 1) / (256 * NT);
    auto raw_weights = [&](int pass, uint2 (&v)[8]) __attribute__((always_inline)) {
        const int i = pass * (256 * NT) + threadIdx.x;
        const int col = (i & 3) * 4, oct = (i >> 2) & 3, ks = (i >> 4) % KS, cb = (i >> 4) / KS % CB, k = (i >> 4) / KS / CB;
        const uint16_t* src = reinterpret_cast<const uint16_t*>(wraw) + ((int64_t)k * C_in + ks * 32 + 8 * oct) * C_out + cb * 16 + col;
        if (i < ITEMS) {
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = *reinterpret_cast<const uint2*>(src + j * C_out);
        }
    };
    auto weights_to_lds = [&](int pass, const uint2 (&v)[8]) __attribute__((always_inline)) {
        const int i = pass * (256 * NT) + threadIdx.x;
        if (i >= ITEMS) return;
        const int col = (i & 3) * 4, oct = (i >> 2) & 3;
        uint4* dst = w_lds + (i >> 4) * 64 + oct * 16 + col;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const uint32_t take = (c & 1) ? 0x07060302u : 0x05040100u;     // the upper or the lower halves of two words
            uint32_t o[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                o[j] = c < 2 ? __builtin_amdgcn_perm(v[2 * j + 1].x, v[2 * j].x, take) : __builtin_amdgcn_perm(v[2 * j + 1].y, v[2 * j].y, take);
            dst[c] = make_uint4(o[0], o[1], o[2], o[3]);
        }
    };
    // Look-ups have to be back before anything behind them is asked for, so the weights are asked for before them (us of fused layers, behind and before,
    // sweeps 36 k / 53 k / 110 k / 200 k 13.0 / 15.0 / 25.7 / 45.8 and 12.9 / 14.6 / 25.0 / 44.7, indoor 53 k / 110 k 15.8 / 26.2 and 15.3 / 25.0; 16 k 10.3 and 10.7).
    constexpr bool AHEAD = FUSED && !WPACKED;
    uint2 ahead[AHEAD ? PASSES : 1][8];
    if constexpr (AHEAD) {
#pragma unroll
        for (int i = 0; i < PASSES; ++i) raw_weights(i, ahead[i]);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll 1
    for (;;) {
        // what depends on the lane is made anew for each round: kept over the rounds it costs the registers that the gathers need
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        const int r = lane & 15, qq = lane >> 4;
        const int at = done + turn * each + (wv >> 2);
        const bool mine = (wv >> 2) < each && at < share;
        const int64_t tile = mine ? first + at : 0;
        const int64_t row = tile * TILE + q * 16 + r;
        const bool group_ok = mine && tile * TILE + q * 16 < n_out;     // uniform per wavefront

        // the group's offset-table lines (all K3 of them) and its mask word: one round trip
        int32_t e[K3];
        uint32_t m = 0;
        if constexpr (FUSED) {
            // the four lanes that serve a row look up every fourth offset each and trade the results
            // through LDS (a wavefront's LDS operations execute in order: no barrier needed)
            __shared__ int32_t found_s[FUSED ? 4 * NT : 1][28][16];
            if (group_ok) {
                int32_t part[7];
                grid_neighbours_part<3, 4>(ms, row, n_out, qq, part);
#pragma unroll
                for (int u = 0; u < 7; ++u) found_s[wv][qq + 4 * u][r] = part[u];
#pragma unroll
                for (int k = 0; k < K3; ++k) e[k] = found_s[wv][k][r];
#pragma unroll
                for (int k = 0; k < K3; ++k) m |= (__ballot(e[k] >= 0) != 0ull ? 1u : 0u) << k;
            } else {
#pragma unroll
                for (int k = 0; k < K3; ++k) e[k] = -1;
            }
        } else if (group_ok) {
            const int32_t* line = nbr + tile * (int64_t)(K3 * TILE) + q * 16 + r;
#pragma unroll
            for (int k = 0; k < K3; ++k) e[k] = line[k * TILE];
            if (gmask != nullptr) {
                m = gmask[tile * 4 + q];
            } else {
                m = __builtin_amdgcn_readfirstlane(mask_of_entries(e));
            }
        } else {
#pragma unroll
            for (int k = 0; k < K3; ++k) e[k] = -1;
        }
        if (done == 0) {
            if constexpr (WPACKED) {
                __builtin_amdgcn_s_waitcnt(0x0f70);        // vmcnt(0)
            } else {
#pragma unroll
                for (int i = 0; i < PASSES; ++i) {
                    uint2 v[8];
                    if constexpr (!AHEAD) raw_weights(i, v);
                    weights_to_lds(i, AHEAD ? ahead[AHEAD ? i : 0] : v);
                }
            }
        }
        SC_MARK(1);
        m = __builtin_amdgcn_readfirstlane(m);

        if constexpr (UP) {
            uint4 own[KS];                       // the coarse row itself: no gather
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                own[ks] = (group_ok && row < n_out) ? reinterpret_cast<const uint4*>(feat + row * C_in)[qq + ks * 4]
                                                    : make_uint4(0, 0, 0, 0);
            if (done == 0) __syncthreads();
            SC_MARK(2);
#pragma unroll
            for (int k = 0; k < K3; ++k) {
                if (m & (1u << k)) {
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb) {
                        f32x4 d = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks)
                            d = mfma16x16x32<DT>(w_lds[((k * CB + cb) * KS + ks) * 64 + lane], own[ks], d);
                        if (e[k] >= 0) store_acc<DT>(out, out_f32, e[k], C_out, cb * 16 + qq * 4, d);
                    }
                }
            }
        } else {
            // every gather of the group in flight at once
            uint4 fb[K3][KS];
#pragma unroll
            for (int k = 0; k < K3; ++k) {
                if (m & (1u << k)) {
                    const uint4* frow = reinterpret_cast<const uint4*>(feat + (int64_t)(e[k] < 0 ? 0 : e[k]) * C_in) + qq;
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) fb[k][ks] = e[k] >= 0 ? frow[ks * 4] : make_uint4(0, 0, 0, 0);
                }
            }
            if (done == 0) __syncthreads();
            SC_MARK(2);

            f32x4 acc[CB];
#pragma unroll
            for (int cb = 0; cb < CB; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < K3; ++k) {
                if (m & (1u << k)) {
#pragma unroll
                    for (int cb = 0; cb < CB; ++cb)
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks)
                            acc[cb] = mfma16x16x32<DT>(w_lds[((k * CB + cb) * KS + ks) * 64 + lane], fb[k][ks], acc[cb]);
                }
            }
            SC_MARK(3);
            if (group_ok && row < n_out) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) store_acc<DT>(out, out_f32, row, C_out, cb * 16 + qq * 4, acc[cb]);
            }
        }
        done += team * each;
        if (!LOOP || done >= share) break;
        each = tiles_per_workgroup(share - done, team, NT);
    }
    SC_MARK(4);
    SC_MARK(5);
}

// A row of zeros that stands in for "no neighbour" in the streaming kernels: a lane without an
// input row reads its operand from here, so every lane issues every load.  The compiler can then
// count, at each use, exactly how many younger loads may still be in flight (s_waitcnt vmcnt(n));
// a load that is skipped under a condition makes that count unknown and every wait becomes
// vmcnt(0), which drains the loads that were issued ahead on purpose.
__device__ __align__(256) uint4 g_zero_row[32];      // 512 bytes: a row of up to 256 16-bit channels

// ---- larger layers: W[k] streamed through LDS, one offset at a time ------------------------------
// One wavefront per 64-row tile (four 16-row groups), NWV tiles per workgroup.  The workgroup
// walks the K3 offsets in lockstep; W[k] reaches the matrix cores through a double-buffered LDS
// tile, each weight operand read once and applied to every group of the wavefront that has a
// neighbour at k.  Everything else is arranged so that loads stay in flight across steps:
//  * the tile's offset-table lines are copied to LDS once, up front, so the loop reads neighbour
//    indices through the LDS counter and never has to wait on the vector-memory counter for them
//    (that counter retires in order: waiting for a young index load would drain every older
//    gather and weight fetch with it);
//  * gathered rows live in a ring of D register slots: as soon as a 32-channel slice of slot
//    k % D has been used it is refilled with the rows of offset k + D;
//  * W[k + D] is fetched into registers at the top of step k and stored to LDS at the end of step
//    k + D - 1;
//  * every load is issued by every lane (rows without a neighbour read the zero row), only the
//    multiplies are skipped, so all waits are exact counts.
// Accumulators (64 rows x C_out per wavefront) never leave the registers.  KS = C_in/32,
// CB = C_out/16.
// Rows are gathered in the operand's own lane order (16 rows x four 16-byte pieces of a 32-channel
// slice per load: 64 contiguous bytes of a row).  Gathering whole 128-byte lines with eight
// consecutive lanes per row is cheaper for the address unit, but the rows then have to pass
// through LDS to reach operand layout (k_conv_gather does), where this kernel's weights already
// keep the LDS busy; an in-register shuffle (lane-swap + quad-permute instructions, 20 VALU
// operations per 16 bytes) was measured slower than either.
// FUSED: as in k_conv_rows16, the offset-table lines come from the dense location table directly.
template <int DT, int K3, int KS, int CB, int NWV, int D, int FUSED>
__global__ void __launch_bounds__(64 * NWV, 2)
k_conv_stream(const uint16_t* __restrict__ feat, const uint4* wp, void* __restrict__ out, int out_f32,
              const MapSource ms, const int64_t* __restrict__ n_out_ptr, int64_t n_out_cap) {
    static_assert(K3 <= 32, "one mask word per group");
    static_assert(!FUSED || K3 == 27, "fused look-ups: 3x3x3 layers");
    const uint32_t* __restrict__ gmask = ms.gmask;
    const int32_t* __restrict__ nbr = ms.nbr;
    constexpr int NTH = 64 * NWV;
    constexpr int C_in = KS * 32, C_out = CB * 16;
    constexpr int WK = CB * KS * 64;                  // uint4 per packed W[k]
    static_assert(WK % NTH == 0, "a weight matrix is a whole number of passes of the workgroup");
    constexpr int WPT = WK / NTH;                     // uint4 per thread per W[k]
    constexpr int CBG = CB < 4 ? CB : 4;              // weight operands held at a time
    static_assert(CB % CBG == 0, "whole operand batches");
    extern __shared__ __align__(16) uint4 smem[];     // w_lds[2][WK] | e_lds[NWV][K3][64]

    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int r = lane & 15, qq = lane >> 4;
    uint4* w_lds = smem;
    int32_t* e_lds = reinterpret_cast<int32_t*>(smem + 2 * WK) + wv * (K3 * TILE);
    SC_MARK(0);
    const int64_t n_out = FUSED ? n_out_cap : output_rows(n_out_ptr, n_out_cap);
    // the grid covers the caller's row capacity; the rows that exist are spread over all XCDs and
    // a workgroup that gets none leaves at once (the same decision in every wavefront, before
    // any barrier)
    // a workgroup's tiles are spread over the whole row range (tile = wavefront * units + unit):
    // its steps last as long as its busiest wavefront's, and neighbouring tiles are alike in how
    // many offsets they take part in (10^6 voxels, 128 channels: -2 %)
    const int64_t units = (n_out + NWV * TILE - 1) / (NWV * TILE);
    const int64_t unit = xcd_unit_of(blockIdx.x, units);
    if (unit < 0) return;
    const int64_t tile = wv * units + unit;
    const bool tile_ok = tile * TILE < n_out;

    uint32_t mg[4] = {0u, 0u, 0u, 0u};
    {   // the tile's offset-table lines -> LDS (read back below by other lanes of this wavefront)
        int32_t v[K3];
        if constexpr (FUSED) {
            if (tile_ok) {
                grid_neighbours<3>(ms, tile * TILE + lane, n_out, v);
#pragma unroll
                for (int k = 0; k < K3; ++k) {
                    const uint64_t vote = __ballot(v[k] >= 0);
#pragma unroll
                    for (int g = 0; g < 4; ++g) mg[g] |= (((vote >> (16 * g)) & 0xffffull) != 0ull ? 1u : 0u) << k;
                }
            } else {
#pragma unroll
                for (int k = 0; k < K3; ++k) v[k] = -1;
            }
        } else if (tile_ok) {
            const int32_t* line = nbr + tile * (int64_t)(K3 * TILE) + lane;
#pragma unroll
            for (int k = 0; k < K3; ++k) v[k] = line[k * TILE];
#pragma unroll
            for (int g = 0; g < 4; ++g) mg[g] = gmask != nullptr ? gmask[tile * 4 + g] : 0u;
            if (gmask == nullptr) {
                const uint32_t m = mask_of_entries(v);
#pragma unroll
                for (int g = 0; g < 4; ++g) mg[g] = __builtin_amdgcn_readlane(m, 16 * g);
            }
        } else {
#pragma unroll
            for (int k = 0; k < K3; ++k) v[k] = -1;
        }
#pragma unroll
        for (int k = 0; k < K3; ++k) e_lds[k * TILE + lane] = v[k];
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) mg[g] = __builtin_amdgcn_readfirstlane(mg[g]);
    SC_MARK(1);

    const u32x4* wsrc = reinterpret_cast<const u32x4*>(wp) + threadIdx.x;
    u32x4 wr[D][WPT];
#pragma unroll
    for (int j = 0; j < D && j < K3; ++j)
#pragma unroll
        for (int i = 0; i < WPT; ++i) wr[j][i] = wsrc[(int64_t)j * WK + i * NTH];

    // a lane gathers row lane % 16 of a group, the (lane / 16)-th 16-byte piece of a 32-channel slice
    auto rowptr = [&](int32_t e) -> const uint4* {
        return (e >= 0 ? reinterpret_cast<const uint4*>(feat + (int64_t)e * C_in) : g_zero_row) + qq;
    };
    uint4 fb[D][4][KS];
#pragma unroll
    for (int j = 0; j < D && j < K3; ++j) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const uint4* frow = rowptr(e_lds[j * TILE + g * 16 + r]);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) fb[j][g][ks] = frow[ks * 4];
        }
    }
    f32x4 acc[4][CB];
#pragma unroll
    for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int cb = 0; cb < CB; ++cb) acc[g][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < WPT; ++i) reinterpret_cast<u32x4*>(w_lds)[threadIdx.x + i * NTH] = wr[0][i];
    lds_barrier();
    SC_MARK(2);

#pragma unroll
    for (int k = 0; k < K3; ++k) {
        const bool more = k + D < K3;
        if (more) {
#pragma unroll
            for (int i = 0; i < WPT; ++i) wr[k % D][i] = wsrc[(int64_t)(k + D) * WK + i * NTH];
        }
        int32_t e4[4] = {-1, -1, -1, -1};
        if (more) {
#pragma unroll
            for (int g = 0; g < 4; ++g) e4[g] = e_lds[(k + D) * TILE + g * 16 + r];
        }
        __builtin_amdgcn_sched_barrier(0);            // the fetches are issued here, not next to their use
        const uint4* wk = w_lds + (k & 1) * WK + lane;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int c0 = 0; c0 < CB; c0 += CBG) {
                uint4 a[CBG];
#pragma unroll
                for (int c = 0; c < CBG; ++c) a[c] = wk[wtile(KS, CB, c0 + c, ks) * 64];
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    if ((mg[g] >> k) & 1u) {
#pragma unroll
                        for (int c = 0; c < CBG; ++c)
                            acc[g][c0 + c] = mfma16x16x32<DT>(a[c], fb[k % D][g][ks], acc[g][c0 + c]);
                    }
                }
            }
            if (more && D == 1) {   // this slice is free: refill it with the rows of offset k + D
#pragma unroll
                for (int g = 0; g < 4; ++g) fb[k % D][g][ks] = rowptr(e4[g])[ks * 4];
            }
        }
        if (more && D > 1) {
            // with a deeper ring there is no hurry: refill the whole slot at once, so that the loads
            // which share a cache line (the 64-byte slices of one row) are issued back to back
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const uint4* frow = rowptr(e4[g]);
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) fb[k % D][g][ks] = frow[ks * 4];
            }
        }
        if (k + 1 < K3) {
#pragma unroll
            for (int i = 0; i < WPT; ++i)
                reinterpret_cast<u32x4*>(w_lds)[((k + 1) & 1) * WK + threadIdx.x + i * NTH] = wr[(k + 1) % D][i];
            lds_barrier();
        }
    }
    SC_MARK(3);
    if (tile_ok) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int64_t row = tile * TILE + g * 16 + r;
            if (row < n_out) {
#pragma unroll
                for (int cb = 0; cb < CB; ++cb) store_acc<DT>(out, out_f32, row, C_out, cb * 16 + qq * 4, acc[g][cb]);
            }
        }
    }
    SC_MARK(4);
    SC_MARK(5);
}

constexpr int CB_MAX = 16;
// The mask word of a 16-row group of a map without masks (K^3 <= 32): line = its first entry, at the lane's row.  The four lanes of a
// row take every fourth offset each, so it is one round trip; offset after offset, each behind the one before, it was up to 27 (us of whole
// strided fp32 layers, K = 3, stride 2: masks made by the build / offset after offset / now: 16 -> 16 2 k / 20 k / 100 k inputs 26.3 / 29.9 / 24.2, 30.8 / 34.3 /
// 28.2, 69.5 / 71.1 / 65.7; 32 -> 32 2 k 32.9 / 35.8 / 30.4; 5 -> 7 100 k 90.1 / 107.1 / 89.5; K = stride = 3, 16 -> 16 100 k 33.7 / 35.9 / 29.8).
__device__ inline uint32_t vote_mask(const int32_t* __restrict__ line, int K3, int qq) {
    uint32_t found = 0u;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = 4 * j + qq;
        const int32_t e = k < K3 ? line[k * TILE] : -1;
        found |= ((uint32_t)~e >> 31) << (4 * j);
    }
    found = or_of_group(found << qq);
    return __builtin_amdgcn_readlane(found, 0) | __builtin_amdgcn_readlane(found, 16) | __builtin_amdgcn_readlane(found, 32) |
           __builtin_amdgcn_readlane(found, 48);
}
// ---- fp32 features and weights -------------------------------------------------------------------
// Same scheme with the fp32 matrix instruction (v_mfma_f32_16x16x4_f32: true fp32 products and
// sums): one wavefront per 16 output rows, offsets walked by mask bit, operands read straight from
// the [K3][C_in][C_out] weights and the feature rows, four input channels per step.  Any C_in,
// C_out <= 256 (edges are zero-filled).
// MASKED: the map has masks.  The mask word is in a vector register either way: walked in a scalar one, the loop over channels took
// 3 to 6 % longer (48 -> 48 on 100 k rows, submanifold 305 -> 318 us, K = 3, stride 3 131 -> 139).
template <int MASKED>
__global__ void __launch_bounds__(256)
k_conv_f32(const float* __restrict__ feat, const float* __restrict__ w, float* __restrict__ out,
           const uint32_t* __restrict__ gmask, const int32_t* __restrict__ nbr, int K3, int mw, int C_in, int C_out,
           const int64_t* __restrict__ n_out_ptr, int64_t n_out_cap) {
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int r = lane & 15, qq = lane >> 4;
    const int CB = (C_out + 15) / 16;
    const int64_t tile = blockIdx.x;
    const int64_t n_out = output_rows(n_out_ptr, n_out_cap);
    const int64_t row = tile * TILE + q * 16 + r;
    if (tile * TILE + q * 16 >= n_out) return;                       // uniform per wavefront

    f32x4 acc[CB_MAX];
#pragma unroll
    for (int cb = 0; cb < CB_MAX; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int32_t* line = nbr + tile * (int64_t)K3 * TILE + q * 16 + r;
    for (int wi = 0; wi < mw; ++wi) {
        uint32_t m;
        if constexpr (MASKED) {
            m = gmask[(tile * 4 + q) * mw + wi];
        } else {
            m = vote_mask(line, K3, qq);
            asm volatile("" : "+v"(m));
        }
        while (m) {
            const int k = wi * 32 + __builtin_ctz(m);
            m &= m - 1;
            const int32_t e = line[(int64_t)k * TILE];
            const float* frow = feat + (int64_t)(e < 0 ? 0 : e) * C_in;
            const float* wk = w + (int64_t)k * C_in * C_out;
            for (int ci0 = 0; ci0 < C_in; ci0 += 4) {
                const int ci = ci0 + qq;
                const bool ci_ok = ci < C_in;
                const float b = (e >= 0 && ci_ok) ? frow[ci] : 0.f;
#pragma unroll
                for (int cb = 0; cb < CB_MAX; ++cb) {
                    if (cb < CB) {
                        const int co = cb * 16 + r;
                        const float a = (ci_ok && co < C_out) ? wk[(int64_t)ci * C_out + co] : 0.f;
                        acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[cb], 0, 0, 0);
                    }
                }
            }
        }
    }
    if (row < n_out) {
        float* orow = out + row * C_out;
#pragma unroll
        for (int cb = 0; cb < CB_MAX; ++cb) {
            if (cb < CB) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int co = cb * 16 + qq * 4 + i;
                    if (co < C_out) orow[co] = acc[cb][i];
                }
            }
        }
    }
}

// fp32 layers of at most four input channels (a network's first layer: coordinates, intensity), K = 2 or 3: the four
// channels of an offset are exactly one 16x16x4 multiply, so the layer is K^3 multiplies per group and output block.
// What it costs is latency, so a group's table lines, then all its rows (one 4-byte load per offset: the four
// lanes of a row read 16 bytes), are in flight together, and the weights come from LDS.  Sums in the order
// of k_conv_f32, whose table entry, row and weights were loaded at their use (whole layers 4 -> 32 on 3 k / 80 k sweep
// voxels 25.2 / 51.3 -> 14.2 / 30.6 us).
template <int K3, int CB>
__global__ void __launch_bounds__(256)
k_conv_f32_first(const float* __restrict__ feat, const float* __restrict__ w, float* __restrict__ out,
                 const uint32_t* __restrict__ gmask, const int32_t* __restrict__ nbr, int C_in,
                 const int64_t* __restrict__ n_out_ptr, int64_t n_out_cap) {
    static_assert(K3 <= 32, "one mask word per group");
    constexpr int C_out = 16 * CB;
    __shared__ __align__(16) float w_s[K3 * 4 * C_out];              // [K3][4][C_out], zero past C_in
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int r = lane & 15, qq = lane >> 4;
    const int64_t n_out = output_rows(n_out_ptr, n_out_cap);
    const int64_t tile = xcd_run_of(blockIdx.x, (n_out + TILE - 1) / TILE);
    if (tile < 0) return;                                            // the whole workgroup
    const int64_t row = tile * TILE + q * 16 + r;

    const int32_t* line = nbr + tile * (int64_t)(K3 * TILE) + q * 16 + r;
    int32_t e[K3];
#pragma unroll
    for (int k = 0; k < K3; ++k) e[k] = row < n_out ? line[k * TILE] : -1;
    uint32_t m = 0u;
    if (gmask != nullptr) {
        m = __builtin_amdgcn_readfirstlane(gmask[tile * 4 + q]);
    } else {
        m = __builtin_amdgcn_readfirstlane(mask_of_entries(e));
    }
    for (int i = threadIdx.x; i < K3 * C_out; i += 256) {           // 16 bytes each
        const int col = i % (C_out / 4), kc = i / (C_out / 4), ci = kc & 3;
        reinterpret_cast<float4*>(w_s)[i] =
            ci < C_in ? reinterpret_cast<const float4*>(w + ((kc >> 2) * C_in + ci) * C_out)[col] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
    float f[K3];
#pragma unroll
    for (int k = 0; k < K3; ++k) f[k] = e[k] >= 0 && qq < C_in ? feat[(int64_t)e[k] * C_in + qq] : 0.f;
    __syncthreads();
    f32x4 acc[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < K3; ++k) {
        if (m & (1u << k)) {
#pragma unroll
            for (int cb = 0; cb < CB; ++cb)
                acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(w_s[(k * 4 + qq) * C_out + cb * 16 + r], f[k], acc[cb], 0, 0, 0);
        }
    }
    if (row < n_out) {
        float* orow = out + row * C_out;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
            *reinterpret_cast<float4*>(orow + cb * 16 + qq * 4) = make_float4(acc[cb][0], acc[cb][1], acc[cb][2], acc[cb][3]);
    }
}

// fp32 layers with few channels (C_in = 16*CI16 <= 64, C_out = 16*CB <= 64, K^3 <= 32): the same
// instruction, loads batched.  A lane reads 16 bytes (4 channels) of its row per 16-channel chunk
// and feeds component j to the j-th of four multiplies, so input channel 16c + 4q + j sits at
// position q of multiply (c, j); the weight operand is read to match.  The offsets that exist are
// taken four at a time: their four table entries are in flight together, then all their feature
// loads, so a group costs two dependent round trips per batch instead of two per offset.
template <int CI16, int CB>
__global__ void __launch_bounds__(256)
k_conv_f32_small(const float* __restrict__ feat, const float* __restrict__ w, float* __restrict__ out,
                 const uint32_t* __restrict__ gmask, const int32_t* __restrict__ nbr, int K3,
                 const int64_t* __restrict__ n_out_ptr, int64_t n_out_cap) {
    constexpr int C_in = 16 * CI16, C_out = 16 * CB, NB = 4;
    const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int r = lane & 15, qq = lane >> 4;
    const int64_t tile = blockIdx.x;
    const int64_t n_out = output_rows(n_out_ptr, n_out_cap);
    const int64_t row = tile * TILE + q * 16 + r;
    if (tile * TILE + q * 16 >= n_out) return;                       // uniform per wavefront

    f32x4 acc[CB];
#pragma unroll
    for (int cb = 0; cb < CB; ++cb) acc[cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int32_t* line = nbr + tile * (int64_t)K3 * TILE + q * 16 + r;
    uint32_t m = gmask != nullptr ? __builtin_amdgcn_readfirstlane(gmask[tile * 4 + q]) : vote_mask(line, K3, qq);
    while (m) {
        int kk[NB];
        int32_t e[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            kk[j] = m ? __builtin_ctz(m) : -1;
            if (m) m &= m - 1;
            e[j] = kk[j] >= 0 ? line[kk[j] * TILE] : -1;
        }
        float4 f[NB][CI16];
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const float4* frow = reinterpret_cast<const float4*>(feat + (int64_t)(e[j] < 0 ? 0 : e[j]) * C_in) + qq;
#pragma unroll
            for (int c = 0; c < CI16; ++c) f[j][c] = e[j] >= 0 ? frow[c * 4] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (kk[j] >= 0) {                                        // uniform
                const float* wk = w + (int64_t)kk[j] * C_in * C_out + r;
#pragma unroll
                for (int c = 0; c < CI16; ++c) {
                    const float b[4] = {f[j][c].x, f[j][c].y, f[j][c].z, f[j][c].w};
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float* wrow = wk + (int64_t)(c * 16 + 4 * qq + t) * C_out;
#pragma unroll
                        for (int cb = 0; cb < CB; ++cb)
                            acc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(wrow[cb * 16], b[t], acc[cb], 0, 0, 0);
                    }
                }
            }
        }
    }
    if (row < n_out) {
        float* orow = out + row * C_out;
#pragma unroll
        for (int cb = 0; cb < CB; ++cb)
            *reinterpret_cast<float4*>(orow + cb * 16 + qq * 4) = make_float4(acc[cb][0], acc[cb][1], acc[cb][2], acc[cb][3]);
    }
}

template <int DT, int K3, int KS, int CB, int NT, int FUSED, int UP = 0, int WPACKED = 0>
static int launch_rows16(int64_t tiles, hipStream_t s, const uint16_t* feat, const uint4* wp, void* out, int out_f32,
                         const MapSource& ms, const int64_t* counts, int64_t n_out_cap) {
    auto fn = k_conv_rows16<DT, K3, KS, CB, NT, FUSED, UP, WPACKED>;
    const size_t lds = (size_t)K3 * CB * KS * 64 * sizeof(uint4);
    static bool allowed[MAX_DEVICES] = {};  // per instantiation
    if (int rc = allow_lds((const void*)fn, lds, allowed)) return rc;
    // workgroups per XCD and round: one per compute unit; without the loop as many as there are at NT tiles each
    const int team = (compute_units() + NUM_XCD - 1) / NUM_XCD;
    const int64_t share = (tiles + NUM_XCD - 1) / NUM_XCD, all = resident_loop(K3, KS, CB, UP) ? 0 : (share + NT - 1) / NT;
    const int64_t most = all > team ? all : team, turns = share < most ? share : most;
    SC_LAUNCH(KID_CONV_MFMA, fn, dim3((unsigned)(turns * NUM_XCD)), dim3(256 * NT), lds, s, feat, wp, out, out_f32, ms, team, counts, n_out_cap);
    return SC_OK;
}

// Shapes whose packed weights fit in LDS as a whole.  The resident kernel's LDS layout of the
// weights is the packed layout itself (tile (k, cb, ks) at ((k CB + cb) KS + ks): one 64-channel
// half at most), so packed weights are copied and raw ones re-laid out on the way in.
static bool resident_shape(int K3, int C_in, int C_out, bool fused) {
    if (K3 == 27 && C_in == 32 && C_out == 32) return true;
    if (fused) return false;
    return K3 == 8 && ((C_in == 32 && C_out == 64) || (C_in == 32 && C_out == 32) || (C_in == 64 && C_out == 64) ||
                       (C_in == 64 && C_out == 32));
}
template <int DT, int FUSED, int WPACKED>
static int launch_resident(int K3, int C_in, int C_out, int64_t tiles, int64_t likely, hipStream_t s, const uint16_t* feat,
                           const uint4* wp, void* out, int out_f32, const MapSource& ms, const int64_t* counts,
                           int64_t n_out_cap, bool* handled) {
    *handled = true;
    const int64_t cus = compute_units();
#define SC_ROWS16(K3V, KSV, CBV, NTV) \
    return launch_rows16<DT, K3V, KSV, CBV, NTV, FUSED, 0, WPACKED>(tiles, s, feat, wp, out, out_f32, ms, counts, n_out_cap)
    // 3x3x3: up to four tiles per workgroup where that is one workgroup per CU for the likely tiles, and two where two do that or there are more than one
    // round of four: with 16 wavefronts of 124 registers a CU has no second workgroup to go on with (us of whole layers, four and two tiles, sweeps: packed
    // 36 k / 48 k / 53 k / 60 k 19.4 / 20.8 / 23.4 / 25.0 and 20.4 / 21.7 / 23.6 / 25.2, 70 k / 80 k / 110 k / 130 k 30.2 / 31.8 / 38.2 / 42.0 and 28.3 / 29.7 / 37.2 / 40.9; fused 36 k / 53 k 12.7 / 14.8
    // and 14.3 / 15.5, 80 k / 200 k 23.4 / 51.0 and 20.5 / 46.0; indoor 80 k 34.4 and 30.1).  The likely ones: the bound of a strided layer is up to eight times what there is.
    if (K3 == 27 && C_in == 32 && C_out == 32 && likely > 2 * cus && likely <= 4 * cus) SC_ROWS16(27, 1, 2, 4);
    if (K3 == 27 && C_in == 32 && C_out == 32) SC_ROWS16(27, 1, 2, 2);
    if constexpr (!FUSED) {
        // 32 -> 64: up to four tiles and all rounds in one workgroup against a workgroup per two tiles (us of the convolution, packed weights, sweeps 2 k / 30 k / 53 k / 80 k / 110 k / 150 k / 200 k 4.3 /
        // 4.6 / 4.9 / 6.0 / 6.3 / 8.2 / 9.0 with two, now 3.8 / 3.9 / 4.5 / 5.4 / 6.6 / 8.1 / 8.9, indoor 53 k / 200 k / 600 k 5.0 / 6.9 / 17.3 and 4.1 / 7.3 / 15.9, random cells 20 k / 100 k 4.9 / 8.9 and 4.6 / 9.0): shares of three
        // tiles, as 110 k sweep and 200 k indoor rows give, leave a quarter of the CUs without any.  Two tiles and the loop 6.1 at 80 k and 18.2 indoor, four without it 9.7 at 150 k.
        if (K3 == 8 && C_in == 32 && C_out == 64) SC_ROWS16(8, 1, 4, 4);
        if (K3 == 8 && C_in == 32 && C_out == 32) SC_ROWS16(8, 1, 2, 2);
        if (K3 == 8 && C_in == 64 && C_out == 64) SC_ROWS16(8, 2, 4, 4);
        if (K3 == 8 && C_in == 64 && C_out == 32) SC_ROWS16(8, 2, 2, 4);      // the up-sampling twin of 32 -> 64
    }
#undef SC_ROWS16
    *handled = false;
    return SC_OK;
}

template <int DT, int K3, int KS, int CB, int NWV, int D, int FUSED>
static int launch_stream(int64_t tiles, hipStream_t s, const uint16_t* feat, const uint4* wp, void* out, int out_f32,
                         const MapSource& ms, const int64_t* counts, int64_t n_out_cap) {
    auto fn = k_conv_stream<DT, K3, KS, CB, NWV, D, FUSED>;
    const size_t lds = (size_t)2 * CB * KS * 64 * sizeof(uint4) +
                       (size_t)NWV * K3 * TILE * sizeof(int32_t);
    static bool allowed[MAX_DEVICES] = {};
    if (int rc = allow_lds((const void*)fn, lds, allowed)) return rc;
    SC_LAUNCH(KID_CONV_MFMA, fn, dim3(xcd_grid((tiles + NWV - 1) / NWV)), dim3(64 * NWV), lds, s, feat, wp, out, out_f32,
              ms, counts, n_out_cap);
    return SC_OK;
}

// Compute units of the current device, asked once (a race between host threads stores the same value).
int compute_units() {
    static int cu_count[MAX_DEVICES] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return 256;
    if (cu_count[dev] == 0) {
        int n = 0;
        cu_count[dev] = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && n > 0 ? n : 256;
    }
    return cu_count[dev];
}

// Up-sampling straight from the strided layer's map: shapes with a dedicated kernel.
template <int DT>
static int launch_up(int K3, int C_in, int C_out, int64_t tiles, hipStream_t s, const uint16_t* feat, const uint4* wp,
                     void* out, int out_f32, const MapSource& ms, const int64_t* counts, int64_t n_out_cap,
                     bool* handled) {
    *handled = true;
#define SC_UP16(K3V, KSV, CBV, NTV) \
    return launch_rows16<DT, K3V, KSV, CBV, NTV, 0, 1>(tiles, s, feat, wp, out, out_f32, ms, counts, n_out_cap)
    // 64 -> 32, a workgroup per two tiles and now: 30 k / 80 k / 110 k / 150 k / 200 k / 260 k 5.1 / 7.0 / 7.5 / 9.8 / 10.6 / 13.0 and 4.9 / 6.4 / 7.9 / 9.4 / 10.2 / 12.5, indoor 200 k / 600 k 8.9 / 20.5 and 9.3 / 18.0, random
    // cells 100 k 8.7 and 8.9; four tiles without the loop 7.4 at 110 k, but 10.9 at 150 k
    if (K3 == 8 && C_in == 64 && C_out == 32) SC_UP16(8, 2, 2, 4);
    if (K3 == 8 && C_in == 32 && C_out == 32) SC_UP16(8, 1, 2, 2);
    if (K3 == 8 && C_in == 64 && C_out == 64) SC_UP16(8, 2, 4, 4);
    if (K3 == 8 && C_in == 128 && C_out == 64) SC_UP16(8, 4, 4, 4);
    if (K3 == 27 && C_in == 32 && C_out == 32) SC_UP16(27, 1, 2, 4);
#undef SC_UP16
    *handled = false;
    return SC_OK;
}

// Shapes with a streaming kernel.
template <int DT, int FUSED>
static int launch_streamed(int K3, int C_in, int C_out, int64_t tiles, hipStream_t s, const uint16_t* feat,
                           const uint4* wp, void* out, int out_f32, const MapSource& ms, const int64_t* counts,
                           int64_t n_out_cap, bool* handled) {
    *handled = true;
#define SC_STREAM(K3V, KSV, CBV, NWV, DV) \
    return launch_stream<DT, K3V, KSV, CBV, NWV, DV, FUSED>(tiles, s, feat, wp, out, out_f32, ms, counts, n_out_cap)
    if (K3 == 27 && C_in == 128 && C_out == 128) SC_STREAM(27, 4, 8, 8, 1);
    if constexpr (!FUSED) {
        if (K3 == 27 && C_in == 32 && C_out == 64) SC_STREAM(27, 1, 4, 4, 3);
        if (K3 == 8 && C_in == 128 && C_out == 128) SC_STREAM(8, 4, 8, 8, 1);
    }
#undef SC_STREAM
    *handled = false;
    return SC_OK;
}

static bool mfma_channels_ok(int C_in, int C_out) {
    return (C_in == 32 || C_in == 64 || C_in == 128 || C_in == 256) && C_out >= 16 && C_out <= 256 && C_out % 16 == 0;
}

// Packed form of 16-bit weights [K3][C_in][C_out] for sc_conv_fwd's kernels (operand tiles, see k_weight_pack).
static int pack_weights(int K3, int C_in, int C_out, const void* d_weight, void* d_packed, hipStream_t s) {
    const int64_t pack_threads = (int64_t)K3 * (C_out / 16) * (C_in / 32) * 64;
    SC_LAUNCH(KID_WEIGHT_PACK, k_weight_pack, dim3((unsigned)((pack_threads + 255) / 256)), dim3(256), 0, s,
              (const uint16_t*)d_weight, (uint4*)d_packed, K3, C_in, C_out);
    return SC_OK;
}

// A 16-bit layer.  `packed`: d_weight is what sc_conv_weight_pack made; otherwise the raw weights,
// which the resident kernels re-lay out themselves and the others have packed into the workspace
// first.  FUSED (dense table, no map) always takes raw weights.  Of strided
// layers the number of output rows is known on the device only.  `sets`: two sets of wavefronts where the general kernel takes it.
template <int FUSED>
static int conv_16bit(int dtype_in, int K3, int mw, int C_in, int C_out, int64_t tiles, int64_t likely, LayerKind kind, bool sets, hipStream_t s,
                      const void* d_feat_in, const void* d_weight, bool packed, void* d_workspace, void* d_feat_out,
                      int out_f32, const MapSource& ms, const int64_t* n_out_ptr, int64_t n_out_cap) {
    const uint16_t* feat = (const uint16_t*)d_feat_in;
    bool handled = false;
    // The resident kernel takes its shapes at every size (us of whole layers, general and resident, packed weights, sweeps: 64 -> 64, K = 2, 110 k / 148 k / 160 k / 175 k /
    // 196 k / 300 k 26.9 / 29.7 / 29.8 / 31.5 / 32.9 / 50.1 and 25.9 / 30.3 / 30.5 / 31.5 / 32.8 / 46.9, indoor 148 k / 196 k / 400 k / 800 k 25.0 / 28.1 / 52.2 / 86.0 and 24.7 / 28.3 / 48.5 / 81.3, random
    // cells 148 k / 175 k / 196 k 45.7 / 50.0 / 53.6 and 43.4 / 46.9 / 49.5; convolutions of inverse maps,
    // sweeps 110 k / 148 k / 196 k / 300 k 14.1 / 18.0 / 20.3 / 28.8 and 12.3 / 14.8 / 16.4 / 23.1, indoor 16.1 / 19.2 / 23.4 / 34.2 and 14.3 / 17.6 / 19.6 / 27.6; 32 -> 32, K = 3, 150 k / 200 k / 400 k 46.7 / 61.9 / 124.0 and 45.2 / 60.2 / 121.2, indoor 50.2 / 62.3 / 124.3 and
    // 46.5 / 59.9 / 116.9).
    if (resident_shape(K3, C_in, C_out, FUSED)) {
        if constexpr (!FUSED) {
            if (packed)
                return dtype_in == SC_F16 ? launch_resident<SC_F16, 0, 1>(K3, C_in, C_out, tiles, likely, s, feat, (const uint4*)d_weight, d_feat_out,
                                                                          out_f32, ms, n_out_ptr, n_out_cap, &handled)
                                          : launch_resident<SC_BF16, 0, 1>(K3, C_in, C_out, tiles, likely, s, feat, (const uint4*)d_weight, d_feat_out,
                                                                           out_f32, ms, n_out_ptr, n_out_cap, &handled);
        }
        return dtype_in == SC_F16 ? launch_resident<SC_F16, FUSED, 0>(K3, C_in, C_out, tiles, likely, s, feat, (const uint4*)d_weight, d_feat_out,
                                                                      out_f32, ms, n_out_ptr, n_out_cap, &handled)
                                  : launch_resident<SC_BF16, FUSED, 0>(K3, C_in, C_out, tiles, likely, s, feat, (const uint4*)d_weight, d_feat_out,
                                                                       out_f32, ms, n_out_ptr, n_out_cap, &handled);
    }
    const bool fused_gather = (C_in == 32 && C_out == 64) || (C_in == 64 && (C_out == 64 || C_out == 128)), wide = C_in == 128 && C_out == 128;
    if (FUSED && !fused_gather && !wide) return SC_EINVAL;     // no fused kernel for this shape: use the three calls
    const uint4* wp = (const uint4*)d_weight;
    if (!packed) {
        if (int prc = pack_weights(K3, C_in, C_out, d_weight, d_workspace, s)) return prc;
        wp = (const uint4*)d_workspace;
    }
    // general or streaming kernel (sc_rules.h).  Fused 32 -> 64, where the look-ups would add to the walk of a wavefront with 64 rows, through
    // the general one at every size (whole layers, us, general and streaming: 2 k 13.1 / 22.3, 53 k 22.5 / 27.0, 200 k 60.3 / 77.6, 400 k 114 / 142, 10^6 257 /
    // 309; indoor 200 k 50.2 / 58.2, 400 k 104 / 115, 800 k 213.6 / 216.9, 10^6 266.9 / 269.0)
    const bool general = FUSED && fused_gather ? true
                         : wide                ? general_128_to_128(K3 == 27 ? 3 : 2, likely, kind == CELLS || kind == OVERLAPPING, compute_units())
                                               : !FUSED && K3 == 27 && C_in == 32 && C_out == 64 &&
                                                     general_32_to_64(likely, kind == OVERLAPPING, compute_units());
    if (general && FUSED)
        return launch_gather_fused(dtype_in, C_in, C_out, tiles, sets, compute_units(), s, feat, wp, d_feat_out, out_f32, ms, n_out_cap);
    if (general)
        return launch_gather(dtype_in, K3, mw, C_in, C_out, tiles, likely, kind, sets, compute_units(), s, feat, wp, d_feat_out, out_f32, ms, n_out_ptr, n_out_cap);
    const int rc = dtype_in == SC_F16 ? launch_streamed<SC_F16, FUSED>(K3, C_in, C_out, tiles, s, feat, wp, d_feat_out, out_f32, ms,
                                                                       n_out_ptr, n_out_cap, &handled)
                                      : launch_streamed<SC_BF16, FUSED>(K3, C_in, C_out, tiles, s, feat, wp, d_feat_out, out_f32, ms,
                                                                        n_out_ptr, n_out_cap, &handled);
    if (handled || rc != SC_OK) return rc;
    if (FUSED) return SC_EINVAL;
    return launch_gather(dtype_in, K3, mw, C_in, C_out, tiles, likely, kind, sets, compute_units(), s, feat, wp, d_feat_out, out_f32, ms, n_out_ptr, n_out_cap);
}

}  // namespace sc

using namespace sc;

extern "C" size_t sc_conv_workspace_bytes(int K, int C_in, int C_out, int dtype_in) {
    if (K < 1 || K > SC_K_MAX || C_in < 1 || C_out < 1) return 0;
    if (dtype_in == SC_F32) return 0;
    return align_up((size_t)K * K * K * C_in * C_out * 2, 256);
}

static int conv_fwd(const void* d_feat_in, int64_t n_map, const void* d_weight, bool packed, void* d_feat_out,
                    int64_t n_out_cap, const void* d_kmap, size_t kmap_bytes, const sc_counts* d_counts, int K, int stride,
                    int mode, int C_in, int C_out, int dtype_in, int dtype_out, void* d_workspace, size_t workspace_bytes,
                    void* stream) {
    if (n_map < 0 || n_map > SC_N_MAX || n_out_cap < 0 || K < 1 || K > SC_K_MAX || C_in < 1 || C_out < 1) return SC_EINVAL;
    if (d_weight == nullptr || d_kmap == nullptr || d_counts == nullptr) return SC_EINVAL;
    if ((n_map > 0 && d_feat_in == nullptr) || (n_out_cap > 0 && d_feat_out == nullptr)) return SC_EINVAL;
    if (!aligned16(d_feat_in) || !aligned16(d_weight) || !aligned16(d_feat_out) || !aligned16(d_kmap) ||
        !aligned16(d_counts) || !aligned16(d_workspace))
        return SC_EINVAL;
    if (dtype_in != SC_F32 && dtype_in != SC_F16 && dtype_in != SC_BF16) return SC_EINVAL;
    if (dtype_out != SC_F32 && dtype_out != dtype_in) return SC_EINVAL;
    const int64_t bound = sc_out_bound(n_map, K, stride, mode);
    if (bound < 0) return SC_EINVAL;
    if (kmap_bytes < sc_kmap_bytes(n_map, K, stride, mode)) return SC_ECAP;
    // rows of the output: of a strided layer what the map build counted, otherwise the rows the map was built from
    const int64_t* n_out_ptr = mode == SC_STRIDED ? &d_counts->n_out : nullptr;
    if (mode != SC_STRIDED && n_out_cap > n_map) n_out_cap = n_map;
    const KmapLayout L = kmap_layout(bound, K, stride, mode);
    int64_t tiles = (n_out_cap + TILE - 1) / TILE;
    if (tiles > L.tiles) tiles = L.tiles;
    if (tiles == 0) return SC_OK;
    // tiles to expect: strided layers on surfaces have about as many output rows as input rows, their bound is up to 8 times that
    const int64_t n_map_tiles = (n_map + TILE - 1) / TILE, likely = tiles < n_map_tiles ? tiles : n_map_tiles;
    const uint32_t* gmask = kmap_masked(mode, L.K3) ? (const uint32_t*)((const char*)d_kmap + L.off_mask) : nullptr;
    const int32_t* nbr = (const int32_t*)((const char*)d_kmap + L.off_nbr);
    const uint32_t* density = (const uint32_t*)map_density(d_kmap, L);
    const LayerKind kind = mode == SC_SUBM ? SUBMANIFOLD : mode == SC_INVERSE ? INVERSE : K == stride ? CELLS : OVERLAPPING;
    hipStream_t s = (hipStream_t)stream;

    if (dtype_in == SC_F32) {           // fp32 weights are used as they are: packed == raw
        if (C_out > 256) return SC_EINVAL;
        // The general kernel where a layer has enough work for it; its steps are mostly latency below that.  us of the convolution,
        // the kernel of small layers (with an instantiation for 32 -> 64 and more) and the general one, on sweeps (K = 3), sets of
        // random cells (few neighbours) and strided layers (K = 3, stride 2, rows of the input):
        //   64 -> 64  sweeps 500 20.0 / 11.7, 4 k 43 / 18, 53 k 121 / 73; random 300 12.3 / 9.2, 16 k 17.6 / 18.7; strided 2 k 33 / 31, 53 k 160 / 114
        //   32 -> 64  sweeps 500 11.6 / 8.6, 16 k 26.5 / 25.2, 53 k 66 / 45; random 300 7.7 / 6.8, 16 k 10.7 / 12.7
        //   64 -> 32  sweeps 500 12.2 / 11.6, 8 k 27.8 / 18.3, 53 k 69 / 46; random 300 7.7 / 9.1, 16 k 10.7 / 13.5
        //   32 -> 32  sweeps 500 7.7 / 8.5, 8 k 16.5 / 13.0, 24 k 25.6 / 19.4; random 2 k 5.8 / 6.9, 16 k 7.0 / 9.0; strided 8 k 15.6 / 12.8, 16 k 15.9 / 15.3
        //   16 -> 64  sweeps 4 k 14.8 / 10.0, 16 k 16.3 / 19.3, 24 k 24.7 / 22.8; random 16 k 7.2 / 12.2; strided 8 k 15.3 / 16.9, 16 k 15.8 / 21.0, 24 k 25.1 / 24.0
        //   64 -> 16  sweeps 8 k 18.4 / 18.0, 24 k 28.6 / 24.2; random 16 k 7.2 / 12.6; strided 16 k 17.3 / 18.3, 24 k 27.3 / 23.0
        //   16 -> 16  random 8 k 5.7 / 9.2
        // So from 2,048 channel products on at every size, and 1,024 from a tile per CU on: below that the small kernel loses
        // up to a quarter on sweeps and wins that on random cells.  Tiles are the ones to expect; the shapes that the small kernel
        // does not have (16 -> 80 to 112, 32 -> 48) have only k_conv_f32 below the line and keep the bound, which draws it lower
        // (strided 4 k rows, k_conv_f32 and general: 32 -> 48 95 / 16, 16 -> 80 72 / 19).
        const int64_t line_tiles = C_out == 16 || C_out == 32 || C_out == 64 ? likely : tiles;
        const bool slices = C_in == 16 || C_in == 32 || C_in == 64 || C_in == 128 || C_in == 256;
        if (slices && C_out % 16 == 0 && (C_in * C_out >= 2048 || (C_in * C_out >= 1024 && line_tiles >= compute_units()) || L.K3 > 32)) {
            const MapSource ms{gmask, nbr, nullptr, nullptr, GridDims{0, 0, 0, 0}, 0u, density};
            return launch_gather(SC_F32, L.K3, L.mw, C_in, C_out, tiles, likely, kind, false, compute_units(), s, d_feat_in, d_weight, d_feat_out, 1, ms, n_out_ptr,
                                 n_out_cap);
        }
        if (C_in <= 4) {
#define SC_F32_FIRST(K3V, CBV)                                                                                                \
    if (L.K3 == K3V && C_out == 16 * CBV) {                                                                                   \
        SC_LAUNCH(KID_CONV_F32, (k_conv_f32_first<K3V, CBV>), dim3(xcd_run_grid(tiles)), dim3(256), 0, s, (const float*)d_feat_in, \
                  (const float*)d_weight, (float*)d_feat_out, gmask, nbr, C_in, n_out_ptr, n_out_cap);                         \
        return SC_OK;                                                                                                         \
    }
            SC_F32_FIRST(27, 1) SC_F32_FIRST(27, 2) SC_F32_FIRST(27, 4) SC_F32_FIRST(8, 1) SC_F32_FIRST(8, 2) SC_F32_FIRST(8, 4)
#undef SC_F32_FIRST
        }
        if (L.K3 <= 32 && C_in % 16 == 0 && C_in <= 64 && C_out % 16 == 0 && C_out <= 64) {
#define SC_F32_SMALL(CI, CBV)                                                                                         \
    if (C_in == 16 * CI && C_out == 16 * CBV) {                                                                       \
        SC_LAUNCH(KID_CONV_F32, (k_conv_f32_small<CI, CBV>), dim3((unsigned)tiles), dim3(256), 0, s,                  \
                  (const float*)d_feat_in, (const float*)d_weight, (float*)d_feat_out, gmask, nbr, L.K3, n_out_ptr,   \
                  n_out_cap);                                                                                         \
        return SC_OK;                                                                                                 \
    }
            SC_F32_SMALL(1, 1) SC_F32_SMALL(1, 2) SC_F32_SMALL(1, 4) SC_F32_SMALL(2, 1) SC_F32_SMALL(2, 2) SC_F32_SMALL(4, 1)
#undef SC_F32_SMALL
        }
        const auto any = gmask != nullptr ? k_conv_f32<1> : k_conv_f32<0>;
        SC_LAUNCH(KID_CONV_F32, any, dim3((unsigned)tiles), dim3(256), 0, s, (const float*)d_feat_in,
                  (const float*)d_weight, (float*)d_feat_out, gmask, nbr, L.K3, L.mw, C_in, C_out, n_out_ptr,
                  n_out_cap);
        return SC_OK;
    }

    if (!mfma_channels_ok(C_in, C_out)) return SC_EINVAL;
    if (!packed) {
        const size_t need = sc_conv_workspace_bytes(K, C_in, C_out, dtype_in);
        if (d_workspace == nullptr || workspace_bytes < need) return SC_ECAP;
    }
    const MapSource ms{gmask, nbr, nullptr, nullptr, GridDims{0, 0, 0, 0}, 0u, density};
    // by the rows of the map, not by the caller's capacity: the order of a row's sums is not to depend on how large a buffer is
    const bool sets = two_sets(n_map_tiles, L.K3, C_out / 16, C_in, mode == SC_STRIDED && K >= 2 * stride, compute_units());
    return conv_16bit<0>(dtype_in, L.K3, L.mw, C_in, C_out, tiles, likely, kind, sets, s, d_feat_in, d_weight, packed,
                         d_workspace, d_feat_out, dtype_out == SC_F32, ms, n_out_ptr, n_out_cap);
}

extern "C" int sc_conv_fwd(const void* d_feat_in, int64_t n_map, const void* d_weight, void* d_feat_out,
                           int64_t n_out_cap, const void* d_kmap, size_t kmap_bytes, const sc_counts* d_counts, int K,
                           int stride, int mode, int C_in, int C_out, int dtype_in, int dtype_out, void* d_workspace,
                           size_t workspace_bytes, void* stream) {
    return conv_fwd(d_feat_in, n_map, d_weight, false, d_feat_out, n_out_cap, d_kmap, kmap_bytes, d_counts, K, stride, mode,
                    C_in, C_out, dtype_in, dtype_out, d_workspace, workspace_bytes, stream);
}

extern "C" int sc_conv_fwd_packed(const void* d_feat_in, int64_t n_map, const void* d_packed, void* d_feat_out,
                                  int64_t n_out_cap, const void* d_kmap, size_t kmap_bytes, const sc_counts* d_counts,
                                  int K, int stride, int mode, int C_in, int C_out, int dtype_in, int dtype_out,
                                  void* stream) {
    return conv_fwd(d_feat_in, n_map, d_packed, true, d_feat_out, n_out_cap, d_kmap, kmap_bytes, d_counts, K, stride, mode,
                    C_in, C_out, dtype_in, dtype_out, nullptr, 0, stream);
}

extern "C" size_t sc_conv_packed_bytes(int K, int C_in, int C_out, int dtype_in) {
    if (K < 1 || K > SC_K_MAX || C_in < 1 || C_out < 1) return 0;
    if (dtype_in == SC_F32) return align_up((size_t)K * K * K * C_in * C_out * 4, 256);
    if (dtype_in != SC_F16 && dtype_in != SC_BF16) return 0;
    return align_up((size_t)K * K * K * C_in * C_out * 2, 256);
}

extern "C" int sc_conv_weight_pack(const void* d_weight, int K, int C_in, int C_out, int dtype_in, void* d_packed,
                                   size_t packed_bytes, void* stream) {
    const size_t need = sc_conv_packed_bytes(K, C_in, C_out, dtype_in);
    if (need == 0 || d_weight == nullptr || d_packed == nullptr || !aligned16(d_weight) || !aligned16(d_packed))
        return SC_EINVAL;
    if (packed_bytes < need) return SC_ECAP;
    hipStream_t s = (hipStream_t)stream;
    const int K3 = K * K * K;
    if (dtype_in == SC_F32) {
        if (C_out > 256) return SC_EINVAL;
        return hipMemcpyAsync(d_packed, d_weight, (size_t)K3 * C_in * C_out * 4, hipMemcpyDeviceToDevice, s) == hipSuccess
                   ? SC_OK : SC_EHIP;
    }
    if (!mfma_channels_ok(C_in, C_out)) return SC_EINVAL;
    return pack_weights(K3, C_in, C_out, d_weight, d_packed, s);
}

extern "C" int sc_conv_up_fwd(const void* d_feat_coarse, int64_t n_map, const void* d_weight, void* d_feat_fine,
                              const void* d_kmap, size_t kmap_bytes, const sc_counts* d_counts, int K, int C_in,
                              int C_out, int dtype_in, int dtype_out, void* stream) {
    if (n_map < 0 || n_map > SC_N_MAX || K < 2 || K > 4 || C_in < 1 || C_out < 1) return SC_EINVAL;
    if (d_weight == nullptr || d_kmap == nullptr || d_counts == nullptr) return SC_EINVAL;
    if (n_map > 0 && (d_feat_coarse == nullptr || d_feat_fine == nullptr)) return SC_EINVAL;
    if (!aligned16(d_feat_coarse) || !aligned16(d_weight) || !aligned16(d_feat_fine) || !aligned16(d_kmap) ||
        !aligned16(d_counts))
        return SC_EINVAL;
    if (dtype_in != SC_F16 && dtype_in != SC_BF16) return SC_EINVAL;
    if (dtype_out != SC_F32 && dtype_out != dtype_in) return SC_EINVAL;
    if (kmap_bytes < sc_kmap_bytes(n_map, K, K, SC_STRIDED)) return SC_ECAP;
    const KmapLayout L = kmap_layout(sc_out_bound(n_map, K, K, SC_STRIDED), K, K, SC_STRIDED);
    if (L.tiles == 0) return SC_OK;
    MapSource ms{};
    ms.gmask = kmap_masked(SC_STRIDED, L.K3) ? (const uint32_t*)((const char*)d_kmap + L.off_mask) : nullptr;
    ms.nbr = (const int32_t*)((const char*)d_kmap + L.off_nbr);
    bool handled = false;
    // the kernel walks the coarse rows: counts->n_out of them, at most the map's bound
    const int rc = dtype_in == SC_F16
                       ? launch_up<SC_F16>(L.K3, C_in, C_out, L.tiles, (hipStream_t)stream, (const uint16_t*)d_feat_coarse,
                                           (const uint4*)d_weight, d_feat_fine, dtype_out == SC_F32 ? 1 : 0, ms,
                                           &d_counts->n_out, n_map, &handled)
                       : launch_up<SC_BF16>(L.K3, C_in, C_out, L.tiles, (hipStream_t)stream, (const uint16_t*)d_feat_coarse,
                                            (const uint4*)d_weight, d_feat_fine, dtype_out == SC_F32 ? 1 : 0, ms,
                                            &d_counts->n_out, n_map, &handled);
    if (rc != SC_OK) return rc;
    return handled ? SC_OK : SC_EINVAL;
}

extern "C" int sc_conv_fwd_grid(const void* d_feat_in, const int32_t* d_coords, int64_t n, const void* d_grid,
                                size_t grid_bytes, int32_t B, int32_t X, int32_t Y, int32_t Z, uint32_t epoch,
                                const void* d_weight, void* d_feat_out, int K, int C_in, int C_out, int dtype_in,
                                int dtype_out, void* d_workspace, size_t workspace_bytes, void* stream) {
    const size_t gneed = sc_grid_bytes(B, X, Y, Z);
    if (gneed == 0 || n < 0 || n > SC_N_MAX || epoch == 0 || K != 3) return SC_EINVAL;
    if (d_weight == nullptr || d_grid == nullptr) return SC_EINVAL;
    if (n > 0 && (d_feat_in == nullptr || d_feat_out == nullptr || d_coords == nullptr)) return SC_EINVAL;
    if (!aligned16(d_feat_in) || !aligned16(d_weight) || !aligned16(d_feat_out) || !aligned16(d_grid) ||
        !aligned16(d_coords) || !aligned16(d_workspace))
        return SC_EINVAL;
    if (dtype_in != SC_F16 && dtype_in != SC_BF16) return SC_EINVAL;
    if (dtype_out != SC_F32 && dtype_out != dtype_in) return SC_EINVAL;
    if (grid_bytes < gneed) return SC_ECAP;
    const size_t need = sc_conv_workspace_bytes(K, C_in, C_out, dtype_in);
    if (d_workspace == nullptr || workspace_bytes < need) return SC_ECAP;
    if (n == 0) return SC_OK;
    const MapSource ms{nullptr, nullptr, (const int4*)d_coords, (const unsigned long long*)d_grid, GridDims{B, X, Y, Z}, epoch, nullptr};
    if (!mfma_channels_ok(C_in, C_out)) return SC_EINVAL;
    return conv_16bit<1>(dtype_in, 27, 1, C_in, C_out, (n + TILE - 1) / TILE, (n + TILE - 1) / TILE, SUBMANIFOLD, two_sets((n + TILE - 1) / TILE, 27, C_out / 16, C_in, false, compute_units()), (hipStream_t)stream, d_feat_in,
                         d_weight, false, d_workspace, d_feat_out, dtype_out == SC_F32, ms, nullptr, n);
}
