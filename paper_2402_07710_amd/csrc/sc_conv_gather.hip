// The general 16-bit convolution kernel: every shape without a kernel of its own in sc_conv.hip
// (kernel sizes other than 3, 256 channels, unequal channel counts).
#include "sc_conv.h"

namespace sc {

// A row of zeros that stands in for "no neighbour": 512 bytes, up to 256 16-bit channels.
static __device__ __align__(512) uint4 g_zero_row[32];

// 16 bytes per lane from global memory straight into LDS: lane l's land at byte lds + 16 l.  The
// instruction takes its LDS address from M0, which nothing else on this target uses.  Inline
// assembly, because the compiler would put a wait for all loads in front of every later LDS read.
__device__ inline void load_to_lds(const void* src, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds) : "memory");
}

// One workgroup of four wavefronts per 64-row tile and block of output channels.  The sum over
// (offset, input channel) is walked in steps of SL 32-channel slices: one offset of 256 or 128 channels, 2
// of 64 or 4 of 32 per step, only the offsets at which the tile has a neighbour.
//  * The rows of the next step are gathered straight into the other half of a double LDS buffer
//    while this step multiplies, each wavefront fetching its 16-row group with eight (four at 32
//    channels) consecutive lanes on one row: whole lines, a quarter of the address cycles of a
//    gather in operand order.  The 16-byte pieces of a row are placed XOR-ed with the row number, so
//    the operand reads (16 rows x one piece) use all banks.
//  * The weight operands of the next step go from the packed tiles in global memory (whole lines,
//    the same for all tiles: cache hits) to a second set of registers.  A wavefront owns CT
//    16-channel output blocks, so no two wavefronts of a tile load the same weights unless the layer
//    has fewer than 64 output channels (then they split the rows: WR).
//  * One wait for everything and one barrier per step.
// Groups without a neighbour are skipped where an offset is at least four slices (KS >= 4); below that
// the test costs more than the multiplies: they read the row of zeros, and the places of the last
// step that have no offset are fetched like the others (of offset 0, rows of zeros) and not multiplied.
// Before (one wavefront per 16 rows, weights and rows loaded at their use): 14 k voxels 256 -> 256
// 555 us, 53 k voxels K = 5 32 -> 32 116 us.
template <int DT, int KS, int WR, int CT, int SL>
__global__ void __launch_bounds__(256, 2)
k_conv_gather(const uint16_t* feat, const uint4* wp, void* __restrict__ out, int out_f32, const uint32_t* __restrict__ gmask,
              const int32_t* __restrict__ nbr, int K3, int mw, int CB, const int64_t* __restrict__ n_out_ptr, int64_t n_out_cap) {
    constexpr int C_in = KS * 32;
    constexpr int OPS = SL / KS;                       // offsets per step
    constexpr int CH = KS == 1 ? 1 : KS / 2;           // chunks per offset: 64 rows x 64 (32) channels
    constexpr int CHB = KS == 1 ? 4096 : 8192;         // bytes per chunk
    constexpr int NI = KS == 1 ? 1 : 2;                // gather instructions per wavefront and chunk
    constexpr int STEP_BYTES = SL * 4096;
    constexpr int WC = 4 / WR, RG = 4 / WR;            // wavefronts across channels, 16-row groups per wavefront
    constexpr bool SKIP = KS >= 4;
    static_assert(SL % KS == 0, "a step is whole offsets");
    extern __shared__ __align__(16) char smem[];       // [2][STEP_BYTES]

    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, qq = lane >> 4;
    const int wr = wv / WC, cb0 = (int)blockIdx.y * (WC * CT) + (wv % WC) * CT;
    int64_t n_out = n_out_cap;
    if (*n_out_ptr < n_out) n_out = *n_out_ptr;
    const int64_t tile = xcd_unit_of(blockIdx.x, (n_out + TILE - 1) / TILE);
    if (tile < 0) return;                              // the whole workgroup

    // the offsets the tile takes part in, in increasing order: number and 4-bit pattern of groups.  The
    // tile's mask words are held by the lanes of one register.
    const uint32_t mvec = lane < 4 * mw ? gmask[tile * (4 * mw) + lane] : 0u;
    uint32_t mg[4] = {0u, 0u, 0u, 0u}, rest = 0u;
    int wi = -1;
    auto next_offset = [&](int& k, uint32_t& pat) __attribute__((always_inline)) {
        while (rest == 0u && wi + 1 < mw) {
            ++wi;
#pragma unroll
            for (int g = 0; g < 4; ++g) mg[g] = __builtin_amdgcn_readlane(mvec, g * mw + wi);
            rest = mg[0] | mg[1] | mg[2] | mg[3];
        }
        k = -1;
        pat = 0u;
        if (rest != 0u) {
            const int b = __builtin_ctz(rest);
            rest &= rest - 1u;
            k = wi * 32 + b;
#pragma unroll
            for (int g = 0; g < 4; ++g) pat |= ((mg[g] >> b) & 1u) << g;
        }
    };

    // gathers: this wavefront fetches group wv; its lane's row inside the group and 16-byte piece
    int grow[NI], gpiece;
    if constexpr (KS == 1) {
        const int logical = (lane & 7) ^ (lane >> 3);  // line = two 64-byte rows, slots XOR-ed with the line number
        grow[0] = (lane >> 3) * 2 + (logical >> 2);
        gpiece = logical & 3;
    } else {
#pragma unroll
        for (int i = 0; i < NI; ++i) grow[i] = i * 8 + (lane >> 3);
        gpiece = (lane & 7) ^ (lane >> 3);
    }
    const int32_t* line = nbr + tile * (int64_t)K3 * TILE + wv * 16;
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
                if (!SKIP || k[o] >= 0) ev[o][i] = line[(int64_t)(k[o] >= 0 ? k[o] : 0) * TILE + grow[i]];
    };
    auto gather = [&](const int (&k)[OPS], const uint32_t (&p)[OPS], int buf) {
#pragma unroll
        for (int o = 0; o < OPS; ++o) {
            if (!SKIP || ((p[o] >> wv) & 1u) != 0u) {
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    const char* src = (SKIP || k[o] >= 0) && ev[o][i] >= 0 ? fbase + (int64_t)ev[o][i] * (C_in * 2) : zbase;
#pragma unroll
                    for (int c = 0; c < CH; ++c)
                        load_to_lds(src + c * 128, __builtin_amdgcn_readfirstlane(lds_base + buf * STEP_BYTES + (o * CH + c) * CHB +
                                                                                  wv * (CHB / 4) + i * 1024));
                }
            }
        }
    };
    auto weights = [&](u32x4 (&a)[SL][CT], const int (&k)[OPS]) {
#pragma unroll
        for (int o = 0; o < OPS; ++o)
            if (!SKIP || k[o] >= 0) {
                const u32x4* wk = reinterpret_cast<const u32x4*>(wp) + (int64_t)(k[o] >= 0 ? k[o] : 0) * (CB * KS * 64) + lane;
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        const int cb = cb0 + ct < CB ? cb0 + ct : CB - 1;      // past the last block: not stored
                        a[o * KS + ks][ct] = wk[(KS == 1 ? cb : ((ks >> 1) * CB + cb) * 2 + (ks & 1)) * 64];
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
#pragma unroll
        for (int o = 0; o < OPS; ++o) {
            if (p[o] == 0u) continue;
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                const int gg = wr * RG + g;
                if (SKIP && ((p[o] >> gg) & 1u) == 0u) continue;
                const char* rows = smem + buf * STEP_BYTES + o * CH * CHB + gg * (CHB / 4);
                uint4 b[KS];
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) b[ks] = *reinterpret_cast<const uint4*>(rows + (ks >> 1) * CHB + ((ks & 1) ? op1 : op0));
#pragma unroll
                for (int ks = 0; ks < KS; ++ks)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        acc[g][ct] = mfma16x16x32<DT>(__builtin_bit_cast(uint4, a[o * KS + ks][ct]), b[ks], acc[g][ct]);
            }
        }
    };
    auto next_step = [&](int (&k)[OPS], uint32_t (&p)[OPS]) __attribute__((always_inline)) {
#pragma unroll
        for (int o = 0; o < OPS; ++o) next_offset(k[o], p[o]);
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
    weights(a0, k1);
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
        weights(a_next, k1);
        entries(k2);
        __builtin_amdgcn_sched_barrier(0);             // requested here, not next to their use
        compute(a, p0, buf);
        step_end();
    };
#pragma unroll 1
    while (p1[0] != 0u) {
        step(a0, a1, 0);
        if (p1[0] == 0u) break;
        step(a1, a0, 1);
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

template <int DT, int KS, int WR, int CT, int SL>
static int launch_gather_as(int K3, int mw, int CB, int64_t tiles, hipStream_t s, const uint16_t* feat, const uint4* wp, void* out,
                            int out_f32, const MapSource& ms, const int64_t* n_out_ptr, int64_t n_out_cap) {
    const unsigned blocks_y = (unsigned)((CB + 4 / WR * CT - 1) / (4 / WR * CT));
    SC_LAUNCH(KID_CONV_MFMA, (k_conv_gather<DT, KS, WR, CT, SL>), dim3(xcd_grid(tiles), blocks_y), dim3(256), 2 * SL * 4096, s, feat, wp,
              out, out_f32, ms.gmask, ms.nbr, K3, mw, CB, n_out_ptr, n_out_cap);
    return SC_OK;
}

template <int DT, int KS, int SL>
static int launch_gather_ks(int K3, int mw, int CB, int64_t tiles, int cus, hipStream_t s, const uint16_t* feat, const uint4* wp, void* out,
                            int out_f32, const MapSource& ms, const int64_t* n_out_ptr, int64_t n_out_cap) {
#define SC_GATHER(WR, CT) return launch_gather_as<DT, KS, WR, CT, SL>(K3, mw, CB, tiles, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap)
    if (CB == 1) SC_GATHER(4, 1);
    if (CB == 2) SC_GATHER(2, 1);
    // two output blocks per wavefront halve how often a tile's rows are gathered; one, where the
    // launch would otherwise leave CUs idle (256 input channels, 219 tiles: -> 128 29.0 us with one,
    // 34.2 with two; -> 256, twice the workgroups, 49.1 and 44.1)
    if (CB <= 4 || 2 * tiles * ((CB + 7) / 8) < 3 * (int64_t)cus) SC_GATHER(1, 1);
    SC_GATHER(1, 2);
#undef SC_GATHER
}

int launch_gather(int dtype_in, int K3, int mw, int C_in, int C_out, int64_t tiles, int cus, hipStream_t s, const uint16_t* feat,
                  const uint4* wp, void* out, int out_f32, const MapSource& ms, const int64_t* n_out_ptr, int64_t n_out_cap) {
    const int CB = C_out / 16;
    // slices per step: a whole offset at 256 channels; four elsewhere, where twice as many workgroups
    // per CU (32 KB of LDS each) are worth more than fewer barriers (53 k voxels K = 5 32 -> 32: 39.3 us,
    // with eight 44.6; 14 k voxels 128 -> 256: 25.2, 26.3)
#define SC_GATHER_KS(KS, SL)                                                                                                      \
    return dtype_in == SC_F16                                                                                                     \
               ? launch_gather_ks<SC_F16, KS, SL>(K3, mw, CB, tiles, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap)    \
               : launch_gather_ks<SC_BF16, KS, SL>(K3, mw, CB, tiles, cus, s, feat, wp, out, out_f32, ms, n_out_ptr, n_out_cap)
    switch (C_in) {
        case 32: SC_GATHER_KS(1, 4);
        case 64: SC_GATHER_KS(2, 4);
        case 128: SC_GATHER_KS(4, 4);
        case 256: SC_GATHER_KS(8, 8);
    }
#undef SC_GATHER_KS
    return SC_EINVAL;
}

}  // namespace sc
