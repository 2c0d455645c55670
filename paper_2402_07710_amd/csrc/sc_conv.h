// Definitions shared by the convolution kernels (sc_conv*.hip).
#pragma once

#include "sc_internal.h"

namespace sc {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Packed weights: W [K3][C_in][C_out] (16-bit elements) as MFMA A-operand tiles of W[k]^T.  A tile
// is 64 lanes x 16 bytes: lane l of tile (k, cb, ks) holds W[k][ks*32 + 8*(l/16) + j][cb*16 + l%16],
// j = 0..7.  Inside one offset k the tiles are ordered by 64-channel half of C_in first, then
// output block, then 32-channel slice of the half, so the tiles a kernel needs for one half of the
// input channels are one contiguous piece: tile number wtile(KS, CB, cb, ks) below (for C_in = 32
// there is one slice and the order is just cb).
__host__ __device__ constexpr int wtile(int KS, int CB, int cb, int ks) {
    return KS == 1 ? cb : ((ks >> 1) * CB + cb) * 2 + (ks & 1);
}
// Rows of the output: counted on the device (strided layers) or known to the caller, who then spares the kernel a round trip in
// front of everything else.
__device__ inline int64_t output_rows(const int64_t* __restrict__ counted, int64_t cap) {
    return counted != nullptr && *counted < cap ? *counted : cap;
}

// Group masks from a line of the offset table (lane = row of the tile): bit of each group that has a neighbour.  Maps of
// strided layers up to K^3 = 32 come without masks (MapSource::gmask null): the kernels read the lines anyway.
__device__ inline uint32_t line_pattern(int32_t entry) {
    const uint64_t vote = __ballot(entry >= 0);
    uint32_t pat = 0u;
#pragma unroll
    for (int g = 0; g < 4; ++g) pat |= (((vote >> (16 * g)) & 0xffffull) != 0ull ? 1u : 0u) << g;
    return pat;
}
// Words OR-ed over the 16 lanes that hold a group's rows (a row of the data-parallel instructions).
__device__ inline uint32_t or_of_group(uint32_t v) {
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true);      // rotated by 8, 4, 2 and 1 lanes
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x124, 0xf, 0xf, true);
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x122, 0xf, 0xf, true);
    v |= (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x121, 0xf, 0xf, true);
    return v;
}
// The mask word of a lane's group from its row's entries, of maps without masks: an instruction an offset shifts the sign in.
// Voting offset by offset (a compare and three scalar instructions each) was 0.3 us of a kernel.
template <int N>
__device__ inline uint32_t mask_of_entries(const int32_t (&e)[N]) {
    static_assert(N < 32, "bits of a word");
    uint32_t none = 0u;
#pragma unroll
    for (int k = N - 1; k >= 0; --k) none = __builtin_amdgcn_alignbit(none, (uint32_t)e[k], 31);
    return or_of_group(~none & ((1u << N) - 1u));
}
// Workgroup barrier for data exchanged through LDS only.  __syncthreads() also waits until every
// outstanding global load of the wavefront has returned (vmcnt(0)), which would drain the gathers
// and weight fetches that were issued ahead on purpose; here only the wavefront's LDS operations
// have to be complete before it arrives.
__device__ inline void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

template <int DT>
__device__ inline f32x4 mfma16x16x32(uint4 a, uint4 b, f32x4 c) {
    if constexpr (DT == SC_F16)
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

__device__ inline uint32_t f32_to_bf16_rne(float f) {
    uint32_t u = __builtin_bit_cast(uint32_t, f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;     // NaN stays NaN
    return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
template <int DT>
__device__ inline uint32_t pack2(float lo, float hi) {
    if constexpr (DT == SC_F16) {
        const _Float16 a = (_Float16)lo, b = (_Float16)hi;              // round to nearest even
        return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
    } else {
        return f32_to_bf16_rne(lo) | (f32_to_bf16_rne(hi) << 16);
    }
}

// Store one accumulator block: the lane holds channels cb*16 + 4*qq .. +3 of output row `row`.
template <int DT>
__device__ inline void store_acc(void* __restrict__ out, int out_f32, int64_t row, int C_out, int col, f32x4 d) {
    if (out_f32) {
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(out) + row * C_out + col) = make_float4(d[0], d[1], d[2], d[3]);
    } else {
        *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(out) + row * C_out + col) =
            make_uint2(pack2<DT>(d[0], d[1]), pack2<DT>(d[2], d[3]));
    }
}

// 16 bytes per lane from global memory straight into LDS: lane l's land at byte lds + 16 l.  The
// instruction takes its LDS address from M0 and needs one wait state after a write of it (s_nop).  Inline
// assembly, because the compiler would put a wait for all loads in front of every later LDS read.
__device__ inline void load_to_lds(const void* src, uint32_t lds) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds) : "m0", "memory");
}

// Large dynamic LDS has to be allowed per kernel, once on every device the kernel runs on: a flag
// per device (a repeated call would be harmless, so a race between host threads is too).
constexpr int MAX_DEVICES = 64;
inline int allow_lds(const void* fn, size_t lds, bool (&done)[MAX_DEVICES]) {
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return SC_EHIP;
    if (!done[dev]) {
        if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) return SC_EHIP;
        done[dev] = true;
    }
    return SC_OK;
}

// The general kernel (sc_conv_gather.hip): any K^3 <= 343, C_out a multiple of 16; 16-bit layers with C_in 32, 64,
// 128 or 256 and packed weights, fp32 layers with C_in 16, 32, 64, 128 or 256 and weights as they are.  `tiles` covers the
// caller's row capacity, `likely` is how many of them to expect (the input's, where the output count is known on the device only).
// `sets`: two sets of wavefronts (two_sets).
int launch_gather(int dtype_in, int K3, int mw, int C_in, int C_out, int64_t tiles, int64_t likely, LayerKind kind, bool sets, int cus, hipStream_t s, const void* feat,
                  const void* wp, void* out, int out_f32, const MapSource& ms, const int64_t* n_out_ptr, int64_t n_out_cap);
int launch_gather_fused(int dtype_in, int C_in, int C_out, int64_t tiles, bool sets, int cus, hipStream_t s, const void* feat, const void* wp,
                        void* out, int out_f32, const MapSource& ms, int64_t n);

}  // namespace sc
