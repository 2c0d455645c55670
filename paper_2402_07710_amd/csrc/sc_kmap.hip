// Offset table / kernel map (paper Section III-C.2 for submanifold layers, Section III-B
// eq. 1-5 and Section III-D for strided layers).
//
// The paper writes a dense N x K^3 table of neighbour rows (-1 where there is none) with one
// thread per point probing the location table K^3 times in a loop, and for strided layers counts
// the distinct output cells with an atomic exchange on a status table plus an atomic counter.
// Here the table is the same offset table, laid out for the matrix cores: outputs are cut into
// tiles of 64 rows, a tile stores its K^3 x 64 neighbour rows offset-major, and a bit per
// (16-row group, offset) records whether the group has any neighbour there, so the convolution
// only touches groups that exist.  Look-ups are issued many at a time (they are independent), not
// one after the other.  Strided layers number their output cells in order of first occurrence
// (min input row per cell + prefix sum), so the result does not depend on thread timing, unlike
// an atomic counter.  The plain per-offset pair lists are produced on demand (sc_kmap_export) by
// ballot + prefix-count compaction of the table.
#include <cstdlib>

#include "sc_internal.h"
#include "sc_rules.h"

namespace sc {

__device__ inline uint64_t lanemask_lt() { return (1ull << (threadIdx.x & 63)) - 1ull; }

__global__ void __launch_bounds__(64)
k_kmap_header(KmapHeader* hdr, KmapHeader value) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *hdr = value;
}

__global__ void __launch_bounds__(64)
k_set_n_out(sc_counts* counts, int64_t n_out) {
    if (threadIdx.x == 0 && blockIdx.x == 0) counts->n_out = n_out;
}

// Submanifold, K = 1 and 7: output row = input row.  One workgroup of WPT wavefronts per 64-row tile; lane =
// row, and the K^3 offsets are dealt to the wavefronts CH at a time.  The probes of a row do not
// depend on each other, so a wavefront issues the loads of its CH offsets together and afterwards
// re-probes only the offsets whose slot held another key: a tile's K^3 x 64 look-ups cost a few
// memory round trips instead of K^3.  Each wavefront then stores its offsets' 64 results as one
// 256-byte line of the tile and votes (ballot) on which 16-row groups have a neighbour.
template <int K, int WPT, int CH, int AT>
__global__ void __launch_bounds__(64 * WPT)
k_kmap_subm(const int4* __restrict__ coords, int64_t n, const uint4* __restrict__ slots,
            const TableHeader* __restrict__ th, uint32_t* __restrict__ gmask, int32_t* __restrict__ nbr,
            uint8_t* __restrict__ density, sc_counts* counts, KmapHeader* hdr, KmapHeader hdr_value) {
    constexpr int K3 = K * K * K, pad = (K - 1) / 2, centre = (K3 - 1) / 2;
    constexpr int PER_PASS = WPT * CH;
    constexpr int PASSES = (K3 + PER_PASS - 1) / PER_PASS;
    constexpr int MW = (K3 + 31) / 32;
    __shared__ uint32_t mask_s[4 * MW];

    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t tile = xcd_unit(blockIdx.x, gridDim.x);
    SC_MARK(0);
    if (tile * TILE >= n) return;                    // padding workgroup of the XCD-aware grid
    if (threadIdx.x < 4 * MW) mask_s[threadIdx.x] = 0u;
    const int64_t row = tile * TILE + lane;
    const bool valid = row < n;
    int4 c = make_int4(0, 0, 0, 0);
    if (valid) c = coords[row];
    const uint32_t mask = th->mask;
    const uint64_t tag = epoch_tag(th->epoch);       // slots of other epochs are free
    if (tile == 0 && threadIdx.x == 0) {
        counts->n_out = n;
        *hdr = hdr_value;
        fold_table_error(th, counts);
    }
    __syncthreads();

    auto neighbour_key = [&](int k, bool& inside) -> uint64_t {
        const int dx = k / (K * K) - pad, dy = (k / K) % K - pad, dz = k % K - pad;
        const int x = c.y + dx, y = c.z + dy, z = c.w + dz;
        inside = in_domain(x) && in_domain(y) && in_domain(z);
        return pack_key(c.x, x, y, z);
    };
    auto load_slot = [&](uint32_t slot) -> uint3 { return *reinterpret_cast<const uint3*>(&slots[slot]); };

    int32_t* tile_nbr = nbr + tile * (int64_t)(K3 * TILE);
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        const int k_base = (p * WPT + w) * CH;
        uint32_t pending = 0;          // bit u: offset k_base+u still has to be looked up
        int32_t found[CH];
        uint3 got[CH][AT];             // AT consecutive attempts of the probe sequence per round
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int k = k_base + u;
            bool inside;
            const uint64_t key = neighbour_key(k, inside);
            found[u] = -1;
            if (valid && k < K3) {
                if (k == centre) found[u] = (int32_t)row;                  // the centre is the row itself
                else if (inside) pending |= 1u << u;
            }
            // the first AT attempts of every offset at once (harmless loads where nothing is pending)
#pragma unroll
            for (int a = 0; a < AT; ++a) got[u][a] = load_slot(probe_slot(key, a, mask));
        }
        SC_MARK(1);
        for (uint32_t t = 0; __any(pending != 0); t += AT) {   // ends: every probe sequence reaches an empty slot
            if (t == AT) SC_MARK(2);
            if (t > 0) {
#pragma unroll
                for (int u = 0; u < CH; ++u) {
                    if (pending & (1u << u)) {
                        bool inside;
                        const uint64_t key = neighbour_key(k_base + u, inside);
#pragma unroll
                        for (int a = 0; a < AT; ++a) got[u][a] = load_slot(probe_slot(key, t + a, mask));
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < CH; ++u) {
                if (pending & (1u << u)) {
                    bool inside;
                    const uint64_t key = neighbour_key(k_base + u, inside);
#pragma unroll
                    for (int a = 0; a < AT; ++a) {
                        if (pending & (1u << u)) {
                            const uint64_t cur = (uint64_t)got[u][a].x | ((uint64_t)got[u][a].y << 32);
                            if (cur == (key | tag)) { found[u] = (int32_t)got[u][a].z; pending &= ~(1u << u); }
                            else if (!same_epoch(cur, tag)) pending &= ~(1u << u);
                        }
                    }
                }
            }
        }
        SC_MARK(3);
#pragma unroll
        for (int u = 0; u < CH; ++u) {
            const int k = k_base + u;
            if (k < K3) {
                tile_nbr[k * TILE + lane] = found[u];
                const uint64_t vote = __ballot(found[u] >= 0);
                if (lane < 4 && ((vote >> (16 * lane)) & 0xffffull) != 0) atomicOr(&mask_s[lane * MW + (k >> 5)], 1u << (k & 31));
            }
        }
    }
    __syncthreads();
    SC_MARK(4);
    if (threadIdx.x < 4 * MW) {
        const uint32_t word = mask_s[threadIdx.x];
        gmask[tile * (4 * MW) + threadIdx.x] = word;
        if (K > 1 && density != nullptr) {
            const uint8_t offsets = density_of<MW, K3>(word, mask_s);
            if (threadIdx.x == 0) density[tile] = offsets;
        }
    }
    SC_MARK(5);
}

// K = 3 and 5, the same tile layout with far fewer instructions.  The kernel above hashes every one of
// a row's K^3 keys from scratch; at about 155 vector instructions per look-up, many of them quarter-rate
// multiplies, issuing them took 81 % of its cycles (300 k voxels).  The K cells of an axis lie in at
// most two blocks of four, so here a wavefront takes one x offset of a tile and forms four block hashes
// per attempt; a look-up is then a select, a few bit operations for its place and a comparison.  What
// bounds it now is the address unit (a random slot per lane and look-up) and the table's lines from L2.
// 10^6 indoor voxels: 104 -> 75 us; sweeps of 110 k: 15.6 -> 13.7, 261 k: 37.7 -> 35.0, 53 k with K = 5:
// 28.2 -> 24.0, 6 k with K = 5: 12 -> 8.4.  All five y offsets of K = 5 at once spill or leave room for
// too few wavefronts (35 us).
// Tiles to the XCDs: contiguous eighths, or runs of MAP_RUN (map_in_runs; of 4 and 64 tiles at 262 k rows 34.4 and 35.5 us against 34.3
// with 16, at 10^6 78.0 and 73.5 against 74.4).
constexpr int MAP_RUN = 16;
template <int K, int YG, int YB, int RUNS>             // YG wavefronts share an x offset's y offsets, each takes YB of its at a time
__global__ void __launch_bounds__(64 * K * YG)
k_kmap_subm_blocks(const int4* __restrict__ coords, int64_t n, const uint4* __restrict__ slots, const TableHeader* __restrict__ th,
                   uint32_t* __restrict__ gmask, int32_t* __restrict__ nbr, uint8_t* __restrict__ density, sc_counts* counts, KmapHeader* hdr,
                   KmapHeader hdr_value) {
    static_assert(K == 3 || K == 5, "K cells in a row lie in at most two blocks of four");
    constexpr int K3 = K * K * K, pad = (K - 1) / 2, MW = (K3 + 31) / 32, YC = (K + YG - 1) / YG, U = YB * K;
    static_assert(YC % YB == 0, "the passes of a wavefront are whole");
    __shared__ uint32_t mask_s[4 * MW];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int w = wave % K, dy_first = wave / K * YC;
    const int64_t tile = RUNS ? xcd_run_of<MAP_RUN>(blockIdx.x, (n + TILE - 1) / TILE) : xcd_unit(blockIdx.x, gridDim.x);
    if (tile < 0 || tile * TILE >= n) return;                              // padding workgroup of the XCD-aware grid
    if (threadIdx.x < 4 * MW) mask_s[threadIdx.x] = 0u;
    const int64_t row = tile * TILE + lane;
    const bool valid = row < n;
    int4 c = make_int4(0, 0, 0, 0);
    if (valid) c = coords[row];
    const uint32_t mask = th->mask, tag = th->epoch << 24;             // slots of other epochs are free
    if (tile == 0 && threadIdx.x == 0) {
        counts->n_out = n;
        *hdr = hdr_value;
        fold_table_error(th, counts);
    }
    __syncthreads();

    const int x = c.y + w - pad;
    const bool x_ok = valid && in_domain(x);
    const uint32_t hi = ((uint32_t)c.x << 16) | (uint32_t)x, want_hi = hi | tag, lx = local_x((uint32_t)x);
    // the two blocks of an axis: that of the first and that of the last cell
    const uint32_t y0 = (uint32_t)(c.z - pad) & ~3u, y1 = (uint32_t)(c.z + pad) & ~3u;
    const uint32_t z0 = (uint32_t)(c.w - pad) & ~3u, z1 = (uint32_t)(c.w + pad) & ~3u;
    const uint32_t px = (hi & ~3u) * BLOCK_MUL_HI, py0 = (y0 << 16) * BLOCK_MUL_LO, py1 = (y1 << 16) * BLOCK_MUL_LO;
    const uint32_t pz0 = z0 * BLOCK_MUL_LO, pz1 = z1 * BLOCK_MUL_LO;
    const uint32_t base[2][2] = {{px ^ (py0 + pz0), px ^ (py0 + pz1)}, {px ^ (py1 + pz0), px ^ (py1 + pz1)}};

    uint32_t bits[4] = {0u, 0u, 0u, 0u};               // this wavefront's bits of the four groups
#pragma unroll 1
    for (int pass = 0; pass < YC / YB; ++pass) {
        const int dy0 = dy_first + pass * YB;
        if (dy0 >= K) break;
        uint3 got[U];
        bool pending[U];
        int32_t found[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int dy = dy0 + u / K, dz = u % K;
            const bool centre = w == pad && dy == pad && dz == pad;
            found[u] = centre && valid ? (int32_t)row : -1;                      // the centre is the row itself
            pending[u] = dy < K && !centre && x_ok && in_domain(c.z + dy - pad) && in_domain(c.w + dz - pad);
        }
        bool any = true;
        for (uint32_t t = 0; any; ++t) {                   // ends: every probe sequence reaches a free slot
            const uint32_t tt = t < REHASH_MAX ? t : REHASH_MAX - 1;
            uint32_t h[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) h[i][j] = block_mix(base[i][j], tt);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int dy = dy0 + u / K, dz = u % K;
                if (t == 0 || pending[u]) {                // a look-up outside the domain reads a slot and ignores it
                    const uint32_t y = (uint32_t)(c.z + dy - pad), z = (uint32_t)(c.w + dz - pad);
                    const bool first_y = (y & ~3u) == y0, first_z = dz == 0 || (dz < K - 1 && (z & ~3u) == z0);
                    const uint32_t hh = first_z ? (first_y ? h[0][0] : h[1][0]) : (first_y ? h[0][1] : h[1][1]);
                    const uint32_t slot = (region_slot(hh, lx | local_y(y) | local_z(z)) + (t - tt)) & mask;
                    got[u] = *reinterpret_cast<const uint3*>(&slots[slot]);
                }
            }
            any = false;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int dy = dy0 + u / K, dz = u % K;
                const uint32_t want_lo = ((uint32_t)(c.z + dy - pad) << 16) | (uint32_t)(c.w + dz - pad);
                const bool hit = got[u].x == want_lo && got[u].y == want_hi, free_slot = ((got[u].y ^ tag) >> 24) != 0u;
                if (pending[u] && hit) found[u] = (int32_t)got[u].z;
                pending[u] = pending[u] && !hit && !free_slot;
                any = any || pending[u];
            }
            any = __any(any);
        }
        int32_t* lines = nbr + tile * (int64_t)(K3 * TILE) + (int64_t)(w * K + dy0) * (K * TILE) + lane;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (dy0 + u / K < K) {
                lines[u * TILE] = found[u];
                const uint64_t vote = __ballot(found[u] >= 0);
#pragma unroll
                for (int g = 0; g < 4; ++g) bits[g] |= ((vote >> (16 * g)) & 0xffffull) != 0ull ? 1u << ((pass * YB * K) + u) : 0u;
            }
    }
    // they start at bit (w K + dy_first) K of the tile's masks
    const int at = (w * K + dy_first) * K;
    if (lane < 4) {
        const uint32_t b = lane == 0 ? bits[0] : lane == 1 ? bits[1] : lane == 2 ? bits[2] : bits[3];
        const uint64_t placed = (uint64_t)b << (at & 31);
        atomicOr(&mask_s[lane * MW + (at >> 5)], (uint32_t)placed);
        if (MW > 1 && (uint32_t)(placed >> 32) != 0u) atomicOr(&mask_s[lane * MW + (at >> 5) + 1], (uint32_t)(placed >> 32));
    }
    __syncthreads();
    if (threadIdx.x < 4 * MW) {
        const uint32_t word = mask_s[threadIdx.x];
        gmask[tile * (4 * MW) + threadIdx.x] = word;
        if (density != nullptr) {
            const uint8_t offsets = density_of<MW, K3>(word, mask_s);
            if (threadIdx.x == 0) density[tile] = offsets;
        }
    }
}

// ---- strided layers ----------------------------------------------------------------------------
// An input p pairs with output cell q at offset d whenever p = q*s + d, d in [0,K)^3 (eq. 1-5 for K ==
// stride, in general the enumeration of Algorithm 1's getOutputCoord with no padding), so it belongs to
// one cell if K == stride and to up to MAXC = ceil(K/s)^3 cells otherwise.  Its valid (offset, cell)
// candidates are numbered j = 0.. in ascending offset order; candidate id c = i*MAXC + j therefore
// orders all candidates by input row and then by offset, and a cell's number is the rank of its lowest
// candidate id among all cells' lowest ids.
// scratch: output-cell table (lowest candidate id of the cell), the candidates' slots, flag words,
// in-block word prefix, block sums / prefixes.
struct StridedScratch {
    int32_t* oslots;         // output-cell table: smallest candidate id of the cell, or CELL_EMPTY
    uint32_t omask;
    int32_t* slot_of;        // [n]
    uint64_t* flagword;      // [ceil(n/64)]  bit i%64 set iff candidate i is the first of its cell
    int32_t* word_prefix;    // [ceil(n/64)]  flags before this word inside its 1024-block
    int32_t* block_sum;      // [nblk]
    int32_t* block_prefix;   // [nblk]
    int32_t* cells;          // [CELL_COUNTERS x 32] distinct output cells claimed so far, one 128-byte line per counter
    size_t bytes;
};
constexpr int CELL_COUNTERS = 64;
constexpr int32_t CELL_EMPTY = 0x7fffffff;
// n = candidates; slots_per_key sizes the output-cell table: 8 where every input is a distinct cell at
// worst (K == stride), 2 for longer candidate lists, whose n is a bound that real voxel sets stay far below
inline StridedScratch strided_scratch(void* p, int64_t n, uint64_t slots_per_key) {
    StridedScratch s;
    const uint64_t cap = hash_capacity(n, slots_per_key);
    const int64_t words = (n + 63) / 64, nblk = (n + 1023) / 1024;
    size_t off = 0;
    char* b = (char*)p;
    // 16 bytes of room per slot, of which the build touches 4: the size of the scratch buffer, and with it which sets
    // sc_kmap_build_noalloc refuses, is what callers were promised when a slot held the cell's key too
    s.oslots = (int32_t*)(b + off); off = align_up(off + cap * 16, 256);
    s.omask = (uint32_t)(cap - 1);
    s.slot_of = (int32_t*)(b + off); off = align_up(off + (size_t)n * 4, 256);
    s.flagword = (uint64_t*)(b + off); off = align_up(off + (size_t)words * 8, 256);
    s.word_prefix = (int32_t*)(b + off); off = align_up(off + (size_t)words * 4, 256);
    s.block_sum = (int32_t*)(b + off); off = align_up(off + (size_t)nblk * 4, 256);
    s.block_prefix = (int32_t*)(b + off); off = align_up(off + (size_t)nblk * 4, 256);
    s.cells = (int32_t*)(b + off); off = align_up(off + (size_t)CELL_COUNTERS * 128, 256);
    s.bytes = off + 256;
    return s;
}

// Prepares a strided build: output-cell table <- empty, claim counters <- 0; short builds: flag words <- 0, offset table <- -1.
__global__ void __launch_bounds__(256)
k_strided_fill(int4* __restrict__ oslots4, uint64_t cap, int32_t* __restrict__ cells, uint64_t* __restrict__ flagword, int64_t words,
               int4* __restrict__ nbr16, int64_t nbr_vec, sc_counts* counts, int reset, int64_t n_in, const TableHeader* th) {
    const int64_t nthr = (int64_t)gridDim.x * blockDim.x;
    const int64_t tid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (reset && blockIdx.x == 0) {                  // a build without a location table starts the counts block itself
        int32_t* w = reinterpret_cast<int32_t*>(counts);
        for (int i = threadIdx.x; i < (int)(sizeof(sc_counts) / 4); i += blockDim.x) w[i] = 0;
        __syncthreads();
        if (threadIdx.x == 0) counts->n_in = n_in;
    }
    // after a location-table build that could not report into the counts block, report for it
    if (th != nullptr && tid == 0) fold_table_error(th, counts);
    if (cells != nullptr && tid < CELL_COUNTERS) cells[tid * 32] = 0;
    for (int64_t i = tid; i < (int64_t)(cap / 4); i += nthr) oslots4[i] = make_int4(CELL_EMPTY, CELL_EMPTY, CELL_EMPTY, CELL_EMPTY);
    for (int64_t i = tid; i < words; i += nthr) flagword[i] = 0ull;
    for (int64_t i = tid; i < nbr_vec; i += nthr) nbr16[i] = make_int4(-1, -1, -1, -1);
}

// Candidate j of the input at c, or k < 0 if it has fewer.  Along one axis the offsets that can
// pair coordinate p with a cell are d = p mod s, p mod s + s, ... below K and not above p (the
// cell coordinate (p - d)/s must not be negative); candidates are numbered with x slowest and z
// fastest, offsets ascending, i.e. in ascending order of the offset number k.
struct Candidate {
    int k;                 // offset number, -1: no such candidate
    int qx, qy, qz;        // the output cell
};
__device__ inline int axis_options(int p, int K, int s) {
    const int top = p < K - 1 ? p : K - 1;
    return (top - p % s) / s + 1;                  // p mod s <= top always: s <= K and p mod s <= p
}
__device__ inline Candidate candidate(const int4 c, int K, int s, int j) {
    const int cy = axis_options(c.z, K, s), cz = axis_options(c.w, K, s), cx = axis_options(c.y, K, s);
    Candidate r;
    r.k = -1; r.qx = r.qy = r.qz = 0;
    if (j >= cx * cy * cz) return r;
    const int dz = c.w % s + (j % cz) * s, dy = c.z % s + ((j / cz) % cy) * s, dx = c.y % s + (j / (cz * cy)) * s;
    r.k = (dx * K + dy) * K + dz;
    r.qx = (c.y - dx) / s; r.qy = (c.z - dy) / s; r.qz = (c.w - dz) / s;
    return r;
}

// Kernel size, stride and candidates per input of a strided layer.  The common shapes are compiled in: the
// enumeration above is a dozen integer divisions, each ~40 instructions when the divisor is not a constant.
template <int KT, int ST>
struct StridedShape {
    static constexpr int MT = ST ? ((KT + ST - 1) / ST) * ((KT + ST - 1) / ST) * ((KT + ST - 1) / ST) : 0;
    int k_, s_, m_;
    __device__ int K() const { return KT ? KT : k_; }
    __device__ int s() const { return ST ? ST : s_; }
    __device__ int maxc() const { return MT ? MT : m_; }
};

// The cell of candidate `id` (input id / maxc, its candidate id % maxc), as a key.
template <class Shape>
__device__ inline uint64_t candidate_key(const int4* __restrict__ coords, const Shape& sh, int32_t id) {
    const int4 c = coords[(uint32_t)id / (uint32_t)sh.maxc()];
    const Candidate q = candidate(c, sh.K(), sh.s(), (uint32_t)id % (uint32_t)sh.maxc());
    return pack_key(c.x, q.qx, q.qy, q.qz);
}

// Claim (or find) the slot of output cell `key` for candidate `id`; returns the slot, or -1 if the table is
// full.  `fresh`: this call claimed it; `ousted`: the id that stood there until this call's smaller one took its place, or -1.  A slot is one word, the smallest id seen of its cell: which cell
// that is follows from the id's coordinates, so claiming a cell is a single compare-and-swap.  It is not preceded by a read: most entries that
// come here, merged by workgroup, are their cell's first, and for them that was a round trip more (us of whole layers on sweeps, with the read and without:
// K = 3, stride 2 2 k / 53 k / 120 k / 200 k 21.9 / 38.8 / 63.5 / 92.0 and 21.2 / 37.8 / 61.6 / 88.6, K = 2 10 k / 200 k 16.3 / 30.0 and 15.6 / 28.9; indoor 200 k 73.9 and 72.2;
// builds alone, sweep 53 k, indoor 53 k and random 20 k: K = 4, stride 2 44.8, 38.6, 49.3 and 44.2, 37.2, 47.9; K = 5, stride 2 80.2, 82.2, 77.4 and 79.9, 78.9, 76.9, stride 3 43.6, 42.6, 47.6 and 43.0, 41.4, 45.6;
// K = 7, stride 2 198, 194, 306 and 197, 175, 306, stride 3 93.9, 102, 87.6 and 93.7, 96.0, 86.8).
template <class Shape>
__device__ inline int32_t claim_cell(int32_t* oslots, uint32_t omask, const int4* __restrict__ coords, const Shape& sh, uint64_t key,
                                     int32_t id, bool& fresh, int32_t& ousted) {
    fresh = false;
    ousted = -1;
    for (uint32_t t = 0; t <= omask + REHASH_MAX; ++t) {
        const uint32_t slot = probe_slot(key, t, omask);
        const int32_t cur = atomicCAS(&oslots[slot], CELL_EMPTY, id);
        if (cur == CELL_EMPTY) {
            fresh = true;
            return (int32_t)slot;
        }
        if (candidate_key(coords, sh, cur) == key) {
            if (id < cur) {
                const int32_t old = atomicMin(&oslots[slot], id);
                if (id < old) ousted = old;
            }
            return (int32_t)slot;
        }
    }
    return -1;
}

// The same for a workgroup's entries at once.  What claiming costs is the rate of global atomics
// (~20 per ns on the whole chip), and entries that are close in order mostly share cells: the workgroup's
// cells are first merged in LDS (key and smallest id; LDS atomics), and only distinct ones go to the table.
// With
// a compare-and-swap on the key and a minimum on the id per entry, 53 k rows took 18.0 us (K = 3, stride
// 2) and 8.5 us (K = 2), 200 k rows 51.8 and 21.0; now 9.7, 7.1, 21.0 and 10.5.  `key` is KEY_EMPTY for a thread without an entry; ids rise
// with the thread.  Returns the thread's slot, -1 if it has none or the table is full (l.full is then set);
// l.fresh counts the cells this workgroup claimed first.
// FLAGS: the bits of the ids that stand in the table, in flag words that start out zero: an id's bit is turned when it comes and
// when a smaller one takes its place.  Turns commute, so the words are right when the last workgroup is done, and who comes
// sets only bits of the workgroup's own ids, gathered in LDS.
constexpr int CLAIM_WG = 256;                          // with 1024 the fixed part (barriers, few workgroups) outweighs the merging: 10.6 us
struct ClaimLds {
    static constexpr int SLOTS = 2 * CLAIM_WG;              // at most half full
    unsigned long long key[SLOTS];
    int32_t id[SLOTS];                                 // smallest id, later the slot in the global table
    int32_t fresh, full;
    uint32_t flags[CLAIM_WG / 32];
};
template <int FLAGS, class Shape>
__device__ inline int32_t claim_cells_of_workgroup(ClaimLds& l, int32_t* oslots, uint32_t omask, const int4* __restrict__ coords,
                                                   const Shape& sh, uint64_t key, int32_t id, uint32_t* flags) {
    constexpr int SLOTS = ClaimLds::SLOTS;
#pragma unroll
    for (int i = 0; i < SLOTS / CLAIM_WG; ++i) {
        l.key[i * CLAIM_WG + threadIdx.x] = KEY_EMPTY;
        l.id[i * CLAIM_WG + threadIdx.x] = CELL_EMPTY;
    }
    if (threadIdx.x == 0) l.fresh = l.full = 0;
    if (FLAGS && threadIdx.x < CLAIM_WG / 32) l.flags[threadIdx.x] = 0u;
    __syncthreads();
    int at = -1;
    bool owner = false;                                // the thread that brought the key in claims the cell
    if (key != KEY_EMPTY) {
        uint32_t e = mix_block((uint32_t)(key >> 32), (uint32_t)key, 0) % SLOTS;
        for (;;) {                                     // ends: at most one key per thread, twice as many slots
            const uint64_t cur = atomicCAS(&l.key[e], (unsigned long long)KEY_EMPTY, (unsigned long long)key);
            owner = cur == KEY_EMPTY;
            if (owner || cur == key) break;
            e = (e + 1) % SLOTS;
        }
        atomicMin(&l.id[e], id);
        at = (int)e;
    }
    __syncthreads();
    bool fresh = false;
    if (owner) {
        const int32_t first = l.id[at];
        int32_t ousted;
        const int32_t slot = claim_cell(oslots, omask, coords, sh, key, first, fresh, ousted);
        if (slot < 0) l.full = 1;
        if (FLAGS && (fresh || ousted >= 0)) atomicXor(&l.flags[(uint32_t)first % CLAIM_WG / 32], 1u << ((uint32_t)first % 32));
        if (FLAGS && ousted >= 0) atomicXor(&flags[(uint32_t)ousted / 32], 1u << ((uint32_t)ousted % 32));
        l.id[at] = slot;
    }
    const uint64_t vote = __ballot(fresh);
    if ((threadIdx.x & 63) == 0 && vote != 0ull) atomicAdd(&l.fresh, __popcll(vote));
    __syncthreads();
    if (FLAGS && threadIdx.x < CLAIM_WG / 32 && l.flags[threadIdx.x] != 0u)
        atomicXor(&flags[(size_t)blockIdx.x * (CLAIM_WG / 32) + threadIdx.x], l.flags[threadIdx.x]);
    return at >= 0 ? l.id[at] : -1;
}

// One thread per candidate (input i = id / maxc, candidate j = id % maxc; one per input for K == stride: the
// cell floor(p/s) of eq. 2, eq. 4): the inputs' candidates are independent, and with a thread each their
// claims are all in flight together.
template <int FLAGS, class Shape>
__global__ void __launch_bounds__(CLAIM_WG)
k_strided_insert(const int4* __restrict__ coords, int64_t n, Shape sh, int32_t* oslots, uint32_t omask, int32_t* __restrict__ cand_slot,
                 int32_t* __restrict__ cells, uint32_t* flags, sc_counts* counts) {
    __shared__ ClaimLds l;
    const int64_t id = (int64_t)blockIdx.x * CLAIM_WG + threadIdx.x, nc = n * sh.maxc();
    uint64_t key = KEY_EMPTY;
    if (id < nc) {
        const uint32_t i = (uint32_t)id / (uint32_t)sh.maxc();         // candidate ids stay below 2^26
        const int j = (int)((uint32_t)id - i * (uint32_t)sh.maxc());
        const int4 c = coords[i];
        if (!in_domain4(c.x, c.y, c.z, c.w)) {
            if (j == 0) latch_status(counts, SC_ERANGE);
        } else {
            const Candidate q = candidate(c, sh.K(), sh.s(), j);
            if (q.k >= 0) key = pack_key(c.x, q.qx, q.qy, q.qz);
        }
    }
    const int32_t slot = claim_cells_of_workgroup<FLAGS>(l, oslots, omask, coords, sh, key, (int32_t)id, flags);
    if (id < nc) cand_slot[id] = slot;
    if (threadIdx.x == 0) {
        if (l.full) latch_status(counts, SC_EFULL);
        // how many cells there are, before they are numbered: the next kernel clears that many table rows
        if (!FLAGS && l.fresh != 0) atomicAdd(&cells[(blockIdx.x % CELL_COUNTERS) * 32], l.fresh);
    }
}

// flag(c) = candidate c is the first (lowest id) of its cell; one bit per candidate, plus the exclusive
// prefix of the flag counts of the words of each block of U x 1024 candidates.  Also clears the offset
// table.  U = 4 for long lists: every workgroup of the pairs kernel scans the block counts for itself.
template <int U>
__global__ void __launch_bounds__(1024)
k_strided_flags(int64_t n, const int32_t* __restrict__ slot_of, const int32_t* __restrict__ oslots, uint64_t* __restrict__ flagword,
                int32_t* __restrict__ word_prefix, int32_t* __restrict__ block_sum, const int32_t* __restrict__ cells,
                int4* __restrict__ nbr16, int K3) {
    __shared__ int32_t count_s[16 * U], total_s;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint64_t vote[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t c = ((int64_t)blockIdx.x * U + u) * 1024 + threadIdx.x;
        bool first = false;
        if (c < n) {
            const int32_t sl = slot_of[c];
            first = sl >= 0 && oslots[sl] == (int32_t)c;
        }
        vote[u] = __ballot(first);
        if (lane == 0) count_s[u * 16 + wave] = __popcll(vote[u]);
    }
    if (wave == 0) {
        int32_t v = cells[lane * 32];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
        if (lane == 0) total_s = v;
    }
    __syncthreads();
    if (lane == 0) {
        int32_t before = 0;
        int w = 0;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            for (; w < u * 16 + wave; ++w) before += count_s[w];
            const int64_t word = ((int64_t)blockIdx.x * U + u) * 16 + wave;
            if (word * 64 < n) {
                flagword[word] = vote[u];
                word_prefix[word] = before;
            }
        }
        if (wave == 15) block_sum[blockIdx.x] = before + count_s[16 * U - 1];
    }
    // offset table <- -1 for the tiles of the output rows, which the insert kernel counted: the bound is
    // ceil(K/s)^3 rows per input, real sets need about one
    const int64_t vec = ((int64_t)total_s + TILE - 1) / TILE * K3 * (TILE / 4), nthr = (int64_t)gridDim.x * 1024;
    for (int64_t v = (int64_t)blockIdx.x * 1024 + threadIdx.x; v < vec; v += nthr) nbr16[v] = make_int4(-1, -1, -1, -1);
}
static_assert(CELL_COUNTERS == 64, "one lane per counter");

// Exclusive prefix of the block sums (one workgroup walks the array), total -> counts->n_out.
__global__ void __launch_bounds__(1024)
k_scan_blocks(const int32_t* __restrict__ block_sum, int32_t* __restrict__ block_prefix, int64_t nblk,
              sc_counts* counts) {
    __shared__ int32_t part[1024];
    __shared__ int32_t carry_s;
    if (threadIdx.x == 0) carry_s = 0;
    __syncthreads();
    for (int64_t base = 0; base < nblk; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const int32_t v = i < nblk ? block_sum[i] : 0;
        part[threadIdx.x] = v;
        __syncthreads();
        for (int off = 1; off < 1024; off <<= 1) {           // Hillis-Steele inclusive scan
            int32_t add = threadIdx.x >= (unsigned)off ? part[threadIdx.x - off] : 0;
            __syncthreads();
            part[threadIdx.x] += add;
            __syncthreads();
        }
        const int32_t carry = carry_s;
        if (i < nblk) block_prefix[i] = carry + part[threadIdx.x] - v;
        __syncthreads();
        if (threadIdx.x == 1023) carry_s = carry + part[1023];
        __syncthreads();
    }
    if (threadIdx.x == 0) counts->n_out = carry_s;
}

// Exclusive prefix of the per-block counts, computed by every workgroup for itself into LDS (the
// counts of up to a thousand blocks: cheaper than a kernel of its own,
// which is one workgroup long).  Returns the total.  All threads of the workgroup call it.
constexpr int SCAN_IN_PAIRS_MAX = 1024;              // blocks (4 M candidates); more: k_scan_blocks
__device__ inline int32_t block_prefix_to_lds(const int32_t* __restrict__ block_sum, int nblk, int32_t* prefix_s,
                                              int32_t* wave_s) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwaves = blockDim.x >> 6;
    const int per = (nblk + (int)blockDim.x - 1) / (int)blockDim.x;
    const int lo = threadIdx.x * per, hi = lo + per < nblk ? lo + per : nblk;
    int32_t sum = 0;
    for (int i = lo; i < hi; ++i) sum += block_sum[i];
    int32_t incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) wave_s[wave] = incl;
    __syncthreads();
    int32_t before = 0, total = 0;
    for (int w = 0; w < nwaves; ++w) {
        if (w < wave) before += wave_s[w];
        total += wave_s[w];
    }
    int32_t run = before + incl - sum;
    for (int i = lo; i < hi; ++i) {
        prefix_s[i] = run;
        run += block_sum[i];
    }
    __syncthreads();
    return total;
}

// Every candidate finds its output row (rank of its cell's first candidate among all first candidates),
// and its input's row goes to that row's entry at the candidate's offset (K == stride: in-cell offset,
// eq. 3, kernel offset, eq. 5).
// SCAN: the prefix of the block counts is made here (block_prefix is then unused) and workgroup 0
// writes the number of output rows.
template <int SCAN, int U, class Shape>
__global__ void __launch_bounds__(256)
k_strided_pairs(const int4* __restrict__ coords, int64_t n, Shape sh, const int32_t* __restrict__ cand_slot,
                const int32_t* __restrict__ oslots, const uint64_t* __restrict__ flagword, const int32_t* __restrict__ word_prefix,
                const int32_t* __restrict__ block_prefix, const int32_t* __restrict__ block_sum, int nblk, int32_t* __restrict__ nbr,
                uint32_t* __restrict__ parent, int4* __restrict__ out_coords, sc_counts* counts, KmapHeader* hdr, KmapHeader hdr_value) {
    __shared__ int32_t prefix_s[SCAN ? SCAN_IN_PAIRS_MAX : 1];
    __shared__ int32_t wave_s[4];
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id == 0) *hdr = hdr_value;
    if constexpr (SCAN) {
        const int32_t total = block_prefix_to_lds(block_sum, nblk, prefix_s, wave_s);
        if (id == 0) counts->n_out = total;
        block_prefix = prefix_s;
    }
    if (id >= n * sh.maxc()) return;
    const int32_t sl = cand_slot[id];
    if (sl < 0) {
        if (parent != nullptr) parent[id] = ~0u;
        return;
    }
    const uint32_t i = (uint32_t)id / (uint32_t)sh.maxc();
    const int4 c = coords[i];
    const int32_t r = oslots[sl];                              // the cell's first candidate
    const Candidate q = candidate(c, sh.K(), sh.s(), (int)((uint32_t)id - i * (uint32_t)sh.maxc()));
    const int32_t o = block_prefix[r >> (U == 4 ? 12 : 10)] + word_prefix[r >> 6] +
                      __popcll(flagword[r >> 6] & ((1ull << (r & 63)) - 1ull));
    // one input per (output row, offset): a plain store is enough; repeated input coordinates are the
    // location table's business (sc_hash_build latches SC_EDUP)
    nbr[((int64_t)(o >> 6) * (sh.K() * sh.K() * sh.K()) + q.k) * TILE + (o & 63)] = (int32_t)i;
    if (parent != nullptr) parent[id] = (uint32_t)o << 6 | (uint32_t)q.k;      // one candidate per input: id is its row
    if (r == (int32_t)id) out_coords[o] = make_int4(c.x, q.qx, q.qy, q.qz);
}

// The same for short builds with one candidate per input (K == stride), whose flag words the insert kernel has made: every
// workgroup counts all words for itself, and there is no kernel between claiming and numbering (a launch of 4 us; whole layers K = 2
// 32 -> 64, 2 k / 10 k / 53 k / 200 k voxels 18.3 / 19.7 / 22.6 / 32.6 -> 16.0 / 17.2 / 20.1 / 30.3 us).  Words and counts of the largest set that comes here are 48 KB of LDS.
template <class Shape>
__global__ void __launch_bounds__(1024)
k_strided_pairs_short(const int4* __restrict__ coords, int n, Shape sh, const int32_t* __restrict__ cand_slot, const int32_t* __restrict__ oslots,
                      const uint64_t* __restrict__ flagword, int32_t* __restrict__ nbr, uint32_t* __restrict__ parent, int4* __restrict__ out_coords,
                      sc_counts* counts, KmapHeader* hdr, KmapHeader hdr_value) {
    __shared__ uint64_t word_s[SHORT_WORDS];
    __shared__ int32_t before_s[SHORT_WORDS], wave_s[16];
    const int id = (int)(blockIdx.x * 1024 + threadIdx.x), lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (id == 0) *hdr = hdr_value;
    // what does not need the words is requested before their barriers
    const int32_t sl = id < n ? cand_slot[id] : -1;
    int4 c = make_int4(0, 0, 0, 0);
    int32_t r = 0;                                             // the cell's first input
    if (sl >= 0) {
        c = coords[id];
        r = oslots[sl];
    }
    constexpr int PER = SHORT_WORDS / 1024;
    const int words = (n + 63) / 64;
    uint64_t word[PER];
    int32_t mine = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int w = threadIdx.x * PER + u;
        word[u] = w < words ? flagword[w] : 0ull;
        mine += __popcll(word[u]);
    }
    int32_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int32_t v = __shfl_up(incl, off);
        if (lane >= off) incl += v;
    }
    if (lane == 63) wave_s[wave] = incl;
    __syncthreads();
    int32_t run = incl - mine, total = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        const int32_t v = wave_s[w];
        if (w < wave) run += v;
        total += v;
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        word_s[threadIdx.x * PER + u] = word[u];
        before_s[threadIdx.x * PER + u] = run;
        run += __popcll(word[u]);
    }
    __syncthreads();
    if (id == 0) counts->n_out = total;
    if (id >= n) return;
    if (sl < 0) {
        if (parent != nullptr) parent[id] = ~0u;
        return;
    }
    const Candidate q = candidate(c, sh.K(), sh.s(), 0);
    const int32_t o = before_s[r >> 6] + __popcll(word_s[r >> 6] & ((1ull << (r & 63)) - 1ull));
    nbr[((int64_t)(o >> 6) * (sh.K() * sh.K() * sh.K()) + q.k) * TILE + (o & 63)] = id;
    if (parent != nullptr) parent[id] = (uint32_t)o << 6 | (uint32_t)q.k;
    if (r == id) out_coords[o] = make_int4(c.x, q.qx, q.qy, q.qz);
}

// Group masks of a finished offset table: one workgroup per tile; its four wavefronts share the
// offset lines, eight lines in flight each, vote on them and merge their bits in LDS.
__global__ void __launch_bounds__(256)
k_masks_from_table(const int32_t* __restrict__ nbr, int K3, int mw, int64_t tiles, uint32_t* __restrict__ gmask,
                   const sc_counts* __restrict__ counts) {
    __shared__ uint32_t mask_s[4 * ((343 + 31) / 32)];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t tile = blockIdx.x;
    // tiles past the last output row are never read
    if (tile >= tiles || tile * TILE >= counts->n_out) return;
    if (threadIdx.x < 4 * mw) mask_s[threadIdx.x] = 0u;
    __syncthreads();
    const int32_t* tile_nbr = nbr + tile * (int64_t)K3 * TILE;
    for (int k0 = w * 8; k0 < K3; k0 += 32) {       // the eight lines k0..k0+7 lie in one mask word
        int32_t v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = k0 + u < K3 ? tile_nbr[(k0 + u) * TILE + lane] : -1;
        uint32_t bits = 0;                          // lanes 0..3: group `lane`
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint64_t vote = __ballot(v[u] >= 0);
            if (lane < 4 && ((vote >> (16 * lane)) & 0xffffull) != 0) bits |= 1u << ((k0 + u) & 31);
        }
        if (lane < 4 && bits) atomicOr(&mask_s[lane * mw + (k0 >> 5)], bits);
    }
    __syncthreads();
    if (threadIdx.x < 4 * mw) gmask[tile * (4 * mw) + threadIdx.x] = mask_s[threadIdx.x];
}

// ---- reading a map back -----------------------------------------------------------------------
__global__ void __launch_bounds__(256)
k_counts_clear_pairs(sc_counts* counts) {
    for (int i = threadIdx.x; i < 343; i += blockDim.x) counts->per_offset[i] = 0;
    if (threadIdx.x == 0) counts->n_pairs = 0;
}

// One wavefront per (tile, offset) line of the table: count the rows that have a neighbour.
__global__ void __launch_bounds__(256)
k_count_pairs(const int32_t* __restrict__ nbr, int K3, int64_t tiles_bound, sc_counts* counts, int inverse) {
    __shared__ int32_t hist[343];
    for (int i = threadIdx.x; i < K3; i += blockDim.x) hist[i] = 0;
    __syncthreads();
    int64_t tiles = ((inverse ? counts->n_in : counts->n_out) + TILE - 1) / TILE;
    if (tiles > tiles_bound) tiles = tiles_bound;
    const int64_t items = tiles * K3;
    const int lane = threadIdx.x & 63;
    const int64_t nwaves = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t it = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); it < items; it += nwaves) {
        const int k = (int)(it % K3);
        const int c = __popcll(__ballot(nbr[it * TILE + lane] >= 0));
        if (lane == 0 && c) atomicAdd(&hist[k], c);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < K3; i += blockDim.x) {
        if (hist[i]) {
            atomicAdd(&counts->per_offset[i], hist[i]);
            atomicAdd((unsigned long long*)&counts->n_pairs, (unsigned long long)hist[i]);
        }
    }
}

// Plain pair lists: one workgroup per offset k walks the tiles in order, 16 tiles (one per
// wavefront) at a time; the rows with a neighbour are compacted by ballot + prefix count behind
// those of the earlier tiles, so the pairs of an offset come out ordered by output row.
__global__ void __launch_bounds__(1024)
k_export(const int32_t* __restrict__ nbr, int K3, int64_t tiles, const int32_t* __restrict__ offset_start,
         int32_t* __restrict__ pairs_in, int32_t* __restrict__ pairs_out) {
    __shared__ int32_t cnt_s[16];
    __shared__ int32_t carry_s;
    const int k = blockIdx.x;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (threadIdx.x == 0) carry_s = offset_start[k];
    __syncthreads();
    for (int64_t t0 = 0; t0 < tiles; t0 += 16) {
        const int64_t t = t0 + w;
        int32_t v = -1;
        if (t < tiles) v = nbr[(t * K3 + k) * TILE + lane];
        const uint64_t vote = __ballot(v >= 0);
        if (lane == 0) cnt_s[w] = __popcll(vote);
        __syncthreads();
        int32_t base = carry_s;
        for (int ww = 0; ww < w; ++ww) base += cnt_s[ww];
        if (v >= 0) {
            const int32_t dst = base + __popcll(vote & lanemask_lt());
            pairs_in[dst] = v;
            pairs_out[dst] = (int32_t)(t * TILE + lane);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int32_t total = 0;
            for (int ww = 0; ww < 16; ++ww) total += cnt_s[ww];
            carry_s += total;
        }
        __syncthreads();
    }
}

struct StartArg {
    int32_t v[344];
};
__global__ void __launch_bounds__(256)
k_write_starts(StartArg a, int count, int32_t* __restrict__ dst) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) dst[i] = a.v[i];
}

// Inverse layer (Section III-E): the pairs of a strided map with input and output swapped.  Every fine row has one parent
// (K == stride); the strided build leaves (coarse row, offset) in one word per fine row, and this kernel expands the 64
// words of a tile to its K^3 lines and group masks.  Finding the words again by scattering the strided table was a kernel of its
// own, a launch of 4 us (transpose and 64 -> 32 convolution on 53 k rows 12.1 -> 9.5 us).
// One wavefront per fine tile, lane = row.  A word counts only if the strided map confirms it: of inputs with the same
// coordinate the map holds one.
__global__ void __launch_bounds__(256)
k_transpose_expand(const int32_t* __restrict__ nbr, const uint32_t* __restrict__ parent, int K3, int mw, int64_t n,
                   const sc_counts* __restrict__ counts, int32_t* __restrict__ inv_nbr, uint32_t* __restrict__ inv_mask, KmapHeader* hdr,
                   KmapHeader hdr_value) {
    const int lane = threadIdx.x & 63;
    if (blockIdx.x == 0 && threadIdx.x == 0) *hdr = hdr_value;
    const int64_t tile = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (tile * TILE >= n) return;
    const int64_t row = tile * TILE + lane, n_out = counts->n_out;
    int32_t* lines = inv_nbr + tile * (int64_t)(K3 * TILE) + lane;
    const uint32_t word = row < n ? parent[row] : ~0u;
    const int64_t o = word >> 6;
    int k = (int)(word & 63u);
    if (o >= n_out || k >= K3 || nbr[((o >> 6) * K3 + k) * TILE + (o & 63)] != (int32_t)row) k = -1;
    for (int w = 0; w < mw; ++w) {
        uint32_t bits = 0;                            // lanes 0..3: group `lane`
        for (int kk = w * 32; kk < K3 && kk < w * 32 + 32; ++kk) {
            lines[kk * TILE] = k == kk ? (int32_t)o : -1;
            const uint64_t vote = __ballot(k == kk);
            if (lane < 4 && ((vote >> (16 * lane)) & 0xffffull) != 0) bits |= 1u << (kk & 31);
        }
        if (lane < 4) inv_mask[(tile * 4 + lane) * mw + w] = bits;
    }
}

// candidates per input of a strided layer: ceil(K/s)^3
static int strided_maxc(int K, int stride) {
    const int m = (K + stride - 1) / stride;
    return m * m * m;
}

static bool kmap_args_ok(int64_t n, int K, int stride, int mode) {
    if (n < 0 || n > SC_N_MAX || K < 1 || K > SC_K_MAX) return false;
    if (mode == SC_SUBM) return stride == 1 && (K % 2) == 1;
    if (mode == SC_INVERSE) return K == stride && K >= 2 && K <= 4;
    if (mode == SC_STRIDED) {
        if (K < 2 || stride < 1 || stride > K) return false;
        return n * (int64_t)strided_maxc(K, stride) <= SC_N_MAX;     // candidate ids and output rows fit
    }
    return false;
}
// slots of the output-cell table per candidate
static uint64_t strided_slots(int K, int stride) { return K == stride && K <= 4 ? 8 : 2; }

// The strided build (arguments checked by the caller): clear the cell table -> claim cells -> flag first
// candidates, clear the rows of the offset table -> number cells, write pairs (-> group masks, K^3 > 32).
template <class Shape>
static int build_strided(const Shape& sh, const int32_t* d_coords, int64_t n, const void* d_table, int K, int stride, int32_t* d_out_coords,
                         void* d_kmap, const KmapLayout& L, const KmapHeader& h, void* d_scratch, sc_counts* d_counts, hipStream_t s) {
    uint32_t* gmask = (uint32_t*)((char*)d_kmap + L.off_mask);
    int32_t* nbr = (int32_t*)((char*)d_kmap + L.off_nbr);
    uint32_t* parent = L.off_parent != 0 ? (uint32_t*)((char*)d_kmap + L.off_parent) : nullptr;
    const int64_t nc = n * strided_maxc(K, stride);            // candidates
    StridedScratch g = strided_scratch(d_scratch, nc, strided_slots(K, stride));
    const uint64_t cap = (uint64_t)g.omask + 1;
    // Short builds clear all the table rows there could be beside the cell table.
    const int64_t nbr_vec = L.tiles * L.K3 * (TILE / 4);
    const bool is_short = short_strided_build(n, K, stride, nbr_vec * 16);
    // workgroups for the larger of the two (K = 5 on 5 k inputs, with workgroups for the cell table only 40.6 us, now 39.9; K = 7 on 3 k
    // 69.3, now 66.1; K <= 3 the same)
    const int64_t cell_vec = (int64_t)(cap / 4), fill_vec = is_short && nbr_vec > cell_vec ? nbr_vec : cell_vec;
    unsigned fb = (unsigned)((fill_vec + 255) / 256);
    if (fb > 4096) fb = 4096;
    SC_LAUNCH(KID_FILL_I32, k_strided_fill, dim3(fb), dim3(256), 0, s, (int4*)g.oslots, cap, g.cells, is_short ? g.flagword : (uint64_t*)nullptr,
              is_short ? (n + 63) / 64 : (int64_t)0, (int4*)nbr, is_short ? nbr_vec : (int64_t)0, d_counts, d_table == nullptr ? 1 : 0, n,
              (const TableHeader*)d_table);
#define SC_STRIDED_INSERT(FLAGS)                                                                                                       \
    SC_LAUNCH(KID_STRIDED_INSERT, (k_strided_insert<FLAGS, Shape>), dim3((unsigned)((nc + CLAIM_WG - 1) / CLAIM_WG)), dim3(CLAIM_WG), 0, s, \
              (const int4*)d_coords, n, sh, g.oslots, g.omask, g.slot_of, g.cells, (uint32_t*)g.flagword, d_counts)
    if (is_short) {
        SC_STRIDED_INSERT(1);
        SC_LAUNCH(KID_STRIDED_PAIRS, k_strided_pairs_short<Shape>, dim3((unsigned)((n + 1023) / 1024)), dim3(1024), 0, s, (const int4*)d_coords, (int)n,
                  sh, (const int32_t*)g.slot_of, (const int32_t*)g.oslots, (const uint64_t*)g.flagword, nbr, parent, (int4*)d_out_coords, d_counts,
                  (KmapHeader*)d_kmap, h);
        if (kmap_masked(SC_STRIDED, L.K3))
            SC_LAUNCH(KID_KMAP_FROM_OFT, k_masks_from_table, dim3((unsigned)L.tiles), dim3(256), 0, s, (const int32_t*)nbr, L.K3, L.mw, L.tiles, gmask,
                      (const sc_counts*)d_counts);
        return SC_OK;
    }
    SC_STRIDED_INSERT(0);
#undef SC_STRIDED_INSERT
    const unsigned gp = (unsigned)((nc + 255) / 256);
#define SC_STRIDED_NUMBER(SCAN, U)                                                                                                     \
    do {                                                                                                                               \
        const int64_t nblk = (nc + U * 1024 - 1) / (U * 1024);                                                                         \
        SC_LAUNCH(KID_STRIDED_FLAGS, k_strided_flags<U>, dim3((unsigned)nblk), dim3(1024), 0, s, nc, (const int32_t*)g.slot_of,        \
                  (const int32_t*)g.oslots, g.flagword, g.word_prefix, g.block_sum, (const int32_t*)g.cells, (int4*)nbr, L.K3);        \
        if (!SCAN)                                                                                                                     \
            SC_LAUNCH(KID_SCAN_BLOCKS, k_scan_blocks, dim3(1), dim3(1024), 0, s, (const int32_t*)g.block_sum, g.block_prefix, nblk,    \
                      d_counts);                                                                                                       \
        SC_LAUNCH(KID_STRIDED_PAIRS, (k_strided_pairs<SCAN, U, Shape>), dim3(gp), dim3(256), 0, s, (const int4*)d_coords, n, sh,       \
                  (const int32_t*)g.slot_of, (const int32_t*)g.oslots, (const uint64_t*)g.flagword, (const int32_t*)g.word_prefix,     \
                  (const int32_t*)g.block_prefix, (const int32_t*)g.block_sum, (int)nblk, nbr, parent, (int4*)d_out_coords, d_counts,          \
                  (KmapHeader*)d_kmap, h);                                                                                             \
    } while (0)
    if (nc <= 512 * 1024) SC_STRIDED_NUMBER(1, 1);
    else if (nc <= (int64_t)SCAN_IN_PAIRS_MAX * 4096) SC_STRIDED_NUMBER(1, 4);
    else SC_STRIDED_NUMBER(0, 4);
#undef SC_STRIDED_NUMBER
    if (kmap_masked(SC_STRIDED, L.K3))
        SC_LAUNCH(KID_KMAP_FROM_OFT, k_masks_from_table, dim3((unsigned)L.tiles), dim3(256), 0, s, (const int32_t*)nbr, L.K3, L.mw, L.tiles, gmask,
                  (const sc_counts*)d_counts);
    return SC_OK;
}

}  // namespace sc

using namespace sc;

extern "C" int64_t sc_out_bound(int64_t n, int K, int stride, int mode) {
    if (!kmap_args_ok(n, K, stride, mode)) return -1;
    return mode == SC_STRIDED ? n * (int64_t)strided_maxc(K, stride) : n;
}

extern "C" size_t sc_kmap_bytes(int64_t n, int K, int stride, int mode) {
    if (!kmap_args_ok(n, K, stride, mode)) return 0;
    return kmap_layout(sc_out_bound(n, K, stride, mode), K, stride, mode).bytes;
}

extern "C" size_t sc_kmap_scratch_bytes(int64_t n, int K, int stride, int mode) {
    if (!kmap_args_ok(n, K, stride, mode)) return 0;
    if (mode == SC_SUBM) return 256;
    if (mode == SC_INVERSE) return strided_scratch(nullptr, n, 8).bytes;
    return strided_scratch(nullptr, sc_out_bound(n, K, stride, mode), strided_slots(K, stride)).bytes;    // one entry per candidate
}

static int kmap_build(const int32_t* d_coords, int64_t n, const void* d_table, int K, int stride, int mode,
                      int32_t* d_out_coords, void* d_kmap, size_t kmap_bytes, void* d_scratch, size_t scratch_bytes,
                      sc_counts* d_counts, void* stream) {
    if (!kmap_args_ok(n, K, stride, mode) || mode == SC_INVERSE) return SC_EINVAL;   // inverse maps: sc_kmap_transpose
    if (d_kmap == nullptr || d_counts == nullptr || (n > 0 && d_coords == nullptr)) return SC_EINVAL;
    if (!aligned16(d_coords) || !aligned16(d_kmap) || !aligned16(d_counts) || !aligned16(d_out_coords) ||
        !aligned16(d_scratch) || !aligned16(d_table))
        return SC_EINVAL;
    if (mode == SC_SUBM && d_table == nullptr) return SC_EINVAL;
    if (mode == SC_STRIDED && (d_out_coords == nullptr || d_scratch == nullptr)) return SC_EINVAL;
    if (kmap_bytes < sc_kmap_bytes(n, K, stride, mode)) return SC_ECAP;
    if (scratch_bytes < sc_kmap_scratch_bytes(n, K, stride, mode) && mode == SC_STRIDED) return SC_ECAP;

    hipStream_t s = (hipStream_t)stream;
    const int64_t bound = sc_out_bound(n, K, stride, mode);
    const KmapLayout L = kmap_layout(bound, K, stride, mode);
    uint32_t* gmask = (uint32_t*)((char*)d_kmap + L.off_mask);
    int32_t* nbr = (int32_t*)((char*)d_kmap + L.off_nbr);
    KmapHeader h{};
    h.magic = KMAP_MAGIC; h.K = K; h.stride = stride; h.mode = mode;
    h.n_in = n; h.n_out_bound = bound; h.tiles = L.tiles; h.mw = L.mw;
    if (n == 0) {
        if (mode == SC_STRIDED && d_table == nullptr)
            SC_LAUNCH(KID_FILL_I32, k_strided_fill, dim3(1), dim3(256), 0, s, (int4*)nullptr, (uint64_t)0, (int32_t*)nullptr,
                      (uint64_t*)nullptr, (int64_t)0, (int4*)nullptr, (int64_t)0, d_counts, 1, (int64_t)0, (const TableHeader*)nullptr);
        SC_LAUNCH(KID_KMAP_HEADER, k_kmap_header, dim3(1), dim3(64), 0, s, (KmapHeader*)d_kmap, h);
        SC_LAUNCH(KID_MISC, k_set_n_out, dim3(1), dim3(64), 0, s, d_counts, (int64_t)0);
        return SC_OK;
    }

    if (mode == SC_SUBM) {
        uint8_t* density = map_density(d_kmap, L);
        HashTable t = table_view(const_cast<void*>(d_table), n);
#define SC_SUBM_LAUNCH(KV, WPT, CH, AT)                                                                           \
    SC_LAUNCH(KID_KMAP_SUBM, (k_kmap_subm<KV, WPT, CH, AT>), dim3(xcd_grid(L.tiles)), dim3(64 * WPT), 0, s,      \
              (const int4*)d_coords, n, (const uint4*)t.slots, (const TableHeader*)t.hdr, gmask, nbr, density, d_counts,          \
              (KmapHeader*)d_kmap, h)
#define SC_SUBM_BLOCKS_AS(KV, YG, YB, RUNS, GRID)                                                                  \
    SC_LAUNCH(KID_KMAP_SUBM, (k_kmap_subm_blocks<KV, YG, YB, RUNS>), dim3(GRID), dim3(64 * KV * YG), 0, s,         \
              (const int4*)d_coords, n, (const uint4*)t.slots, (const TableHeader*)t.hdr, gmask, nbr, density, d_counts,    \
              (KmapHeader*)d_kmap, h)
#define SC_SUBM_BLOCKS(KV, YG, YB)                                                                                 \
    do {                                                                                                           \
        if (map_in_runs(L.tiles, KV, compute_units())) SC_SUBM_BLOCKS_AS(KV, YG, YB, 1, xcd_run_grid<MAP_RUN>(L.tiles));            \
        else SC_SUBM_BLOCKS_AS(KV, YG, YB, 0, xcd_grid(L.tiles));                                                  \
    } while (0)
        switch (K) {
            case 1: SC_SUBM_LAUNCH(1, 1, 1, 1); break;
            case 3:
                // nine wavefronts a tile up to 16 tiles per CU, where their shorter chains still show (8 k rows:
                // 5.3 against 6.8 us, 261 k: 35.0 against 37.4); past it the block hashes that the wavefronts of
                // an x offset repeat cost more (300 k: 33.4 against 30.7, 10^6: 98 against 75)
                if (L.tiles <= 16 * (int64_t)compute_units()) SC_SUBM_BLOCKS(3, 3, 1);
                else SC_SUBM_BLOCKS(3, 1, 3);
                break;
            case 5: SC_SUBM_BLOCKS(5, 3, 1); break;
            case 7: SC_SUBM_LAUNCH(7, 8, 4, 1); break;
            default: return SC_EINVAL;
        }
#undef SC_SUBM_LAUNCH
#undef SC_SUBM_BLOCKS
#undef SC_SUBM_BLOCKS_AS
        if (d_out_coords != nullptr && d_out_coords != d_coords) {
            if (hipMemcpyAsync(d_out_coords, d_coords, (size_t)n * 16, hipMemcpyDeviceToDevice, s) != hipSuccess)
                return SC_EHIP;
        }
        return SC_OK;
    }

    // the common shapes are compiled in, the others take K and stride as arguments
    if (K == 2 && stride == 2)
        return build_strided(StridedShape<2, 2>{}, d_coords, n, d_table, K, stride, d_out_coords, d_kmap, L, h, d_scratch, d_counts, s);
    if (K == 3 && stride == 2)
        return build_strided(StridedShape<3, 2>{}, d_coords, n, d_table, K, stride, d_out_coords, d_kmap, L, h, d_scratch, d_counts, s);
    return build_strided(StridedShape<0, 0>{K, stride, strided_maxc(K, stride)}, d_coords, n, d_table, K, stride, d_out_coords, d_kmap, L, h,
                         d_scratch, d_counts, s);
}

extern "C" int sc_kmap_build(const int32_t* d_coords, int64_t n, const void* d_table, int K, int stride, int mode,
                             int32_t* d_out_coords, void* d_kmap, size_t kmap_bytes, void* d_scratch,
                             size_t scratch_bytes, sc_counts* d_counts, void* stream) {
    return kmap_build(d_coords, n, d_table, K, stride, mode, d_out_coords, d_kmap, kmap_bytes, d_scratch, scratch_bytes,
                      d_counts, stream);
}

// ---- the same build for callers that cannot allocate ------------------------------------------
// The scratch of a strided build (output-cell table, per-input slots, flag words, prefixes) lives
// in one device array of the library instead of a caller's buffer.  Every device holds its own
// copy of the array at its own address; the name below is only a host-side handle, so the
// address is asked for once per device (with that device current) and that pointer is what the
// kernels receive.  The build clears what it needs itself (k_strided_fill), so the contents a
// previous call left behind do not matter; two calls that overlap on one device would race.
static __device__ __align__(256) unsigned char scratch[SC_NOALLOC_SCRATCH_BYTES];

static int noalloc_scratch(void** out) {
    constexpr int MAX_DEVICES = 64;
    static void* ptr[MAX_DEVICES] = {};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return SC_EHIP;
    if (ptr[dev] == nullptr) {
        void* p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) return SC_EHIP;
        ptr[dev] = p;
    }
    *out = ptr[dev];
    return SC_OK;
}

extern "C" int sc_kmap_build_noalloc(const int32_t* d_coords, int64_t n, const void* d_table, int K, int stride,
                                     int mode, int32_t* d_out_coords, void* d_kmap, size_t kmap_bytes,
                                     sc_counts* d_counts, void* stream) {
    if (!kmap_args_ok(n, K, stride, mode) || mode == SC_INVERSE) return SC_EINVAL;
    const size_t need = sc_kmap_scratch_bytes(n, K, stride, mode);
    if (need > (size_t)SC_NOALLOC_SCRATCH_BYTES) return SC_ECAP;
    void* p = nullptr;
    if (int rc = noalloc_scratch(&p)) return rc;
    return kmap_build(d_coords, n, d_table, K, stride, mode, d_out_coords, d_kmap, kmap_bytes, p,
                      (size_t)SC_NOALLOC_SCRATCH_BYTES, d_counts, stream);
}

extern "C" int sc_kmap_transpose(const void* d_kmap, int64_t n, int K, int stride, const sc_counts* d_counts,
                                 void* d_kmap_inv, size_t kmap_inv_bytes, void* stream) {
    if (!kmap_args_ok(n, K, stride, SC_INVERSE)) return SC_EINVAL;
    if (d_kmap == nullptr || d_kmap_inv == nullptr || d_counts == nullptr || d_kmap == d_kmap_inv) return SC_EINVAL;
    if (!aligned16(d_kmap) || !aligned16(d_kmap_inv) || !aligned16(d_counts)) return SC_EINVAL;
    if (kmap_inv_bytes < sc_kmap_bytes(n, K, stride, SC_INVERSE)) return SC_ECAP;
    hipStream_t s = (hipStream_t)stream;
    const KmapLayout L = kmap_layout(n, K, stride, SC_STRIDED);      // offset table and masks lie alike in both directions
    KmapHeader h{};
    h.magic = KMAP_MAGIC; h.K = K; h.stride = stride; h.mode = SC_INVERSE;
    h.n_in = n; h.n_out_bound = n; h.tiles = L.tiles; h.mw = L.mw;
    if (n == 0) {
        SC_LAUNCH(KID_KMAP_HEADER, k_kmap_header, dim3(1), dim3(64), 0, s, (KmapHeader*)d_kmap_inv, h);
        return SC_OK;
    }
    const int32_t* nbr = (const int32_t*)((const char*)d_kmap + L.off_nbr);
    int32_t* inv_nbr = (int32_t*)((char*)d_kmap_inv + L.off_nbr);
    uint32_t* inv_mask = (uint32_t*)((char*)d_kmap_inv + L.off_mask);
    const uint32_t* parent = (const uint32_t*)((const char*)d_kmap + L.off_parent);
    SC_LAUNCH(KID_KMAP_FROM_OFT, k_transpose_expand, dim3((unsigned)((L.tiles + 3) / 4)), dim3(256), 0, s, nbr, parent, L.K3, L.mw, n, d_counts,
              inv_nbr, inv_mask, (KmapHeader*)d_kmap_inv, h);
    return SC_OK;
}

extern "C" int sc_counts_read(sc_counts* d_counts, sc_counts* h_counts, const void* d_kmap, int64_t n, int K,
                              int stride, int mode, void* stream) {
    if (d_counts == nullptr || h_counts == nullptr) return SC_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    if (d_kmap != nullptr) {
        if (!kmap_args_ok(n, K, stride, mode)) return SC_EINVAL;
        const KmapLayout L = kmap_layout(sc_out_bound(n, K, stride, mode), K, stride, mode);
        SC_LAUNCH(KID_MISC, k_counts_clear_pairs, dim3(1), dim3(256), 0, s, d_counts);
        if (L.tiles > 0) {
            int64_t items = L.tiles * L.K3;
            unsigned gb = (unsigned)((items + 3) / 4);
            if (gb > 2048) gb = 2048;
            SC_LAUNCH(KID_COUNT_PAIRS, k_count_pairs, dim3(gb), dim3(256), 0, s,
                      (const int32_t*)((const char*)d_kmap + L.off_nbr), L.K3, L.tiles, d_counts,
                      mode == SC_INVERSE ? 1 : 0);
        }
    }
    if (hipMemcpyAsync(h_counts, d_counts, sizeof(sc_counts), hipMemcpyDeviceToHost, s) != hipSuccess) return SC_EHIP;
    if (hipStreamSynchronize(s) != hipSuccess) return SC_EHIP;
    return h_counts->status < 0 ? h_counts->status : SC_OK;
}

extern "C" int sc_kmap_export(const void* d_kmap, int64_t n, int K, int stride, int mode, const sc_counts* h_counts,
                              int32_t* d_pairs_in, int32_t* d_pairs_out, int32_t* d_offset_start, void* stream) {
    if (d_kmap == nullptr || h_counts == nullptr || d_offset_start == nullptr) return SC_EINVAL;
    if (!kmap_args_ok(n, K, stride, mode)) return SC_EINVAL;
    if (h_counts->n_pairs > 0 && (d_pairs_in == nullptr || d_pairs_out == nullptr)) return SC_EINVAL;
    if (h_counts->n_pairs > 0x7fffffffLL) return SC_ECAP;
    hipStream_t s = (hipStream_t)stream;
    const KmapLayout L = kmap_layout(sc_out_bound(n, K, stride, mode), K, stride, mode);
    StartArg h_start{};
    int32_t acc = 0;
    for (int k = 0; k < L.K3; ++k) {
        h_start.v[k] = acc;
        acc += h_counts->per_offset[k];
    }
    h_start.v[L.K3] = acc;
    if ((int64_t)acc != h_counts->n_pairs) return SC_EINVAL;
    SC_LAUNCH(KID_MISC, k_write_starts, dim3(1), dim3(256), 0, s, h_start, L.K3 + 1, d_offset_start);
    const int64_t tiles = ((mode == SC_INVERSE ? h_counts->n_in : h_counts->n_out) + TILE - 1) / TILE;
    if (tiles > 0 && acc > 0)
        SC_LAUNCH(KID_EXPORT, k_export, dim3((unsigned)L.K3), dim3(1024), 0, s,
                  (const int32_t*)((const char*)d_kmap + L.off_nbr), L.K3, tiles, (const int32_t*)d_offset_start, d_pairs_in, d_pairs_out);
    return SC_OK;
}
