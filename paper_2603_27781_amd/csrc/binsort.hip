// Tile binning and depth sort (GS^3LAM Sec. 3.2.1: the tile-based rasterizer
// of the cited 3DGS work sorts Gaussians in depth order per tile).
//
// Every visible (view, Gaussian) pair emits one instance per tile of its
// rectangle; the instances are then grouped by tile and each tile's list is
// sorted by (binary32 depth bits, emission index).  Emission runs in (view,
// index) order and a Gaussian is in a tile's list once, so that key is
// distinct and orders like (depth, Gaussian index): grouping by tile needs no
// stable sort, and the final order (view, tile, depth, index) does not
// depend on the order in which the groups were filled.  Six launches:
//   1. k_bin_reset, or k_chunk_sums where there are many chunks of pairs: the
//      call's state, and the second the instances of every chunk;
//   2. k_emit: one workgroup per chunk of pairs of one view: instance offsets
//      and emission; each instance counts itself into its tile in LDS, what
//      the counter held is its place among the chunk's, and the chunk's
//      counts become a row of a (chunk, tile) table (or, for a view of more
//      tiles than fit, into one counter per tile in memory);
//   3. k_tile_scan (k_tile_scan_one): the table's columns to [start, end) of
//      every tile and the first place of every (chunk, tile);
//   4. k_place: each instance's sort key to its place;
//   5. k_tile_sort_short, 6. k_tile_sort_long: the lists in order.
// (An LSD radix sort by tile id before them, with the visible pairs compacted
// and their offsets scanned first, took 19 launches, most of them of a few
// microseconds.  Alone: one 1200x680 view of 1M Gaussians 87 -> 45 us, eight
// such views 232 -> 147, 640x480 / 200k 134 -> 80, 320x240 / 60k 62 -> 28,
// 16 mixed views of 2M 740 -> 502.  The kernels move 56 bytes per instance, 20
// per visible pair and 8 per pair, about 40 us of the eight views' 147 at the
// rate of a copy; the rest is latency and, in the sort, vector work.)
//
// Every count that the host does not know (visible pairs, instances) stays on
// the device; grids are sized for the capacity and blocks beyond the count
// exit early, so the whole pipeline is graph-capturable.
//
// Blocks that wait (the look-back of k_emit and the tile scans, the merges of
// k_tile_sort_long) take a ticket first and wait only for blocks with earlier
// tickets, which are already running and wait for none after them, so every
// wait ends (the spin is bounded all the same).
#include <cstdlib>

#include "sgs_common.h"

namespace sgs {

namespace {

// Value of v held by lane (lane ^ J), for wavefront sums and the
// compare-exchanges of the bitonic network.  No LDS round trip where the hardware has a register
// path: J = 1, 2 are DPP quad permutations, J = 8 a DPP row rotation (within
// a row of 16 lanes that is lane ^ 8), J = 16, 32 permlane swaps of v with
// itself (which give the values of the lanes with the bit clear and set);
// J = 4 goes through the LDS crossbar (ds_swizzle, no address operand).
template <int J>
__device__ __forceinline__ uint32_t lane_xor_u32(uint32_t v, int lane) {
    if constexpr (J == 1) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
    } else if constexpr (J == 2) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
    } else if constexpr (J == 8) {
        return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xF, 0xF, true);  // row_ror:8
    } else if constexpr (J == 4) {
        return (uint32_t)__builtin_amdgcn_ds_swizzle((int)v, (4 << 10) | 0x1F);  // xor_mask 4
    } else if constexpr (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);  // v(l & ~16), v(l | 16)
        return (lane & 16) ? r[0] : r[1];
    } else {
        static_assert(J == 32, "lane_xor_u32: J is a power of two up to 32");
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);  // v(l & ~32), v(l | 32)
        return (lane & 32) ? r[0] : r[1];
    }
}

// Sum of x over the 64 lanes, in every lane (integer: the order does not
// matter), with one LDS crossbar step (J = 4) instead of six shuffles.
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t x, int lane) {
    x += lane_xor_u32<1>(x, lane);
    x += lane_xor_u32<2>(x, lane);
    x += lane_xor_u32<4>(x, lane);
    x += lane_xor_u32<8>(x, lane);
    x += lane_xor_u32<16>(x, lane);
    x += lane_xor_u32<32>(x, lane);
    return x;
}

// Sum of a[0 .. m) by the whole block (all threads get it).
template <int NT>
__device__ __forceinline__ uint32_t block_sum(const uint32_t* __restrict__ a, int m, uint32_t* s_tmp) {
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    uint32_t x = 0;
    for (int i = tid; i < m; i += NT) x += a[i];
    x = wave_sum_u32(x, lane);
    if (lane == 0) s_tmp[wave] = x;
    __syncthreads();
    uint32_t t = 0;
#pragma unroll
    for (int w = 0; w < NT / kWave; ++w) t += s_tmp[w];
    __syncthreads();
    return t;
}

// ----------------------------------------------------------------------------
// decoupled look-back
// ----------------------------------------------------------------------------
// Status word of a block: bits 62-63 the state (0 not ready, 1 the block's
// totals, 2 inclusive prefixes), bits 32-61 one count (visible pairs), bits
// 0-31 the other (instances).
constexpr uint64_t LB_AGG = 1ull << 62;
constexpr uint64_t LB_INC = 2ull << 62;
constexpr uint64_t LB_VALUE = LB_AGG - 1;
constexpr int LB_SPIN_MAX = 1 << 20;

__device__ __forceinline__ void lb_publish(uint64_t* st, uint64_t word) {
    __hip_atomic_store(st, word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t lb_read(const uint64_t* st) {
    return __hip_atomic_load(st, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Where a wait that gave up is recorded: the call's flag and the caller's
// sticky flag (the low words of counts[3] and counts[4]), and how many reads
// a wait may take.
struct LbGiveUp {
    uint32_t* flag;
    uint32_t* sticky;
    int spin_limit;
};

__device__ __forceinline__ void give_up(LbGiveUp gu) {
    atomicOr(gu.flag, 1u);
    atomicOr(gu.sticky, 1u);
}

// Exclusive prefix (both counts) of block `b` (> 0) from the status words of
// the blocks before it; called by one whole wavefront, which reads 64 of them
// at a time, newest first.  Positions before block 0 count as an inclusive 0.
// A predecessor that has not published after gu.spin_limit further reads is
// counted as 0 -- a short prefix -- and the give-up is recorded, so that the
// binning's later kernels stand down and the caller sees it.
__device__ uint64_t lb_lookback(const uint64_t* status, int b, LbGiveUp gu) {
    const int lane = threadIdx.x & (kWave - 1);
    uint64_t prefix = 0;
    for (int j = b - 1;; j -= kWave) {
        const int k = j - lane;
        uint64_t s = k >= 0 ? lb_read(status + k) : LB_INC;
        for (int spin = 0; __any((s >> 62) == 0) && spin < gu.spin_limit; ++spin)
            if ((s >> 62) == 0) s = lb_read(status + k);
        if (__any((s >> 62) == 0) && lane == 0) give_up(gu);
        const uint64_t inc = __ballot((s >> 62) == 2);
        uint64_t v = s & LB_VALUE;
        if (inc != 0 && lane > __builtin_ctzll(inc)) v = 0;  // stop at the nearest inclusive prefix
        prefix += ((uint64_t)wave_sum_u32((uint32_t)(v >> 32), lane) << 32) + wave_sum_u32((uint32_t)v, lane);
        if (inc != 0) return prefix;
    }
}

// Publishes the block's totals, looks back and publishes its inclusive
// prefix; every thread gets the exclusive one.
__device__ __forceinline__ uint64_t lb_exchange(uint64_t totals, int b, uint64_t* status, uint64_t* s_prefix,
                                                LbGiveUp gu) {
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        uint64_t prefix = 0;
        if (b > 0) {
            if (lane == 0) lb_publish(status + b, LB_AGG | totals);
            prefix = lb_lookback(status, b, gu);
        }
        if (lane == 0) {
            lb_publish(status + b, LB_INC | ((prefix + totals) & LB_VALUE));
            *s_prefix = prefix;
        }
    }
    __syncthreads();
    return *s_prefix;
}

__device__ __forceinline__ int lb_ticket(uint32_t* ticket, int* s_block) {
    if (threadIdx.x == 0) *s_block = (int)atomicAdd(ticket, 1u);
    __syncthreads();
    return *s_block;
}

// ----------------------------------------------------------------------------
// instance offsets and emission
// ----------------------------------------------------------------------------
constexpr int EM_THREADS = 1024, EM_WAVES = EM_THREADS / kWave;
constexpr int EM_ITEMS = 16;                         // pairs per lane and pass at most (none for some lanes in small chunks)
constexpr int EM_PASS = EM_THREADS * EM_ITEMS;       // pairs per workgroup and pass at most
constexpr int EM_RING = 2 * kWave;                   // queued visible pairs per wavefront
constexpr int EM_LOOKBACK = 128;                     // up to this many chunks, offsets by look-back
constexpr int EM_LDS_TILES = 32768;                  // 16-bit tile counters per workgroup at most (64 of 160 KB a CU)
constexpr int64_t EM_CHUNK = 32768;                  // pairs of a chunk at most, so that they count to 16 bits
constexpr int SC_WAVES = 16, SC_THREADS = SC_WAVES * kWave;
constexpr int SC_MAXBLK = 4096;                      // blocks of k_tile_scan at most

// The words one call clears before it uses them.
struct BinState {
    uint32_t emit_ticket, scan_ticket, long_ticket;
    uint32_t wholes, parts, levels;  // lists of one workgroup, parts of longer ones, most levels of a merge
    int64_t instances, placed;  // all of them; those below the capacity
    uint64_t emit_status[EM_LOOKBACK];
    uint64_t scan_status[SC_MAXBLK];
};
static_assert(sizeof(BinState) % 4 == 0, "cleared as words");

// Clears the call's state, the give-up flag and the tiles' counters in memory,
// if k_emit counts there (with a kernel, not a memset, so that graph replays
// stay correct).
__device__ __forceinline__ void bin_reset(BinState* st, int64_t* counts, uint32_t* tiles, int64_t n_tiles) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x, i0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    uint32_t* w = reinterpret_cast<uint32_t*>(st);
    for (int64_t i = i0; i < (int64_t)(sizeof(BinState) / 4); i += stride) w[i] = 0;
    for (int64_t i = i0; i < n_tiles; i += stride) tiles[i] = 0;
    if (i0 == 0) counts[3] = 0;
}

__global__ void __launch_bounds__(256) k_bin_reset(BinState* st, int64_t* counts, uint32_t* tiles, int64_t n_tiles) {
    bin_reset(st, counts, tiles, n_tiles);
}

// Instances and visible pairs of every chunk of pairs.
__global__ void __launch_bounds__(EM_THREADS) k_chunk_sums(const int32_t* __restrict__ touched, int n, int per_view,
                                                           int64_t chunk, uint32_t* __restrict__ inst_sums,
                                                           uint32_t* __restrict__ vis_sums, BinState* st,
                                                           int64_t* counts, uint32_t* tiles, int64_t n_tiles) {
    __shared__ uint32_t s_w[2][EM_WAVES];
    bin_reset(st, counts, tiles, n_tiles);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const int v = (int)blockIdx.x / per_view;
    const int64_t i0 = (int64_t)((int)blockIdx.x - v * per_view) * chunk, i1 = min(i0 + chunk, (int64_t)n);
    const int32_t* src = touched + (int64_t)v * n;
    uint32_t a = 0, b = 0;
    for (int64_t j = i0; j < i1; j += EM_PASS) {
#pragma unroll
        for (int k = 0; k < EM_ITEMS; ++k) {
            const int64_t i = j + k * EM_THREADS + tid;
            const int32_t c = i < i1 ? src[i] : 0;
            a += (uint32_t)c;
            b += c > 0 ? 1u : 0u;
        }
    }
    a = wave_sum_u32(a, lane);
    b = wave_sum_u32(b, lane);
    if (lane == 0) {
        s_w[0][wave] = a;
        s_w[1][wave] = b;
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t x = 0, y = 0;
        for (int w = 0; w < EM_WAVES; ++w) {
            x += s_w[0][w];
            y += s_w[1][w];
        }
        inst_sums[blockIdx.x] = x;
        vis_sums[blockIdx.x] = y;
    }
}

struct EmitArgs {
    const int32_t* touched;
    const uint4* rect;
    const gs_view* views;
    int n, n_views, tile, per_view;  // per_view: chunks of each view
    int64_t chunk, capacity;
    int per_wave;    // pairs per wavefront and pass
    int items;       // the same per lane, rounded up
    const uint32_t *inst_sums, *vis_sums;  // not read with the look-back
    BinState* st;
    uint32_t* table;
    int stride;      // words between the table's entries
    uint32_t *cell_e, *rank_e, *depth_e;
    int32_t *inst_gid, *pair_first;
    int64_t* counts;
    LbGiveUp gu;
};

// The table: row b of view v (chunk b of it) starts at entry
// per_view * tile_offset + b * (tiles of the view).
__device__ __forceinline__ int64_t table_row(const gs_view& vw, int per_view, int b, int tiles_v) {
    return (int64_t)per_view * vw.tile_offset + (int64_t)b * tiles_v;
}

// Emission of one chunk of pairs of one view.  The visible pair whose first
// instance has emission index o writes one instance per tile of its
// rectangle at o, o + 1, ... (row-major): its Gaussian (inst_gid), its
// depth's binary32 bits (depth_e, which the projection stored with the
// rectangle), its table entry (cell_e) and its place among the entry's
// (rank_e).  pair_first[pair] = o, so the instances of a pair stay contiguous
// in emission space whatever the tile lists do.
//
// The chunk's offset: with LOOKBACK (few chunks) a single-pass scan over the
// chunks before it, otherwise the sums k_chunk_sums left (with many chunks
// the chain of waits costs more than a second reading of the tile counts).
//
// Each wavefront walks its own contiguous part of the chunk, queues the
// visible pairs in LDS and takes them up to 64 at a time, a pair per lane;
// the lanes then stride over all of the group's instances together, so a pair
// with many tiles does not stall its wavefront and the writes are contiguous
// across lanes.  The pair of each instance: every pair whose first instance
// falls in the current 64 marks that slot with its lane in LDS, and a
// max-scan over the wavefront (DPP) carries the latest mark to every later
// slot.
//
// Counting in LDS where it can be: a returning atomic per instance on
// counters in memory (eight sets, one per XCD) made this kernel 128 us at
// eight 1200x680 views, 26 G atomics/s, against 57 us now.  The counters
// are 16 bits wide (a pair is in a tile once, so a count is at most the
// chunk's pairs), two to a word.  LDS false, for views of more tiles than that
// holds (and where the table would not fit): one counter per tile in memory,
// cleared by the launch before, for all chunks.  (Walking the pairs again for
// every 32,768 tiles took 43 ms for a 3840x2160 view of 300 k Gaussians at
// tile 8, 52.6 M instances, and 900 ms at 7680x4320; now 3.3 and 4.3.)
template <bool LOOKBACK, bool LDS>
__global__ void __launch_bounds__(EM_THREADS) __attribute__((amdgpu_waves_per_eu(8, 8))) k_emit(EmitArgs A) {
    extern __shared__ uint32_t s_cnt[];
    __shared__ uint32_t s_tmp[EM_WAVES];
    __shared__ uint64_t s_prefix;
    __shared__ int s_block;
    __shared__ uint16_t s_qpair[EM_WAVES][EM_RING];   // queued pairs: index in the wavefront's part of the pass,
    __shared__ uint32_t s_qfirst[EM_WAVES][EM_RING];  // first instance in the pass
    __shared__ uint2 s_info[EM_WAVES][kWave];  // (x0 | y0 << 16, rect width)
    __shared__ uint2 s_who[EM_WAVES][kWave];   // (Gaussian, depth bits)
    __shared__ int32_t s_mark[EM_WAVES][kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int total_chunks = A.per_view * A.n_views;
    const int ch = LOOKBACK ? lb_ticket(&A.st->emit_ticket, &s_block) : (int)blockIdx.x;
    const int v = ch / A.per_view, cb = ch - v * A.per_view;
    const gs_view& vw = A.views[v];
    const int tiles_x = ceil_div(vw.width, A.tile), tiles_v = tiles_x * ceil_div(vw.height, A.tile);
    const int64_t row = LDS ? table_row(vw, A.per_view, cb, tiles_v) : vw.tile_offset;
    const int64_t c0 = (int64_t)cb * A.chunk, c1 = min(c0 + A.chunk, (int64_t)A.n);
    const int64_t vbase = (int64_t)v * A.n;
    const int pass = EM_WAVES * A.per_wave;
    // this wavefront's pairs of the pass that starts at j: item k of lane l is
    // pair j + wave * per_wave + 64 k + l; `live` of them are there
    auto live_of = [&](int64_t j) {
        const int64_t left = c1 - j - (int64_t)wave * A.per_wave;
        return left < A.per_wave ? (int)left : A.per_wave;
    };
    auto tiles_of = [&](const int32_t* pairs, int live, int k) {
        const int q = k * kWave + lane;
        return q < live ? pairs[q] : 0;
    };
    auto pairs_of = [&](int64_t j) { return A.touched + (vbase + j + (int64_t)wave * A.per_wave); };
    // first instance of this wavefront within the pass, and the pass's totals
    auto pass_offsets = [&](int64_t j, uint32_t& off, uint32_t& tot_i, uint32_t& tot_v) {
        uint32_t ni = 0, nv = 0;
        const int32_t* pairs = pairs_of(j);
        const int live = live_of(j);
#pragma unroll
        for (int k = 0; k < EM_ITEMS; ++k) {
            const int32_t c = tiles_of(pairs, live, k);
            ni += (uint32_t)c;
            nv += c > 0 ? 1u : 0u;
        }
        const uint32_t e = block_exclusive<EM_THREADS>(ni, s_tmp, &tot_i);
        off = (uint32_t)__builtin_amdgcn_readlane((int)e, 0);  // the lanes' pairs are interleaved
        tot_v = 0;
        if (LOOKBACK) block_exclusive<EM_THREADS>(nv, s_tmp, &tot_v);
    };
    // 1. the chunk's offset
    uint64_t prefix;
    uint32_t off = 0, tot_i = 0, tot_v = 0;
    pass_offsets(c0, off, tot_i, tot_v);
    if constexpr (LOOKBACK) {
        uint64_t tot = ((uint64_t)tot_v << 32) + tot_i;
        for (int64_t j = c0 + pass; j < c1; j += pass) {  // uniform
            uint32_t o2, ti, tv;
            pass_offsets(j, o2, ti, tv);
            tot += ((uint64_t)tv << 32) + ti;
        }
        prefix = lb_exchange(tot, ch, A.st->emit_status, &s_prefix, A.gu);
        if (ch == total_chunks - 1 && tid == 0) {
            const int64_t I = (int64_t)(uint32_t)(prefix + tot);
            A.st->instances = I;
            A.counts[1] = (int64_t)((prefix + tot) >> 32);
        }
    } else {
        prefix = block_sum<EM_THREADS>(A.inst_sums, ch, s_tmp);
        if (ch == total_chunks - 1) {  // uniform
            const uint32_t nv = block_sum<EM_THREADS>(A.vis_sums, total_chunks, s_tmp);
            if (tid == 0) {
                A.st->instances = (int64_t)(uint32_t)prefix + A.inst_sums[ch];
                A.counts[1] = nv;
            }
        }
    }
    if (ch == total_chunks - 1 && tid == 0) {
        const int64_t I = A.st->instances;
        A.st->placed = I < A.capacity ? I : A.capacity;
        A.counts[0] = I;
        A.counts[2] = I > A.capacity ? 1 : 0;
        if (I > A.capacity) atomicOr(A.gu.sticky, 1u);  // sticky: only the caller clears it
    }
    const int64_t first = (int64_t)(uint32_t)prefix;

    // 2. the walk
    if constexpr (LDS) {
        for (int i = tid; i < (tiles_v + 1) / 2; i += EM_THREADS) s_cnt[i] = 0;
        __syncthreads();
    }
    int64_t done = 0;  // instances of the passes before
    for (int64_t j = c0; j < c1; j += pass) {
        if (j != c0) pass_offsets(j, off, tot_i, tot_v);
        uint32_t run = off;  // first instance of the next pair, within the pass
        int head = 0, tail = 0;
        const uint32_t wpair = (uint32_t)(j + (int64_t)wave * A.per_wave);
        // emits the queued pairs [head, head + ng), one per lane
        auto emit = [&](int ng) {
            uint32_t my_start = 0, my_end = 0;
            const int q0 = head & (EM_RING - 1);
            const uint32_t gstart = s_qfirst[wave][q0];
            if (lane < ng) {
                const int q = (head + lane) & (EM_RING - 1);
                const uint32_t i = wpair + s_qpair[wave][q], f = s_qfirst[wave][q];
                const uint4 r = A.rect[vbase + i];
                const uint32_t x0 = r.x & 0xffffu, y0 = r.x >> 16, x1 = r.y & 0xffffu, y1 = r.y >> 16;
                const uint32_t wr = x1 - x0 + 1, hr = y1 - y0 + 1;
                my_start = f - gstart;
                my_end = my_start + wr * hr;
                A.pair_first[vbase + i] = (int32_t)(first + done + f);
                s_info[wave][lane] = make_uint2(x0 | (y0 << 16), wr);
                s_who[wave][lane] = make_uint2(i, r.z);
            }
            const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)my_end, ng - 1);
            const int64_t o_g = first + done + gstart;
            int carry = 0;  // the pair of the last instance before the current 64
            for (uint32_t b0 = 0; b0 < total; b0 += kWave) {
                s_mark[wave][lane] = -1;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                // starts strictly increase (a visible pair has an
                // instance), so a slot is marked at most once
                if (lane < ng && my_start >= b0 && my_start < b0 + kWave) s_mark[wave][my_start - b0] = lane;
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                const int lo = max(wave_max_scan(s_mark[wave][lane]), carry);
                carry = __builtin_amdgcn_readlane(lo, kWave - 1);
                const uint32_t k = b0 + lane;
                const int64_t o = o_g + k;
                const uint2 info = s_info[wave][lo], who = s_who[wave][lo];
                // row and column of the instance in the rectangle (width
                // info.y): the quotient is below 2^16, so a float estimate
                // is within one of it and one correction step makes it exact
                const uint32_t li = k - (s_qfirst[wave][(head + lo) & (EM_RING - 1)] - gstart);
                uint32_t q = (uint32_t)((float)li * __builtin_amdgcn_rcpf((float)info.y));
                int32_t r = (int32_t)(li - q * info.y);
                if (r < 0) {
                    --q;
                    r += (int32_t)info.y;
                } else if (r >= (int32_t)info.y) {
                    ++q;
                    r -= (int32_t)info.y;
                }
                const int t = (int)((info.x >> 16) + q) * tiles_x + (int)(info.x & 0xffffu) + r;
                if (k < total && o < A.capacity) {
                    uint32_t rank;
                    if constexpr (LDS) {
                        const int sh = (t & 1) * 16;
                        rank = (atomicAdd(&s_cnt[t >> 1], 1u << sh) >> sh) & 0xffffu;
                    } else {
                        rank = atomicAdd(&A.table[(row + t) * A.stride], 1u);
                    }
                    A.inst_gid[o] = (int32_t)who.x;
                    A.depth_e[o] = who.y;
                    A.cell_e[o] = (uint32_t)(row + t);
                    A.rank_e[o] = rank;
                }
            }
            head += ng;
            // the next group rewrites this wavefront's LDS
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        // one round per 64 pairs (the next ones' counts in flight), and a
        // last one for what is left in the queue
        const int32_t* pairs = pairs_of(j);
        const int live = live_of(j);
        int32_t next = tiles_of(pairs, live, 0);
        for (int k = 0; k <= A.items; ++k) {
            const int32_t c = next;
            next = tiles_of(pairs, live, k + 1);
            const uint32_t incl = (uint32_t)wave_add_scan(c);
            const uint64_t m = __builtin_amdgcn_ballot_w64(c > 0);
            if (c > 0) {
                const int before = __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                const int q = (tail + before) & (EM_RING - 1);
                s_qpair[wave][q] = (uint16_t)(k * kWave + lane);
                s_qfirst[wave][q] = run + incl - (uint32_t)c;
            }
            run += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
            tail += (int)__popcll(m);
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            const int ng = min(tail - head, kWave);
            if (ng == kWave || (k == A.items && ng > 0)) emit(ng);
        }
        done += tot_i;
    }
    if constexpr (LDS) {
        __syncthreads();
        for (int i = tid; i < tiles_v; i += EM_THREADS)
            A.table[row + i] = (s_cnt[i >> 1] >> ((i & 1) * 16)) & 0xffffu;
    }
}

// ----------------------------------------------------------------------------
// tile ranges and placement
// ----------------------------------------------------------------------------
// [start, end) of every tile (0, 0 where it has no instance, and everywhere
// when a wait gave up), and each table entry <- the first place of its
// instances: a single-pass scan over blocks of `rounds` groups of 64 tiles.
// A group's tiles lie across the lanes of a wavefront, its chunks are shared
// out over the wavefronts.
__global__ void __launch_bounds__(SC_THREADS) k_tile_scan(uint32_t* table, const gs_view* views,
                                                          int n_views, int tile, int per_view, int tiles, int rounds,
                                                          int2* ranges, BinState* st, LbGiveUp gu) {
    __shared__ uint32_t s_part[SC_WAVES][kWave];
    __shared__ uint32_t s_at[kWave];
    __shared__ uint32_t s_sum;
    __shared__ uint64_t s_prefix;
    __shared__ int s_block;
    const int b = lb_ticket(&st->scan_ticket, &s_block);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const bool off = *gu.flag != 0;  // of an earlier launch
    const int seg = (per_view + SC_WAVES - 1) / SC_WAVES;
    const int r0 = min(wave * seg, per_view), r1 = min(r0 + seg, per_view);
    constexpr int KEEP = 16;
    uint32_t c[KEEP];
    int64_t col = 0, step = 0;  // this lane's column: its entry of row 0, the distance of the rows
    // the column sums of group r by wavefront, in s_part; the first KEEP of
    // the wavefront's entries stay in c
    auto group_sums = [&](int r) {
        const int64_t t = ((int64_t)b * rounds + r) * kWave + lane;
        const bool in = !off && t < tiles;
        if (in) {
            const int v = view_of_tile(views, n_views, (int)t);
            const gs_view& vw = views[v];
            const int tiles_v = ceil_div(vw.width, tile) * ceil_div(vw.height, tile);
            col = table_row(vw, per_view, 0, tiles_v) + (t - vw.tile_offset);
            step = tiles_v;
        }
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < KEEP; ++k) {
            c[k] = in && r0 + k < r1 ? table[col + (r0 + k) * step] : 0u;
            sum += c[k];
        }
        if (in)
            for (int q = r0 + KEEP; q < r1; ++q) sum += table[col + q * step];
        s_part[wave][lane] = sum;
        __syncthreads();
    };
    uint32_t total = 0;  // of the block (wavefront 0)
    for (int r = 0; r < rounds; ++r) {
        group_sums(r);
        if (wave == 0) {
            uint32_t x = 0;
            for (int w = 0; w < SC_WAVES; ++w) x += s_part[w][lane];
            total += wave_sum_u32(x, lane);
        }
        if (rounds > 1) __syncthreads();
    }
    uint32_t start = (uint32_t)lb_exchange(total, b, st->scan_status, &s_prefix, gu);
    for (int r = 0; r < rounds; ++r) {
        if (rounds > 1) group_sums(r);
        const int64_t t = ((int64_t)b * rounds + r) * kWave + lane;
        if (wave == 0) {
            uint32_t x = 0;
            for (int w = 0; w < SC_WAVES; ++w) x += s_part[w][lane];
            const uint32_t incl = (uint32_t)wave_add_scan((int)x);
            const uint32_t at = start + incl - x;
            s_at[lane] = at;
            if (lane == kWave - 1) s_sum = incl;
            if (t < tiles) ranges[t] = x > 0 ? make_int2((int)at, (int)(at + x)) : make_int2(0, 0);
        }
        __syncthreads();
        if (!off && t < tiles) {
            uint32_t at = s_at[lane];
            for (int w = 0; w < wave; ++w) at += s_part[w][lane];
#pragma unroll
            for (int k = 0; k < KEEP; ++k) {
                if (r0 + k < r1) table[col + (r0 + k) * step] = at;
                at += c[k];
            }
            for (int q = r0 + KEEP; q < r1; ++q) {
                const uint32_t x = table[col + q * step];
                table[col + q * step] = at;
                at += x;
            }
        }
        start += s_sum;
        __syncthreads();
    }
}

// The same for a table of one entry per tile: a thread takes SC_ITEMS tiles a
// round, instead of one column of which 15 of 16 wavefronts have no row (a
// 16384x16384 view at tile 16, 1 M tiles: 11 us, 253 that way).
constexpr int SC_ITEMS = 8, SC_ROUND = SC_THREADS * SC_ITEMS;
__global__ void __launch_bounds__(SC_THREADS) k_tile_scan_one(uint32_t* table, int stride, int tiles, int rounds,
                                                              int2* ranges, BinState* st, LbGiveUp gu) {
    __shared__ uint32_t s_tmp[SC_WAVES];
    __shared__ uint64_t s_prefix;
    __shared__ int s_block;
    const int b = lb_ticket(&st->scan_ticket, &s_block);
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid / kWave;
    const bool off = *gu.flag != 0;  // of an earlier launch
    // the counts of round r: item k of the thread is tile tile_of(r, k)
    auto tile_of = [&](int r, int k) {
        return ((int64_t)b * rounds + r) * SC_ROUND + wave * (kWave * SC_ITEMS) + k * kWave + lane;
    };
    uint32_t c[SC_ITEMS];
    auto load = [&](int r) {
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < SC_ITEMS; ++k) {
            const int64_t t = tile_of(r, k);
            c[k] = !off && t < tiles ? table[t * stride] : 0u;
            sum += c[k];
        }
        return sum;
    };
    uint32_t total = 0, tot;
    for (int r = 0; r < rounds; ++r) {
        block_exclusive<SC_THREADS>(load(r), s_tmp, &tot);
        total += tot;
    }
    uint32_t start = (uint32_t)lb_exchange(total, b, st->scan_status, &s_prefix, gu);
    for (int r = 0; r < rounds; ++r) {
        const uint32_t e = block_exclusive<SC_THREADS>(load(r), s_tmp, &tot);
        uint32_t at = start + (uint32_t)__builtin_amdgcn_readlane((int)e, 0);  // the lanes' tiles are interleaved
#pragma unroll
        for (int k = 0; k < SC_ITEMS; ++k) {
            const int64_t t = tile_of(r, k);
            const uint32_t incl = (uint32_t)wave_add_scan((int)c[k]), p = at + incl - c[k];
            at += (uint32_t)__builtin_amdgcn_readlane((int)incl, kWave - 1);
            if (t < tiles) {
                ranges[t] = c[k] > 0 ? make_int2((int)p, (int)(p + c[k])) : make_int2(0, 0);
                if (stride == 1) table[t] = p;
            }
        }
        start += tot;
    }
}

// Every instance's sort key, (depth bits << 32 | emission index), to its
// place in its tile's list.
constexpr int PL_THREADS = 256, PL_ITEMS = 4;
__global__ void __launch_bounds__(PL_THREADS) k_place(const uint32_t* __restrict__ cell_e,
                                                      const uint32_t* __restrict__ rank_e,
                                                      const uint32_t* __restrict__ depth_e,
                                                      const uint32_t* __restrict__ table, int stride,
                                                      const BinState* __restrict__ st, int64_t capacity,
                                                      uint64_t* __restrict__ slab,
                                                      const uint32_t* __restrict__ gave_up) {
    const int64_t I = st->placed;
    if (*gave_up) return;
    // XCD x takes the x-th eighth of the instances: with several views the
    // lists they go to are then few enough to be filled in its own L2 (eight
    // 1200x680 views: 30 us, 46 with the instances dealt to all XCDs)
    constexpr int64_t TILE = PL_THREADS * PL_ITEMS;
    const int64_t share = (I + kXcds * TILE - 1) / (kXcds * TILE) * TILE;
    const int64_t x0 = (int64_t)(blockIdx.x & (kXcds - 1)) * share, x1 = x0 + share < I ? x0 + share : I;
    for (int64_t b0 = x0 + (int64_t)(blockIdx.x / kXcds) * TILE; b0 < x1; b0 += (int64_t)(gridDim.x / kXcds) * TILE) {
        uint32_t ci[PL_ITEMS], rk[PL_ITEMS], d[PL_ITEMS];
#pragma unroll
        for (int k = 0; k < PL_ITEMS; ++k) {
            const int64_t e = b0 + k * PL_THREADS + threadIdx.x;
            const int64_t ec = e < x1 ? e : x1 - 1;
            ci[k] = cell_e[ec];
            rk[k] = rank_e[ec];
            d[k] = depth_e[ec];
        }
#pragma unroll
        for (int k = 0; k < PL_ITEMS; ++k) {
            const int64_t e = b0 + k * PL_THREADS + threadIdx.x;
            const int64_t p = (int64_t)table[(size_t)ci[k] * stride] + rk[k];
            if (e < x1 && p < capacity) slab[p] = ((uint64_t)d[k] << 32) | (uint64_t)e;
        }
    }
}

// ----------------------------------------------------------------------------
// per-tile sort
// ----------------------------------------------------------------------------
// Each tile's keys (depth bits << 32 | emission index; depths are positive, so
// the bits order like the values) in ascending order: distinct keys, so any
// correct sort is the one.  A list is cut into runs of 64 keys, one key per
// lane; each run is sorted across the lanes of a wavefront by a bitonic
// network; the rank of a key among up to eight runs (a chunk of 512) is its
// lane plus, for every other run, the number of that run's keys below it (a
// 6-step binary search in LDS); chunks of a longer list merge the same way
// (8- or 9-step searches in the other sorted chunks).  k_tile_sort_short
// gives each list of up to kTsShort one wavefront and queues the longer ones
// for k_tile_sort_long, which gives each up to kTsLong a workgroup; beyond
// that, one workgroup sorts each kTsLong keys of it, and pairs of sorted runs
// are merged, level by level, a workgroup for each kTsLong keys that come out.
constexpr int kTsShort = 512, kTsLong = 4096;
constexpr int kTsChunk = 512;  // keys a wavefront sorts at once (8 runs of 64)

constexpr int TSS_THREADS = kWave;  // short lists: one wavefront per tile
constexpr int TSL_THREADS = 256;    // long lists: one workgroup per kTsLong keys
constexpr uint64_t kNoKey = ~0ull;  // padding, above every real key

template <int J>
__device__ __forceinline__ uint64_t lane_xor_u64(uint64_t v, int lane) {
    const uint32_t lo = lane_xor_u32<J>((uint32_t)v, lane);
    const uint32_t hi = lane_xor_u32<J>((uint32_t)(v >> 32), lane);
    return ((uint64_t)hi << 32) | lo;
}

// Bitonic sort of one key per lane: afterwards lane l holds the l-th
// smallest of the wavefront's 64 keys.  Blocks of SIZE = 2, 4, ..., 64, each
// merged by compare-exchanges at distances J = SIZE/2, ..., 1; in each, the
// lane with bit J clear keeps the smaller key inside an ascending block (bit
// SIZE clear) and the larger inside a descending one.
template <int SIZE, int J>
__device__ __forceinline__ uint64_t bitonic_merge(uint64_t x, int lane) {
    const uint64_t y = lane_xor_u64<J>(x, lane);
    const bool keep_min = ((lane & J) == 0) == ((lane & SIZE) == 0);
    x = keep_min ? (y < x ? y : x) : (y > x ? y : x);
    if constexpr (J > 1) x = bitonic_merge<SIZE, J / 2>(x, lane);
    return x;
}

template <int SIZE>
__device__ __forceinline__ uint64_t bitonic_sort(uint64_t x, int lane) {
    if constexpr (SIZE > 2) x = bitonic_sort<SIZE / 2>(x, lane);
    return bitonic_merge<SIZE, SIZE / 2>(x, lane);
}

__device__ __forceinline__ uint64_t wave_bitonic_u64(uint64_t x, int lane) { return bitonic_sort<kWave>(x, lane); }

// Number of keys of the sorted array a[0 .. 2^LOG) below `key`
// (branch-free binary search; a is padded with kNoKey).
template <int LOG>
__device__ __forceinline__ int count_below(const uint64_t* a, uint64_t key) {
    int p = 0;
#pragma unroll
    for (int s = 1 << (LOG - 1); s > 0; s >>= 1) p += a[p + s - 1] < key ? s : 0;
    return p + (a[p] < key ? 1 : 0);
}

// One wavefront sorts the keys k[0 .. R) (run r holds list positions
// r*64 .. r*64+63, kNoKey past the end): every run across the lanes, the
// runs stored in s_run, then each key's rank among all R runs.  Returns, in
// k[r], the sorted keys of run r and, in rank[r], their ranks in the chunk.
template <int R>
__device__ __forceinline__ void wave_sort_chunk(uint64_t (&k)[8], int (&rank)[8], uint64_t* s_run, int lane) {
#pragma unroll
    for (int r = 0; r < R; ++r) {
        k[r] = wave_bitonic_u64(k[r], lane);
        s_run[r * kWave + lane] = k[r];
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
    for (int r = 0; r < R; ++r) {
        int rk = lane;
#pragma unroll
        for (int r2 = 0; r2 < R; ++r2)
            if (r2 != r) rk += count_below<6>(s_run + r2 * kWave, k[r]);
        rank[r] = rk;
    }
}

// Runs R of a chunk of n keys, dispatched to a compile-time count.
__device__ __forceinline__ void wave_sort_chunk_n(int n, uint64_t (&k)[8], int (&rank)[8], uint64_t* s_run,
                                                  int lane) {
    switch ((n + kWave - 1) / kWave) {
        case 1: wave_sort_chunk<1>(k, rank, s_run, lane); break;
        case 2: wave_sort_chunk<2>(k, rank, s_run, lane); break;
        case 3: wave_sort_chunk<3>(k, rank, s_run, lane); break;
        case 4: wave_sort_chunk<4>(k, rank, s_run, lane); break;
        case 5: wave_sort_chunk<5>(k, rank, s_run, lane); break;
        case 6: wave_sort_chunk<6>(k, rank, s_run, lane); break;
        case 7: wave_sort_chunk<7>(k, rank, s_run, lane); break;
        default: wave_sort_chunk<8>(k, rank, s_run, lane); break;
    }
}

// Part `part` of a list of more than kTsLong keys, slab[begin .. begin + len).
// The parts of one list are consecutive; `first` is the index of the first of
// them, and done[first] counts those that are through a level.
struct ListPart {
    int32_t tile, part, first, begin, len;
};
__device__ __forceinline__ int log2_ceil(int n) { return n > 1 ? 32 - __clz(n - 1) : 0; }

// Tiles in the XCD-aware order of the compositing launches (tile_of_block).
// After a wait gave up, every list is left empty.
__global__ void __launch_bounds__(TSS_THREADS) k_tile_sort_short(int2* __restrict__ ranges, int total_tiles,
                                                                  int run_log2, const uint64_t* __restrict__ slab,
                                                                  uint32_t* __restrict__ tile_keys,
                                                                  int32_t* __restrict__ inst,
                                                                  uint32_t* __restrict__ wholes,
                                                                  ListPart* __restrict__ list_parts,
                                                                  uint32_t* __restrict__ done, BinState* st,
                                                                  const uint32_t* __restrict__ gave_up) {
    static_assert(kTsShort == kTsChunk && kTsChunk == 8 * kWave, "a short list is one chunk of eight runs");
    __shared__ uint64_t s_run[kTsChunk];
    const int t = tile_of_block(blockIdx.x, total_tiles, run_log2);
    if (t < 0) return;
    const int lane = threadIdx.x;
    if (*gave_up) {
        if (lane == 0) ranges[t] = make_int2(0, 0);
        return;
    }
    const int2 rg = ranges[t];
    const int L = rg.y - rg.x;
    if (L <= 0) return;
    if (L > kTsShort) {  // uniform across the wavefront: left to k_tile_sort_long
        if (L <= kTsLong) {
            if (lane == 0) wholes[atomicAdd(&st->wholes, 1u)] = (uint32_t)t;
            return;
        }
        const uint32_t parts = (uint32_t)(L + kTsLong - 1) / kTsLong;
        uint32_t at = 0;
        if (lane == 0) {
            at = atomicAdd(&st->parts, parts);
            done[at] = 0;
            atomicMax(&st->levels, (uint32_t)log2_ceil((int)parts));
        }
        at = (uint32_t)__builtin_amdgcn_readlane((int)at, 0);
        for (uint32_t k = lane; k < parts; k += kWave) list_parts[at + k] = {t, (int)k, (int)at, rg.x, L};
        return;
    }
    const uint64_t* in = slab + rg.x;
    uint64_t k[8];
    int rank[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        const int i = r * kWave + lane;
        k[r] = i < L ? in[i] : kNoKey;
    }
    wave_sort_chunk_n(L, k, rank, s_run, lane);
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        if (r * kWave < L && k[r] != kNoKey) inst[rg.x + rank[r]] = (int32_t)(uint32_t)k[r];
        if (r * kWave + lane < L) tile_keys[rg.x + r * kWave + lane] = (uint32_t)t;
    }
}

struct LongLds {
    uint64_t sorted[kTsLong];
    uint64_t run[TSL_THREADS / kWave][kTsChunk];
};

// The L (<= kTsLong) keys at `in`, sorted by the whole block: put(place, key)
// is called for each.
template <class Put>
__device__ __forceinline__ void sort_long_chunk(const uint64_t* __restrict__ in, int L, LongLds& S, Put put) {
    constexpr int NW = TSL_THREADS / kWave;
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    // chunks of 256 keys (four runs) up to 1024, so that all four wavefronts
    // sort; of 512 beyond, where more chunks would make the final merge's
    // searches the larger cost
    const bool small = L <= 4 * (kTsChunk / 2);
    const int CH = small ? kTsChunk / 2 : kTsChunk;
    const int nchunk = (L + CH - 1) / CH;
    for (int c = wave; c < nchunk; c += NW) {
        const int c0 = c * CH;
        const int nc = min(CH, L - c0);
        uint64_t k[8];
        int rank[8];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const int i = c0 + r * kWave + lane;
            k[r] = r * kWave < CH && i < L ? in[i] : kNoKey;
        }
        wave_sort_chunk_n(nc, k, rank, S.run[wave], lane);
#pragma unroll
        for (int r = 0; r < 8; ++r)
            if (r * kWave + lane < nc) S.sorted[c0 + rank[r]] = k[r];
        // pad the last chunk to a full CH for the searches
        for (int i = nc + lane; i < CH; i += kWave) S.sorted[c0 + i] = kNoKey;
        // S.run is rewritten by this wavefront's next chunk
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    __syncthreads();
    for (int j = threadIdx.x; j < L; j += TSL_THREADS) {
        const uint64_t key = S.sorted[j];
        const int c = j / CH;
        int pos = j - c * CH;
        for (int c2 = 0; c2 < nchunk; ++c2) {
            if (c2 == c) continue;
            pos += small ? count_below<8>(S.sorted + c2 * CH, key) : count_below<9>(S.sorted + c2 * CH, key);
        }
        put(pos, key);
    }
}

// Number of keys of the ascending a[0 .. n) below `key`.
__device__ __forceinline__ int lower_bound(const uint64_t* a, int n, uint64_t key) {
    int lo = 0;
    while (n > 0) {
        const int h = n >> 1;
        const bool below = a[lo + h] < key;
        lo = below ? lo + h + 1 : lo;
        n = below ? n - h - 1 : h;
    }
    return lo;
}

// How many of the first d keys of the merge of a[0 .. na) and b[0 .. nb) are
// a's, by a whole wavefront: 64 candidates a round.
__device__ __forceinline__ int merge_split(const uint64_t* a, int na, const uint64_t* b, int nb, int d) {
    const int lane = threadIdx.x & (kWave - 1);
    int lo = d > nb ? d - nb : 0, hi = d < na ? d : na;
    while (lo < hi) {
        const int step = (hi - lo + kWave - 1) / kWave, m = lo + lane * step;
        // true up to the last candidate below the answer (m < na and
        // 0 <= d - 1 - m < nb in [lo, hi))
        const int c = (int)__popcll(__ballot(m < hi && a[m] < b[d - 1 - m]));
        if (c == 0) return lo;
        hi = min(hi, lo + c * step);
        lo += (c - 1) * step + 1;
    }
    return lo;
}

// The queued lists.  A fixed grid of workgroups takes tickets: the parts'
// sorts, the whole lists, then the levels of the merges, every part once in
// each.  A merge waits until all parts of its list are through the level
// before, whose tickets are earlier.  Level l merges pairs of runs of
// kTsLong 2^(l-1) keys between slab and slab2 (the last one into inst): the
// workgroup's kTsLong keys of the result are a stretch of either run, which it
// finds by bisection and merges in LDS.  (Each key looked up in every other
// part of its list in memory, and every wavefront fencing for itself, took 9.7
// ms for four lists of 717 k keys and 11.4 for 336 of 54 k, now 0.6 and 2.1; one
// workgroup's counting passes over a list, before that, 21.0 and 5.4.)
__global__ void __launch_bounds__(TSL_THREADS) k_tile_sort_long(int2* __restrict__ ranges,
                                                                 const uint32_t* __restrict__ wholes,
                                                                 const ListPart* __restrict__ list_parts,
                                                                 uint32_t* done, BinState* st, uint64_t* slab,
                                                                 uint64_t* slab2, uint32_t* __restrict__ tile_keys,
                                                                 int32_t* __restrict__ inst, LbGiveUp gu) {
    __shared__ LongLds S;
    __shared__ int s_item;
    __shared__ int s_ok;
    __shared__ int s_split[2];
    const int n_parts = (int)st->parts, n_wholes = (int)st->wholes;
    const int64_t count = n_wholes + (int64_t)n_parts * (1 + (int)st->levels);
    if (count == 0) return;
    // the workgroup's writes are visible to the next level before they count:
    // the barrier orders them before thread 0's release, which (one per
    // workgroup, not one per wavefront) writes the XCD's L2 back
    auto through = [&](int first) {
        __syncthreads();
        if (threadIdx.x == 0) __hip_atomic_fetch_add(done + first, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
    };
    for (;;) {
        __syncthreads();  // the LDS is reused by the next entry
        const int item = lb_ticket(&st->long_ticket, &s_item);
        if (item >= count) return;
        if (item >= n_parts && item < n_parts + n_wholes) {
            const uint32_t tile = wholes[item - n_parts];
            const int2 rg = ranges[tile];
            sort_long_chunk(slab + rg.x, rg.y - rg.x, S, [&](int pos, uint64_t key) {
                inst[rg.x + pos] = (int32_t)(uint32_t)key;
                tile_keys[rg.x + pos] = tile;
            });
            continue;
        }
        const int m = item - n_parts - n_wholes;
        const int level = item < n_parts ? 0 : m / n_parts + 1;
        const ListPart lp = list_parts[item < n_parts ? item : m % n_parts];
        const int p0 = lp.part * kTsLong, np = min(kTsLong, lp.len - p0);
        if (level == 0) {
            // in place: every key is in LDS before the first is written
            uint64_t* mine = slab + lp.begin + p0;
            sort_long_chunk(mine, np, S, [&](int pos, uint64_t key) { mine[pos] = key; });
            through(lp.first);
            continue;
        }
        const int parts = (lp.len + kTsLong - 1) / kTsLong, levels = log2_ceil(parts);
        if (level > levels) continue;
        if (threadIdx.x == 0) {
            const auto ready = [&] {
                return (int)__hip_atomic_load(done + lp.first, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >=
                       parts * level;
            };
            bool ok = ready();
            const int spins = __hip_atomic_load(gu.flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ? 0 : gu.spin_limit;
            for (int spin = 0; !ok && spin < spins; ++spin) ok = ready();
            if (!ok) {  // the list is left empty; the caller discards the call's results
                give_up(gu);
                ranges[lp.tile] = make_int2(0, 0);
            }
            s_ok = ok;
            // the whole workgroup reads the other parts after this and the barrier
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        if (!s_ok) continue;
        const uint64_t* src = ((level & 1) ? slab : slab2) + lp.begin;
        const int run = kTsLong << (level - 1), r0 = (lp.part >> level << level) * kTsLong;
        const int na = min(run, lp.len - r0), nb = min(run, max(lp.len - r0 - run, 0)), d = p0 - r0;
        const uint64_t *a = src + r0, *b = a + run;
        const int wave = threadIdx.x / kWave;
        if (wave < 2) {
            const int i = merge_split(a, na, b, nb, d + wave * np);
            if ((threadIdx.x & (kWave - 1)) == 0) s_split[wave] = i;
        }
        __syncthreads();
        const int i0 = s_split[0], ca = s_split[1] - i0, cb = np - ca;
        for (int j = threadIdx.x; j < np; j += TSL_THREADS) S.sorted[j] = j < ca ? a[i0 + j] : b[d - i0 + (j - ca)];
        __syncthreads();
        uint64_t* dst = ((level & 1) ? slab2 : slab) + lp.begin + p0;
        for (int j = threadIdx.x; j < np; j += TSL_THREADS) {
            const uint64_t key = S.sorted[j];
            const int pos = j < ca ? j + lower_bound(S.sorted + ca, cb, key) : j - ca + lower_bound(S.sorted, ca, key);
            if (level < levels) {
                dst[pos] = key;
            } else {
                inst[lp.begin + p0 + pos] = (int32_t)(uint32_t)key;
                tile_keys[lp.begin + p0 + pos] = (uint32_t)lp.tile;
            }
        }
        if (level < levels) through(lp.first);
    }
}

struct WsLayout {
    size_t slab, cell_e, rank_e, depth_e, inst_sums, vis_sums, state, wholes, parts, done, table, total;
    int64_t table_words;
};

// Chunks of a view of n pairs: of 256 pairs while the look-back reaches
// over all of them, of 1024 up to a workgroup per CU, then 4096, then 16384 or,
// where those would be more than a thousand, EM_CHUNK, so that their table
// stays small.  (Few pairs can be many instances, which two chunks of 1024 would
// leave to two workgroups: of 2000 Gaussians that reach most of a 1200x680
// view, 6.4 M instances, the binning takes 720 us instead of 1970.  Chunks of 64
// pairs: 370, but 3 us more for 1000 Gaussians in a 64x64 view.)
// lds: k_emit counts in LDS (a chunk's tiles fit there and the table, with
// larger chunks where it has to be, in table_words).
struct Chunks {
    int64_t chunk;
    int per_view, per_wave;
    bool lds;
};
Chunks chunks_of(int n, int n_views, int64_t total_tiles, int max_tiles, int64_t table_words) {
    auto per_view = [&](int64_t c) { return (int)((n + c - 1) / c); };
    auto count = [&](int64_t c) { return (int64_t)n_views * per_view(c); };
    auto fits = [&](int64_t c) { return per_view(c) * total_tiles <= table_words; };
    int64_t c = EM_CHUNK;
    if (count(256) <= EM_LOOKBACK) c = 256;
    else if (count(1024) <= 256) c = 1024;
    else if (count(4096) <= 512) c = 4096;
    else if (count(EM_PASS) <= 1024) c = EM_PASS;
    int64_t larger = c;
    while (!fits(larger) && larger < EM_CHUNK) larger *= 2;
    const bool lds = max_tiles <= EM_LDS_TILES && fits(larger);
    if (lds) c = larger;
    return {c, per_view(c), (int)(c < EM_PASS ? c : EM_PASS) / EM_WAVES, lds};
}

WsLayout ws_layout(int n, int n_views, int64_t capacity) {
    auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
    const int64_t vn = (int64_t)n * n_views;
    const size_t cap = (size_t)(capacity > 0 ? capacity : 1);
    const size_t chunks = (size_t)n_views * (size_t)((n + 1023) / 1024);  // that need sums, at most
    // a list of L > kTsLong keys has ceil(L / kTsLong) <= L / (kTsLong / 2) parts
    const size_t wholes = cap / (kTsShort + 1) + 1, parts = cap / (kTsLong / 2) + 1;
    WsLayout L;
    // the (chunk, tile) table: the tiles are not known here, so four words per
    // pair, at most 16 MB, or a byte per instance, at most 128 MB (few pairs
    // with many instances reach many tiles), and 4 MB at least; a call whose
    // tiles need more takes larger chunks or counts in memory
    const int64_t by_pairs = 4 * vn < (4 << 20) ? 4 * vn : (4 << 20);
    const int64_t want = by_pairs > (int64_t)cap / 4 ? by_pairs : (int64_t)cap / 4;
    L.table_words = want < (1 << 20) ? (1 << 20) : (want > (32 << 20) ? (32 << 20) : want);
    size_t o = 0;
    L.slab = o; o += al(8 * cap);
    L.cell_e = o; o += al(4 * cap);  // these two, read for the last time by k_place, are slab2 of the merges
    L.rank_e = o; o += al(4 * cap);
    L.depth_e = o; o += al(4 * cap);
    L.inst_sums = o; o += al(4 * chunks);
    L.vis_sums = o; o += al(4 * chunks);
    L.state = o; o += al(sizeof(BinState));
    L.wholes = o; o += al(4 * wholes);
    L.parts = o; o += al(sizeof(ListPart) * parts);
    L.done = o; o += al(4 * parts);
    L.table = o; o += al(4 * (size_t)L.table_words);
    L.total = o;
    return L;
}

}  // namespace

size_t binsort_workspace_bytes(int n, int n_views, int64_t capacity) { return ws_layout(n, n_views, capacity).total; }

// Reads a wait may take before it gives up (LB_SPIN_MAX, or the value of
// SGS_LOOKBACK_SPIN, which tests set to force the give-up path).
int lookback_spin_limit() {
    const char* v = std::getenv("SGS_LOOKBACK_SPIN");
    if (v == nullptr || *v == 0) return LB_SPIN_MAX;
    const long x = std::strtol(v, nullptr, 10);
    return x < 0 ? 0 : (x > LB_SPIN_MAX ? LB_SPIN_MAX : (int)x);
}

hipError_t launch_binsort(const uint32_t* rect, const int32_t* touched, int n,
                          const gs_view* views_dev, int n_views, int total_tiles, int max_tiles, int tile, void* ws,
                          int64_t capacity, uint32_t* tile_keys, int32_t* inst, int32_t* inst_gid,
                          int32_t* pair_first, int32_t* ranges, int64_t* counts, hipStream_t s) {
    if (n <= 0 || n_views <= 0 || total_tiles <= 0) return hipErrorInvalidValue;
    const WsLayout L = ws_layout(n, n_views, capacity);
    const Chunks ck = chunks_of(n, n_views, total_tiles, max_tiles, L.table_words);
    char* w = static_cast<char*>(ws);
    auto words = [&](size_t off) { return reinterpret_cast<uint32_t*>(w + off); };
    BinState* st = reinterpret_cast<BinState*>(w + L.state);
    uint64_t* slab = reinterpret_cast<uint64_t*>(w + L.slab);
    ListPart* parts = reinterpret_cast<ListPart*>(w + L.parts);
    uint32_t* done = words(L.done);
    int2* rg = reinterpret_cast<int2*>(ranges);

    // a wait past the spin limit (SGS_LOOKBACK_SPIN overrides it, for tests)
    // records the give-up in counts[3] and counts[4]
    LbGiveUp gu;
    gu.flag = reinterpret_cast<uint32_t*>(counts + 3);
    gu.sticky = reinterpret_cast<uint32_t*>(counts + 4);
    gu.spin_limit = lookback_spin_limit();

    EmitArgs A;
    A.touched = touched;
    A.rect = reinterpret_cast<const uint4*>(rect);
    A.views = views_dev;
    A.n = n;
    A.n_views = n_views;
    A.tile = tile;
    A.per_view = ck.per_view;
    A.chunk = ck.chunk;
    A.capacity = capacity;
    A.per_wave = ck.per_wave;
    A.items = (ck.per_wave + kWave - 1) / kWave;
    A.inst_sums = words(L.inst_sums);
    A.vis_sums = words(L.vis_sums);
    A.st = st;
    // counted in memory, the table has one entry per tile; where that does not
    // fit, the first words of the tile ranges
    const int rows = ck.lds ? ck.per_view : 1;
    const bool own = (int64_t)rows * total_tiles <= L.table_words;
    A.table = own ? words(L.table) : reinterpret_cast<uint32_t*>(ranges);
    A.stride = own ? 1 : 2;
    const int64_t clear = ck.lds ? 0 : (int64_t)total_tiles * A.stride;
    A.cell_e = words(L.cell_e);
    A.rank_e = words(L.rank_e);
    A.depth_e = words(L.depth_e);
    A.inst_gid = inst_gid;
    A.pair_first = pair_first;
    A.counts = counts;
    A.gu = gu;
    // 1. and 2.
    const size_t lds = ck.lds ? 4 * (((size_t)max_tiles + 1) / 2) : 0;
    const unsigned chunks = (unsigned)(n_views * ck.per_view);
    const dim3 eb(EM_THREADS);
    if (chunks <= EM_LOOKBACK) {
        const int64_t rb = (clear + 4095) / 4096;
        hipLaunchKernelGGL(k_bin_reset, dim3((unsigned)(rb < 8 ? 8 : (rb < 1024 ? rb : 1024))), dim3(256), 0, s, st,
                           counts, A.table, clear);
        hipLaunchKernelGGL((ck.lds ? k_emit<true, true> : k_emit<true, false>), dim3(chunks), eb, lds, s, A);
    } else {
        hipLaunchKernelGGL(k_chunk_sums, dim3(chunks), eb, 0, s, touched, n, ck.per_view, ck.chunk,
                           words(L.inst_sums), words(L.vis_sums), st, counts, A.table, clear);
        hipLaunchKernelGGL((ck.lds ? k_emit<false, true> : k_emit<false, false>), dim3(chunks), eb, lds, s, A);
    }
    // 3.
    const int64_t round = rows > 1 ? kWave : SC_ROUND;
    int rounds = 1;
    while (SC_MAXBLK * round * rounds < (int64_t)total_tiles) ++rounds;
    const dim3 sb((unsigned)((total_tiles + round * rounds - 1) / (round * rounds)));
    if (rows > 1)
        hipLaunchKernelGGL(k_tile_scan, sb, dim3(SC_THREADS), 0, s, A.table, views_dev, n_views, tile, rows,
                           total_tiles, rounds, rg, st, gu);
    else
        hipLaunchKernelGGL(k_tile_scan_one, sb, dim3(SC_THREADS), 0, s, A.table, A.stride, total_tiles, rounds, rg, st,
                           gu);
    if (capacity <= 0) return hipGetLastError();
    // 4.
    const int64_t pb = (capacity + PL_THREADS * PL_ITEMS * kXcds - 1) / (PL_THREADS * PL_ITEMS * kXcds);
    hipLaunchKernelGGL(k_place, dim3((unsigned)(pb < 1024 ? pb : 1024) * kXcds), dim3(PL_THREADS), 0, s, A.cell_e,
                       A.rank_e, A.depth_e, A.table, A.stride, st, capacity, slab, gu.flag);
    // 5. and 6. (no list is longer than the Gaussians)
    const int run_log2 = tile_run_log2(tile, total_tiles);
    hipLaunchKernelGGL(k_tile_sort_short, dim3(tile_grid(total_tiles, run_log2)), dim3(TSS_THREADS), 0, s, rg,
                       total_tiles, run_log2, slab, tile_keys, inst, words(L.wholes), parts, done, st, gu.flag);
    if (n > kTsShort) {
        const int64_t max_long = capacity / (kTsShort + 1) + 1;
        hipLaunchKernelGGL(k_tile_sort_long, dim3((unsigned)(max_long < 768 ? max_long : 768)), dim3(TSL_THREADS), 0,
                           s, rg, words(L.wholes), parts, done, st, slab, reinterpret_cast<uint64_t*>(w + L.cell_e),
                           tile_keys, inst, gu);
    }
    return hipGetLastError();
}

}  // namespace sgs
