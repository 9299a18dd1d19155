// Wavefront- and workgroup-level building blocks for gfx950 (64-wide wavefronts) and the two device-wide
// primitives the planner and the backward pass share: a tiled scan and a stable LSD radix sort.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "common.h"

namespace bp {

// ---------------------------------------------------------------------------------------------
// wavefront helpers
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return threadIdx.x & (kWave - 1); }

__device__ __forceinline__ uint64_t lanemask_lt() { return (uint64_t(1) << lane_id()) - 1; }

struct AddOp {
    template <typename T>
    __device__ __forceinline__ T operator()(T a, T b) const { return a + b; }
};
// Lane movements as operands of vector instructions (DPP) instead of trips through the LDS (what __shfl compiles to).
// CTRL names the movement; a lane without a source, or in a row that ROWS leaves out, keeps `old`.
template <int CTRL, int ROWS, typename T>
__device__ __forceinline__ T dpp_move(T old, T x) {
    static_assert(sizeof(T) == 4 || sizeof(T) == 8, "whole registers");
    if constexpr (sizeof(T) == 4) {
        return (T)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, ROWS, 0xf, false);
    } else {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)old, (int)(uint32_t)x, CTRL, ROWS, 0xf, false);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)((uint64_t)old >> 32),
                                                                  (int)(uint32_t)((uint64_t)x >> 32), CTRL, ROWS, 0xf, false);
        return (T)(((uint64_t)hi << 32) | lo);
    }
}
constexpr int kDppRowShr = 0x110, kDppWaveShl1 = 0x130, kDppWaveShr1 = 0x138, kDppRowBcast15 = 0x142, kDppRowBcast31 = 0x143;

// The value of the lane below; lane 0 gets `first`.
template <typename T>
__device__ __forceinline__ T lane_below(T x, T first) {
    return dpp_move<kDppWaveShr1, 0xf>(first, x);
}
// The value of the lane above; the last lane gets `last`.
template <typename T>
__device__ __forceinline__ T lane_above(T x, T last) {
    return dpp_move<kDppWaveShl1, 0xf>(last, x);
}
// The value of lane `from` (the same in every lane).
template <typename T>
__device__ __forceinline__ T lane_value(T x, int from) {
    if constexpr (sizeof(T) == 4) {
        return (T)__builtin_amdgcn_readlane((int)x, from);
    } else {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, from);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)x >> 32), from);
        return (T)(((uint64_t)hi << 32) | lo);
    }
}

// Integers only, and 0 must be the operation's identity.  Rows of 16 lanes are
// scanned by themselves, then the row totals are passed on to the rows behind.  All 64 lanes take part.
template <typename T, typename Op>
__device__ __forceinline__ T wave_inclusive_scan(T x, Op op) {
    x = op(x, dpp_move<kDppRowShr + 1, 0xf>(T(0), x));
    x = op(x, dpp_move<kDppRowShr + 2, 0xf>(T(0), x));
    x = op(x, dpp_move<kDppRowShr + 4, 0xf>(T(0), x));
    x = op(x, dpp_move<kDppRowShr + 8, 0xf>(T(0), x));
    x = op(x, dpp_move<kDppRowBcast15, 0xa>(T(0), x));
    x = op(x, dpp_move<kDppRowBcast31, 0xc>(T(0), x));
    return x;
}

// Scan of one value per thread over a workgroup of BLOCK threads (BLOCK % 64 == 0), thread order.
// `wave_tot` is LDS scratch of BLOCK/64 entries.  Writes the exclusive and inclusive values and the
// reduction over the whole workgroup.  Ends with a barrier, so wave_tot can be reused at once.
template <int BLOCK, typename T, typename Op>
__device__ __forceinline__ void block_scan(T x, Op op, T identity, T* wave_tot, T* exclusive, T* inclusive,
                                           T* block_total) {
    constexpr int WAVES = BLOCK / kWave;
    const int w = threadIdx.x / kWave, lane = lane_id();
    T inc = wave_inclusive_scan(x, op);
    T exc = lane_below(inc, identity);
    if (lane == kWave - 1) wave_tot[w] = inc;
    __syncthreads();
    T prefix = identity, total = identity;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) {
        T t = wave_tot[i];
        if (i < w) prefix = op(prefix, t);
        total = op(total, t);
    }
    __syncthreads();
    *exclusive = op(prefix, exc);
    *inclusive = op(prefix, inc);
    *block_total = total;
}

// ---------------------------------------------------------------------------------------------
// device-wide scan:  out(i, exclusive_prefix_i, inclusive_prefix_i)  for value_i = in(i), i in [0, n)
//   pass 1  per-tile reduction                   -> partials[tile]
//   pass 2  one workgroup scans the partials in place (exclusive) and appends the grand total; left out where the
//           tiles are few: every workgroup of pass 3 then adds up the partials before its own
//   pass 3  per-tile scan seeded with its partial
// A tile is kScanBlock * ROUNDS consecutive elements; each wavefront owns a contiguous stretch of it and takes it in
// ROUNDS rounds of 64 consecutive elements (lane l holds element r*64 + l of the stretch), so loads coalesce
// and a round is scanned with lane shuffles alone; the workgroup meets at one barrier per tile.
// Op must be associative and commutative, with 0 its identity.
// ---------------------------------------------------------------------------------------------
constexpr int kScanBlock = 256;
// Rounds of a tile by the number of elements.  The rounds of pass 3 follow one another (what `out` fetches for one is
// asked for after the stores of the one before), so small inputs are dealt to as many workgroups as they fill: 40 K
// rows took 12.4 us on 20 workgroups of 8 rounds, 4.4 us on 160 of one.  Large ones take long tiles, which keep the
// partials few.
constexpr int64_t kScanSmall = int64_t(1) << 18, kScanMiddle = int64_t(1) << 21;
inline int scan_rounds(int64_t n) { return n <= kScanSmall ? 1 : n <= kScanMiddle ? 4 : 8; }
// Up to here pass 2 is left out: the partials are 8 KB at most, or 16 KB of 64-bit ones, read from L2 by every workgroup at
// once, where the one workgroup of pass 2 is a launch of its own (2.5 to 4 us, with the gaps on both sides).
constexpr int64_t kScanFewTiles = 2048;

template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T x, Op op) {
    return lane_value(wave_inclusive_scan(x, op), kWave - 1);
}

template <int ROUNDS, typename T, typename Op, typename In>
__global__ __launch_bounds__(kScanBlock) void scan_reduce_kernel(In in, int64_t n, T* partials, Op op, T identity) {
    __shared__ T wave_tot[kScanBlock / kWave];
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int64_t base = (int64_t)blockIdx.x * (kScanBlock * ROUNDS) + w * (kWave * ROUNDS) + lane;
    T acc = identity;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t i = base + r * kWave;
        if (i < n) acc = op(acc, in(i));
    }
    acc = wave_reduce(acc, op);
    if (lane == 0) wave_tot[w] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        T total = identity;
#pragma unroll
        for (int k = 0; k < kScanBlock / kWave; ++k) total = op(total, wave_tot[k]);
        partials[blockIdx.x] = total;
    }
}

// One workgroup: it is the serial part of every scan.  A thread takes kSpinePerThread consecutive partials per round
// and moves them in 16-byte accesses: with one 4-byte access per partial and thread the kernel's time follows the
// number of memory instructions, whatever the rounds (41,600 partials, the spine of a scan over 85 M elements: 42 us
// element by element, 12 us this way).
constexpr int kSpinePerThread = 8;
template <typename T, typename Op>
__global__ __launch_bounds__(1024) void scan_spine_kernel(T* partials, int64_t nparts, Op op, T identity) {
    constexpr int VEC = kSpinePerThread * (int)sizeof(T) / 16;
    static_assert(kSpinePerThread * sizeof(T) % 16 == 0, "a thread's partials are a whole number of 16-byte pieces");
    __shared__ T wave_tot[1024 / kWave];
    const bool aligned = (reinterpret_cast<uintptr_t>(partials) & 15) == 0;
    T carry = identity;
    for (int64_t base = 0; base < nparts; base += 1024 * kSpinePerThread) {
        const int64_t i0 = base + (int64_t)threadIdx.x * kSpinePerThread;
        const bool whole = aligned && i0 + kSpinePerThread <= nparts;
        union {
            T v[kSpinePerThread];
            uint4 q[VEC];
        } mine;
        if (whole) {
            const uint4* src = reinterpret_cast<const uint4*>(partials + i0);
#pragma unroll
            for (int k = 0; k < VEC; ++k) mine.q[k] = src[k];
        } else {
#pragma unroll
            for (int k = 0; k < kSpinePerThread; ++k) mine.v[k] = i0 + k < nparts ? partials[i0 + k] : identity;
        }
        T sum = identity;
#pragma unroll
        for (int k = 0; k < kSpinePerThread; ++k) sum = op(sum, mine.v[k]);
        T exc, inc, total;
        block_scan<1024>(sum, op, identity, wave_tot, &exc, &inc, &total);
        T run = op(carry, exc);
#pragma unroll
        for (int k = 0; k < kSpinePerThread; ++k) {       // every partial becomes the scan of those before it
            const T next = op(run, mine.v[k]);
            mine.v[k] = run;
            run = next;
        }
        if (whole) {
            uint4* dst = reinterpret_cast<uint4*>(partials + i0);
#pragma unroll
            for (int k = 0; k < VEC; ++k) dst[k] = mine.q[k];
        } else {
#pragma unroll
            for (int k = 0; k < kSpinePerThread; ++k)
                if (i0 + k < nparts) partials[i0 + k] = mine.v[k];
        }
        carry = op(carry, total);
    }
    if (threadIdx.x == 0) partials[nparts] = carry;
}

// Pass 3, what comes before a wavefront's stretch.  `mine`: the stretch's own reduction.  SPINE: pass 2 has run.  Without it,
// `partials` holds the bare sums of the tiles, the workgroup adds up those before its own (scan_tiles_before, asked for
// ahead), and the last one writes the grand total behind them (where no other workgroup reads).
template <typename T>
struct ScanShared {
    T wave_tot[kScanBlock / kWave];
    T wave_before[kScanBlock / kWave];
};
template <bool SPINE, typename T, typename Op>
__device__ __forceinline__ T scan_tiles_before(const T* partials, Op op, T identity) {
    T before = identity;
    if constexpr (!SPINE)
        for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kScanBlock) before = op(before, partials[t]);
    return before;
}
template <bool SPINE, typename T, typename Op>
__device__ __forceinline__ T scan_carry(T mine, T before, T* partials, Op op, T identity, ScanShared<T>& sh) {
    constexpr int WAVES = kScanBlock / kWave;
    const int w = threadIdx.x / kWave, lane = lane_id();
    if constexpr (!SPINE) {
        before = wave_reduce(before, op);
        if (lane == 0) sh.wave_before[w] = before;
    }
    if (lane == 0) sh.wave_tot[w] = mine;
    __syncthreads();
    T carry;
    if constexpr (SPINE) {
        carry = partials[blockIdx.x];
    } else {
        carry = identity;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) carry = op(carry, sh.wave_before[k]);
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
            T total = carry;
#pragma unroll
            for (int k = 0; k < WAVES; ++k) total = op(total, sh.wave_tot[k]);
            partials[gridDim.x] = total;
        }
    }
    for (int k = 0; k < w; ++k) carry = op(carry, sh.wave_tot[k]);
    return carry;
}

template <int ROUNDS, bool SPINE, typename T, typename Op, typename In, typename Out>
__global__ __launch_bounds__(kScanBlock) void scan_apply_kernel(In in, Out out, int64_t n, T* partials, Op op, T identity) {
    __shared__ ScanShared<T> sh;
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int64_t base = (int64_t)blockIdx.x * (kScanBlock * ROUNDS) + w * (kWave * ROUNDS) + lane;
    T v[ROUNDS];
    T mine = identity;
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t i = base + r * kWave;
        v[r] = i < n ? in(i) : identity;
    }
    const T before = scan_tiles_before<SPINE>(partials, op, identity);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) mine = op(mine, v[r]);
    T carry = scan_carry<SPINE>(wave_reduce(mine, op), before, partials, op, identity, sh);
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const int64_t i = base + r * kWave;
        const T inc = wave_inclusive_scan(v[r], op);
        const T exc = lane_below(inc, identity);
        if (i < n) out(i, op(carry, exc), op(carry, inc));
        carry = op(carry, lane_value(inc, kWave - 1));
    }
}

inline int64_t scan_num_tiles(int64_t n) { return n > 0 ? ceil_div(n, (int64_t)kScanBlock * scan_rounds(n)) : 1; }
// Partials needed by the scans of up to n elements: one per tile, of which a shorter input may have more, plus the
// grand total.
inline size_t scan_partials(int64_t n) {
    int64_t most = scan_num_tiles(n);
    if (n > kScanSmall) most = std::max(most, scan_num_tiles(kScanSmall));
    if (n > kScanMiddle) most = std::max(most, scan_num_tiles(kScanMiddle));
    return (size_t)most + 1;
}

static_assert(kScanSmall <= kScanFewTiles * kScanBlock && kScanMiddle <= kScanFewTiles * kScanBlock * 4, "no spine for these");
// Passes 2 and 3 behind the per-tile reductions in `partials`.  apply(rounds, spine, grid) launches pass 3.
template <typename T, typename Op, typename Apply>
int scan_finish(int64_t n, T* partials, Op op, T identity, hipStream_t stream, Apply&& apply) {
    const int64_t tiles = scan_num_tiles(n);
    const dim3 grid((unsigned)tiles);
    switch (scan_rounds(n)) {                             // fewer than 8 rounds: at most kScanFewTiles tiles
        case 1: return apply(std::integral_constant<int, 1>{}, std::false_type{}, grid);
        case 4: return apply(std::integral_constant<int, 4>{}, std::false_type{}, grid);
        default: break;
    }
    if (tiles <= kScanFewTiles) return apply(std::integral_constant<int, 8>{}, std::false_type{}, grid);
    BP_LAUNCH(K_SCAN_SPINE, (scan_spine_kernel<T, Op>), dim3(1), dim3(1024), 0, stream, partials, tiles, op, identity);
    return apply(std::integral_constant<int, 8>{}, std::true_type{}, grid);
}

// Pass 1.
template <typename T, typename Op, typename In>
int scan_reduce(In in, int64_t n, T* partials, Op op, T identity, hipStream_t stream) {
    const dim3 grid((unsigned)scan_num_tiles(n)), block(kScanBlock);
    switch (scan_rounds(n)) {
        case 1: BP_LAUNCH(K_SCAN_REDUCE, (scan_reduce_kernel<1, T, Op, In>), grid, block, 0, stream, in, n, partials, op, identity); break;
        case 4: BP_LAUNCH(K_SCAN_REDUCE, (scan_reduce_kernel<4, T, Op, In>), grid, block, 0, stream, in, n, partials, op, identity); break;
        default: BP_LAUNCH(K_SCAN_REDUCE, (scan_reduce_kernel<8, T, Op, In>), grid, block, 0, stream, in, n, partials, op, identity); break;
    }
    return BP_OK;
}

// All passes on `stream`.  partials[scan_num_tiles(n)] holds the grand total afterwards.
template <typename T, typename Op, typename In, typename Out>
int device_scan(In in, Out out, int64_t n, T* partials, Op op, T identity, hipStream_t stream) {
    BP_TRY((scan_reduce<T, Op, In>(in, n, partials, op, identity, stream)));
    return scan_finish(n, partials, op, identity, stream, [&](auto rounds, auto spine, dim3 grid) {
        BP_LAUNCH(K_SCAN_APPLY, (scan_apply_kernel<rounds(), spine(), T, Op, In, Out>), grid, dim3(kScanBlock), 0, stream, in, out,
                  n, partials, op, identity);
        return (int)BP_OK;
    });
}

// ---------------------------------------------------------------------------------------------
// stable LSD radix sort of (key, 32-bit value) pairs, RB = 8 or 9 bits per pass
//   upsweep    per-tile digit histogram              -> counts[digit][tile]
//   scan       every digit's counts by one workgroup  -> the digit's elements before every tile, and its total
//              (left out where the tiles are few)
//   downsweep  per-tile stable ranking in LDS, coalesced scatter; a tile adds the totals of the lower digits itself
// Ranking inside a tile: each wavefront owns a contiguous 64*IPT stretch, lane l holds elements
// j*64+l; for every j the lanes that share a digit find each other with ballots (one per digit bit),
// rank = running per-wave digit count + number of lower lanes among the peers.
// The bits to sort are spread evenly over the fewest passes of at most 9 bits (34 bits: 9+9+8+8).
// ---------------------------------------------------------------------------------------------
// The tiles of a sort: elements per thread, threads of the workgroup that takes one.  The widest are for sorts of keys alone:
// two workgroups a CU, as many wavefronts as four of 256 threads, but a tile leaves runs of 16 keys a digit at 9 bits
// where one of 4096 leaves 8, and half the counts (85 M words: the scatter that makes its keys 377 -> 284 us, at 9 bits from
// arrays 289 -> 277, its histogram 190 -> 164, the scan of the counts 16.7 -> 9.2).
template <int ITEMS, int THREADS>
struct SortTiles {
    static constexpr int IPT = ITEMS, BLOCK = THREADS, TILE = ITEMS * THREADS;
};
typedef SortTiles<4, 256> SmallTiles;
typedef SortTiles<16, 256> LargeTiles;
typedef SortTiles<16, 512> WideTiles;
// Tile of this workgroup.  Workgroups go to the eight XCDs round-robin; with the mapping below XCD x takes the x-th
// eighth of the tiles in order, so the tiles whose scattered runs are neighbours in memory meet in one L2.
__device__ __forceinline__ uint32_t sort_tile_of_block(uint32_t ntiles) {
    const uint32_t per = (ntiles + 7u) / 8u;
    return (blockIdx.x % 8u) * per + blockIdx.x / 8u;
}
inline uint32_t sort_grid(uint32_t ntiles) { return (ntiles + 7u) / 8u * 8u; }
constexpr int kMaxRadixBits = 9;
constexpr int kMaxRadix = 1 << kMaxRadixBits;
// A sort of few (small) tiles has no launch for the digit counts: the upsweep leaves them tile by tile, and every
// workgroup of the scatter adds them up for its digits, sixteen tiles in flight together.  19 tiles: the scatter takes
// 6.0 instead of 4.6 us and a launch of 3.6 us and its gap are gone; 100 tiles: 7 to 16 instead of 5 to 6 us, no gain.
constexpr uint32_t kSortFewTiles = 32;

// Where a pass reads its elements.  Plain arrays are the common case; a pass may also make its keys on the fly from
// something else (and so save writing them out first).  A source loads what it needs for element i with load(i),
// which depends on nothing but i, so a thread's loads all go out together (the value of element i likewise with
// load_val(i, at) and then val(); element i is a wavefront's at + lane, `at` the same in every lane); a cursor, made for a stretch of elements
// [first, end) that the whole workgroup shares, then turns what was loaded into the key: load<true> and key<true> where plain(), which is
// the same in every lane, says that the stretch needs no test element by element; done() follows the last of them.  Where a part of the key does not
// decide the digit and takes a second load, that load is late(): asked for before the tile is ranked, and merged
// into the key only when the key leaves its registers.
template <typename K>
struct SortArrays {
    const K* keys;
    const uint32_t* vals;     // NULL for a sort of keys alone
    typedef K Raw;
    static constexpr bool kLate = false;
    template <bool PLAIN>
    __device__ __forceinline__ K load(int64_t i) const { return keys[i]; }
    typedef uint32_t RawVal;
    __device__ __forceinline__ uint32_t load_val(int64_t i, int64_t) const { return vals[i]; }
    __device__ __forceinline__ uint32_t val(uint32_t raw, int64_t) const { return raw; }
    struct Cursor {
        __device__ __forceinline__ Cursor(const SortArrays&, int64_t, int64_t) {}
        __device__ __forceinline__ bool plain() const { return true; }
        template <bool PLAIN>
        __device__ __forceinline__ K key(int64_t, K raw) { return raw; }
        __device__ __forceinline__ void done() const {}
    };
};

// Keys whose values are their own places in the array (a sort that is to return the permutation it applied).
template <typename K>
struct SortKeysNumbered {
    const K* keys;
    typedef K Raw;
    static constexpr bool kLate = false;
    template <bool PLAIN>
    __device__ __forceinline__ K load(int64_t i) const { return keys[i]; }
    typedef uint32_t RawVal;
    __device__ __forceinline__ uint32_t load_val(int64_t i, int64_t) const { return (uint32_t)i; }
    __device__ __forceinline__ uint32_t val(uint32_t raw, int64_t) const { return raw; }
    struct Cursor {
        __device__ __forceinline__ Cursor(const SortKeysNumbered&, int64_t, int64_t) {}
        __device__ __forceinline__ bool plain() const { return true; }
        template <bool PLAIN>
        __device__ __forceinline__ K key(int64_t, K raw) { return raw; }
        __device__ __forceinline__ void done() const {}
    };
};

// Counts the digits of a wavefront's lanes; if any lane is here, lane 0 is.  Skewed keys put many lanes on one counter:
// those that share lane 0's digit are counted by lane 0 with one addition, the others add one by one.
__device__ __forceinline__ void count_digit(uint32_t* hist, uint32_t d) {
    const uint32_t d0 = __builtin_amdgcn_readfirstlane(d);
    const uint32_t same = (uint32_t)__popcll(__ballot(d == d0));
    const bool first = lane_id() == 0;
    if (first || d != d0) atomicAdd(&hist[d], first ? same : 1u);
}

template <typename K, int RB, typename Tiles, typename Src>
__global__ __launch_bounds__(Tiles::BLOCK) void sort_upsweep_kernel(Src src, uint32_t n, int shift, uint32_t mask,
                                                                  uint32_t* __restrict__ counts, uint32_t ntiles,
                                                                  int by_tile) {
    constexpr int RADIX = 1 << RB, IPT = Tiles::IPT, BLOCK = Tiles::BLOCK;
    __shared__ uint32_t hist[RADIX];
    const uint32_t tile = sort_tile_of_block(ntiles);
    if (tile >= ntiles) return;
    for (int d = threadIdx.x; d < RADIX; d += BLOCK) hist[d] = 0;
    __syncthreads();
    const int64_t base = (int64_t)tile * (BLOCK * IPT);
    const int64_t end = base + BLOCK * IPT < (int64_t)n ? base + BLOCK * IPT : (int64_t)n;
    const int64_t mine = base + threadIdx.x;
    typename Src::Cursor cur(src, base, end);
    const auto count = [&](int64_t i, const typename Src::Raw& raw) {
        count_digit(hist, (uint32_t)(cur.template key<false>(i, raw) >> shift) & mask);
    };
    typename Src::Raw raw[IPT];
    if (end - base == BLOCK * IPT) {
#pragma unroll
        for (int j = 0; j < IPT; ++j) raw[j] = src.template load<false>(mine + j * BLOCK);
#pragma unroll
        for (int j = 0; j < IPT; ++j) count(mine + j * BLOCK, raw[j]);
    } else {
#pragma unroll
        for (int j = 0; j < IPT; ++j) raw[j] = src.template load<false>(mine + j * BLOCK < end ? mine + j * BLOCK : end - 1);
#pragma unroll
        for (int j = 0; j < IPT; ++j)
            if (mine + j * BLOCK < end) count(mine + j * BLOCK, raw[j]);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < RADIX; d += BLOCK)
        counts[by_tile ? (size_t)tile * RADIX + d : (size_t)d * ntiles + tile] = hist[d];
}

// Digit d's counts, one per tile, lie side by side: one workgroup per digit turns them into the counts of the tiles
// before (from `in` to `out`, which may be the same array) and leaves their sum in totals[d].  Nothing here meets
// another workgroup, so this is one launch where a scan over all digits and tiles at once takes three.  A round takes
// BLOCK * SCAN_ROUNDS counts, the next round's loads out before this one's sums; it is bound by the launch where the
// tiles are few (25 tiles: 3 us for 10.5 us of reduce, spine and apply) and by memory where they are many (20,800
// tiles and 512 digits: 20 us for 33 us).
template <int BLOCK, int SCAN_ROUNDS>
__global__ __launch_bounds__(BLOCK) void sort_digit_scan_kernel(const uint32_t* in, uint32_t* out, uint32_t ntiles,
                                                                uint32_t* __restrict__ totals) {
    constexpr int WAVES = BLOCK / kWave;
    __shared__ uint32_t wave_tot[2][WAVES];
    const int w = threadIdx.x / kWave, lane = lane_id();
    const size_t row = (size_t)blockIdx.x * ntiles;
    const uint32_t mine = w * (kWave * SCAN_ROUNDS) + lane;
    uint32_t v[SCAN_ROUNDS], carry = 0;
#pragma unroll
    for (int r = 0; r < SCAN_ROUNDS; ++r) v[r] = mine + r * kWave < ntiles ? in[row + mine + r * kWave] : 0u;
    for (uint32_t base = 0, turn = 0; base < ntiles; base += BLOCK * SCAN_ROUNDS, turn ^= 1u) {
        uint32_t next[SCAN_ROUNDS];
        uint32_t sum = 0;
#pragma unroll
        for (int r = 0; r < SCAN_ROUNDS; ++r) {
            const uint32_t i = base + BLOCK * SCAN_ROUNDS + mine + r * kWave;
            next[r] = i < ntiles ? in[row + i] : 0u;
        }
#pragma unroll
        for (int r = 0; r < SCAN_ROUNDS; ++r) sum += v[r];
        sum = wave_reduce(sum, AddOp());
        if (lane == 0) wave_tot[turn][w] = sum;          // two sets in turn: one barrier a round
        __syncthreads();
        uint32_t run = carry;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            const uint32_t t = wave_tot[turn][k];
            if (k < w) run += t;
            carry += t;
        }
#pragma unroll
        for (int r = 0; r < SCAN_ROUNDS; ++r) {
            const uint32_t i = base + mine + r * kWave;
            const uint32_t inc = wave_inclusive_scan(v[r], AddOp());
            if (i < ntiles) out[row + i] = run + inc - v[r];
            run += lane_value(inc, kWave - 1);
            v[r] = next[r];
        }
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = carry;
}

// Of the lanes in peers_lo / peers_hi, those with this lane's digit.  One ballot per bit: a lane whose bit is set keeps
// the lanes of the ballot, the others those outside it, i.e. peers &= ~(ballot ^ bit), the bit spread over a word.  The
// scatter is bound by its vector instructions (a wave64 instruction for every element of 85 M costs 2.2 us, and this was
// nine a bit): written as one three-input instruction per half a bit takes four.
template <int RB>
__device__ __forceinline__ void same_digit_lanes(uint32_t d, uint32_t* peers_lo, uint32_t* peers_hi) {
    constexpr uint32_t kAndXnor = 0x90;         // a & ~(b ^ c) as a truth table over a, b, c
    uint32_t lo = *peers_lo, hi = *peers_hi;
    int32_t bits[RB];
    uint64_t ballots[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        bits[b] = __builtin_amdgcn_sbfe((int32_t)d, b, 1);                // 0 or -1
        asm("" : "+v"(bits[b]));                // or the compiler shifts the digit once more for the test
        ballots[b] = __ballot(bits[b] != 0);
    }
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const int32_t bit = bits[b];
        const uint64_t m = ballots[b];
        lo = __builtin_amdgcn_bitop3_b32(lo, (uint32_t)m, (uint32_t)bit, kAndXnor);
        hi = __builtin_amdgcn_bitop3_b32(hi, (uint32_t)(m >> 32), (uint32_t)bit, kAndXnor);
    }
    *peers_lo = lo;
    *peers_hi = hi;
}

typedef uint32_t __attribute__((may_alias)) TwoCounters;      // two 16-bit counters, cleared with one store

// Bound by memory at 8 bits (85 M words: 250 us for 1.36 GB), at 9 by vector and LDS instructions beside it (277).  What hides
// latency is the number of wavefronts a CU holds: 16 of keys alone (76 KB of LDS a workgroup of 512), 12 of keys and values (8
// at 9 bits).
template <typename K, int RB, typename Tiles, typename Src, bool VALS>
__global__ __launch_bounds__(Tiles::BLOCK, !VALS ? 4 : RB > 8 ? 2 : 3) void sort_downsweep_kernel(Src src, K* __restrict__ kout,
                                                                    uint32_t* __restrict__ vout, uint32_t n, int shift,
                                                                    uint32_t mask, const uint32_t* __restrict__ before,
                                                                    const uint32_t* __restrict__ totals, uint32_t ntiles) {
    constexpr int RADIX = 1 << RB;
    constexpr int IPT = Tiles::IPT, BLOCK = Tiles::BLOCK;
    constexpr int DPT = RADIX > BLOCK ? RADIX / BLOCK : 1;     // consecutive digits owned by a thread in the digit scan
    constexpr int WAVES = BLOCK / kWave;
    constexpr int TILE = Tiles::TILE;
    constexpr int WTILE = kWave * IPT;
    static_assert(TILE < 65536, "places in a tile fit 16 bits");
    static_assert(RADIX % DPT == 0 && RADIX / DPT <= BLOCK, "every digit has an owner");
    __shared__ __attribute__((aligned(4))) uint16_t wcnt[WAVES][RADIX];    // per-wave digit counts, then where the wave's elements start in the tile
    __shared__ uint32_t gbase[RADIX];          // global base of the digit for this tile, minus its start in the tile
    __shared__ uint64_t wave_tot[WAVES];
    __shared__ K skeys[TILE];
    __shared__ uint32_t svals[VALS ? TILE : 1];

    const int tid = threadIdx.x, lane = tid & (kWave - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid / kWave);      // the same in every lane: scalar addresses follow
    const uint32_t tile = sort_tile_of_block(ntiles);
    if (tile >= ntiles) return;
    for (int d = tid; d < WAVES * RADIX / 2; d += BLOCK) reinterpret_cast<TwoCounters*>(&wcnt[0][0])[d] = 0;
    // asked for now, used after the ranking
    uint32_t all[DPT], earlier[DPT];           // elements of the thread's digits: in all tiles, in the tiles before
    const bool owner = RADIX / DPT == BLOCK || tid < RADIX / DPT;
#pragma unroll
    for (int k = 0; k < DPT; ++k) all[k] = earlier[k] = 0;
    if (!owner) {
    } else if (IPT > SmallTiles::IPT || totals) {
#pragma unroll
        for (int k = 0; k < DPT; ++k) {
            all[k] = totals[tid * DPT + k];
            earlier[k] = before[(size_t)(tid * DPT + k) * ntiles + tile];
        }
    } else {                                   // few tiles: `before` holds the bare counts, tile by tile
        constexpr int STEP = 16;               // tiles whose counts are in flight together
        for (uint32_t t0 = 0; t0 < ntiles; t0 += STEP) {
            uint32_t c[STEP][DPT];
#pragma unroll
            for (int u = 0; u < STEP; ++u)
#pragma unroll
                for (int k = 0; k < DPT; ++k) c[u][k] = t0 + u < ntiles ? before[(size_t)(t0 + u) * RADIX + tid * DPT + k] : 0u;
#pragma unroll
            for (int u = 0; u < STEP; ++u)
#pragma unroll
                for (int k = 0; k < DPT; ++k) {
                    all[k] += c[u][k];
                    earlier[k] += t0 + u < tile ? c[u][k] : 0u;
                }
        }
    }
    __syncthreads();

    const int64_t tile_base = (int64_t)tile * TILE;
    const int64_t tile_end = tile_base + TILE < (int64_t)n ? tile_base + TILE : (int64_t)n;
    const int64_t wbase = tile_base + w * WTILE;
    const int64_t mine = wbase + lane;
    typename Src::Cursor cur(src, tile_base, tile_end);
    // A full tile (every one but the last) has no elements to leave out; the test is the same in every lane.
    const auto run = [&](auto full_tile) {
        constexpr bool FULL = decltype(full_tile)::value;
        const auto in = [&](int j) { return FULL || mine + j * kWave < tile_end; };
        K key[IPT];
        uint32_t val[VALS ? IPT : 1], late[Src::kLate ? IPT : 1];
        uint32_t rank[IPT];
        {
            typename Src::Raw raw[IPT];
#pragma unroll
            for (int j = 0; j < IPT; ++j) {
                const int64_t i = in(j) ? mine + j * kWave : tile_end - 1;
                raw[j] = src.template load<FULL>(i);
            }
            if constexpr (VALS) {
                const auto first_of = [&](int j) {          // of the round's elements; one that is there
                    const int64_t at = wbase + j * kWave;
                    return FULL || at < tile_end ? at : (tile_end - 1) / kWave * kWave;
                };
                typename Src::RawVal raw_val[IPT];
#pragma unroll
                for (int j = 0; j < IPT; ++j) raw_val[j] = src.load_val(in(j) ? mine + j * kWave : tile_end - 1, first_of(j));
#pragma unroll
                for (int j = 0; j < IPT; ++j) val[j] = src.val(raw_val[j], first_of(j));
            }
            if constexpr (Src::kLate) {
#pragma unroll
                for (int j = 0; j < IPT; ++j) late[j] = in(j) ? src.late(wbase + j * kWave) : 0u;
            }
#pragma unroll
            for (int j = 0; j < IPT; ++j) key[j] = cur.template key<FULL>(in(j) ? mine + j * kWave : tile_end - 1, raw[j]);
            cur.done();
        }
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const uint32_t d = (uint32_t)(key[j] >> shift) & mask;
            uint32_t peers_lo = ~0u, peers_hi = ~0u;
            if constexpr (!FULL) {
                const uint64_t here = __ballot(in(j));
                peers_lo = (uint32_t)here;
                peers_hi = (uint32_t)(here >> 32);
            }
            same_digit_lanes<RB>(d, &peers_lo, &peers_hi);
            const uint32_t seen = wcnt[w][d];
            rank[j] = __builtin_amdgcn_mbcnt_hi(peers_hi, __builtin_amdgcn_mbcnt_lo(peers_lo, seen));
            __builtin_amdgcn_wave_barrier();
            if (in(j) && rank[j] == seen)              // the lowest of the peers
                wcnt[w][d] = (uint16_t)(seen + (uint32_t)__popc(peers_lo) + (uint32_t)__popc(peers_hi));
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();

        {   // thread tid owns digits tid*DPT .. tid*DPT+DPT-1: offsets of the waves inside each digit, then digit starts
            // (one scan for both the tile's own digit counts, low word, and the digits' totals, high word)
            uint32_t tot[DPT], start[DPT][WAVES];
            uint64_t sum = 0;
#pragma unroll
            for (int k = 0; k < DPT; ++k) {
                const int d = tid * DPT + k;
                uint32_t before_wave = 0;
#pragma unroll
                for (int i = 0; i < WAVES; ++i) {
                    start[k][i] = before_wave;
                    if (owner) before_wave += wcnt[i][d];
                }
                tot[k] = before_wave;
                sum += ((uint64_t)all[k] << 32) | before_wave;
            }
            uint64_t exc2, inc2, total2;
            block_scan<BLOCK>(sum, AddOp(), uint64_t(0), wave_tot, &exc2, &inc2, &total2);
            uint32_t exc = (uint32_t)exc2, below = (uint32_t)(exc2 >> 32);
#pragma unroll
            for (int k = 0; k < DPT && owner; ++k) {
                const int d = tid * DPT + k;
#pragma unroll
                for (int i = 0; i < WAVES; ++i) wcnt[i][d] = (uint16_t)(exc + start[k][i]);
                gbase[d] = below + earlier[k] - exc;
                exc += tot[k];
                below += all[k];
            }
        }
        __syncthreads();

#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            if (in(j)) {
                const uint32_t d = (uint32_t)(key[j] >> shift) & mask;
                const uint32_t pos = wcnt[w][d] + rank[j];
                if constexpr (Src::kLate) skeys[pos] = src.merge(key[j], late[j]);
                else skeys[pos] = key[j];
                if constexpr (VALS) svals[pos] = val[j];
            }
        }
        __syncthreads();

        const uint32_t tile_n = FULL ? (uint32_t)TILE : (uint32_t)(tile_end - tile_base);
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            const uint32_t pos = j * BLOCK + tid;
            if (FULL || pos < tile_n) {
                const K k = skeys[pos];
                const uint32_t dst = gbase[(uint32_t)(k >> shift) & mask] + pos;
                kout[dst] = k;
                if constexpr (VALS) vout[dst] = svals[pos];
            }
        }
    };
    if (tile_end - tile_base == TILE && cur.plain()) run(std::true_type{});
    else run(std::false_type{});
}

template <typename Tiles>
inline uint32_t sort_num_tiles(int64_t n) { return (uint32_t)(n > 0 ? ceil_div(n, Tiles::TILE) : 1); }

// uint32 words of temporary storage for the sort of n elements in such tiles, or larger ones
template <typename Tiles>
inline size_t sort_temp_words(int64_t n) {
    return (((size_t)kMaxRadix * sort_num_tiles<Tiles>(n) + 63) & ~size_t(63)) + kMaxRadix;
}

// One pass.  The histogram reads `up`, the scatter reads `src`: the same elements, but a source that has to fetch
// more than the digit needs may leave that to the scatter alone.
// `ready`: the pass's histogram made by a kernel of the caller's that read the same elements anyway, counts[digit][tile], or
// in `counts` itself, laid out as the upsweep would; NULL: the upsweep makes it.
template <typename Tiles>
inline bool sort_counts_by_tile(uint32_t ntiles) { return Tiles::IPT <= SmallTiles::IPT && ntiles <= kSortFewTiles; }

template <typename K, int RB, typename Tiles, typename Up, typename Src, bool VALS>
int radix_sort_pass(const Up& up, const Src& src, K* kout, uint32_t* vout, int64_t n, int bit, int nb, uint32_t* counts,
                    uint32_t* totals, uint32_t ntiles, hipStream_t stream, const uint32_t* ready) {
    const uint32_t mask = (1u << nb) - 1u;
    const bool few = sort_counts_by_tile<Tiles>(ntiles) && (!ready || ready == counts);
    if (!ready)
        BP_LAUNCH(K_SORT_UPSWEEP, (sort_upsweep_kernel<K, RB, Tiles, Up>), dim3(sort_grid(ntiles)), dim3(Tiles::BLOCK), 0, stream,
                  up, (uint32_t)n, bit, mask, counts, ntiles, few ? 1 : 0);
    // few tiles: one round of a small workgroup; many: large workgroups, which keep their number of rounds down
    const uint32_t* digit_counts = ready ? ready : counts;
    if (!few) {
        if (ntiles <= 4 * 256)
            BP_LAUNCH(K_SORT_SCAN, (sort_digit_scan_kernel<256, 4>), dim3(1 << RB), dim3(256), 0, stream, digit_counts, counts,
                      ntiles, totals);
        else
            BP_LAUNCH(K_SORT_SCAN, (sort_digit_scan_kernel<1024, 4>), dim3(1 << RB), dim3(1024), 0, stream, digit_counts, counts,
                      ntiles, totals);
    }
    BP_LAUNCH(K_SORT_DOWNSWEEP, (sort_downsweep_kernel<K, RB, Tiles, Src, VALS>), dim3(sort_grid(ntiles)), dim3(Tiles::BLOCK), 0,
              stream, src, kout, vout, (uint32_t)n, bit, mask, (const uint32_t*)counts,
              (const uint32_t*)(few ? nullptr : totals), ntiles);
    return BP_OK;
}

template <typename K, typename Tiles, typename Up, typename Src, bool VALS>
int radix_sort_one_pass(const Up& up, const Src& src, K* kout, uint32_t* vout, int64_t n, int bit, int nb,
                        uint32_t* counts, uint32_t* totals, uint32_t ntiles, hipStream_t stream,
                        const uint32_t* ready = nullptr) {
    if (nb > 8)
        return radix_sort_pass<K, 9, Tiles, Up, Src, VALS>(up, src, kout, vout, n, bit, nb, counts, totals, ntiles, stream,
                                                         ready);
    return radix_sort_pass<K, 8, Tiles, Up, Src, VALS>(up, src, kout, vout, n, bit, nb, counts, totals, ntiles, stream, ready);
}

// Bits the first pass of a sort over [begin_bit, end_bit) takes (the passes share the bits evenly).
inline int radix_first_pass_bits(int begin_bit, int end_bit) {
    const int total = end_bit - begin_bit;
    if (total <= 0) return 0;
    const int passes = (total + kMaxRadixBits - 1) / kMaxRadixBits;
    return (total + passes - 1) / passes;
}

// Stable sort of n elements by key bits [begin_bit, end_bit).  The first pass reads `first` (any source; its
// histogram reads `first_up`, which must give the same sorted bits) and writes buffer 0, every later pass reads the
// buffer the one before wrote and writes the other one; *result says which buffer holds the sorted output (-1: no
// pass ran, nothing was written).  VALS: 32-bit values travel with the keys.  n < 2^32 - 8192.
// first_counts: the first pass's histogram where a kernel of the caller's has made it already (radix_sort_pass).
template <typename K, typename Tiles, typename Up, typename Src, bool VALS>
int radix_sort_from(const Up& first_up, const Src& first, K* const kbuf[2], uint32_t* const vbuf[2], int64_t n,
                    int begin_bit, int end_bit, uint32_t* temp, hipStream_t stream, int* result,
                    const uint32_t* first_counts = nullptr) {
    *result = -1;
    if (n <= 0 || end_bit <= begin_bit) return BP_OK;
    const uint32_t ntiles = sort_num_tiles<Tiles>(n);
    uint32_t* counts = temp;
    uint32_t* totals = temp + (((size_t)kMaxRadix * ntiles + 63) & ~size_t(63));
    const int total = end_bit - begin_bit;
    const int passes = (total + kMaxRadixBits - 1) / kMaxRadixBits;
    int bit = begin_bit;
    for (int p = 0; p < passes; ++p) {
        const int left = end_bit - bit;
        const int nb = (left + (passes - p) - 1) / (passes - p);      // spread the remaining bits evenly
        const int out = p & 1;
        if (p == 0) {
            BP_TRY((radix_sort_one_pass<K, Tiles, Up, Src, VALS>(first_up, first, kbuf[out], VALS ? vbuf[out] : nullptr, n, bit,
                                                               nb, counts, totals, ntiles, stream, first_counts)));
        } else {
            const SortArrays<K> in{kbuf[out ^ 1], VALS ? vbuf[out ^ 1] : nullptr};
            BP_TRY((radix_sort_one_pass<K, Tiles, SortArrays<K>, SortArrays<K>, VALS>(in, in, kbuf[out],
                                                                                    VALS ? vbuf[out] : nullptr, n, bit, nb,
                                                                                    counts, totals, ntiles, stream)));
        }
        bit += nb;
        *result = out;
    }
    return BP_OK;
}

// Sorts n (key, value) pairs by key bits [begin_bit, end_bit), stable.  The data ping-pongs between
// (keys_a, vals_a) and (keys_b, vals_b); input is in the `a` buffers; *result_in_b tells where the
// sorted output ended up.  n < 2^32 - 8192.
template <typename K, typename Tiles>
int radix_sort_pairs(K* keys_a, K* keys_b, uint32_t* vals_a, uint32_t* vals_b, int64_t n, int begin_bit, int end_bit,
                     uint32_t* temp, hipStream_t stream, bool* result_in_b, const uint32_t* first_counts = nullptr) {
    K* const kbuf[2] = {keys_b, keys_a};
    uint32_t* const vbuf[2] = {vals_b, vals_a};
    int result = -1;
    const SortArrays<K> in{keys_a, vals_a};
    BP_TRY((radix_sort_from<K, Tiles, SortArrays<K>, SortArrays<K>, true>(in, in, kbuf, vbuf, n, begin_bit, end_bit, temp, stream,
                                                                        &result, first_counts)));
    *result_in_b = result == 0;
    return BP_OK;
}

// The same with the values 0 .. n-1 in the order of the input: vals_a is scratch, nobody has to fill it.
template <typename K, typename Tiles>
int radix_sort_numbered(K* keys_a, K* keys_b, uint32_t* vals_a, uint32_t* vals_b, int64_t n, int begin_bit, int end_bit,
                        uint32_t* temp, hipStream_t stream, bool* result_in_b) {
    K* const kbuf[2] = {keys_b, keys_a};
    uint32_t* const vbuf[2] = {vals_b, vals_a};
    int result = -1;
    const SortArrays<K> up{keys_a, nullptr};
    const SortKeysNumbered<K> in{keys_a};
    BP_TRY((radix_sort_from<K, Tiles, SortArrays<K>, SortKeysNumbered<K>, true>(up, in, kbuf, vbuf, n, begin_bit, end_bit, temp,
                                                                              stream, &result)));
    *result_in_b = result == 0;
    return BP_OK;
}

}  // namespace bp
