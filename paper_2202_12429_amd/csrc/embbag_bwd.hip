// bp_embbag_bwd_update: deterministic backward + fused sparse optimizer step on cached rows.
//
// Gradients, not embeddings, are combined (Section 6), so any per-row optimizer can follow; the update
// rules are SGD, element-wise Adagrad and row-wise Adagrad.
//
// The work of a batch is described by two lists of records (the planner emits them with its optional grouping;
// bp_embbag_bwd_update builds them itself after a stable sort of the lookups by slot):
//   row records    one per distinct row: where its lookups start in the grouped order, how many they are, its
//                  slot, its first lookup.  A row of up to BP_BWD_ROW_MAX lookups is summed (fp64) and updated by
//                  one lane group, which needs nothing but its record to ask for the cache row and the first
//                  gradient row.
//   piece records  a row with more lookups is cut into pieces of BP_BWD_PIECE lookups; one workgroup (narrow rows: one
//                  wavefront) takes a piece, its lane groups add their shares and meet.  A one-piece row is updated
//                  at once.  For a row of several pieces the piece's sum is stored, and whoever finds, by a counter,
//                  that all the others have stored theirs adds the sums and updates the row (of very many pieces: in
//                  stretches first).
// ONE launch does all of it: workgroups [0, piece_blocks) take pieces, the rest take rows.
// Every order of addition is fixed by the row's own records and its type and width, never by timing or by the rest of the batch:
// results are bit-identical run to run, and from one entry point to the other.
// The summed gradient is rounded to fp32 once; the optimizer step itself is fp32 arithmetic.
#include <algorithm>
#include <type_traits>

#include "bwd_records.h"
#include "common.h"
#include "device_prims.h"
#include "row_access.h"

namespace bp {
namespace {

// ---- 1. keys ---------------------------------------------------------------------------------
// Keys (slots) and values (bags) of the sort, and its first histogram on the way, which reads the same keys: a workgroup takes
// one tile of that sort.  The searches of a thread's lookups go step by step together, so that a step costs one round trip.
// Clears the counters of bwd_records_kernel.  Bound by the searches' round trips (19,000 lookups in 4,291 bags: 8.2 us, where keys
// and histogram by themselves took 4.9 and 2.9 and a launch more).
template <int RB, typename Tiles>
__global__ __launch_bounds__(Tiles::BLOCK) void bwd_keys_kernel(const int32_t* __restrict__ slots, const int64_t* __restrict__ bag_off,
                                                                uint32_t n, uint32_t bags, int64_t C, uint32_t* __restrict__ keys,
                                                                uint32_t* __restrict__ vals, uint32_t mask,
                                                                uint32_t* __restrict__ counts, uint32_t ntiles, int by_tile,
                                                                uint64_t* __restrict__ counters) {
    constexpr int IPT = Tiles::IPT, BLOCK = Tiles::BLOCK, RADIX = 1 << RB;
    __shared__ uint32_t hist[RADIX];
    const uint32_t tile = blockIdx.x;
    for (int d = threadIdx.x; d < RADIX; d += BLOCK) hist[d] = 0;
    if (tile == 0 && threadIdx.x < 2) counters[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t first = tile * (uint32_t)Tiles::TILE + threadIdx.x;
    uint32_t s[IPT], bag[IPT];
#pragma unroll
    for (int j = 0; j < IPT; ++j) s[j] = first + j * BLOCK < n ? (uint32_t)slots[first + j * BLOCK] : 0u;
#pragma unroll
    for (int j = 0; j < IPT; ++j) bag[j] = first + j * BLOCK;
    if (bag_off) {                                       // largest b with bag_off[b] <= the lookup
        uint32_t hi[IPT];                                // bag_off[bag] <= lookup < bag_off[hi]
#pragma unroll
        for (int j = 0; j < IPT; ++j) {
            bag[j] = 0;
            hi[j] = bags;
        }
        for (uint32_t range = bags; range > 1; range = (range + 1) / 2) {
            int64_t at[IPT];
#pragma unroll
            for (int j = 0; j < IPT; ++j) at[j] = bag_off[bag[j] + (hi[j] - bag[j]) / 2];      // asked for by all, done or not
#pragma unroll
            for (int j = 0; j < IPT; ++j) {
                const uint32_t mid = bag[j] + (hi[j] - bag[j]) / 2;
                const bool below = at[j] <= (int64_t)first + j * BLOCK;
                if (hi[j] - bag[j] > 1) {
                    bag[j] = below ? mid : bag[j];
                    hi[j] = below ? hi[j] : mid;
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < IPT; ++j) {
        const uint32_t k = first + j * BLOCK;
        if (k < n) {
            const uint32_t key = s[j] < (uint64_t)C ? s[j] : (uint32_t)C;     // out-of-range slots sort behind every real one
            keys[k] = key;
            vals[k] = bag[j];
            count_digit(hist, key & mask);
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < RADIX; d += BLOCK) counts[by_tile ? (size_t)tile * RADIX + d : (size_t)d * ntiles + tile] = hist[d];
}

// Grouped variant: the plan lists lookup positions grouped by row; the gradient row of a position is its bag.
// First every bag writes its number over its own stretch of positions -- a wavefront takes 64 bags and goes through
// them one by one, its lanes writing side by side (one lane per bag would scatter 64 short runs per store) --, then
// the grouped positions pick their bag up from that map, which stays in L2.
__global__ __launch_bounds__(256) void bwd_bag_of_lookup_kernel(const int64_t* __restrict__ bag_off, int64_t bags, int64_t n,
                                                                uint32_t* __restrict__ bag_of_lookup) {
    const int lane = threadIdx.x % kWave;
    const int64_t b0 = ((int64_t)blockIdx.x * (256 / kWave) + threadIdx.x / kWave) * kWave;      // wave-uniform
    if (b0 >= bags) return;
    const int64_t b = b0 + lane;
    int64_t k = b < bags ? bag_off[b] : 0, end = b < bags ? bag_off[b + 1] : 0;
    if (k < 0) k = 0;
    if (end > n) end = n;
    if (k > end) k = end;                                // before lanes are added to it: k + lane cannot wrap
    const int here = (int)(bags - b0 < kWave ? bags - b0 : kWave);
    for (int t = 0; t < here; ++t) {
        const int64_t first = __shfl(k, t, kWave), stop = __shfl(end, t, kWave);
        for (int64_t q = first + lane; q < stop; q += kWave) bag_of_lookup[q] = (uint32_t)(b0 + t);
    }
}

__global__ __launch_bounds__(256) void bwd_bags_of_positions_kernel(const int32_t* __restrict__ positions,
                                                                    const uint32_t* __restrict__ bag_of_lookup, int64_t n,
                                                                    int64_t bags, uint32_t* __restrict__ bag_of) {
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p >= n) return;
    const uint32_t k = (uint32_t)positions[p];
    const uint32_t b = k < (uint64_t)n ? bag_of_lookup[k] : 0u;
    bag_of[p] = b < (uint64_t)bags ? b : 0u;      // offsets that do not cover every lookup leave holes in the map
}

// The same for bags of five lookups and more in the mean.  The gather above runs at the rate of the lines it finds in a map of
// four bytes a lookup; sixteen bytes tell the bags of 64 lookups: the bag of the first, a mask of the lookups at which another
// one starts, and whether those bags follow one another without an empty one between.  Where they don't, the position looks
// for its bag in the offsets, up to the next stretch's first.  Map / list, us a grouped call on one row, positions at random:
// bags of 1 to 49, 4.2 M lookups 82 / 28, 0.26 M 15.9 / 8.1; of 0 to 12, 4.2 M 103 / 79, 16 K 13.4 / 11.4; of 0 to 10, 4.2 M 109 /
// 97; of 0 to 8, 4.2 M 115 / 120, 1 M 30.3 / 30.5: there most stretches hold an empty bag.
struct BagsOf64 {
    static constexpr uint32_t kGaps = 1;
    uint32_t mask_lo, mask_hi, first, flags;
};
static_assert(sizeof(BagsOf64) == 16, "one load");
__device__ __forceinline__ BagsOf64 bags_of_64(const int64_t* __restrict__ bag_off, int64_t bags, int64_t b, int64_t from, int64_t end) {
    // `from`: the stretch's first lookup; bag b holds it and ends at `end`
    BagsOf64 r{0u, 0u, (uint32_t)b, 0u};
    const int64_t stop = from + 64;
    uint64_t mask = 0;
    while (end < stop && ++b < bags) {          // bag b starts at `end`, which lies behind the start before it: 63 steps at most
        const int64_t next = bag_off[b + 1];
        if (next <= end) {
            r.flags = BagsOf64::kGaps;
            break;
        }
        mask |= uint64_t(1) << (end - from);
        end = next;
    }
    r.mask_lo = (uint32_t)mask;
    r.mask_hi = (uint32_t)(mask >> 32);
    return r;
}
// A wavefront takes 64 bags: every lane writes the stretches that start in its own short one, and those of a long one are
// written by all lanes together.
__global__ __launch_bounds__(256) void bwd_list_bags_kernel(const int64_t* __restrict__ bag_off, int64_t bags, int64_t n,
                                                            BagsOf64* __restrict__ list) {
    constexpr int64_t kLong = 4;                                 // stretches
    const int lane = threadIdx.x % kWave;
    const int64_t b0 = ((int64_t)blockIdx.x * (256 / kWave) + threadIdx.x / kWave) * kWave;      // wave-uniform
    if (b0 >= bags) return;
    const int64_t b = b0 + lane;
    int64_t k = b < bags ? bag_off[b] : 0, end = b < bags ? bag_off[b + 1] : 0;
    if (k < 0) k = 0;
    if (end > n) end = n;
    if (k > end) k = end;
    const int64_t t0 = (k + 63) >> 6, t1 = (end + 63) >> 6;      // stretches [t0, t1) start inside the bag
    const bool is_long = t1 - t0 > kLong;
    if (!is_long)
        for (int64_t t = t0; t < t1; ++t) list[t] = bags_of_64(bag_off, bags, b, t * 64, end);
    for (uint64_t left = __ballot(is_long); left; left &= left - 1) {
        const int who = __ffsll((unsigned long long)left) - 1;
        const int64_t first = __shfl(t0, who, kWave), stop = __shfl(t1, who, kWave), e = __shfl(end, who, kWave);
        for (int64_t t = first + lane; t < stop; t += kWave) list[t] = bags_of_64(bag_off, bags, b0 + who, t * 64, e);
    }
}
// Offsets that do not cover every lookup leave entries unwritten: whatever is found there is taken into [0, bags).
__global__ __launch_bounds__(256) void bwd_bags_from_list_kernel(const int32_t* __restrict__ positions,
                                                                 const BagsOf64* __restrict__ list,
                                                                 const int64_t* __restrict__ bag_off, int64_t n, int64_t bags,
                                                                 uint32_t* __restrict__ bag_of) {
    constexpr int U = 4;                                         // positions of a thread, in flight together
    const int64_t p0 = (int64_t)blockIdx.x * (256 * U) + threadIdx.x;
    const uint32_t last = (uint32_t)(bags > 0 ? bags - 1 : 0);
    uint32_t k[U];
    uint4 e[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int64_t p = p0 + u * 256;
        k[u] = p < n ? (uint32_t)positions[p] : 0u;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) e[u] = *reinterpret_cast<const uint4*>(list + (k[u] < (uint64_t)n ? k[u] >> 6 : 0u));
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const uint64_t upto = (((uint64_t)e[u].y << 32) | e[u].x) & (~uint64_t(0) >> (63 - (k[u] & 63u)));
        uint32_t bag = min(e[u].z + (uint32_t)__popcll(upto), last);
        if (k[u] >= (uint64_t)n) {
            bag = 0;                                             // not a position
        } else if (e[u].w & BagsOf64::kGaps) {
            // the last bag of those up to the next stretch's first that starts at or before the lookup
            const int64_t t = (int64_t)(k[u] >> 6) + 1;
            uint32_t hi = t * 64 < n ? min(list[t].first, last) : last;
            while (bag < hi) {
                const uint32_t mid = bag + (hi - bag + 1) / 2;
                if (bag_off[mid] <= (int64_t)k[u]) bag = mid; else hi = mid - 1;
            }
        }
        const int64_t p = p0 + u * 256;
        if (p < n) bag_of[p] = bag;
    }
}
constexpr int64_t kListedBags = 5;      // mean lookups a bag

// ---- 3./4. reduce and update -----------------------------------------------------------------
struct UpdateParams {
    int optimizer;
    float lr, eps;
    int lpr;
    int dim;
    uint32_t bags;      // rows of the upstream gradient: a bag number beyond them reads row 0 instead
    int64_t wst;        // stride of a cache row, in pieces
    int64_t sst;        // stride of a row's optimizer state, in floats
};

// Running sum of one lane's piece of gradient rows.  Sums are carried in fp64 and rounded to fp32 once,
// which makes the result independent of how a slot's lookups were cut into items (fp64 addition of
// fp32 values is exact until the partial sums outgrow 53 bits); everything after the sum is fp32.
template <int N>
struct SumPiece {
    double v[N];
    __device__ __forceinline__ void zero() {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = 0.0;
    }
    template <bool BF16, bool SPLIT>
    __device__ __forceinline__ void add(const Piece<BF16, N, SPLIT>& p) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += (double)p.v[i];
    }
    __device__ __forceinline__ void add(const SumPiece& o) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] += o.v[i];
    }
    // fp64 [.. D] partial rows, the piece of lane c from element c * N on, through device-coherent accesses: written
    // through to memory and read from it, past the caches that the GPU's dies do not share, so that a sum stored by one
    // workgroup can be read by any other without either of them writing back or dropping everything else its cache
    // holds (what a device-wide fence would cost).
    __device__ __forceinline__ void store_device(double* row, int c) const {
        uint64_t* p = reinterpret_cast<uint64_t*>(row + (size_t)c * N);
#pragma unroll
        for (int i = 0; i < N; ++i)
            __hip_atomic_store(p + i, (uint64_t)__double_as_longlong(v[i]), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __device__ __forceinline__ void load_device(const double* row, int c) {
        const uint64_t* p = reinterpret_cast<const uint64_t*>(row + (size_t)c * N);
#pragma unroll
        for (int i = 0; i < N; ++i)
            v[i] = __longlong_as_double((long long)__hip_atomic_load(p + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    template <typename P>
    __device__ __forceinline__ P rounded() const {
        P p;
#pragma unroll
        for (int i = 0; i < N; ++i) p.v[i] = (float)v[i];
        return p;
    }
};

template <int GW>
__device__ __forceinline__ double group_sum(double x) {
#pragma unroll
    for (int off = GW / 2; off >= 1; off >>= 1) x += __shfl_xor(x, off, GW);
    return x;
}

// The piece of lane c of row `slot` and of its optimizer state, loaded ahead of the gradient sum so that the row's
// latency hides behind the gradient loads.
template <typename P>
struct RowPiece {
    typename P::Raw w_raw;
    P s;       // element-wise Adagrad state
    float s_row;         // row-wise Adagrad state
};

template <typename P>
__device__ __forceinline__ RowPiece<P> load_row(const UpdateParams& u, const typename P::Unit* cache_w, const float* cache_s,
                                                   int64_t slot, int c, bool active) {
    RowPiece<P> r;
    r.w_raw = P::none();
    r.s.zero();
    r.s_row = 0.f;
    if (active) {
        r.w_raw = P::fetch(cache_w + slot * u.wst, c, u.lpr);
        if (u.optimizer == BP_ADAGRAD) r.s.load_f32(cache_s + slot * u.sst, c, u.lpr);
    }
    if (u.optimizer == BP_ADAGRAD_ROWWISE) r.s_row = cache_s[slot * u.sst];
    return r;
}

// Applies one optimizer step to the piece of lane c of row `slot`; g is the row's summed gradient in fp32, r the
// piece as loaded by load_row.  All lanes of the group call this (the row-wise rule reduces over the group); lanes
// with c >= lpr carry zeros and touch no memory, and neither do the lanes of a group that is not the writer.
// One fp32 operation per statement: step = lr*g, then for Adagrad s += g*g, den = sqrt(s) + eps, step /= den,
// and w -= step.
template <int GW, typename P>
__device__ __forceinline__ void finish_update(const UpdateParams& u, typename P::Unit* cache_w, float* cache_s, int64_t slot, int c,
                                              const RowPiece<P>& r, const P& g, bool active) {
    constexpr int N = P::N;
    P w;
    w.decode(r.w_raw);
    if (u.optimizer == BP_SGD) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float step = u.lr * g.v[i];
            w.v[i] = w.v[i] - step;
        }
    } else if (u.optimizer == BP_ADAGRAD) {
        P s = r.s;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float gg = g.v[i] * g.v[i];
            s.v[i] = s.v[i] + gg;
            const float den = sqrtf(s.v[i]) + u.eps;
            const float step = (u.lr * g.v[i]) / den;
            w.v[i] = w.v[i] - step;
        }
        if (active) s.store_f32(cache_s + slot * u.sst, c, u.lpr);
    } else {
        // mean of squares over the row: an fp64 sum, rounded once.  bf16 rows: in fours of elements, the i-th of the row's
        // first half with the i-th of its second, and then over the lanes; a lane by eights holds both, by fours one of them.
        double ss = 0.0;
#pragma unroll
        for (int i = 0; i < 4; ++i) ss += (double)g.v[i] * (double)g.v[i];
        if constexpr (N == 8) {
            double second = 0.0;
#pragma unroll
            for (int i = 4; i < N; ++i) second += (double)g.v[i] * (double)g.v[i];
            ss += second;
        } else if constexpr (P::BF16) {
            const int half = u.lpr / 2;
            const double second = __shfl(ss, c + half, GW);
            ss = c < half ? ss + second : 0.0;
        }
        ss = group_sum<GW>(ss);
        const float mean = (float)(ss / (double)u.dim);
        const float s = r.s_row + mean;
        const float den = sqrtf(s) + u.eps;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const float step = (u.lr * g.v[i]) / den;
            w.v[i] = w.v[i] - step;
        }
        if (c == 0 && active) cache_s[slot * u.sst] = s;
    }
    if (active) P::put(cache_w + slot * u.wst, w.encode(), c, u.lpr);
}

// Adds the gradient rows of the grouped lookups [p0, p1) into acc: bursts of four rows, the indices of the next
// burst loaded while the rows of this one arrive.  idx holds the bag numbers of the first four lookups; FOLLOWED: and afterwards
// those of the first four of [q0, q1), unless [p0, p1) is empty.
template <bool FOLLOWED, typename P, int N>
__device__ __forceinline__ void add_gradient_rows(SumPiece<N>& acc, uint32_t (&idx)[4], uint32_t p0, uint32_t p1, uint32_t q0,
                                                  uint32_t q1, const uint32_t* __restrict__ bag_of,
                                                  const float* __restrict__ grad, const UpdateParams& u, int c) {
    for (uint32_t p = p0; p < p1; p += 4) {
        P t[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)     // the bag number is clamped where it is used: its load stays in flight until then
            if (p + j < p1) t[j].load_f32(grad + (size_t)min(idx[j], u.bags - 1u) * u.dim, c, u.lpr);
        const bool more = !FOLLOWED || p + 4 < p1;
        const uint32_t next = more ? p + 4 : q0, end = more ? p1 : q1;
#pragma unroll
        for (int j = 0; j < 4; ++j) idx[j] = next + j < end ? bag_of[next + j] : 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            if (p + j < p1) acc.add(t[j]);
    }
}

// Who takes a piece.  Rows of up to four lanes: one wavefront, whose 16 or more lane groups have a piece's lookups in flight
// in a burst or four; its groups' sums meet by lane shuffles, without LDS or barriers, and four pieces are under way a
// workgroup.  Wider rows: the workgroup.  (64-byte rows, a Criteo-shaped batch: 22.0 us with a workgroup a piece, whose 64 sums
// four lanes added one after the other, 14.2 this way.)
template <int GW>
constexpr bool kWavePieces = GW <= 4;
// A workgroup of 256 threads, or one of sixteen lane groups, where a group's share of a piece is sixteen lookups at most: four
// bursts one behind the other where 64-lane rows have sixteen in 256 threads (BwdLaunch has the rule).  Eight groups for the
// widest bf16 rows, which have no form by fours: four shares a group of 256 threads would wait in 32 KB of LDS, one workgroup
// a CU less (58,000 rows of dim 512: 49.2 us, 43.6 with two shares).
template <int GW, typename P>
constexpr int kBwdWideBlock = GW <= 16 ? 256 : P::N == 8 && GW == 64 ? 512 : 16 * GW;
template <int GW, int BLOCK>
constexpr int kPieceThreads = kWavePieces<GW> ? kWave : BLOCK;

// The order of a piece's sum, the same in every form of the kernel for a type and a width: kShares shares of lookups one behind
// the other are each summed in lookup order; share i then meets share i + kShares/2, these sums meet in the same way, and so
// on.  A form with fewer lane groups gives group j the shares j, j + groups, ..., which meet there; one with more leaves groups
// without a share.  (The pieces' sums of a row of several are shared out one by one and meet alike.)  So neither the entry
// point nor what else is in the batch changes a row's result.  As many shares as the form by fours has lane groups at most: it
// serves the small launches, which wait for their pieces.  With as many as the form by eights, a second share a group cost them 5
// to 10 % (bf16 rows of dim 16, 2,000 lookups: 4.30 / 4.57 us), and the form by eights gains nothing by them.
constexpr int piece_groups(int gw) { return gw <= 4 ? kWave / gw : gw <= 16 ? 256 / gw : 16; }      // of the form with the most
template <int GW, typename P>
constexpr int kShares = P::N == 4 ? piece_groups(GW) : GW == 64 ? 8 : piece_groups(2 * GW);
// Places of a thread in LDS, N doubles each, for the sums below.
template <int S, int PG, bool WAVE>
constexpr int kHeldSums = S == 4 * PG ? 2 : S == 2 * PG || !WAVE ? 1 : 0;
// The sum of the shares of lane group j, in their order: one(acc, share, next) adds up one of them (from S on there is nothing
// to add) and is told which one follows (S: none).  Shares are of `per` of `count`: those from count / per on are empty, and
// where a group's second is, nothing waits.  Sums that wait for others do so in the thread's places in LDS: the kernel has no
// registers for them.
template <int S, int PG, int N, int R, typename One>
__device__ __forceinline__ SumPiece<N> sum_shares(uint32_t j, uint32_t count, uint32_t per, double (*held)[R], One&& one) {
    constexpr int M = S > PG ? S / PG : 1;
    static_assert((S % PG == 0 || PG % S == 0) && (M == 1 || M == 2 || M == 4), "every group has as many, which meet in pairs");
    const auto put = [&](const SumPiece<N>& acc, int place) {
#pragma unroll
        for (int i = 0; i < N; ++i) held[place * N + i][threadIdx.x] = acc.v[i];
    };
    const auto meet = [&](SumPiece<N>& acc, int place) {
#pragma unroll
        for (int i = 0; i < N; ++i) acc.v[i] += held[place * N + i][threadIdx.x];
    };
    SumPiece<N> acc;
    if constexpr (M == 1) {
        acc.zero();
        one(acc, j, (uint32_t)S);
    } else {
        int turns = 1;                                              // the same in every lane
#pragma unroll
        for (int t = 1; t < M; ++t) turns += count > t * PG * per;
#pragma unroll 1
        for (int t = 0;; ++t) {
            acc.zero();
            one(acc, j + t * PG, t + 1 < M ? j + (t + 1) * PG : (uint32_t)S);
            if (M == 4 && t >= 2) meet(acc, t - 2);                 // of four: 0 and 2, 1 and 3
            if (t + 1 >= turns) break;
            put(acc, M == 4 ? t % 2 : 0);
        }
        if (M == 4 && turns == 3) meet(acc, 1);
        else if (turns > 1) meet(acc, 0);
    }
    return acc;
}
// Sum over the lane groups that took a piece.  The whole sum is in the first group.  By workgroup: the wavefronts behind the
// first four leave their sums in LDS, in the threads' own places, for those, then three of the four for the first, which goes on
// by lane shuffles.  The places may be used again after the call.
template <int GW, int BLOCK, int N, int R>
__device__ __forceinline__ void piece_sum(SumPiece<N>& acc, double (*held)[R]) {
    if constexpr (!kWavePieces<GW>) {
        constexpr uint32_t FOUR = 4 * kWave;
        static_assert(BLOCK == FOUR || BLOCK == 2 * FOUR || BLOCK == 4 * FOUR, "halves of halves");
        const uint32_t tid = threadIdx.x;
        const auto leave = [&](uint32_t from, uint32_t to) {
            if (tid >= from && tid < to) {
#pragma unroll
                for (int i = 0; i < N; ++i) held[i][tid] = acc.v[i];
            }
            __syncthreads();
        };
        const auto meet_four = [&](uint32_t step) {            // this one and those step, 2 * step and 3 * step on
#pragma unroll
            for (int i = 0; i < N; ++i)
                acc.v[i] = (acc.v[i] + held[i][tid + 2 * step]) + (held[i][tid + step] + held[i][tid + 3 * step]);
        };
        if constexpr (BLOCK > FOUR) {
            leave(FOUR, BLOCK);
            if (tid < FOUR) {
                if constexpr (BLOCK == 4 * FOUR) {
                    meet_four(FOUR);
                } else {
#pragma unroll
                    for (int i = 0; i < N; ++i) acc.v[i] += held[i][tid + FOUR];
                }
            }
        }
        leave(kWave, FOUR);
        if (tid < kWave) meet_four(kWave);
        __syncthreads();
    }
#pragma unroll
    for (int off = kWave / 2; off >= GW; off >>= 1)
#pragma unroll
        for (int i = 0; i < N; ++i) acc.v[i] += __shfl_xor(acc.v[i], off, kWave);
}

// counts: the numbers of row and piece records when they were made on the device (bp_embbag_bwd_update), else NULL
// and the host's numbers hold.  use_first: a row record's `first` is the bag of its first lookup (one lookup per bag,
// or records made from sorted bag numbers); otherwise every bag number comes from bag_of.
// Rows a lane group takes per round.  Two would have their requests in flight together, but at eight wavefronts per
// SIMD their state spills (50.7 us), and with the registers for it only six wavefronts fit (40.8 us).
constexpr int kBwdRows = 1;
template <int GW, typename P, int BLOCK>
__global__ __launch_bounds__(BLOCK, P::N == 8 ? 4 : 8) void bwd_rows_kernel(const uint4* __restrict__ row_recs,
                                                            const uint4* __restrict__ piece_recs,
                                                            const uint32_t* __restrict__ n_rows_ptr,
                                                            const uint32_t* __restrict__ n_pieces_ptr,
                                                            uint32_t n_rows_host, uint32_t n_pieces_host,
                                                            uint32_t piece_blocks, const uint32_t* __restrict__ bag_of,
                                                            int use_first, uint32_t n, int64_t C,
                                                            const float* __restrict__ grad, typename P::Unit* cache_w, float* cache_s,
                                                            double* partial, uint32_t partial_rows, uint32_t* tickets,
                                                            UpdateParams u) {
    constexpr int N = P::N;
    constexpr int G = BLOCK / GW;                     // lane groups per workgroup
    const int c = threadIdx.x % GW, j = threadIdx.x / GW;
    const bool active = c < u.lpr;

    if (blockIdx.x >= piece_blocks) {
        // ---- rows of up to kRowMax lookups: kBwdRows per lane group and round.  First every request that needs
        // nothing but the record -- the cache row, its state, the first bag numbers -- then the sums.  The record's
        // test is a value, not a branch in front of the requests: behind an early `continue` the compiler fetches
        // the record word by word, each word behind the test of the one before, and the row's requests leave two
        // round trips later (39.4 instead of 37.3 us on a Criteo-shaped batch).
        const uint32_t R = n_rows_ptr ? *n_rows_ptr : n_rows_host;
        const uint32_t groups = (gridDim.x - piece_blocks) * G;
        for (uint32_t w0 = ((blockIdx.x - piece_blocks) * G + j) * kBwdRows; w0 < R; w0 += groups * kBwdRows) {
            uint4 rec[kBwdRows];
            bool ok[kBwdRows];
            RowPiece<P> row[kBwdRows];
            uint32_t idx[kBwdRows][4];
#pragma unroll
            for (int r = 0; r < kBwdRows; ++r) rec[r] = w0 + r < R ? row_recs[w0 + r] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < kBwdRows; ++r) {
                const uint32_t start = rec[r].x & kPosMask, count = rec[r].y, slot = rec[r].z;
                ok[r] = !(rec[r].x & kLongRow) && (int64_t)slot < C && count != 0 && start < n && count <= n - start;
                row[r] = load_row<P>(u, cache_w, cache_s, ok[r] ? (int64_t)slot : 0, c, active && ok[r]);
                idx[r][0] = use_first ? rec[r].w : (ok[r] ? bag_of[start] : 0u);
#pragma unroll
                for (int k = 1; k < 4; ++k) idx[r][k] = ok[r] && (uint32_t)k < count ? bag_of[start + k] : 0u;
            }
#pragma unroll
            for (int r = 0; r < kBwdRows; ++r) {
                if (!ok[r]) continue;
                const uint32_t start = rec[r].x & kPosMask, count = rec[r].y;
                SumPiece<N> acc;
                acc.zero();
                if (active) add_gradient_rows<false, P, N>(acc, idx[r], start, start + count, 0, 0, bag_of, grad, u, c);
                finish_update<GW, P>(u, cache_w, cache_s, (int64_t)rec[r].z, c, row[r], acc.template rounded<P>(), active);
            }
        }
        return;
    }

    // ---- pieces of longer rows: a wavefront or a workgroup each (kWavePieces)
    constexpr bool WAVE = kWavePieces<GW>;
    constexpr int PG = kPieceThreads<GW, BLOCK> / GW;           // lane groups that share a piece
    constexpr int PER_BLOCK = BLOCK / kPieceThreads<GW, BLOCK>;
    constexpr int S = kShares<GW, P>;
    constexpr int HELD = kHeldSums<S, PG, WAVE>;
    __shared__ double held[HELD ? HELD * N : 1][HELD ? BLOCK : 1];
    const int pj = WAVE ? j % PG : j;
    const uint32_t n_pieces = n_pieces_ptr ? *n_pieces_ptr : n_pieces_host;
    const bool writer = active && pj == 0;
    for (uint32_t pi = blockIdx.x * PER_BLOCK + (WAVE ? threadIdx.x / kWave : 0u); pi < n_pieces; pi += piece_blocks * PER_BLOCK) {
        const uint4 r0 = piece_recs[2 * (size_t)pi], r1 = piece_recs[2 * (size_t)pi + 1];
        const uint32_t start = r0.x, count = r0.y, slot = r0.z, index = r0.w, pieces = r1.x, pbase = r1.y;
        // a record that points outside the batch or the workspace does nothing (the test is the same in every lane)
        if ((int64_t)slot >= C || count == 0 || start >= n || count > n - start || pieces == 0 || index >= pieces) continue;
        const bool direct = pieces == 1;
        if (!direct && (pbase >= partial_rows || pieces > partial_rows - pbase)) continue;
        const uint32_t per = (count + 4 * S - 1) / (4 * S) * 4;      // lookups of a share: whole bursts
        const auto share_at = [&](uint32_t share) { return start + min(share * per, count); };
        uint32_t idx[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) idx[k] = share_at(pj) + k < share_at(pj + 1) ? bag_of[share_at(pj) + k] : 0u;
        SumPiece<N> acc = sum_shares<S, PG, N>((uint32_t)pj, count, per, held, [&](SumPiece<N>& sum, uint32_t share, uint32_t next) {
            if (active)
                add_gradient_rows<(S > PG), P, N>(sum, idx, share_at(share), share_at(share + 1), share_at(next), share_at(next + 1),
                                                 bag_of, grad, u, c);
        });
        piece_sum<GW, BLOCK, N>(acc, held);
        if (direct) {      // the row is asked for only now: one more round trip after a few hundred gradient rows
            if (pj == 0) {
                const RowPiece<P> row = load_row<P>(u, cache_w, cache_s, (int64_t)slot, c, writer);
                finish_update<GW, P>(u, cache_w, cache_s, (int64_t)slot, c, row, acc.template rounded<P>(), writer);
            }
            continue;
        }
        // One of several pieces: leave the sum where whoever takes the last piece will find it, then take a ticket
        // (device-coherent stores, complete before this piece is counted; whoever counts the last piece then reads
        // all the sums with device-coherent loads).  The pieces of a row of very many meet in stretches of kStretch first,
        // and then the stretches: whoever takes the row's last piece would read the sums of thousands one burst behind the other,
        // most of all a wavefront of four-lane rows, with sixteen lane groups (a row's 4.2 M lookups, dim 16: 392 us in one
        // step, 63 in two; dim 64 698 / 313; 262,144 lookups, dim 16: 30.0 / 11.8).  The second step costs 1.2 us: up to five bursts
        // a share there is one (200,000 lookups, the hottest row's 66 pieces, dim 16: 11.5 in one step, 12.6 in two).
        constexpr uint32_t kStretch = 64, kAtOnce = 10 * S;
        const bool at_once = pieces <= kAtOnce;
        uint32_t mine = index, step = 1, first = at_once ? 0u : index / kStretch * kStretch;
        uint32_t members = at_once ? pieces : min(kStretch, pieces - first);
        uint32_t* ticket = tickets + pbase + first;
        bool last;
#pragma unroll 1
        for (;;) {
            // The writers and the lane that draws the ticket are of one wavefront, which waits for its stores here by itself: a
            // fence for the workgroup leaves them on their way, its barrier too.
            static_assert(GW <= kWave, "the writers are lanes of the workgroup's, or the piece's, first wavefront");
            if (writer) acc.store_device(partial + (size_t)(pbase + mine) * u.dim, c);
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            if constexpr (WAVE) {
                uint32_t drawn = 0;
                if (threadIdx.x % kWave == 0) drawn = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                last = __builtin_amdgcn_readfirstlane(drawn) + 1u == members;
            } else {
                __syncthreads();
                if (threadIdx.x == 0)                      // told through its own place in LDS
                    held[0][0] = __hip_atomic_fetch_add(ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1u == members ? 1.0 : 0.0;
                __syncthreads();
                last = held[0][0] != 0.0;
                __syncthreads();                           // everybody has read it before a later sum rewrites it
            }
            if (!last) break;
            acc = sum_shares<S, PG, N>((uint32_t)pj, members, 1, held, [&](SumPiece<N>& sum, uint32_t share, uint32_t) {
                for (uint32_t b = share; b < members && (PG <= S || share < S); b += 2 * S) {
                    SumPiece<N> t[2];
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        t[k].zero();
                        if (active && b + (uint32_t)k * S < members)
                            t[k].load_device(partial + (size_t)(pbase + first + (b + k * S) * step) * u.dim, c);
                    }
#pragma unroll
                    for (int k = 0; k < 2; ++k) sum.add(t[k]);
                }
            });
            piece_sum<GW, BLOCK, N>(acc, held);
            if (threadIdx.x % kPieceThreads<GW, BLOCK> == 0)      // the counter is zero again for the next call
                __hip_atomic_store(ticket, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (step > 1 || at_once) break;
            mine = first;                                         // the stretches, each in the place of its first piece
            step = kStretch;
            first = 0;
            members = (pieces + kStretch - 1) / kStretch;
            ticket = tickets + pbase + 1;                         // counts no stretch
        }
        if (!last) continue;
        if (pj == 0) {
            const RowPiece<P> row = load_row<P>(u, cache_w, cache_s, (int64_t)slot, c, writer);
            finish_update<GW, P>(u, cache_w, cache_s, (int64_t)slot, c, row, acc.template rounded<P>(), writer);
        }
    }
}

// ---- records made on the device (bp_embbag_bwd_update: one batch, lookups sorted by slot) -------------------------
// One launch, without a scan: a workgroup counts the rows and pieces that start among its lookups, draws as many places in the
// two lists from a counter each, and writes them there.  The lists' order follows the draws, and nothing depends on it: every
// record is complete in itself, and a row of several pieces owns a stretch of partial sums of its own.  A row ends where the slot
// changes: within the window as a rule, else it is searched for.  (19,000 lookups: the scans over lookups and rows took four
// launches and 12.7 us, one of 7.0 this way; the whole call on 4 M lookups 565 -> 313 us, on 500 22.0 -> 14.9.)
template <int ROUNDS>
__global__ __launch_bounds__(kScanBlock) void bwd_records_kernel(const uint32_t* __restrict__ keys, const uint32_t* __restrict__ bags,
                                                                 uint32_t n, uint4* __restrict__ row_recs,
                                                                 uint4* __restrict__ piece_recs, unsigned long long* counters) {
    constexpr int WAVES = kScanBlock / kWave;
    constexpr uint32_t TILE = kScanBlock * ROUNDS, WINDOW = TILE + 256;
    __shared__ uint32_t wave_rows[WAVES], row_base;
    __shared__ uint64_t wave_pieces[WAVES], piece_base;
    __shared__ uint32_t win[WINDOW];                     // the tile's keys and the next 256: nearly every row ends in them
    const int w = threadIdx.x / kWave, lane = lane_id();
    const uint32_t tile = blockIdx.x * TILE, end = min(n - tile, WINDOW);
    for (uint32_t t = threadIdx.x; t < end; t += kScanBlock) win[t] = keys[tile + t];
    const uint32_t of_wave = tile + w * (kWave * ROUNDS);
    uint32_t before = of_wave > 0 && of_wave <= n ? keys[of_wave - 1] : 0u;
    __syncthreads();
    uint32_t key[ROUNDS], count[ROUNDS];                 // count: of the row that starts here, 0 where none does
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t p = of_wave + r * kWave + lane;
        key[r] = p < n ? win[p - tile] : 0u;
    }
    uint32_t rows = 0;
    uint64_t pieces = 0;                                 // pieces, and in the high word those of rows of several
    const auto packed = [](uint32_t lookups) {
        const uint32_t pc = pieces_of(lookups);
        return (uint64_t)pc | ((uint64_t)(pc > 1 ? pc : 0u) << 32);
    };
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t p = of_wave + r * kWave + lane;
        const uint32_t left = lane_below(key[r], before);
        before = lane_value(key[r], kWave - 1);
        const bool head = p < n && (p == 0 || key[r] != left);
        count[r] = 0;
        if (head) {
            // the key at lo - 1 is the row's, the one at hi is not (or hi is n)
            uint32_t lo = p - tile + 1, hi = min(end, lo + kRowMax - 1);
            if (hi < end && win[hi] == key[r]) {
                lo = hi + 1;
                hi = end;
            }
            while (lo < hi) {
                const uint32_t mid = lo + (hi - lo) / 2;
                if (win[mid] == key[r]) lo = mid + 1; else hi = mid;
            }
            lo += tile;
            if (lo == tile + end && lo < n) {            // it goes on behind the window
                hi = lo;
                for (uint32_t step = WINDOW; hi < n && keys[hi] == key[r]; step *= 2) {
                    lo = hi + 1;
                    hi = step < n - hi ? hi + step : n;
                }
                while (lo < hi) {
                    const uint32_t mid = lo + (hi - lo) / 2;
                    if (keys[mid] == key[r]) lo = mid + 1; else hi = mid;
                }
            }
            count[r] = lo - p;
        }
        rows += (uint32_t)__popcll(__ballot(head));
        if (__ballot(count[r] > kRowMax)) pieces += wave_reduce(packed(count[r]), AddOp());
    }
    if (lane == 0) {
        wave_rows[w] = rows;
        wave_pieces[w] = pieces;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t r = 0;
        uint64_t pc = 0;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) {
            r += wave_rows[k];
            pc += wave_pieces[k];
        }
        row_base = r ? (uint32_t)atomicAdd(counters, (unsigned long long)r) : 0u;
        piece_base = pc ? (uint64_t)atomicAdd(counters + 1, (unsigned long long)pc) : 0u;
    }
    __syncthreads();
    uint32_t row = row_base;
    uint64_t piece = piece_base;
    for (int k = 0; k < w; ++k) {
        row += wave_rows[k];
        piece += wave_pieces[k];
    }
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) {
        const uint32_t p = of_wave + r * kWave + lane;
        const uint64_t heads = __ballot(count[r] != 0);
        uint64_t mine = piece;
        if (__ballot(count[r] > kRowMax)) {
            const uint64_t inc = wave_inclusive_scan(packed(count[r]), AddOp());
            mine = piece + lane_below(inc, uint64_t(0));
            piece += lane_value(inc, kWave - 1);
        }
        if (count[r]) {
            const uint32_t pc = pieces_of(count[r]);
            const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(heads >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)heads, row));
            row_recs[at] = make_uint4(p | (pc ? kLongRow : 0u), count[r], key[r], bags[p]);
            if (pc) write_pieces(piece_recs, (uint32_t)mine, pc, p, count[r], key[r], (uint32_t)(mine >> 32), 0u);
        }
        row += (uint32_t)__popcll(heads);
    }
}

// ---- workspace -------------------------------------------------------------------------------
constexpr int64_t kLargeSort = int64_t(1) << 21;

struct ReduceScratch {      // what the reduce kernel itself needs, in both entry points
    uint32_t* tickets;      // the caller's counters, one per partial row, zero between calls
    double* partial;
    uint32_t partial_rows;
};
ReduceScratch carve_reduce(Carver& c, int64_t n, int dim) {
    ReduceScratch r{};
    r.partial_rows = (uint32_t)partial_rows_for(n);
    r.partial = c.take<double>((size_t)r.partial_rows * (size_t)dim);
    return r;
}

struct BwdWorkspace {
    ReduceScratch red;
    uint32_t *keys_a, *keys_b, *vals_a, *vals_b, *sort_temp;
    uint64_t* counters;        // rows; pieces, and in the high word those of rows of several
    uint4 *row_recs, *piece_recs;
    size_t bytes;
};

BwdWorkspace carve_bwd(void* base, size_t cap, int64_t n, int dim) {
    Carver c(base, cap);
    BwdWorkspace w{};
    const size_t m = (size_t)(n > 0 ? n : 1);
    w.red = carve_reduce(c, n, dim);
    w.keys_a = c.take<uint32_t>(m);
    w.keys_b = c.take<uint32_t>(m);
    w.vals_a = c.take<uint32_t>(m);
    w.vals_b = c.take<uint32_t>(m);
    w.sort_temp = c.take<uint32_t>(n >= kLargeSort ? sort_temp_words<LargeTiles>(n) : sort_temp_words<SmallTiles>(n));
    w.counters = c.take<uint64_t>(2);
    w.row_recs = c.take<uint4>(m);
    w.piece_recs = c.take<uint4>(2 * piece_capacity_for(n));
    w.bytes = c.used();
    return w;
}

// Two choices that change no bit of the result (kShares above), us of the kernel on caches of hundreds of MB, ids uniform / skewed
// (of 200,000 lookups 181,000 / 53,000 rows distinct).  bp_embbag_bwd_update knows no counts when it launches, only bounds, and so
// takes the forms for batches with long rows and as many rows as lookups:
//   bf16 rows by fours or by eights a lane (dispatch_values).  By fours pieces are quicker in a launch that the chip holds at once
//     (20,000 lookups, dim 64: 3.8 / 6.6 by fours, 3.7 / 8.1 by eights); a larger one has the more bytes in flight by eights
//     (200,000, dim 128, row-wise Adagrad: 50 / 29.5 by fours, 44 / 27.8 by eights; 1.3 M: 249 / 178, 235 / 177).
//   256 threads or sixteen lane groups, for rows of 32 and 64 lanes: the wide workgroup has a piece done sooner, which small
//     launches wait for (fp32, dim 256, row-wise Adagrad, 20,000 lookups, skewed: 18.2 with 256 threads, 11.8 wide); large ones
//     lose, whose rows hold a workgroup's place until its last one ends (200,000: 65.8, 70.3).  Rows that leave lanes idle gain
//     in launches that the chip holds at once (dim 100, 20,000 skewed: 11.1, 9.2; bf16 dim 192, 200,000: 42.2, 45.3), and so few
//     pieces that they are likely short are not worth it (30,000 lookups of 18,000 rows, one piece, dim 256: 14.4, 15.4).
struct BwdLaunch {
    const bp_config* cfg;
    ReduceScratch red;
    const uint4 *row_recs, *piece_recs;
    const uint32_t *n_rows_ptr, *n_pieces_ptr;     // device counts, or NULL when the host's numbers hold
    uint32_t n_rows, n_pieces;                     // host counts, or upper bounds when the device counts
    const uint32_t* bag_of;
    int use_first;
    int64_t n;
    const float* grad;
    void* cache_w;
    void* cache_s;
    hipStream_t stream;
    int64_t bags;
    int64_t chips(int lanes) const { return ceil_div((int64_t)n_rows * lanes, int64_t(256) * 2048); }      // that the rows fill
    bool long_rows() const { return (int64_t)n_pieces * 4096 >= (int64_t)n_rows; }
    int launch() { return dispatch_values<true>(cfg, n_pieces == 0 || chips(group_width(cfg->dim / 4)) > 1, *this); }
    template <int GW, typename P>
    int run(int lpr) {
        if constexpr (kBwdWideBlock<GW, P> != 256) {
            const bool wide = long_rows() && chips(GW) <= (lpr == GW ? 4 : 1);
            if (wide) return run_block<GW, P, kBwdWideBlock<GW, P>>(lpr);
        }
        return run_block<GW, P, 256>(lpr);
    }
    template <int GW, typename P, int BLOCK>
    int run_block(int lpr) {
        const size_t sbytes = cfg->cache_state_stride ? (size_t)cfg->cache_state_stride : state_row_bytes(cfg);
        UpdateParams u{cfg->optimizer, cfg->lr, cfg->eps, lpr, cfg->dim,
                       (uint32_t)(bags > 0 ? bags : 1), cache_w_stride16(cfg) * P::kPerVec, (int64_t)(sbytes / 4)};
        int64_t piece_blocks = ceil_div((int64_t)n_pieces, BLOCK / kPieceThreads<GW, BLOCK>), row_blocks = ceil_div((int64_t)n_rows, BLOCK / GW);
        if (piece_blocks > kMaxGridBlocks / 4) piece_blocks = kMaxGridBlocks / 4;
        if (row_blocks > kMaxGridBlocks) row_blocks = kMaxGridBlocks;
        if (row_blocks < 1) row_blocks = 1;
        BP_LAUNCH(K_BWD_REDUCE_UPDATE, (bwd_rows_kernel<GW, P, BLOCK>), dim3((unsigned)(piece_blocks + row_blocks)), dim3(BLOCK), 0,
                  stream, row_recs, piece_recs, n_rows_ptr, n_pieces_ptr, n_rows, n_pieces, (uint32_t)piece_blocks, bag_of,
                  use_first, (uint32_t)n, cfg->capacity, grad, (typename P::Unit*)cache_w, (float*)cache_s, red.partial,
                  red.partial_rows, red.tickets, u);
        return BP_OK;
    }
};

int check_bwd_args(const bp_config* cfg, int64_t n, int64_t bags) {
    BP_TRY(check_config(cfg));
    if (n < 0 || bags < 0) return fail(BP_ERR_INVALID_ARG, "negative size");
    if (n >= (int64_t(1) << 31) || bags >= (int64_t(1) << 31)) return fail(BP_ERR_UNSUPPORTED, "size >= 2^31");
    return BP_OK;
}

}  // namespace
}  // namespace bp

using namespace bp;

BP_EXPORT size_t bp_embbag_bwd_ticket_bytes(int64_t n_lookups) { return partial_rows_for(n_lookups) * sizeof(uint32_t); }

BP_EXPORT int bp_embbag_bwd_update_workspace_bytes(const bp_config* cfg, int64_t n_lookups, int64_t bags, size_t* bytes) {
    if (!bytes) return fail(BP_ERR_INVALID_ARG, "bytes is NULL");
    BP_TRY(check_bwd_args(cfg, n_lookups, bags));
    // enough for fewer lookups as well, of which those just below kLargeSort need more than those from there on (the
    // call itself asks for no more than its own batch needs)
    *bytes = carve_bwd(nullptr, 0, n_lookups, cfg->dim).bytes;
    if (n_lookups >= kLargeSort) *bytes = std::max(*bytes, carve_bwd(nullptr, 0, kLargeSort - 1, cfg->dim).bytes);
    return BP_OK;
}

BP_EXPORT int bp_embbag_bwd_update(const bp_config* cfg, void* cache_w, void* cache_state, const int32_t* lookup_slots,
                                    const int64_t* bag_offsets, int64_t n_lookups, int64_t bags, const float* grad_out,
                                    void* workspace, size_t workspace_bytes, uint32_t* tickets, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t n = n_lookups;
    BP_TRY(check_bwd_args(cfg, n, bags));
    if (n == 0) return BP_OK;
    if (!bag_offsets && n != bags)
        return fail(BP_ERR_INVALID_ARG, "bag_offsets is NULL but n_lookups %lld != bags %lld", (long long)n, (long long)bags);
    if (!cache_w || !lookup_slots || !grad_out) return fail(BP_ERR_INVALID_ARG, "NULL pointer");
    if (cfg->optimizer != BP_SGD && !cache_state) return fail(BP_ERR_INVALID_ARG, "cache_state is NULL");
    if (((uintptr_t)cache_w | (uintptr_t)cache_state | (uintptr_t)grad_out) & 15)
        return fail(BP_ERR_INVALID_ARG, "cache_w, cache_state and grad_out must be 16-byte aligned");
    if (!workspace || ((uintptr_t)workspace & 255)) return fail(BP_ERR_INVALID_ARG, "workspace NULL or not 256-byte aligned");
    if (!tickets || ((uintptr_t)tickets & 3)) return fail(BP_ERR_INVALID_ARG, "tickets NULL or not 4-byte aligned");
    BwdWorkspace w = carve_bwd(workspace, workspace_bytes, n, cfg->dim);
    if (w.bytes > workspace_bytes)
        return fail(BP_ERR_WORKSPACE_TOO_SMALL, "workspace %zu < required %zu bytes", workspace_bytes, w.bytes);
    w.red.tickets = tickets;

    bool in_b = false;
    const int key_bits = bits_for(cfg->capacity + 1);
    const auto keys_and_sort = [&](auto tiles) {
        typedef decltype(tiles) Tiles;
        const uint32_t ntiles = sort_num_tiles<Tiles>(n);
        const int nb = radix_first_pass_bits(0, key_bits), by_tile = sort_counts_by_tile<Tiles>(ntiles);
        const uint32_t mask = (1u << nb) - 1u;
        if (nb > 8)
            BP_LAUNCH(K_BWD_KEYS, (bwd_keys_kernel<9, Tiles>), dim3(ntiles), dim3(Tiles::BLOCK), 0, stream, lookup_slots, bag_offsets,
                      (uint32_t)n, (uint32_t)bags, cfg->capacity, w.keys_a, w.vals_a, mask, w.sort_temp, ntiles, by_tile, w.counters);
        else
            BP_LAUNCH(K_BWD_KEYS, (bwd_keys_kernel<8, Tiles>), dim3(ntiles), dim3(Tiles::BLOCK), 0, stream, lookup_slots, bag_offsets,
                      (uint32_t)n, (uint32_t)bags, cfg->capacity, w.keys_a, w.vals_a, mask, w.sort_temp, ntiles, by_tile, w.counters);
        return radix_sort_pairs<uint32_t, Tiles>(w.keys_a, w.keys_b, w.vals_a, w.vals_b, n, 0, key_bits, w.sort_temp, stream, &in_b,
                                                 w.sort_temp);
    };
    if (n >= kLargeSort) BP_TRY(keys_and_sort(LargeTiles{}));
    else BP_TRY(keys_and_sort(SmallTiles{}));
    const uint32_t* skeys = in_b ? w.keys_b : w.keys_a;
    const uint32_t* sbags = in_b ? w.vals_b : w.vals_a;

    // the records; the counts stay on the device
    unsigned long long* const counters = reinterpret_cast<unsigned long long*>(w.counters);
    if (n <= kScanSmall)
        BP_LAUNCH(K_BWD_ITEMS, bwd_records_kernel<1>, dim3((unsigned)ceil_div(n, kScanBlock)), dim3(kScanBlock), 0, stream, skeys,
                  sbags, (uint32_t)n, w.row_recs, w.piece_recs, counters);
    else
        BP_LAUNCH(K_BWD_ITEMS, bwd_records_kernel<8>, dim3((unsigned)ceil_div(n, 8 * kScanBlock)), dim3(kScanBlock), 0, stream, skeys,
                  sbags, (uint32_t)n, w.row_recs, w.piece_recs, counters);
    const uint32_t* n_rows = reinterpret_cast<const uint32_t*>(w.counters);              // low words
    const uint32_t* n_pieces = reinterpret_cast<const uint32_t*>(w.counters + 1);

    BwdLaunch l{cfg, w.red, w.row_recs, w.piece_recs, n_rows, n_pieces, (uint32_t)n, (uint32_t)piece_capacity_for(n), sbags,
                1, n, grad_out, cache_w, cache_state, stream, bags};
    return l.launch();
}

// ---- grouped variant: the plan already lists the batch's lookups grouped by row ---------------------------------
namespace bp {
namespace {
struct GroupedWorkspace {
    ReduceScratch red;
    uint32_t* bag_of;          // bag of every grouped position
    uint32_t* bag_of_lookup;   // bag of every lookup, in lookup order
    size_t bytes;
};
GroupedWorkspace carve_grouped(void* base, size_t cap, int64_t n, int dim, bool multi_hot) {
    Carver c(base, cap);
    GroupedWorkspace w{};
    const size_t m = (size_t)(n > 0 ? n : 1);
    w.red = carve_reduce(c, n, dim);
    w.bag_of = multi_hot ? c.take<uint32_t>(m) : nullptr;
    w.bag_of_lookup = multi_hot ? c.take<uint32_t>(m) : nullptr;
    w.bytes = c.used();
    return w;
}
}  // namespace
}  // namespace bp

BP_EXPORT int bp_embbag_bwd_update_grouped_workspace_bytes(const bp_config* cfg, int64_t n_lookups, int64_t bags,
                                                           int32_t multi_hot, size_t* bytes) {
    if (!bytes) return fail(BP_ERR_INVALID_ARG, "bytes is NULL");
    BP_TRY(check_bwd_args(cfg, n_lookups, bags));
    *bytes = carve_grouped(nullptr, 0, n_lookups, cfg->dim, multi_hot != 0).bytes;
    return BP_OK;
}

BP_EXPORT int bp_embbag_bwd_update_grouped(const bp_config* cfg, void* cache_w, void* cache_state,
                                           const int32_t* grouped_lookups, const bp_row_rec* row_recs, int64_t n_rows,
                                           const bp_piece_rec* piece_recs, int64_t n_pieces, const int64_t* bag_offsets,
                                           int64_t n_lookups, int64_t bags, const float* grad_out, void* workspace,
                                           size_t workspace_bytes, uint32_t* tickets, void* stream_) {
    hipStream_t stream = (hipStream_t)stream_;
    const int64_t n = n_lookups;
    BP_TRY(check_bwd_args(cfg, n, bags));
    if (n == 0) return BP_OK;
    if (n_rows < 1 || n_rows > n) return fail(BP_ERR_INVALID_ARG, "n_rows %lld outside [1, n_lookups]", (long long)n_rows);
    if (n_pieces < 0 || n_pieces > (int64_t)piece_capacity_for(n) || (n_pieces && !piece_recs))
        return fail(BP_ERR_INVALID_ARG, "n_pieces %lld outside [0, %lld] or piece_recs is NULL", (long long)n_pieces,
                    (long long)piece_capacity_for(n));
    if (!bag_offsets && n != bags)
        return fail(BP_ERR_INVALID_ARG, "bag_offsets is NULL but n_lookups %lld != bags %lld", (long long)n, (long long)bags);
    if (!cache_w || !grouped_lookups || !row_recs || !grad_out) return fail(BP_ERR_INVALID_ARG, "NULL pointer");
    if (cfg->optimizer != BP_SGD && !cache_state) return fail(BP_ERR_INVALID_ARG, "cache_state is NULL");
    if (((uintptr_t)cache_w | (uintptr_t)cache_state | (uintptr_t)grad_out | (uintptr_t)row_recs | (uintptr_t)piece_recs) & 15)
        return fail(BP_ERR_INVALID_ARG, "cache_w, cache_state, grad_out and the records must be 16-byte aligned");
    if (!workspace || ((uintptr_t)workspace & 255)) return fail(BP_ERR_INVALID_ARG, "workspace NULL or not 256-byte aligned");
    if (!tickets || ((uintptr_t)tickets & 3)) return fail(BP_ERR_INVALID_ARG, "tickets NULL or not 4-byte aligned");
    GroupedWorkspace w = carve_grouped(workspace, workspace_bytes, n, cfg->dim, bag_offsets != nullptr);
    if (w.bytes > workspace_bytes)
        return fail(BP_ERR_WORKSPACE_TOO_SMALL, "workspace %zu < required %zu bytes", workspace_bytes, w.bytes);
    w.red.tickets = tickets;
    const uint32_t* bag_of = reinterpret_cast<const uint32_t*>(grouped_lookups);   // one lookup per bag: position == bag
    if (bag_offsets) {
        const dim3 bag_grid((unsigned)ceil_div(bags > 0 ? bags : 1, 256));
        if (n >= kListedBags * bags) {
            BagsOf64* list = reinterpret_cast<BagsOf64*>(w.bag_of_lookup);         // a quarter of a byte a lookup
            BP_LAUNCH(K_BWD_KEYS, bwd_list_bags_kernel, bag_grid, dim3(256), 0, stream, bag_offsets, bags, n, list);
            BP_LAUNCH(K_BWD_KEYS, bwd_bags_from_list_kernel, dim3((unsigned)ceil_div(n, 1024)), dim3(256), 0, stream, grouped_lookups,
                      (const BagsOf64*)list, bag_offsets, n, bags, w.bag_of);
        } else {
            BP_LAUNCH(K_BWD_KEYS, bwd_bag_of_lookup_kernel, bag_grid, dim3(256), 0, stream, bag_offsets, bags, n, w.bag_of_lookup);
            BP_LAUNCH(K_BWD_KEYS, bwd_bags_of_positions_kernel, dim3((unsigned)ceil_div(n, 256)), dim3(256), 0, stream,
                      grouped_lookups, (const uint32_t*)w.bag_of_lookup, n, bags, w.bag_of);
        }
        bag_of = w.bag_of;
    }
    BwdLaunch l{cfg, w.red, reinterpret_cast<const uint4*>(row_recs), reinterpret_cast<const uint4*>(piece_recs), nullptr,
                nullptr, (uint32_t)n_rows, (uint32_t)n_pieces, bag_of, bag_offsets == nullptr, n, grad_out, cache_w,
                cache_state, stream, bags};
    return l.launch();
}

// ---- the grouped variant for callers that cannot allocate ---------------------------------------------------------
// Same kernels; the scratch (counters, partial sums, the bag numbers of the grouped positions) lives in a fixed array
// in device memory that belongs to the library.  Every GPU the library runs on holds its own copy of the array at
// its own address, found once per device with that device current.
namespace bp {
namespace {
constexpr size_t kStaticScratchBytes = size_t(16) << 20;
// The counters own a stretch of fixed size at the array's start, whatever the batch: partial sums of one call must
// never land where a later, larger call expects zeroed counters.
constexpr size_t kStaticTickets = size_t(1) << 16;
constexpr size_t kStaticTicketBytes = kStaticTickets * sizeof(uint32_t);
static __device__ __align__(256) unsigned char g_static_scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
unsigned char* g_scratch_ptr[kMaxDevices] = {};     // per device: where its copy of the array lives

__global__ __launch_bounds__(256) void bwd_clear_words_kernel(uint32_t* p, size_t n) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// The current device's copy of the scratch array.  On the first call for a device the address is looked up and the
// array cleared once (the counters at its start must be zero; every call leaves them zero).
int static_scratch(hipStream_t stream, unsigned char** out) {
    int dev = -1;
    BP_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(BP_ERR_UNSUPPORTED, "device %d outside [0, %d)", dev, kMaxDevices);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        BP_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_static_scratch)));
        if (!ptr) return fail(BP_ERR_HIP, "the scratch array has no address on device %d", dev);
        const size_t words = kStaticScratchBytes / sizeof(uint32_t);
        BP_LAUNCH(K_FILL, bwd_clear_words_kernel, dim3((unsigned)ceil_div((int64_t)words, 256)), dim3(256), 0, stream,
                  (uint32_t*)ptr, words);
        g_scratch_ptr[dev] = (unsigned char*)ptr;
    }
    *out = g_scratch_ptr[dev];
    return BP_OK;
}
}  // namespace
}  // namespace bp

BP_EXPORT size_t bp_embbag_bwd_update_grouped_static_max_bytes(void) { return kStaticScratchBytes; }

BP_EXPORT int bp_embbag_bwd_update_grouped_static_bytes(const bp_config* cfg, int64_t n_lookups, int64_t bags,
                                                        int32_t multi_hot, size_t* bytes) {
    if (!bytes) return fail(BP_ERR_INVALID_ARG, "bytes is NULL");
    BP_TRY(check_bwd_args(cfg, n_lookups, bags));
    if (partial_rows_for(n_lookups) > kStaticTickets)
        return fail(BP_ERR_UNSUPPORTED, "a batch of %lld lookups needs %zu counters, the library's fixed array holds %zu",
                    (long long)n_lookups, partial_rows_for(n_lookups), kStaticTickets);
    *bytes = kStaticTicketBytes + carve_grouped(nullptr, 0, n_lookups, cfg->dim, multi_hot != 0).bytes;
    return BP_OK;
}

BP_EXPORT int bp_embbag_bwd_update_grouped_static(const bp_config* cfg, void* cache_w, void* cache_state,
                                                  const int32_t* grouped_lookups, const bp_row_rec* row_recs,
                                                  int64_t n_rows, const bp_piece_rec* piece_recs, int64_t n_pieces,
                                                  const int64_t* bag_offsets, int64_t n_lookups, int64_t bags,
                                                  const float* grad_out, void* stream) {
    size_t need = 0;
    BP_TRY(bp_embbag_bwd_update_grouped_static_bytes(cfg, n_lookups, bags, bag_offsets != nullptr, &need));
    if (need > kStaticScratchBytes)
        return fail(BP_ERR_UNSUPPORTED, "a batch of %lld lookups needs %zu bytes of scratch, the library's fixed array holds %zu",
                    (long long)n_lookups, need, kStaticScratchBytes);
    if (n_lookups == 0) return BP_OK;
    unsigned char* base = nullptr;
    BP_TRY(static_scratch((hipStream_t)stream, &base));
    return bp_embbag_bwd_update_grouped(cfg, cache_w, cache_state, grouped_lookups, row_recs, n_rows, piece_recs, n_pieces,
                                        bag_offsets, n_lookups, bags, grad_out, base + kStaticTicketBytes,
                                        kStaticScratchBytes - kStaticTicketBytes, reinterpret_cast<uint32_t*>(base), stream);
}
