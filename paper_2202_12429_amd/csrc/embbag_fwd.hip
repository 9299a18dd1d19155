// bp_embbag_fwd: EmbeddingBag-sum forward over cache slots (the trainer's embedding lookup, Section 2.1,
// served from the GPU-resident cache of Section 3.2).
//  - bags of several lookups: one lane group per bag; every lane owns a piece of the row (16 bytes, or 8 of bf16 rows by
//    fours), accumulates in fp32 in lookup order and writes its piece of the pooled row;
//  - one lookup per bag (a row copy): the output is a flat array of 16-byte pieces (bf16 rows go by fours), one per lane with
//    no idle lanes, several pieces per lane in flight; a wavefront's stores are one contiguous kilobyte.
// bp_embbag_fwd_grouped: the same row copies walked by the plan's row and piece records instead of a slot per
// lookup: every distinct row is fetched once and written to the bags that look it up.
#include <algorithm>

#include "bwd_records.h"
#include "common.h"
#include "row_access.h"

namespace bp {
namespace {

// Bags of several lookups, bounded by the rows' latency where the launch leaves the chip room, else by memory: a burst's
// rows are in flight together, the slots of the next burst come while they arrive, and a bag's last, short burst is one
// round trip like the others (4.2 M rows of 256 bytes in 163,840 bags: 129 us with the last rows one by one and no slots
// fetched ahead, 118 this way, 9.1 TB/s of rows).  How deep a burst pays is the rule at FwdLaunch.
constexpr uint32_t kNoSlot = 0xffffffffu;      // past the end of every cache
template <int GW, typename P, int BURST>
__global__ __launch_bounds__(kRowBlock) void embbag_fwd_kernel(const typename P::Raw* __restrict__ cache_w,
                                                               const int32_t* __restrict__ slots,
                                                               const int64_t* __restrict__ bag_off, int64_t bags,
                                                               int64_t n, int64_t C, int lpr, int64_t wst, int dim,
                                                               float* __restrict__ out) {
    const int64_t bag = ((int64_t)blockIdx.x * kRowBlock + threadIdx.x) / GW;
    const int c = threadIdx.x % GW;
    if (bag >= bags || c >= lpr) return;
    P acc;
    acc.zero();
    int64_t k = bag_off[bag];
    int64_t end = bag_off[bag + 1];
    if (k < 0) k = 0;                           // offsets that point outside the lookups read nothing there
    if (end > n) end = n;
    if (k > end) k = end;                       // before anything is added to it: k + j cannot wrap
    uint32_t s[BURST];
    const auto fetch_slots = [&](int64_t at) {
        // A whole burst's slots in wide loads where every lane has a bag, and loads, of its own (dim 4, 163,840 bags of 8
        // lookups: 13.0 us guarded one by one, 11.3 this way); lanes that share their loads gain nothing by it.
        if (GW == 1 && at + BURST <= end) {
#pragma unroll
            for (int j = 0; j < BURST; ++j) s[j] = (uint32_t)slots[at + j];
        } else {
#pragma unroll
            for (int j = 0; j < BURST; ++j) s[j] = at + j < end ? (uint32_t)slots[at + j] : kNoSlot;
        }
    };
    fetch_slots(k);
    for (; k < end; k += BURST) {
        typename P::Raw raw[BURST];
#pragma unroll
        for (int j = 0; j < BURST; ++j)
            raw[j] = s[j] < (uint64_t)C ? cache_w[(int64_t)s[j] * wst + c] : P::none();
        if (k + BURST < end) fetch_slots(k + BURST);      // one test: bags of a single burst pass it by
#pragma unroll
        for (int j = 0; j < BURST; ++j) {       // in lookup order; a row that is not there adds zeros
            P p;
            p.decode(raw[j]);
            acc.add(p);
        }
    }
    acc.store_f32_stream(out + bag * dim, c);
}

// One lookup per bag.  Piece p of the output belongs to bag p / lpr, piece p % lpr of its row.  A workgroup owns
// kRowBlock * U consecutive pieces; the division by lpr uses inv = floor(2^32 / lpr) + 1, exact for the dividends
// that occur here (below 2^32 / lpr).
constexpr int kFlatPieces = 4;
template <typename P, int U>
__global__ __launch_bounds__(kRowBlock) void embbag_fwd_onehot_kernel(const typename P::Raw* __restrict__ cache_w,
                                                                      const int32_t* __restrict__ slots, int64_t bags,
                                                                      int64_t C, uint32_t lpr, uint32_t inv, int64_t wst,
                                                                      int dim, float* __restrict__ out) {
    const int64_t base = (int64_t)blockIdx.x * (kRowBlock * U);
    const int64_t bag0 = base / lpr;
    const uint32_t r0 = (uint32_t)(base - bag0 * lpr);
    int64_t bag[U];
    uint32_t c[U], s[U];
    typename P::Raw raw[U];
#pragma unroll
    for (int j = 0; j < U; ++j) {
        const uint32_t q = r0 + j * kRowBlock + threadIdx.x;
        const uint32_t dq = lpr == 1 ? q : __umulhi(q, inv);
        c[j] = q - dq * lpr;
        bag[j] = bag0 + dq;
        s[j] = bag[j] < bags ? (uint32_t)slots[bag[j]] : 0xffffffffu;
    }
#pragma unroll
    for (int j = 0; j < U; ++j)
        raw[j] = s[j] < (uint64_t)C ? cache_w[(int64_t)s[j] * wst + c[j]] : P::none();
#pragma unroll
    for (int j = 0; j < U; ++j) {
        if (bag[j] >= bags) continue;
        P p;
        p.decode(raw[j]);
        p.store_f32_stream(out + bag[j] * dim, (int)c[j]);
    }
}

// One lookup per bag, from the plan's grouping: the bag of the grouped lookup at position p is grouped[p].  The output
// rows are written one here, one there, and a 128-byte line is often shared by two of them: plain stores, which meet
// in L2, are quicker here than non-temporal ones (27 against 30 us on a Criteo-shaped batch of 192-byte rows; 183
// against 253 us on 1.3 M rows of 512 bytes, whole lines).  Workgroups
// [0, piece_blocks) take the pieces of long rows (every lane group fetches the row and writes it to its share of the
// piece's bags), the others take one row of up to kRowMax lookups per lane group.
constexpr int kFwdRows = 2;
template <int GW, typename P>
__global__ __launch_bounds__(kRowBlock) void embbag_fwd_rows_kernel(const uint4* __restrict__ row_recs,
                                                                    const uint4* __restrict__ piece_recs, uint32_t n_rows,
                                                                    uint32_t n_pieces, uint32_t piece_blocks,
                                                                    const uint32_t* __restrict__ grouped, uint32_t n,
                                                                    int64_t C, const typename P::Raw* __restrict__ cache_w, int lpr,
                                                                    int64_t wst, int dim, float* __restrict__ out) {
    constexpr int G = kRowBlock / GW;
    static_assert(kPiece <= (uint32_t)kRowBlock, "a lane group's share of a piece is at most one lookup per lane");
    const int c = threadIdx.x % GW, j = threadIdx.x / GW;
    const bool active = c < lpr;
    if (blockIdx.x >= piece_blocks) {
        if (!active) return;
        // kFwdRows consecutive rows per lane group and round: their records first, then their rows and the bags of
        // their first lookups, all in flight together, then the stores
        const uint32_t groups = (gridDim.x - piece_blocks) * G;
        for (uint32_t w0 = ((blockIdx.x - piece_blocks) * G + j) * kFwdRows; w0 < n_rows; w0 += groups * kFwdRows) {
            uint4 rec[kFwdRows];
            typename P::Raw raw[kFwdRows];
            uint32_t start[kFwdRows], count[kFwdRows], bag[kFwdRows][4];
#pragma unroll
            for (int r = 0; r < kFwdRows; ++r) rec[r] = w0 + r < n_rows ? row_recs[w0 + r] : make_uint4(0, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < kFwdRows; ++r) {
                start[r] = rec[r].x & kPosMask;
                count[r] = rec[r].y;
                const uint32_t slot = rec[r].z;
                if ((rec[r].x & kLongRow) || (int64_t)slot >= C || start[r] >= n || count[r] > n - start[r]) count[r] = 0;
                raw[r] = count[r] ? cache_w[(int64_t)slot * wst + c] : P::none();
                bag[r][0] = rec[r].w;                     // the row's first lookup: its position is its bag
#pragma unroll
                for (int k = 1; k < 4; ++k) bag[r][k] = (uint32_t)k < count[r] ? grouped[start[r] + k] : n;
            }
#pragma unroll
            for (int r = 0; r < kFwdRows; ++r) {
                if (count[r] == 0) continue;
                P p;
                p.decode(raw[r]);
#pragma unroll
                for (int k = 0; k < 4; ++k)
                    if ((uint32_t)k < count[r] && bag[r][k] < n) p.store_f32(out + (size_t)bag[r][k] * dim, c, lpr);
                for (uint32_t k = 4; k < count[r]; k += 4) {      // the few rows of 5 .. kRowMax lookups
                    uint32_t more[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) more[q] = k + q < count[r] ? grouped[start[r] + k + q] : n;
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (more[q] < n) p.store_f32(out + (size_t)more[q] * dim, c, lpr);
                }
            }
        }
        return;
    }
    // a piece: lane group j writes the row to the j-th stretch of the piece's bags.  A stretch has at most GW lookups
    // (kPiece <= G * GW), so every lane of the group, idle ones included, fetches one bag number and the group hands
    // them round by lane shuffle: one coalesced load instead of a round trip per bag.
    for (uint32_t pi = blockIdx.x; pi < n_pieces; pi += piece_blocks) {
        const uint4 r0 = piece_recs[2 * (size_t)pi];
        const uint32_t start = r0.x, count = r0.y, slot = r0.z;
        if ((int64_t)slot >= C || count == 0 || count > kPiece || start >= n || count > n - start) continue;
        const uint32_t per = (count + G - 1) / G;
        const uint32_t p0 = min((uint32_t)j * per, count), share = min(per, count - p0);
        const uint32_t mine = (uint32_t)c < share ? grouped[start + p0 + c] : n;
        P p;
        if (active) p.decode(cache_w[(int64_t)slot * wst + c]);
        constexpr int STEP = GW < 16 ? GW : 16;
#pragma unroll
        for (int t0 = 0; t0 < GW; t0 += STEP) {
            if ((uint32_t)t0 >= per) break;              // per <= GW, and the same in the whole workgroup
#pragma unroll
            for (int t = t0; t < t0 + STEP; ++t) {
                const uint32_t bag = __shfl(mine, t, GW);
                if (active && bag < n) p.store_f32(out + (size_t)bag * dim, c, lpr);
            }
        }
    }
}

struct FwdRowsLaunch {
    const bp_config* cfg;
    const void* cache_w;
    const uint32_t* grouped;
    const uint4* row_recs;
    const uint4* piece_recs;
    int64_t n_rows, n_pieces, bags;
    float* out;
    hipStream_t stream;
    template <int GW, typename P>
    int run(int lpr) {
        int64_t piece_blocks = n_pieces, row_blocks = ceil_div(n_rows, (int64_t)(kRowBlock / GW) * kFwdRows);
        if (piece_blocks > kMaxGridBlocks / 4) piece_blocks = kMaxGridBlocks / 4;
        if (row_blocks > kMaxGridBlocks) row_blocks = kMaxGridBlocks;
        if (row_blocks < 1) row_blocks = 1;
        BP_LAUNCH(K_FWD, (embbag_fwd_rows_kernel<GW, P>), dim3((unsigned)(piece_blocks + row_blocks)), dim3(kRowBlock), 0,
                  stream, row_recs, piece_recs, (uint32_t)n_rows, (uint32_t)n_pieces, (uint32_t)piece_blocks, grouped,
                  (uint32_t)bags, cfg->capacity, (const typename P::Raw*)cache_w, lpr, cache_w_stride16(cfg) * P::kPerVec,
                  cfg->dim, out);
        return BP_OK;
    }
};

// How many rows of a bag to have in flight (us in bursts of four / of eight; tables of 2 GB, Zipf rows, bags of 0 to twice
// the mean, unless stated):
//   long bags take eight.  Nothing else hides the rows' latency in small launches (f32 dim 64, 4,096 bags of 25, table in
//     the caches: 6.0 / 5.2), and large ones gain a little (a training pass over six batches of 163,840 bags of 1 to 50:
//     2,688 / 2,673).
//   short bags take four: at a mean of 6.5 the two are about even, and below it the guards of rows that are not there are
//     the cost (f32, 32,768 bags of mean 1: dim 64 3.7 / 4.3, dim 256 8.3 / 9.1).
//   but the shortest bags (a mean of less than 1.75) of bf16 rows by eights that fill a group of 8 lanes or more take eight from
//     2^20 lanes on: such launches are nearly all pooled stores, and the deeper form holds fewer wavefronts on a CU (dim 64,
//     262,144 bags of mean 1: 22.5 / 14.7; dim 512, 131,072 of mean 1.5: 76.2 / 50.8, of mean 2: 51.5 / 52.5).  Rows that leave
//     lanes idle do not gain (dim 96, 262,144 of mean 1: 21.9 / 24.8).
constexpr int64_t kManyLanes = int64_t(1) << 20;            // twice what the chip holds
struct FwdLaunch {
    const bp_config* cfg;
    const void* cache_w;
    const int32_t* slots;
    const int64_t* bag_off;
    int64_t bags, n_lookups;
    float* out;
    hipStream_t stream;
    // HIP takes fewer than 2^32 threads a launch, which 67 M bags of 64 lanes reach: more go in several launches.
    template <int GW, typename P>
    int run(int lpr) {
        const int64_t most = (int64_t(1) << 31) / GW;
        for (int64_t b0 = 0; b0 < bags; b0 += most) BP_TRY((run_bags<GW, P>(lpr, b0, std::min(most, bags - b0))));
        return BP_OK;
    }
    template <int GW, typename P>
    int run_bags(int lpr, int64_t b0, int64_t count) {
        const auto* w = (const typename P::Raw*)cache_w;
        const int64_t wst = cache_w_stride16(cfg) * P::kPerVec;
        float* const to = out + b0 * cfg->dim;
        if (bag_off == nullptr) {
            const uint32_t inv = lpr == 1 ? 0u : (uint32_t)((uint64_t(1) << 32) / (uint32_t)lpr + 1);
            const dim3 flat((unsigned)ceil_div(count * lpr, (int64_t)kRowBlock * kFlatPieces));
            BP_LAUNCH(K_FWD, (embbag_fwd_onehot_kernel<P, kFlatPieces>), flat, dim3(kRowBlock), 0, stream, w, slots + b0, count,
                      cfg->capacity, (uint32_t)lpr, inv, wst, cfg->dim, to);
            return BP_OK;
        }
        const dim3 grid((unsigned)ceil_div(count * GW, kRowBlock));
        const bool long_bags = 2 * n_lookups >= 13 * bags, shortest = 4 * n_lookups < 7 * bags;
        if (long_bags || (P::BF16 && P::N == 8 && GW >= 8 && lpr == GW && shortest && bags * GW >= kManyLanes))
            BP_LAUNCH(K_FWD, (embbag_fwd_kernel<GW, P, 8>), grid, dim3(kRowBlock), 0, stream, w, slots, bag_off + b0, count, n_lookups,
                      cfg->capacity, lpr, wst, cfg->dim, to);
        else
            BP_LAUNCH(K_FWD, (embbag_fwd_kernel<GW, P, 4>), grid, dim3(kRowBlock), 0, stream, w, slots, bag_off + b0, count, n_lookups,
                      cfg->capacity, lpr, wst, cfg->dim, to);
        return BP_OK;
    }
};

// bf16 rows of bags of several lookups: by fours a lane or by eights (row_access.h)?  By fours while the launch is no more than
// the chip holds at once, where latency rules and half the registers and whole lines of pooled rows help.  Larger launches read
// rows at the rate of their requests, which by fours are twice as many, the more the longer the bags and the more lanes idle:
// they stay by fours only where nearly all they do is write pooled rows, up to a limit on lanes * mean^2 that grows with the
// rows that fill their group.  us by eights (in the depth they take) / by fours, bags of a Poisson length, three outputs in turn:
//   dim 64: 32,768 bags of mean 1 4.3 / 3.9, 262,144 14.7 / 14.7; 524,288 of mean 2 30.0 / 39.1
//   dim 128: 65,536 of mean 1 9.1 / 7.5; 131,072 of mean 2 15.7 / 18.5, 524,288 52.5 / 66.9     dim 256: 32,768 of mean 1 9.0 / 7.1
//   dim 24: 1,048,576 of mean 1 25.1 / 33.7     dim 96: 16,384 of mean 1 3.9 / 3.7, 262,144 21.9 / 29.7
bool pooled_by_eights(int dim, int64_t n, int64_t bags) {
    constexpr double kChipLanes = 1 << 19;
    const int lanes = dim / 4, group = group_width(lanes);
    const double all = (double)group * (double)bags;
    if (2 * n >= 5 * bags) return true;
    if (lanes <= 2 || all <= kChipLanes) return false;
    const bool full = lanes == group;
    const double mean = std::max((double)n / (double)bags, full ? 0.0 : 0.7);
    return all * mean * mean > (full && lanes >= 32 ? 8 << 20 : full && lanes >= 16 ? 4 << 20 : 1 << 20);
}

}  // namespace
}  // namespace bp

using namespace bp;

BP_EXPORT int bp_embbag_fwd(const bp_config* cfg, const void* cache_w, const int32_t* lookup_slots,
                             const int64_t* bag_offsets, int64_t n_lookups, int64_t bags, float* out, void* stream) {
    BP_TRY(check_config(cfg));
    if (bags < 0 || n_lookups < 0) return fail(BP_ERR_INVALID_ARG, "negative size");
    if (bags >= (int64_t(1) << 31) || n_lookups >= (int64_t(1) << 31)) return fail(BP_ERR_UNSUPPORTED, "size >= 2^31");
    if (bags == 0) return BP_OK;
    if (!bag_offsets && n_lookups != bags)
        return fail(BP_ERR_INVALID_ARG, "bag_offsets is NULL but n_lookups %lld != bags %lld", (long long)n_lookups, (long long)bags);
    if (!cache_w || !out || (n_lookups && !lookup_slots)) return fail(BP_ERR_INVALID_ARG, "NULL pointer");
    if (((uintptr_t)cache_w | (uintptr_t)out) & 15) return fail(BP_ERR_INVALID_ARG, "cache_w and out must be 16-byte aligned");
    FwdLaunch l{cfg, cache_w, lookup_slots, bag_offsets, bags, n_lookups, out, (hipStream_t)stream};
    return dispatch_values<false>(cfg, bag_offsets && pooled_by_eights(cfg->dim, n_lookups, bags), l);
}

BP_EXPORT int bp_embbag_fwd_grouped(const bp_config* cfg, const void* cache_w, const int32_t* grouped_lookups,
                                     const bp_row_rec* row_recs, int64_t n_rows, const bp_piece_rec* piece_recs,
                                     int64_t n_pieces, int64_t bags, float* out, void* stream) {
    BP_TRY(check_config(cfg));
    if (bags < 0 || n_rows < 0 || n_pieces < 0) return fail(BP_ERR_INVALID_ARG, "negative size");
    if (bags >= (int64_t(1) << 31)) return fail(BP_ERR_UNSUPPORTED, "size >= 2^31");
    if (n_rows > bags || n_pieces > bags) return fail(BP_ERR_INVALID_ARG, "more rows or pieces than lookups");
    if (bags == 0 || n_rows == 0) return BP_OK;
    if (!cache_w || !out || !grouped_lookups || !row_recs || (n_pieces && !piece_recs))
        return fail(BP_ERR_INVALID_ARG, "NULL pointer");
    if (((uintptr_t)cache_w | (uintptr_t)out | (uintptr_t)row_recs | (uintptr_t)piece_recs) & 15)
        return fail(BP_ERR_INVALID_ARG, "cache_w, out, row_recs and piece_recs must be 16-byte aligned");
    FwdRowsLaunch l{cfg, cache_w, reinterpret_cast<const uint32_t*>(grouped_lookups), reinterpret_cast<const uint4*>(row_recs),
                    reinterpret_cast<const uint4*>(piece_recs), n_rows, n_pieces, bags, out, (hipStream_t)stream};
    // bf16 rows of 33 to 64 lanes by fours leave a workgroup four lane groups, which write a piece's bags 64 one behind the other:
    // small launches with pieces wait for that, where eight groups by eights write 32 (dim 160, 4,000 lookups, 19 pieces 6.2 us by
    // fours, 4.5 by eights, 16,000 7.5 / 6.9, 30,000 8.3 / 9.3; dim 256 4,000 6.4 / 6.2, 8,000 7.3 / 7.5; without pieces 3.0 / 3.1).
    const int lanes = cfg->dim / 4;
    return dispatch_values<false>(cfg, lanes > 32 && n_pieces > 0 && bags * lanes <= 700'000, l);
}
