// Stage 1 of the ODB window pipeline: length-aware grouping (Sec. 2.2, Eq. 1).
//
//   rank_form_kernel      ranks of at most 16,384 samples: everything below in one block per
//                         rank and one launch
//   lengths_kernel        l_i = off[i+1] - off[i], validity, window min / max length
//   radix_hist, rank_scan, radix_scatter
//                         segmented stable LSD radix sort of every rank's samples by
//                         (length descending, id ascending): keys are max_l - l, the
//                         segments are the ranks, and stability over the id-ordered input
//                         gives the id tie-break
//   chain_kernel          runs of equal step of every rank and the chain of group starts
//                         through them, G_r
//   chain_index_kernel    formation group index of every position from its run
//   links_kernel, jump_kernel, gidx / groups
//                         where the runs do not fit the table: next-group-start links,
//                         pointer-jumping list ranking that marks every group start
//
// Grouping, restated: visiting a rank's samples longest first with threshold t (1 at
// the start), a group closes once it holds t samples and t becomes B(l) of its last
// (shortest) sample.  So group 0 is position 0 alone and a group starting at position
// p > 0 has B(l[p-1]) members (clipped by the end of the rank): next(0) = 1 and
// next(p) = p + B(l[p-1]).  The group starts are exactly the positions reachable from 0
// along next().
//
// Two equivalent ways to find them.  Lengths are sorted, so the step b(p) = B(l[p-1]) is
// constant on runs of positions, and there are at most ~2 sqrt(budget) distinct values
// of floor(budget / l): inside a run of step b the chain advances by exactly b, so one
// thread per rank can go from run to run (in LDS) with one remainder each, and every
// position's group index follows from its run's first chain position, its step and the group
// starts before the run.  The runs come from the budget alone: the positions where the
// step changes are searched in the sorted lengths, so nobody reads them all.  When the
// number of runs may exceed the LDS table, pointer jumping over the next() links marks
// the chain in O(log G) doubling rounds instead.
#include <climits>
#include <cmath>
#include <vector>

#include "odb_internal.h"
#include "odb_search.h"

namespace odb {

namespace {

// Lanes of this wave whose `valid` digit equals this lane's (ballot per digit bit).
__device__ __forceinline__ uint64_t match_digit(uint32_t d, bool valid, int dbits) {
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < dbits; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t m = __ballot(bit);
        peers &= bit ? m : ~m;
    }
    return peers;
}

// Lengths, their validity and the window's shortest and longest.  Every block ends with two
// atomics on the same two words, ~10 ns each one after the other: 2,048 blocks spent 50 us on
// them whatever the window's size (16 x 65,536 samples: 51 us, now 17; 64 x 262,144: 67, now 43).
constexpr int kLengthsDeep = 8;
constexpr int kLengthsBlocksPerCU = 2;

__global__ void __launch_bounds__(kBlock) lengths_kernel(const int64_t* __restrict__ tok_off, int64_t n,
                                                         int32_t* __restrict__ len, DevStatus* st) {
    uint32_t lmin = 0xFFFFFFFFu, lmax = 0;
    int64_t bad = LLONG_MAX;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    auto one = [&](int64_t p, int64_t a, int64_t b) {
        int64_t l = b - a;
        if (l < 1 || l > INT_MAX || a < 0) {
            bad = bad < p ? bad : p;
            l = 1;
        }
        len[p] = (int32_t)l;
        lmin = (uint32_t)l < lmin ? (uint32_t)l : lmin;
        lmax = (uint32_t)l > lmax ? (uint32_t)l : lmax;
    };
    // kLengthsDeep grid-stride iterations at a time, their loads issued together: the grid is
    // two blocks per compute unit, so the loads in flight come from depth
    int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (; p + (kLengthsDeep - 1) * stride < n; p += kLengthsDeep * stride) {
        int64_t a[kLengthsDeep], b[kLengthsDeep];
#pragma unroll
        for (int k = 0; k < kLengthsDeep; ++k) {
            a[k] = tok_off[p + k * stride];
            b[k] = tok_off[p + k * stride + 1];
        }
#pragma unroll
        for (int k = 0; k < kLengthsDeep; ++k) one(p + k * stride, a[k], b[k]);
    }
    for (; p < n; p += stride) one(p, tok_off[p], tok_off[p + 1]);
    // one pair of atomics per block: lanes -> waves (shuffles) -> block (LDS)
    __shared__ uint32_t s_min[kBlock / kWave], s_max[kBlock / kWave];
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) {
        uint32_t a = __shfl_xor(lmin, d, kWave), b = __shfl_xor(lmax, d, kWave);
        lmin = a < lmin ? a : lmin;
        lmax = b > lmax ? b : lmax;
    }
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_min[threadIdx.x / kWave] = lmin;
        s_max[threadIdx.x / kWave] = lmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int i = 1; i < kBlock / kWave; ++i) {
            lmin = s_min[i] < lmin ? s_min[i] : lmin;
            lmax = s_max[i] > lmax ? s_max[i] : lmax;
        }
        if (lmax > 0) {
            atomicMin(&st->min_len, lmin);
            atomicMax(&st->max_len, lmax);
        }
    }
    if (bad != LLONG_MAX) {
        atomicOr(&st->err, kErrLength);
        atomicMin((unsigned long long*)&st->first_bad, (unsigned long long)bad);
    }
}

__global__ void rank_counts_kernel(const int64_t* __restrict__ off, int W, RankState* ranks) {
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < W; r += gridDim.x * blockDim.x) {
        RankState z = {};
        z.cnt = off[r + 1] - off[r];
        ranks[r] = z;
    }
}

// First radix tile of every rank: tile_first[r] = sum_{r' < r} ceil(n_r' / tile).
// Tiles never straddle ranks.  One block.
__global__ void __launch_bounds__(kBlock) sort_tiles_kernel(const int64_t* __restrict__ off, int W, int tile,
                                                            int64_t* __restrict__ tile_first) {
    __shared__ int64_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int b = 0; b < W; b += kBlock) {
        const int r = b + threadIdx.x;
        const int64_t v = r < W ? (off[r + 1] - off[r] + tile - 1) / tile : 0;
        int64_t tot;
        const int64_t ex = block_excl_sum(v, &tot);
        const int64_t c = carry;
        if (r < W) tile_first[r] = c + ex;
        __syncthreads();
        if (threadIdx.x == 0) carry = c + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) tile_first[W] = carry;
}

struct SortTile {
    int64_t start;       // first position
    int32_t count;       // keys in this tile
    int32_t seg_tiles;   // tiles of this tile's rank
    int64_t first;       // global index of the rank's first tile
    int32_t j;           // index of this tile within its rank
};

template <int kTile>
__device__ __forceinline__ SortTile sort_tile(const int64_t* __restrict__ off,
                                              const int64_t* __restrict__ tile_first, int W, int64_t b) {
    const int r = rank_of(tile_first, W, b);
    SortTile t;
    t.first = tile_first[r];
    t.j = (int32_t)(b - t.first);
    t.seg_tiles = (int32_t)(tile_first[r + 1] - t.first);
    t.start = off[r] + (int64_t)t.j * kTile;
    const int64_t left = off[r + 1] - t.start;
    t.count = (int32_t)(left < kTile ? left : kTile);
    return t;
}

// Keys per thread of a tile: 16 where that still leaves every compute unit four tiles and more,
// else 8.  Longer tiles write longer runs per digit (64 x 262,144 samples: the plan 566 -> 543 us
// with a key and a position per item, 497 -> 491 with both in a word), shorter ones spread a
// smaller window further (16 x 65,536: 204 us against 199).
inline int sort_items(int64_t n) { return n >= (int64_t)4 << 20 ? 2 * kSortItems : kSortItems; }

// How a window's range of lengths is sorted: passes of dbits bits (at least 2, so that a rank's
// counts come in whole vectors of 4) over keys max - length, and whether a key fits one word
// with a position of ibits bits.
struct SortPlan {
    int passes, dbits;
    bool packed;
};

__host__ __device__ inline SortPlan sort_plan(uint32_t min_len, uint32_t max_len, int ibits) {
    int bits = 0;
    while (bits < 32 && ((max_len - min_len) >> bits) != 0) ++bits;
    SortPlan p;
    p.passes = (bits + 7) / 8;
    const int d = p.passes > 0 ? (bits + p.passes - 1) / p.passes : 0;
    p.dbits = d < 2 ? 2 : d;
    p.packed = bits + ibits <= 32;
    return p;
}

// The first pass is launched before the host knows the lengths' range: its kernels then read the
// range on the device (`range`) and leave what they are not made for (equal lengths; a scatter
// that is the only pass, or does not fit one word) to the host.

// Digit counts of every tile.  kHistCopies copies of the table, lane l counting in copy
// l mod kHistCopies with a plain LDS add: equal digits of a wave (the high digit of
// skewed lengths) then meet in groups of at most 8 lanes.  Finding the lanes of equal digit
// first (a ballot per digit bit) for one add per distinct digit took 38 instead of 20 us on
// 16.7 M samples.
constexpr int kHistCopies = 8;

template <int kItems, bool kFirst>
__global__ void __launch_bounds__(kBlock) radix_hist_kernel(const int64_t* __restrict__ off,
                                                            const int64_t* __restrict__ tile_first, int W,
                                                            const uint32_t* __restrict__ keys_in,
                                                            const int32_t* __restrict__ len_in, uint32_t maxl,
                                                            int shift, int dbits, const DevStatus* __restrict__ range,
                                                            uint32_t* __restrict__ counts) {
    if (kFirst && range) {
        maxl = range->max_len;
        const SortPlan p = sort_plan(range->min_len, maxl, 0);
        if (p.passes == 0) return;
        dbits = p.dbits;
    }
    const SortTile b = sort_tile<kBlock * kItems>(off, tile_first, W, blockIdx.x);
    const int radix = 1 << dbits;
    const uint32_t mask = (uint32_t)radix - 1;
    __shared__ uint32_t h[256 * kHistCopies];
    uint32_t key[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int li = it * kBlock + threadIdx.x;
        const int64_t p = b.start + (li < b.count ? li : 0);
        key[it] = kFirst ? maxl - (uint32_t)len_in[p] : keys_in[p];
    }
    for (int i = threadIdx.x; i < radix * kHistCopies; i += kBlock) h[i] = 0;
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kItems; ++it)
        if (it * kBlock + (int)threadIdx.x < b.count)
            atomicAdd(&h[((key[it] >> shift) & mask) * kHistCopies + (threadIdx.x & (kHistCopies - 1))], 1u);
    __syncthreads();
    const int64_t col = (int64_t)b.first << dbits;
    for (int d = threadIdx.x; d < radix; d += kBlock) {
        uint32_t sum = 0;
#pragma unroll
        for (int k = 0; k < kHistCopies; ++k) sum += h[d * kHistCopies + k];
        counts[col + (int64_t)d * b.seg_tiles + b.j] = sum;
    }
}

// Exclusive scan of one rank's digit counts (digit-major, its tiles in order) from the rank's
// first position on: one block per rank, 16 consecutive counts a thread.  The ranks' scans are
// independent because a rank's counts add up to its samples; ranks of many tiles take the
// general scan (three launches, ~20 us) instead.
// 512 threads, not 1,024, so that a block starts beside the collate of the step before (kChainBlock).
constexpr int kRankScanThreads = 512;
constexpr int kRankScanItems = 16;
constexpr int64_t kRankScanMax = 8ll * kRankScanThreads * kRankScanItems;   // about 2 us per 8,192 counts

__global__ void __launch_bounds__(kRankScanThreads) rank_scan_kernel(const int64_t* __restrict__ off,
                                                                     const int64_t* __restrict__ tile_first, int dbits,
                                                                     const DevStatus* __restrict__ range,
                                                                     uint32_t* __restrict__ counts) {
    if (range) {
        const SortPlan p = sort_plan(range->min_len, range->max_len, 0);
        if (p.passes == 0) return;
        dbits = p.dbits;
    }
    const int r = blockIdx.x, t = threadIdx.x;
    const int64_t first = tile_first[r] << dbits, m = (tile_first[r + 1] << dbits) - first;
    __shared__ uint32_t s_w[kRankScanThreads / kWave];
    uint32_t carry = (uint32_t)off[r];
    for (int64_t i0 = 0; i0 < m; i0 += (int64_t)kRankScanThreads * kRankScanItems) {
        // vectors of 4: every rank's counts start at, and number, a multiple of 2^dbits >= 4
        uint4 v[kRankScanItems / 4];
        uint32_t sum = 0;
        uint32_t* c = counts + first + i0 + (int64_t)t * kRankScanItems;
#pragma unroll
        for (int k = 0; k < kRankScanItems / 4; ++k) {
            const bool on = i0 + (int64_t)t * kRankScanItems + 4 * k < m;
            v[k] = on ? reinterpret_cast<const uint4*>(c)[k] : make_uint4(0, 0, 0, 0);
            sum += v[k].x + v[k].y + v[k].z + v[k].w;
        }
        const uint32_t inc = wave_scan_dpp<OpAdd>(sum);
        if ((t & (kWave - 1)) == kWave - 1) s_w[t / kWave] = inc;
        __syncthreads();
        uint32_t at = carry + inc - sum;
#pragma unroll
        for (int k = 0; k < kRankScanThreads / kWave; ++k) {
            at += k < t / kWave ? s_w[k] : 0u;
            carry += s_w[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < kRankScanItems / 4; ++k) {
            const uint4 x = v[k];
            uint4 o;
            o.x = at;
            o.y = o.x + x.x;
            o.z = o.y + x.y;
            o.w = o.z + x.z;
            at = o.w + x.w;
            if (i0 + (int64_t)t * kRankScanItems + 4 * k < m) reinterpret_cast<uint4*>(c)[k] = o;
        }
    }
}

// Scatter one tile, stably.  A wave takes a quarter of the tile, its items in position order,
// and keeps its running count of each digit in LDS: an item's rank among the wave's equal
// digits is that count plus the lower lanes holding the digit (ballot match).  One scan
// over digits and waves then gives every wave's first slot for every digit; the items are placed
// in LDS in that order and written out from it, so each digit's run of the tile goes to
// consecutive addresses (written straight from registers, about two items per digit and
// round, they cost 4.6 B of HBM writes per byte).  The count, slot table and placement done round
// by round, two block barriers each, took 90 and 82 instead of 78 and 59 us for the two passes over
// 16.7 M samples, a key and a position each in tiles of 2,048 (the low digit spreads a tile over
// twice the runs).
//
// Where a key and a position within its rank fit one 32-bit word (kPacked: the position in the
// low `ibits` bits, and `shift` counts from the word's), the passes move that word instead of a
// key and a position: half the bytes between two passes and half the LDS (64 x 262,144 samples:
// the two passes 62 and 62 -> 46 and 48 us).
template <int kItems, bool kPacked, bool kFirst, bool kLast>
__global__ void __launch_bounds__(kBlock) radix_scatter_kernel(
    const int64_t* __restrict__ off, const int64_t* __restrict__ tile_first, int W,
    const uint32_t* __restrict__ keys_in,
    const int32_t* __restrict__ len_in, const int32_t* __restrict__ vals_in, uint32_t maxl, int ibits, int shift,
    int dbits, const DevStatus* __restrict__ range, const uint32_t* __restrict__ offs, uint32_t* __restrict__ keys_out,
    int32_t* __restrict__ vals_out, int32_t* __restrict__ slen_out) {
    if (kPacked && kFirst && !kLast && range) {
        maxl = range->max_len;
        const SortPlan p = sort_plan(range->min_len, maxl, ibits);
        if (p.passes < 2 || !p.packed) return;
        dbits = p.dbits;
    }
    const SortTile b = sort_tile<kBlock * kItems>(off, tile_first, W, blockIdx.x);
    const int radix = 1 << dbits;
    const uint32_t mask = (uint32_t)radix - 1;
    constexpr int kWaves = kBlock / kWave, kTile = kBlock * kItems;
    __shared__ uint32_t s_shift[256];         // global position of the digit's first item less its local one
    __shared__ uint32_t s_cnt[kWaves][256];   // items of a digit in a wave, then the wave's first local slot
    __shared__ uint32_t s_key[kTile];
    __shared__ int32_t s_val[kPacked ? 1 : kTile];
    const int64_t rank0 = b.start - (int64_t)b.j * kTile;   // the rank's first position
    const int w = threadIdx.x / kWave;
    const int p0 = w * (kTile / kWaves) + (threadIdx.x & (kWave - 1));   // item it: p0 + it * 64
    uint32_t key[kItems];
    int32_t val[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int li = p0 + it * kWave;
        const int64_t p = b.start + (li < b.count ? li : 0);
        key[it] = kFirst ? maxl - (uint32_t)len_in[p] : keys_in[p];
        if (kPacked && kFirst) key[it] = key[it] << ibits | (uint32_t)(p - rank0);
        if (!kPacked) val[it] = kFirst ? (int32_t)p : vals_in[p];
    }
    const int64_t col = (int64_t)b.first << dbits;
    uint32_t base = 0;
    if ((int)threadIdx.x < radix) base = offs[col + (int64_t)threadIdx.x * b.seg_tiles + b.j];
#pragma unroll
    for (int k = 0; k < kWaves; ++k) s_cnt[k][threadIdx.x] = 0;
    __syncthreads();
    uint32_t at[kItems];
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const bool valid = p0 + it * kWave < b.count;
        const uint32_t d = (key[it] >> shift) & mask;
        const uint64_t peers = match_digit(d, valid, dbits);
        const uint32_t below = (uint32_t)lanes_below(peers);
        // every lane reads the count before the digit's first lane adds to it: LDS operations of
        // one wave complete in order (the fences keep the compiler to it)
        at[it] = s_cnt[w][d] + below;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (valid && below == 0) s_cnt[w][d] += (uint32_t)__popcll(peers);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    __syncthreads();
    {
        uint32_t c[kWaves], sum = 0, tot;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            c[k] = s_cnt[k][threadIdx.x];
            sum += c[k];
        }
        uint32_t ex = block_excl_sum(sum, &tot);
        s_shift[threadIdx.x] = base - ex;
#pragma unroll
        for (int k = 0; k < kWaves; ++k) {
            s_cnt[k][threadIdx.x] = ex;
            ex += c[k];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        if (p0 + it * kWave < b.count) {
            const uint32_t q = s_cnt[w][(key[it] >> shift) & mask] + at[it];
            s_key[q] = key[it];
            if (!kPacked) s_val[q] = val[it];
        }
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < kItems; ++it) {
        const int q = it * kBlock + threadIdx.x;
        if (q >= b.count) break;
        const uint32_t k = s_key[q];
        const uint32_t pos = s_shift[(k >> shift) & mask] + (uint32_t)q;
        if (!kPacked)
            vals_out[pos] = s_val[q];
        else if (kLast)
            vals_out[pos] = (int32_t)(rank0 + (k & ((1u << ibits) - 1)));
        if (kLast)
            slen_out[pos] = (int32_t)(maxl - (kPacked ? k >> ibits : k));
        else
            keys_out[pos] = k;
    }
}

__global__ void __launch_bounds__(kBlock) identity_order_kernel(int64_t n, const int32_t* __restrict__ len,
                                                                int32_t* __restrict__ order,
                                                                int32_t* __restrict__ slen) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        order[p] = (int32_t)p;
        slen[p] = len[p];
    }
}

// next-group-start links over the current sequences; positions outside every rank's
// live range [off[r], off[r] + cnt_r) and links leaving a rank point to the sentinel n.
__global__ void __launch_bounds__(kBlock) links_kernel(const int32_t* __restrict__ slen,
                                                       const int64_t* __restrict__ off,
                                                       const RankState* __restrict__ ranks, int W, int64_t n,
                                                       int64_t budget, int32_t* __restrict__ jmp,
                                                       uint8_t* __restrict__ marks) {
    __shared__ int64_t s_off[kLdsRanks + 1];
    off = stage_ranks(off, W, s_off);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p <= n; p += stride) {
        if (p == n) {
            jmp[n] = (int32_t)n;
            marks[n] = 0;
            continue;
        }
        const int r = rank_of(off, W, p);
        const int64_t base = off[r];
        const int64_t c = ranks[r].cnt;
        const int64_t q = p - base;
        if (q >= c) {
            jmp[p] = (int32_t)n;
            marks[p] = 0;
            continue;
        }
        const int64_t step = q == 0 ? 1 : batch_size(budget, slen[p - 1]);
        const int64_t t = p + step;
        jmp[p] = (int32_t)(t < base + c ? t : n);
        marks[p] = q == 0 ? 1 : 0;
    }
}

// One doubling round: m <- m U J(m), J <- J o J.  Marks are updated in place (a mark seen
// early only propagates sooner; every marked position is still a chain element), the
// jump table is double-buffered.  A round starts only if the previous one marked
// something new; otherwise the marks are already closed under J and it returns at once.
__global__ void __launch_bounds__(kBlock) jump_kernel(const int32_t* __restrict__ jin,
                                                      int32_t* __restrict__ jout, uint8_t* marks, int64_t n,
                                                      DevStatus* st, int round) {
    if (round > 0 && st->jump_changed[round - 1] == 0) return;
    bool changed = false;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p <= n; p += stride) {
        const int32_t j = jin[p];
        if (p < n && j < n && marks[p] && !marks[j]) {
            marks[j] = 1;
            changed = true;
        }
        jout[p] = j < n ? jin[j] : (int32_t)n;
    }
    if (__ballot(changed) && (threadIdx.x & (kWave - 1)) == 0) st->jump_changed[round] = 1;
}

// ---- chain walk over runs of equal step
// Positions q >= 1 of a rank (q < cnt_r) fall into runs of equal step b = B(l[q - 1]); the
// lengths are sorted, so the step never decreases along the rank.  The chain's group starts
// are q = 0 and, in run k, the positions c_k, c_k + b_k, ... of the run, where c_k is the
// chain's first position in it (none if the chain jumps over the run).  The group index of a
// position is the number of group starts at or before it, minus one: g_k group starts before
// run k (position 0 not counted), plus (q - c_k) / b_k + 1 once q >= c_k.
//
// One block per rank (of kChainThreads in rank_form_kernel, of kChainBlock in chain_kernel):
//   runs    the distinct steps are known without looking at the samples: the values
//           b = B(longest) .. sqrt(budget), and for each length l below budget / sqrt(budget)
//           the step budget / l, at most 2 sqrt(budget) + 2 or the length range; a run starts
//           at the first length at or below a threshold, found by one binary search per
//           candidate (a sample of 1,024 lengths in LDS, then the samples between two of them).
//           Where a rank has fewer samples than there may be steps, its samples are looked at
//           instead
//   chase   one thread follows the chain from run to run: the only serial part, a
//           multiplication by the step's reciprocal per run (computed by all threads before)
//   counts  group starts per run and their prefix, by all threads
// The group index of every position follows in closed form: in the same block for ranks of at
// most kRankBlockMax samples, else by chain_index_kernel over all tiles.
//
// Bound by the chase: ~25 ns per run.  64 ranks x 262,144 samples, ~700 runs per rank: the
// run table from a count, a scan and a write pass over all samples took 105 us and a chase that
// divides 83 us; 38 us here, and the group indices 28 instead of 71 us (nothing is read per
// sample any more).
constexpr int kChainThreads = 1024;
constexpr int kChainWaves = kChainThreads / kWave;
constexpr int kRunCap = 4096;   // runs per rank
// chain_kernel's threads.  A plan runs beside the previous step's collate, which keeps three waves
// of 84 vector registers (88 allocated) on every SIMD: two more waves of a block of 512 fit there, four of a block
// of 1,024 did not at 68, 50 or 48 registers a thread, and the plan waited until the
// collate ended (64 x 262,144: 16 ms a chain in the two-stream schedule).
constexpr int kChainBlock = 512;
constexpr int kChainSamples = 1024;   // lengths of a rank sampled for the search
constexpr int kChaseBatch = 8;        // runs the chase reads at once

// One block: every rank's first global group id (exclusive sum of G_r) and the total in
// gbase[W].
__global__ void __launch_bounds__(kBlock) rank_groups_kernel(RankState* ranks, int W, int64_t* __restrict__ gbase) {
    int64_t carry = 0;
    for (int b = 0; b < W; b += kBlock) {
        const int r = b + threadIdx.x;
        const int64_t G = r < W ? ranks[r].G : 0;
        int64_t tot;
        const int64_t ex = block_excl_sum(G, &tot);
        if (r < W) {
            ranks[r].gbase = carry + ex;
            gbase[r] = carry + ex;
        }
        carry += tot;
    }
    if (threadIdx.x == 0) gbase[W] = carry;
}

__global__ void init_jump_flags(DevStatus* st) {
    if (threadIdx.x < kMaxJumpRounds) st->jump_changed[threadIdx.x] = 0;
}

struct CountLoad {
    const uint32_t* c;
    int64_t n;
    __device__ uint32_t operator()(int64_t i) const { return i < n ? c[i] : 0u; }
};
struct CountStore {
    uint32_t* c;
    __device__ void operator()(int64_t i, uint32_t v) const { c[i] = v; }
};

struct MarkLoad {
    const uint8_t* m;
    __device__ uint32_t operator()(int64_t i) const { return m[i]; }
};
struct InclStore {
    const uint8_t* m;
    int32_t* out;
    __device__ void operator()(int64_t i, uint32_t ex) const { out[i] = (int32_t)(ex + m[i]); }
};

__global__ void __launch_bounds__(kBlock) gidx_kernel(const uint8_t* __restrict__ marks,
                                                      const int32_t* __restrict__ incl,
                                                      const int64_t* __restrict__ off,
                                                      const RankState* __restrict__ ranks, int W, int64_t n,
                                                      int32_t* __restrict__ gidx, int32_t* __restrict__ gstart) {
    __shared__ int64_t s_off[kLdsRanks + 1];
    off = stage_ranks(off, W, s_off);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        const int r = rank_of(off, W, p);
        const int64_t base = off[r];
        if (p - base >= ranks[r].cnt) continue;
        const int32_t before = base > 0 ? incl[base - 1] : 0;
        gidx[p] = incl[p] - before - 1;
        if (marks[p]) gstart[incl[p] - 1] = (int32_t)p;
    }
}

__global__ void groups_kernel(const int32_t* __restrict__ incl, const int64_t* __restrict__ off, int W,
                              RankState* ranks, int64_t* __restrict__ gbase, int32_t* __restrict__ groups_out) {
    for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < W; r += gridDim.x * blockDim.x) {
        const int64_t base = off[r];
        const int64_t c = ranks[r].cnt;
        const int32_t before = base > 0 ? incl[base - 1] : 0;
        const int64_t G = c > 0 ? incl[base + c - 1] - before : 0;
        ranks[r].G = G;
        ranks[r].gbase = before;
        gbase[r] = before;
        if (r == W - 1) gbase[W] = before + G;
        if (groups_out) groups_out[r] = (int32_t)G;
    }
}

// ---- the chain of one rank
// Batch size B(l) (Eq. 1), clipped to 2^31 - 1 (any larger step leaves the rank).
__device__ __forceinline__ uint32_t step_of(int32_t l, int64_t budget) {
    return (uint32_t)batch_size(budget, l);
}

// Calls f(q, step) for every run start q in [lo, hi) (1 <= lo < hi <= cnt), in order: q = 1,
// and every q whose step B(l[q-1]) differs from the previous position's B(l[q-2]).  Loads
// eight lengths at a time, at clamped positions, so the loads of a batch are in flight
// together; equal neighbouring lengths skip the divisions.
template <typename F>
__device__ __forceinline__ void chunk_run_starts(const int32_t* len, int lo, int hi, int64_t budget, F f) {
    int32_t lp = lo >= 2 ? len[lo - 2] : 0;
    uint32_t bp = lo >= 2 ? step_of(lp, budget) : 0u;
    for (int q0 = lo; q0 < hi; q0 += 8) {
        int32_t l8[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int qq = q0 + j < hi ? q0 + j : hi - 1;
            l8[j] = len[qq - 1];
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int q = q0 + j;
            if (q >= hi) break;
            const int32_t l = l8[j];
            if (q == 1) {
                bp = step_of(l, budget);
                f(q, bp);
            } else if (l != lp) {
                const uint32_t b = step_of(l, budget);
                if (b != bp) f(q, b);
                bp = b;
            }
            lp = l;
        }
    }
}

// Exclusive scan of v over the block of NT threads; *total receives the sum.
template <int NT>
__device__ __forceinline__ uint32_t chain_scan(uint32_t v, uint32_t* total) {
    __shared__ uint32_t s_w[NT / kWave];
    const int t = threadIdx.x;
    const uint32_t inc = wave_scan_dpp<OpAdd>(v);
    if ((t & (kWave - 1)) == kWave - 1) s_w[t / kWave] = inc;
    __syncthreads();
    uint32_t pre = 0, tot = 0;
#pragma unroll
    for (int i = 0; i < NT / kWave; ++i) {
        const uint32_t x = s_w[i];
        pre += i < t / kWave ? x : 0u;
        tot += x;
    }
    __syncthreads();
    *total = tot;
    return pre + inc - v;
}

// The run table of a rank longer than one block's share, for chain_index_kernel: rank r's run
// k at position off[r] + k of four position-indexed arrays, and the run that holds the first
// position of every sort tile.
struct RunTable {
    int32_t* start;
    int32_t* step;
    int32_t* first;    // c_k (INT32_MAX if the chain jumps over the run)
    int32_t* before;   // g_k
    uint32_t* tile;    // [sort tiles]
    uint32_t* runs;    // [W]
};

// LDS of chain_rank, in words: run starts, steps, first positions (and, before, candidates),
// reciprocals (later the prefix), and the sample of lengths.
constexpr int kChainStart = 0, kChainStep = kRunCap + 16, kChainFirst = kChainStep + kRunCap + kChaseBatch,
              kChainMore = kChainFirst + kRunCap + kChaseBatch, kChainSample = kChainMore + kRunCap + kChaseBatch,
              kChainWords = kChainSample + kChainSamples;

// The chain of rank r: cnt sorted lengths at `len`, its positions from `base` on.
// kIndex: write the group indices here (short ranks); otherwise leave the run table.
// sq = floor(sqrt(budget)); by_step: at most kRunCap - 2 steps are possible for this budget
// and length range (otherwise the rank holds at most kRunCap samples).
template <bool kIndex, int NT>
__device__ __forceinline__ void chain_rank(uint32_t* lds, const int32_t* len, int r, int64_t base, int cnt,
                                           RankState* ranks, int64_t budget, int64_t sq, int by_step,
                                           int32_t* __restrict__ gidx, int32_t* __restrict__ groups_out,
                                           const RunTable& tbl, const int64_t* __restrict__ tile_first, int tile,
                                           DevStatus* st) {
    uint32_t *s_start = lds + kChainStart, *s_b = lds + kChainStep, *s_c = lds + kChainFirst, *s_m = lds + kChainMore;
    int32_t* s_len = reinterpret_cast<int32_t*>(lds + kChainSample);
    const int t = threadIdx.x;
    if (cnt <= 1) {   // no position >= 1, no run: position 0 (if any) is the only group start
        if (t == 0) {
            if (kIndex && cnt == 1) gidx[base] = 0;
            if (ranks) ranks[r].G = cnt;
            if (groups_out) groups_out[r] = cnt;
        }
        return;
    }
    const int last = cnt - 1;   // lengths [0, last) are the steps of positions [1, cnt)
    int R = 0;
    if (by_step) {
        // the longest of every `stride` lengths
        const uint32_t stride = search_stride(last, kChainSamples);
        for (uint32_t i = t; i < (uint32_t)kChainSamples; i += NT)
            s_len[i] = i * stride < (uint32_t)last ? len[i * stride] : 0;
        __syncthreads();
        const int64_t lmax = len[0], lmin = len[last - 1];
        const int64_t blo = batch_size(budget, (int32_t)lmax), bhi = batch_size(budget, (int32_t)lmin);
        const int64_t na = blo <= sq ? (bhi < sq ? bhi : sq) - blo + 1 : 0;
        const int64_t lhi = lmax < budget / (sq + 1) ? lmax : budget / (sq + 1);
        const int64_t nb = lhi >= lmin ? lhi - lmin + 1 : 0;
        const int64_t nc = na + nb;
        if (nc > kRunCap) {   // cannot happen (the host's bound): report, and leave the rank without groups
            if (t == 0) {
                atomicOr(&st->err, kErrInternal);
                if (ranks) ranks[r].G = 0;
                if (groups_out) groups_out[r] = 0;
            }
            return;
        }
        // first position of every candidate step (s_c), then the runs that hold a position
        for (int i = t; i < (int)nc; i += NT) {
            const int64_t b = i < na ? blo + i : (int64_t)step_of((int32_t)(lhi - (i - na)), budget);
            const int64_t at = i < na ? budget / b : lhi - (i - na);   // step b: lengths at most `at`
            const uint32_t p = i > 0 ? first_at_most([&](uint32_t k) { return s_len[k]; },
                                                     [&](uint32_t k) { return len[k]; }, last, stride, kChainSamples, at)
                                     : 0u;
            s_c[i] = p;
            s_m[i] = (uint32_t)b;
        }
        __syncthreads();
        for (int i0 = 0; i0 < (int)nc; i0 += NT) {
            const int i = i0 + t;
            bool live = false;
            if (i < (int)nc) live = s_c[i] < (i + 1 < (int)nc ? s_c[i + 1] : (uint32_t)last);
            uint32_t tot;
            const uint32_t ex = chain_scan<NT>(live ? 1u : 0u, &tot);
            if (live) {
                s_start[R + ex] = s_c[i] + 1;
                s_b[R + ex] = s_m[i];
            }
            R += (int)tot;
        }
    } else {
        const int per = (last + NT - 1) / NT;
        const int lo = 1 + t * per;
        const int hi = lo + per < cnt ? lo + per : cnt;
        // the step never decreases, so a chunk whose first and last positions have the step of
        // the position before it holds no run start
        const bool busy = lo < hi && (lo == 1 || step_of(len[lo - 2], budget) != step_of(len[hi - 2], budget));
        uint32_t mine = 0, tot;
        if (busy) chunk_run_starts(len, lo, hi, budget, [&](int, uint32_t) { ++mine; });
        uint32_t at = chain_scan<NT>(mine, &tot);
        if (tot > (uint32_t)kRunCap) {   // cannot happen (at most kRunCap samples)
            if (t == 0) {
                atomicOr(&st->err, kErrInternal);
                if (ranks) ranks[r].G = 0;
                if (groups_out) groups_out[r] = 0;
            }
            return;
        }
        if (mine)
            chunk_run_starts(len, lo, hi, budget, [&](int q, uint32_t b) {
                s_start[at] = (uint32_t)q;
                s_b[at] = b;
                ++at;
            });
        R = (int)tot;
    }
    if (t == 0) s_start[R] = (uint32_t)cnt;
    __syncthreads();
    // The chase.  Let x = e + b - 1 - cur for the chain's position cur on entering a run that
    // ends at e.  If cur < e the run holds k = x / b chain positions and the next one is
    // e + b - 1 - x % b; if not, x < b, and the same expression gives cur again.  So the only
    // chain is x' = x % b + (e' - e) + (b' - b).  A step larger than the rank leaves it like one
    // of the rank's size.
    //
    // Ranks of up to 2^19 positions: x < 2^20 and the remainder runs in fp32, exact integers
    // throughout.  inv is 1 / b less 2^-21 of it, so the quotient is at most x / b and less than
    // one below it (b >= 2: x / b * 2^-20 < 1): the remainder comes out in [0, 2 b) and one
    // subtraction brings it below b, taken if it does not turn the sign (the larger unsigned
    // pattern).  Only the first run can have step 1, whose remainder is 0.
    const bool fp = cnt <= (1 << 19);
    for (int i = t; i < R; i += NT) {
        const uint32_t b = s_b[i] < (uint32_t)cnt ? s_b[i] : (uint32_t)cnt;
        const uint32_t bp = i > 0 ? (s_b[i - 1] < (uint32_t)cnt ? s_b[i - 1] : (uint32_t)cnt) : 0u;
        // into run i: x_0 itself (cur = next(0) = 1, the second group starts at position 1), else
        // what is added to the previous run's remainder
        const uint32_t d = i > 0 ? s_start[i + 1] - s_start[i] + b - bp : s_start[1] + b - 2;
        s_c[i] = fp ? __float_as_uint((float)d) : d;
        // ceil(2^32 / b): (x * m) >> 32 is x / b or one more for x < 2^32
        s_m[i] = fp ? __float_as_uint((1.0f / (float)b) * (1.0f - 0x1p-21f)) : 0xFFFFFFFFu / b + 1u;
    }
    __syncthreads();
    if (t == 0) {
        // s_c[i] becomes x of run i; runs come in batches read ahead of their use, so that the
        // chain carries arithmetic only (reads past R return what is never used)
        uint32_t d0[kChaseBatch], b0[kChaseBatch], m0[kChaseBatch], d1[kChaseBatch], b1[kChaseBatch], m1[kChaseBatch];
        auto load = [&](int i0, uint32_t (&d)[kChaseBatch], uint32_t (&b)[kChaseBatch], uint32_t (&m)[kChaseBatch]) {
#pragma unroll
            for (int j = 0; j < kChaseBatch; ++j) {
                d[j] = s_c[i0 + j];
                b[j] = s_b[i0 + j];
                m[j] = s_m[i0 + j];
            }
        };
        auto walk = [&](auto run) {
            load(0, d0, b0, m0);
            for (int i0 = 0; i0 < R; i0 += 2 * kChaseBatch) {
                if (i0 + kChaseBatch < R) load(i0 + kChaseBatch, d1, b1, m1);
                run(i0, d0, b0, m0);
                if (i0 + kChaseBatch >= R) break;
                if (i0 + 2 * kChaseBatch < R) load(i0 + 2 * kChaseBatch, d0, b0, m0);
                run(i0 + kChaseBatch, d1, b1, m1);
            }
        };
        const uint32_t most = (uint32_t)cnt;
        if (fp) {
            float rem = 0.0f;
            walk([&](int i0, const uint32_t (&d)[kChaseBatch], const uint32_t (&b)[kChaseBatch],
                     const uint32_t (&m)[kChaseBatch]) {
                float bf[kChaseBatch];
                uint32_t xs[kChaseBatch];
#pragma unroll
                for (int j = 0; j < kChaseBatch; ++j) bf[j] = (float)(b[j] < most ? b[j] : most);
#pragma unroll
                for (int j = 0; j < kChaseBatch; ++j) {
                    const float x = rem + __uint_as_float(d[j]);
                    xs[j] = (uint32_t)x;
                    const float q = __builtin_truncf(x * __uint_as_float(m[j]));
                    const float ra = __builtin_fmaf(-q, bf[j], x);
                    const uint32_t ua = __float_as_uint(ra), ub = __float_as_uint(ra - bf[j]);
                    rem = __uint_as_float(ua < ub ? ua : ub);
                    if (j == 0 && i0 == 0 && bf[0] == 1.0f) rem = 0.0f;
                }
#pragma unroll
                for (int j = 0; j < kChaseBatch; ++j) s_c[i0 + j] = xs[j];
            });
        } else {
            uint32_t rem = 0;
            walk([&](int i0, const uint32_t (&d)[kChaseBatch], const uint32_t (&b)[kChaseBatch],
                     const uint32_t (&m)[kChaseBatch]) {
                uint32_t xs[kChaseBatch];
#pragma unroll
                for (int j = 0; j < kChaseBatch; ++j) {
                    const uint32_t bj = b[j] < most ? b[j] : most;
                    const uint32_t x = rem + d[j];
                    xs[j] = x;
                    const uint32_t ra = x - __umulhi(x, m[j]) * bj;
                    rem = ra < ra + bj ? ra : ra + bj;   // wrapped below 0 if the quotient was one too many
                    if (j == 0 && i0 == 0 && bj == 1) rem = 0;
                }
#pragma unroll
                for (int j = 0; j < kChaseBatch; ++j) s_c[i0 + j] = xs[j];
            });
        }
    }
    __syncthreads();
    // the chain's first position in every run
    for (int i = t; i < R; i += NT) {
        const uint32_t b = s_b[i] < (uint32_t)cnt ? s_b[i] : (uint32_t)cnt;
        const uint32_t cur = s_start[i + 1] + b - 1 - s_c[i];
        s_c[i] = cur < s_start[i + 1] ? cur : 0x7FFFFFFFu;
    }
    __syncthreads();
    // group starts per run and their exclusive prefix (into s_m)
    uint32_t carry = 0;
    for (int i0 = 0; i0 < R; i0 += NT) {
        const int i = i0 + t;
        uint32_t ng = 0, tot;
        if (i < R) {
            const uint32_t c = s_c[i], e = s_start[i + 1], b = s_b[i];
            ng = c < e ? (e - c + b - 1) / b : 0u;
        }
        const uint32_t ex = chain_scan<NT>(ng, &tot);
        if (i < R) s_m[i] = carry + ex;
        carry += tot;
    }
    if (t == 0) {
        if (ranks) ranks[r].G = 1 + (int64_t)carry;
        if (groups_out) groups_out[r] = (int32_t)(1 + carry);
    }
    __syncthreads();
    auto run_of = [&](uint32_t q) {   // last run with start <= q
        int a = 0, z = R;
        while (z - a > 1) {
            const int m = (a + z) >> 1;
            if (s_start[m] <= q) a = m; else z = m;
        }
        return a;
    };
    if (kIndex) {
        for (int q = t; q < cnt; q += NT) {
            int32_t g = 0;
            if (q > 0) {
                const int a = run_of((uint32_t)q);
                const uint32_t c = s_c[a];
                g = (int32_t)(s_m[a] + ((uint32_t)q >= c ? ((uint32_t)q - c) / s_b[a] + 1u : 0u));
            }
            gidx[base + q] = g;
        }
    } else {
        for (int i = t; i < R; i += NT) {
            tbl.start[base + i] = (int32_t)s_start[i];
            tbl.step[base + i] = (int32_t)s_b[i];
            tbl.first[base + i] = (int32_t)s_c[i];
            tbl.before[base + i] = (int32_t)s_m[i];
        }
        const int64_t t0 = tile_first[r], t1 = tile_first[r + 1];
        for (int64_t j = t0 + t; j < t1; j += NT) {
            const int64_t q = (j - t0) * tile;
            if (q < cnt) tbl.tile[j] = (uint32_t)(q > 0 ? run_of((uint32_t)q) : 0);
        }
        if (t == 0) {
            tbl.start[base + R] = cnt;   // R < cnt: a rank has fewer runs than positions
            tbl.runs[r] = (uint32_t)R;
        }
    }
}

// ranks (or null: whole ranks): an alignment round's buffers; with kIndex the next round's,
// whose count becomes current here.
template <bool kIndex>
__global__ void __launch_bounds__(kChainBlock) chain_kernel(const int64_t* __restrict__ off, RankState* ranks,
                                                              const int32_t* __restrict__ slen, int64_t budget,
                                                              int64_t sq, int by_step, int32_t* __restrict__ gidx,
                                                              int32_t* __restrict__ groups_out, RunTable tbl,
                                                              const int64_t* __restrict__ tile_first, int tile,
                                                              DevStatus* st) {
    __shared__ uint32_t lds[kChainWords];
    const int r = blockIdx.x;
    const int64_t base = off[r];
    const int cnt = (int)(ranks ? (kIndex ? ranks[r].next_cnt : ranks[r].cnt) : off[r + 1] - base);
    if (kIndex && ranks && threadIdx.x == 0) ranks[r].cnt = cnt;
    chain_rank<kIndex, kChainBlock>(lds, slen + base, r, base, cnt, ranks, budget, sq, by_step, gidx, groups_out, tbl, tile_first,
                       tile, st);
}

// ---- one block per rank
// Ranks of at most kRankBlockMax samples are grouped by one block each, in one launch and with
// no host synchronisation: lengths (invalid ones as 1; odb_align_groups reports them), a
// stable LSD radix sort by length descending in LDS, the chain and the group indices.
//
// The sort is that of the streaming rounds: a wave takes KPT groups of 64 consecutive positions
// in order and keeps its running count of each digit (up to 8 bits) in LDS, so an item's rank
// among equal digits is that count plus the lower lanes holding the digit; one scan over
// (digit, wave) places every wave.  The chain then reads the lengths from LDS.  One round of
// 1,024 items at a time with two block barriers each, the ids and keys in global memory, and
// the chain in a second launch took 14 + 10 us on 2 x 2,048 samples and 21 + 13 on 8 x 4,096;
// 17.5 and 23.5 us here.
constexpr int kFormBins = 256;

// Where a digit's count of wave w lies: (digit, wave) order for the scan, a digit's waves rotated
// by a quarter of the digit, so that the digits a wave counts spread over all LDS banks instead of
// every 16th (8 x 1,021 samples: the form 14.9 -> 13.2 us; 8 x 4,096: 24.7 -> 23.5).
__device__ __forceinline__ uint32_t form_bin(uint32_t d, int w) {
    return d * kChainWaves + ((w + (d >> 2)) & (kChainWaves - 1));
}

template <int KPT>
constexpr size_t form_lds_bytes() {
    constexpr size_t P = (size_t)kChainThreads * KPT;
    constexpr size_t sort = 2 * P + 4 * kFormBins * kChainWaves, chain = 4 * kChainWords;
    return 4 * P + (sort > chain ? sort : chain);
}

// off: rank offsets in device memory, or null: in `vals`.
template <int KPT>
__global__ void __launch_bounds__(kChainThreads) rank_form_kernel(Values vals, const int64_t* __restrict__ off,
                                                                  const int64_t* __restrict__ tok_off, int64_t budget,
                                                                  int64_t sq, int by_step,
                                                                  int32_t* __restrict__ order,
                                                                  int32_t* __restrict__ slen,
                                                                  int32_t* __restrict__ gidx,
                                                                  int32_t* __restrict__ groups_out, DevStatus* st) {
    constexpr int P = kChainThreads * KPT;
    constexpr int kPer = kFormBins * kChainWaves / kChainThreads;
    extern __shared__ uint32_t dyn[];
    uint32_t* s_len = dyn;
    uint32_t* s_cnt = dyn + P;                                                       // [digit][wave]
    uint16_t* s_idx = reinterpret_cast<uint16_t*>(s_cnt + kFormBins * kChainWaves);   // [P]
    __shared__ uint32_t s_max;
    const int r = blockIdx.x, t = threadIdx.x, w = t / kWave;
    const int64_t base = off ? off[r] : vals.v[r];
    const int cnt = (int)((off ? off[r + 1] : vals.v[r + 1]) - base);
    if (t == 0) s_max = 0;
    __syncthreads();
    if (cnt > 0) {
        // positions of wave w: [w * KPT * 64, (w + 1) * KPT * 64), item c at + c * 64 + lane
        const int p0 = w * KPT * kWave + (t & (kWave - 1));
        uint32_t len[KPT], idx[KPT], mx = 0;
        int64_t t0[KPT], t1[KPT];
#pragma unroll
        for (int c = 0; c < KPT; ++c) {
            const int p = p0 + c * kWave;
            const int64_t s = base + (p < cnt ? p : cnt - 1);
            t0[c] = tok_off[s];
            t1[c] = tok_off[s + 1];
        }
#pragma unroll
        for (int c = 0; c < KPT; ++c) {
            const int64_t l = t1[c] - t0[c];
            len[c] = l < 1 || l > INT_MAX || t0[c] < 0 ? 1u : (uint32_t)l;
            idx[c] = (uint32_t)(p0 + c * kWave);
            if (p0 + c * kWave < cnt) mx = len[c] > mx ? len[c] : mx;
        }
        mx = wave_scan_dpp<OpMax>(mx);
        if ((t & (kWave - 1)) == kWave - 1) atomicMax(&s_max, mx);
        __syncthreads();
        const int bits = 32 - __clz((int)s_max);
        const int passes = (bits + 7) / 8;
        const int dbits = (bits + passes - 1) / passes;
        const uint32_t mask = (1u << dbits) - 1;
        for (int k = 0, sh = 0; k < passes; ++k, sh += dbits) {
            for (int i = t; i < kFormBins * kChainWaves; i += kChainThreads) s_cnt[i] = 0;
            __syncthreads();
            uint32_t at[KPT];
#pragma unroll
            for (int c = 0; c < KPT; ++c) {
                const bool valid = p0 + c * kWave < cnt;
                const uint32_t d = mask - ((len[c] >> sh) & mask);
                const uint64_t m = match_digit(d, valid, dbits);
                const uint32_t below = (uint32_t)lanes_below(m);
                // every lane reads the count before the digit's first lane adds to it (LDS
                // operations of one wave complete in order; the fences keep the compiler to it)
                at[c] = s_cnt[form_bin(d, w)] + below;
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (valid && below == 0) s_cnt[form_bin(d, w)] += (uint32_t)__popcll(m);
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            }
            __syncthreads();
            {
                // kPer waves of one digit a thread
                const uint32_t d = t * kPer / kChainWaves;
                const int w0 = t * kPer % kChainWaves;
                uint32_t v[kPer], sum = 0, tot;
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    v[i] = s_cnt[form_bin(d, w0 + i)];
                    sum += v[i];
                }
                uint32_t ex = chain_scan<kChainThreads>(sum, &tot);
#pragma unroll
                for (int i = 0; i < kPer; ++i) {
                    s_cnt[form_bin(d, w0 + i)] = ex;
                    ex += v[i];
                }
            }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < KPT; ++c)
                if (p0 + c * kWave < cnt) {
                    const uint32_t to = s_cnt[form_bin(mask - ((len[c] >> sh) & mask), w)] + at[c];
                    s_len[to] = len[c];
                    s_idx[to] = (uint16_t)idx[c];
                }
            __syncthreads();
#pragma unroll
            for (int c = 0; c < KPT; ++c) {
                const int p = p0 + c * kWave;
                len[c] = p < cnt ? s_len[p] : 1u;
                idx[c] = p < cnt ? s_idx[p] : 0u;
            }
        }
#pragma unroll
        for (int c = 0; c < KPT; ++c) {
            const int p = p0 + c * kWave;
            if (p < cnt) {
                order[base + p] = (int32_t)(base + idx[c]);
                slen[base + p] = (int32_t)len[c];
            }
        }
        __syncthreads();   // the chain takes the place of the counters and indices
    }
    chain_rank<true, kChainThreads>(dyn + P, reinterpret_cast<const int32_t*>(s_len), r, base, cnt, nullptr, budget, sq, by_step, gidx,
                     groups_out, RunTable{}, nullptr, 0, st);
}

typedef int32_t I4 __attribute__((ext_vector_type(4), aligned(4)));

// Group index of every live position, and with `gstart` the global position of every group
// start at its global group id, from the run table.  One block per sort tile, kItems
// consecutive positions per thread: one search (between the runs of the tile's first
// positions) and one division, then a step along the run.
template <int kItems>
__global__ void __launch_bounds__(kBlock) chain_index_kernel(const int64_t* __restrict__ off,
                                                             const int64_t* __restrict__ tile_first, int W,
                                                             const RankState* __restrict__ ranks, RunTable tbl,
                                                             int32_t* __restrict__ gidx, int32_t* __restrict__ gstart) {
    constexpr int kTile = kBlock * kItems;
    const int64_t b = blockIdx.x;
    const int r = rank_of(tile_first, W, b);
    const int64_t base = off[r];
    const int64_t cnt = ranks ? ranks[r].cnt : off[r + 1] - base;
    const int64_t tile0 = (b - tile_first[r]) * kTile;
    const int64_t q0 = tile0 + (int64_t)threadIdx.x * kItems;
    if (q0 >= cnt) return;
    const int m = cnt - q0 < kItems ? (int)(cnt - q0) : kItems;
    // the run of position max(q0, 1), between the runs of this tile's and the next tile's first
    // positions
    const int32_t* start = tbl.start + base;
    uint32_t q = q0 > 0 ? (uint32_t)q0 : 1u;
    int a = 0;
    uint32_t end = 0, nxt = 0, step = 1;   // the run's end, the next group start, the step
    int32_t g = 0;                         // group of the current position
    bool head = true;                      // the current position starts its group
    auto enter = [&](uint32_t x) {
        end = (uint32_t)start[a + 1];
        step = (uint32_t)tbl.step[base + a];
        const uint32_t c = (uint32_t)tbl.first[base + a];
        g = tbl.before[base + a];
        nxt = c;
        head = false;
        if (x >= c) {
            const uint32_t k = (x - c) / step;
            g += (int32_t)k + 1;
            nxt = c + (k + 1) * step;
            head = nxt - step == x;
        }
    };
    if (cnt > 1) {
        a = (int)tbl.tile[b];
        int z = tile0 + kTile < cnt ? (int)tbl.tile[b + 1] + 1 : (int)tbl.runs[r];
        while (z - a > 1) {
            const int mid = (a + z) >> 1;
            if ((uint32_t)start[mid] <= q) a = mid; else z = mid;
        }
        enter(q);
    }
    int32_t out[kItems];
    uint32_t heads = 0;
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
        const uint32_t x = (uint32_t)q0 + i;
        if (x == 0) {   // position 0: the first group, of one
            out[i] = 0;
            heads |= 1u;
            continue;
        }
        if (i < m && x > q) {
            if (x >= end) {   // a run holds at least one position
                a += 1;
                enter(x);
            } else if (x == nxt) {
                g += 1;
                nxt += step;
                head = true;
            } else {
                head = false;
            }
            q = x;
        }
        out[i] = g;
        heads |= head && i < m ? 1u << i : 0u;
    }
    int32_t* o = gidx + base + q0;
    if (m == kItems) {
#pragma unroll
        for (int i = 0; i < kItems; i += 4) *reinterpret_cast<I4*>(o + i) = I4{out[i], out[i + 1], out[i + 2], out[i + 3]};
    } else {
#pragma unroll
        for (int i = 0; i < kItems; ++i)
            if (i < m) o[i] = out[i];
    }
    if (gstart) {
        const int64_t gb = ranks[r].gbase;
#pragma unroll
        for (int i = 0; i < kItems; ++i)
            if ((heads >> i) & 1) gstart[gb + out[i]] = (int32_t)(base + q0 + i);
    }
}

}  // namespace

// floor(sqrt(v)).
static int64_t isqrt(int64_t v) {
    uint64_t s = (uint64_t)std::sqrt((double)v);
    while (s * s > (uint64_t)v) --s;
    while ((s + 1) * (s + 1) <= (uint64_t)v) ++s;
    return (int64_t)s;
}

// Whether chain_kernel can list the steps of a rank from the budget and the range of its
// lengths (0: unknown), or has to look at its samples, or (kChainJump) neither fits its table:
// floor(budget / l) takes at most 2 sqrt(budget) values, and one per length plus the few
// that the listing adds.
enum ChainBy { kChainByStep, kChainBySample, kChainJump };

static ChainBy chain_by(int64_t budget, int64_t max_cnt, int64_t len_range) {
    if (2 * (isqrt(budget) + 1) <= kRunCap || (len_range > 0 && len_range + 4 <= kRunCap)) return kChainByStep;
    return max_cnt <= kRunCap ? kChainBySample : kChainJump;
}

// Whether odb_form_groups takes a window by one block per rank.  The limit on the steps is narrower
// than the chain's table: which path a call takes is seen from outside (this one leaves a bad length
// to odb_align_groups, the other waits and reports it), so the line stays where the header has it.
constexpr int64_t kFormSteps = 3840;

static bool form_in_one_block(int64_t budget, int64_t max_cnt) {
    return max_cnt <= kRankBlockMax && (max_cnt <= kFormSteps || 2 * (isqrt(budget) + 1) + 1 <= kFormSteps);
}
static_assert(kFormSteps <= kRunCap, "the one-block grouping's chain fits its table");

bool chain_fits(int64_t budget, int64_t max_cnt) { return chain_by(budget, max_cnt, 0) != kChainJump; }

int group_short_ranks(int W, int64_t budget, int64_t max_cnt, const int64_t* d_rank_off, const int32_t* d_slen,
                      int32_t* d_gidx, RankState* d_ranks, DevStatus* st, hipStream_t s) {
    hipLaunchKernelGGL(chain_kernel<true>, dim3(W), dim3(kChainBlock), 0, s, d_rank_off, d_ranks, d_slen, budget,
                       isqrt(budget), chain_by(budget, max_cnt, 0) == kChainByStep ? 1 : 0, d_gidx, (int32_t*)nullptr,
                       RunTable{}, (const int64_t*)nullptr, 0, st);
    ODB_LAUNCHED();
    return ODB_OK;
}

// Mark scan, group index of every position, global group starts, G_r.
static int finish_groups(const Layout& L, void* ws, int W, int64_t n, const int64_t* d_off, int32_t* d_gidx,
                         int32_t* d_groups_out, RankState* d_ranks, hipStream_t s) {
    uint8_t* marks = ws_at<uint8_t>(ws, L.marks);
    int32_t* incl = ws_at<int32_t>(ws, L.incl);
    int32_t* gstart = ws_at<int32_t>(ws, L.gstart);
    ODB_TRY((device_excl_scan<uint32_t>(MarkLoad{marks}, InclStore{marks, incl}, n,
                                        ws_at<uint32_t>(ws, L.partials), s)));
    hipLaunchKernelGGL(gidx_kernel, dim3(grid_for(n, kBlock, (int64_t)num_cus() * kPlanBlocksPerCU)), dim3(kBlock), 0, s,
                       (const uint8_t*)marks, (const int32_t*)incl, d_off, (const RankState*)d_ranks, W, n,
                       d_gidx, gstart);
    ODB_LAUNCHED();
    hipLaunchKernelGGL(groups_kernel, dim3(grid_for(W, kBlock)), dim3(kBlock), 0, s, (const int32_t*)incl, d_off,
                       W, d_ranks, ws_at<int64_t>(ws, L.gbase), d_groups_out);
    ODB_LAUNCHED();
    return ODB_OK;
}

int group_sequences(const Layout& L, void* ws, int W, int64_t n, int64_t budget, const int64_t* d_off,
                    int64_t max_cnt, int64_t len_range, bool tiles_ready, const int32_t* d_slen, int32_t* d_gidx,
                    int32_t* d_groups_out, RankState* d_ranks, hipStream_t s) {
    int32_t* j0 = ws_at<int32_t>(ws, L.jmp0);
    int32_t* j1 = ws_at<int32_t>(ws, L.jmp1);
    uint8_t* marks = ws_at<uint8_t>(ws, L.marks);
    int32_t* incl = ws_at<int32_t>(ws, L.incl);
    DevStatus* st = ws_at<DevStatus>(ws, L.status);
    const unsigned grid = grid_for(n + 1, kBlock, (int64_t)num_cus() * kPlanBlocksPerCU);
    const ChainBy by = chain_by(budget, max_cnt, len_range);
    if (by != kChainJump) {
        const int items = sort_items(n);
        int64_t* d_tile_first = ws_at<int64_t>(ws, L.tile_first);
        if (!tiles_ready) {
            hipLaunchKernelGGL(sort_tiles_kernel, dim3(1), dim3(kBlock), 0, s, d_off, W, (int)kBlock * items, d_tile_first);
            ODB_LAUNCHED();
        }
        const RunTable tbl{j0, j1, ws_at<int32_t>(ws, L.gsize), incl, ws_at<uint32_t>(ws, L.counts),
                           ws_at<uint32_t>(ws, L.rank_runs)};
        hipLaunchKernelGGL(chain_kernel<false>, dim3(W), dim3(kChainBlock), 0, s, d_off, d_ranks, d_slen, budget,
                           isqrt(budget), by == kChainByStep ? 1 : 0, (int32_t*)nullptr, d_groups_out, tbl,
                           (const int64_t*)d_tile_first, (int)kBlock * items, st);
        ODB_LAUNCHED();
        if (d_ranks) {   // the next round of an alignment numbers its groups over all ranks
            hipLaunchKernelGGL(rank_groups_kernel, dim3(1), dim3(kBlock), 0, s, d_ranks, W, ws_at<int64_t>(ws, L.gbase));
            ODB_LAUNCHED();
        }
        const unsigned tiles = (unsigned)L.num_sort_blocks[items > kSortItems];
        if (tiles > 0) {
            const auto kernel = items > kSortItems ? chain_index_kernel<2 * kSortItems> : chain_index_kernel<kSortItems>;
            hipLaunchKernelGGL(kernel, dim3(tiles), dim3(kBlock), 0, s, d_off, (const int64_t*)d_tile_first,
                               W, (const RankState*)d_ranks, tbl, d_gidx,
                               d_ranks ? ws_at<int32_t>(ws, L.gstart) : (int32_t*)nullptr);
            ODB_LAUNCHED();
        }
        return ODB_OK;
    }
    if (!d_ranks) {   // the jumping kernels read the counts from the rank states
        d_ranks = ws_at<RankState>(ws, L.ranks);
        hipLaunchKernelGGL(rank_counts_kernel, dim3(grid_for(W, kBlock)), dim3(kBlock), 0, s, d_off, W, d_ranks);
        ODB_LAUNCHED();
    }
    hipLaunchKernelGGL(links_kernel, dim3(grid), dim3(kBlock), 0, s, d_slen, d_off,
                       (const RankState*)d_ranks, W, n, budget, j0, marks);
    ODB_LAUNCHED();
    // chains have at most max_cnt elements: ceil(log2(max_cnt + 1)) + 1 doubling rounds
    // always suffice; rounds after convergence return immediately
    int rounds = 1;
    while ((int64_t(1) << (rounds - 1)) <= max_cnt && rounds < kMaxJumpRounds) ++rounds;
    hipLaunchKernelGGL(init_jump_flags, dim3(1), dim3(64), 0, s, st);
    ODB_LAUNCHED();
    for (int k = 0; k < rounds; ++k) {
        const int32_t* jin = (k & 1) ? j1 : j0;
        int32_t* jout = (k & 1) ? j0 : j1;
        hipLaunchKernelGGL(jump_kernel, dim3(grid), dim3(kBlock), 0, s, jin, jout, marks, n, st, k);
        ODB_LAUNCHED();
    }
    return finish_groups(L, ws, W, n, d_off, d_gidx, d_groups_out, d_ranks, s);
}

}  // namespace odb

using namespace odb;

extern "C" int odb_form_groups(const odb_window_t* w, int64_t budget, int32_t* d_order, int32_t* d_sorted_len,
                               int32_t* d_group_index, int32_t* d_groups_per_rank, void* d_ws, size_t ws_bytes,
                               void* stream) {
    Layout L;
    ODB_TRY(check_workspace(w, d_ws, ws_bytes, &L));
    if (budget < 1) return set_error(ODB_E_INVALID_ARG, "budget must be >= 1");
    const int W = w->num_ranks;
    const int64_t n = w->num_samples;
    if (n > 0 && (!d_order || !d_sorted_len || !d_group_index))
        return set_error(ODB_E_INVALID_ARG, "stage-1 output pointers must not be NULL");
    if (!d_groups_per_rank) return set_error(ODB_E_INVALID_ARG, "d_groups_per_rank is NULL");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int64_t* d_off = ws_at<int64_t>(d_ws, L.rank_off);
    DevStatus* st = ws_at<DevStatus>(d_ws, L.status);
    int32_t* len = ws_at<int32_t>(d_ws, L.len);
    int64_t max_cnt = 0;
    for (int r = 0; r < W; ++r) {
        const int64_t c = w->rank_offsets[r + 1] - w->rank_offsets[r];
        if (c > max_cnt) max_cnt = c;
    }

    // one block per rank: one launch, no synchronisation (invalid lengths are grouped as
    // length 1 and reported by odb_align_groups); the rank offsets go along as kernel arguments
    // where they fit
    if (form_in_one_block(budget, max_cnt)) {
        const ChainBy by = chain_by(budget, max_cnt, 0);
        Values v{};
        const int64_t* off = nullptr;
        if (W < kValuesPerLaunch) {
            for (int r = 0; r <= W; ++r) v.v[r] = w->rank_offsets[r];
        } else {
            ODB_TRY(upload_small(w, L, d_ws, nullptr, s));
            off = d_off;
        }
#define ODB_FORM(KPT)                                                                                             \
    hipLaunchKernelGGL(rank_form_kernel<KPT>, dim3(W), dim3(kChainThreads), form_lds_bytes<KPT>(), s, v, off,      \
                       w->d_token_offsets, budget, isqrt(budget), by == kChainByStep ? 1 : 0, d_order, d_sorted_len, \
                       d_group_index, d_groups_per_rank, st)
        // the fewest positions per thread that hold the largest rank
        if (max_cnt <= kChainThreads) ODB_FORM(1);
        else if (max_cnt <= 2 * kChainThreads) ODB_FORM(2);
        else if (max_cnt <= 4 * kChainThreads) ODB_FORM(4);
        else if (max_cnt <= 8 * kChainThreads) ODB_FORM(8);
        else ODB_FORM(16);
#undef ODB_FORM
        static_assert(kRankBlockMax <= 16 * kChainThreads, "positions per thread");
        ODB_LAUNCHED();
        return ODB_OK;
    }
    ODB_TRY(upload_small(w, L, d_ws, nullptr, s));

    // (a2) is a segmented stable radix sort on key = max_l - l, first digit first
    const int items = sort_items(n);
    const bool longer = items > kSortItems;
    const int64_t NB = L.num_sort_blocks[longer];
    const int64_t rank_tiles = (max_cnt + kBlock * items - 1) / (kBlock * items);
    int ibits = 0;   // bits of a position within a rank
    while ((int64_t(1) << ibits) < max_cnt) ++ibits;
    int64_t* d_tile_first = ws_at<int64_t>(d_ws, L.tile_first);
    uint32_t* counts = ws_at<uint32_t>(d_ws, L.counts);
    uint32_t* keys[2] = {ws_at<uint32_t>(d_ws, L.keys0), ws_at<uint32_t>(d_ws, L.keys1)};
    int32_t* vals[2] = {ws_at<int32_t>(d_ws, L.vals0), ws_at<int32_t>(d_ws, L.vals1)};
    auto hist = [&](bool first, const uint32_t* kin, uint32_t maxl, int shift, int dbits, const DevStatus* range) {
        const auto k = first ? (longer ? radix_hist_kernel<2 * kSortItems, true> : radix_hist_kernel<kSortItems, true>)
                             : (longer ? radix_hist_kernel<2 * kSortItems, false> : radix_hist_kernel<kSortItems, false>);
        hipLaunchKernelGGL(k, dim3((unsigned)NB), dim3(kBlock), 0, s, d_off, (const int64_t*)d_tile_first, W, kin,
                           (const int32_t*)len, maxl, shift, dbits, range, counts);
    };
    auto scan = [&](int dbits, const DevStatus* range) {
        hipLaunchKernelGGL(rank_scan_kernel, dim3(W), dim3(kRankScanThreads), 0, s, d_off, (const int64_t*)d_tile_first,
                           dbits, range, counts);
    };
#define ODB_SCATTER(P, F, La, kin, vin, maxl, shift, dbits, range, kout, vout)                                             \
    do {                                                                                                      \
        const auto scatter = longer ? radix_scatter_kernel<2 * kSortItems, P, F, La> : radix_scatter_kernel<kSortItems, P, F, La>; \
        hipLaunchKernelGGL(scatter, dim3((unsigned)NB), dim3(kBlock), 0, s, d_off, (const int64_t*)d_tile_first, W,                \
                           kin, (const int32_t*)len, vin, maxl, ibits, shift, dbits, range, (const uint32_t*)counts, kout, vout,   \
                           d_sorted_len);                                                                     \
    } while (0)

    // (a1) lengths and their validity; the one synchronisation of this call.  While the host waits
    // for the range of lengths and comes back with the launches that depend on it, the stream
    // runs the first digit's pass (8 x 65,536 samples, the whole step: 1,569 -> 1,551 us;
    // 16 x 65,536, the plan: 190 -> 185; 64 x 262,144: 498 -> 493)
    if (n > 0) {
        hipLaunchKernelGGL(sort_tiles_kernel, dim3(1), dim3(kBlock), 0, s, d_off, W, (int)kBlock * items, d_tile_first);
        ODB_LAUNCHED();
    }
    hipLaunchKernelGGL(lengths_kernel, dim3(grid_for(n, kBlock, (int64_t)num_cus() * kLengthsBlocksPerCU)), dim3(kBlock), 0, s,
                       w->d_token_offsets, n, len, st);
    ODB_LAUNCHED();
    DevStatus hs;
    bool ahead = false;
    if (rank_tiles << 8 <= kRankScanMax) ODB_TRY(read_begin(st, sizeof(DevStatus), s, &ahead));
    if (ahead) {
        const DevStatus* range = st;
        hist(true, nullptr, 0, 0, 0, range);
        ODB_LAUNCHED();
        scan(0, range);
        ODB_LAUNCHED();
        ODB_SCATTER(true, true, false, (const uint32_t*)nullptr, (const int32_t*)nullptr, 0u, ibits, 0, range, keys[0], vals[0]);
        ODB_LAUNCHED();
        ODB_TRY(read_end(&hs, sizeof(DevStatus)));
    } else {
        ODB_TRY(read_device(&hs, st, sizeof(DevStatus), s));
    }
    if (hs.err & kErrLength) {
        if (ahead) ODB_TRY_HIP(hipStreamSynchronize(s));   // an error leaves nothing running
        return set_error(ODB_E_INVALID_DATA,
                         "sample %lld has a length outside [1, 2^31) or a negative token offset",
                         (long long)hs.first_bad);
    }
    const uint32_t maxl = hs.max_len, minl = hs.min_len;
    const SortPlan sp = sort_plan(minl, maxl, ibits);
    if (sp.passes == 0) {
        hipLaunchKernelGGL(identity_order_kernel, dim3(grid_for(n, kBlock, (int64_t)num_cus() * kPlanBlocksPerCU)), dim3(kBlock),
                           0, s, n, (const int32_t*)len, d_order, d_sorted_len);
        ODB_LAUNCHED();
    }
    for (int pass = 0; pass < sp.passes; ++pass) {
        const int shift = pass * sp.dbits;
        const bool first = pass == 0, last = pass == sp.passes - 1;
        if (first && !last && ahead && sp.packed) continue;
        const uint32_t* kin = first ? nullptr : keys[(pass - 1) & 1];
        const int32_t* vin = first ? nullptr : vals[(pass - 1) & 1];
        uint32_t* kout = last ? nullptr : keys[pass & 1];
        int32_t* vout = last ? d_order : vals[pass & 1];
        if (!(first && ahead)) {   // else the counts are there
            hist(first, kin, maxl, first || !sp.packed ? shift : shift + ibits, sp.dbits, nullptr);
            ODB_LAUNCHED();
            if (rank_tiles << sp.dbits <= kRankScanMax) {
                scan(sp.dbits, nullptr);
                ODB_LAUNCHED();
            } else {
                ODB_TRY((device_excl_scan<uint32_t>(CountLoad{counts, NB << sp.dbits}, CountStore{counts}, NB << sp.dbits,
                                                    ws_at<uint32_t>(d_ws, L.partials), s)));
            }
        }
        const DevStatus* host = nullptr;
#define ODB_SCATTER_PASS(F, La)                                                                                   \
    do {                                                                                                          \
        if (sp.packed) ODB_SCATTER(true, F, La, kin, vin, maxl, shift + ibits, sp.dbits, host, kout, vout);       \
        else ODB_SCATTER(false, F, La, kin, vin, maxl, shift, sp.dbits, host, kout, vout);                        \
    } while (0)
        if (first && last) ODB_SCATTER_PASS(true, true);
        else if (first) ODB_SCATTER_PASS(true, false);
        else if (last) ODB_SCATTER_PASS(false, true);
        else ODB_SCATTER_PASS(false, false);
#undef ODB_SCATTER_PASS
#undef ODB_SCATTER
        ODB_LAUNCHED();
    }

    // (a3, a4) the group chain
    return group_sequences(L, d_ws, W, n, budget, d_off, max_cnt, (int64_t)maxl - minl + 1, n > 0, d_sorted_len,
                           d_group_index, d_groups_per_rank, nullptr, s);
}
