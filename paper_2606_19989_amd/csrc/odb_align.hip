// Stages 2-3 of the ODB window pipeline: Distributed Group Alignment (Eq. 3,
// Algorithm 1, termination rules of Sec. 2.3) and identity coverage (App. C).
//
// Three paths, equal results: a window that aligns in one round is written from closed forms
// (rows, slots and tiles kernels), join windows of short ranks that overflow run two launches
// a round without waiting for the host (short_round_kernel), and what is left goes round by
// round, as below.
//
// Every rank's buffer is a contiguous run of formation positions; a group is a range
// of them.  One alignment round is:
//   group_sizes        size of every group
//   adjust_kernel      per rank: the simulated all_gather of (G_r, S_r, C_r) and Eq. 3's T,
//                      then split (closed form, below) or overflow (size threshold)
//   slot_records       rows / max length / real tokens of every aligned step, and the
//                      global sample count of every step
//   finalize_kernel    per rank: the round's cut (join: all T steps; non-join: up to the
//                      first step reaching Q), which positions are emitted, where they go
//   emit_kernel        writes emitted ids (rows short to long) and the next buffer
// and rounds repeat on the returned samples until the termination rule fires.
//
// Split in closed form.  Algorithm 1 peels, one at a time, the last sample of the first
// multi-sample group met scanning the short-to-long list from its long end.  In
// formation order (longest first) that is the longest member of the first group with
// at least two samples; after k = T - G_r peels, formation positions [0, X) are
// singletons, [X, end of group j*) is one group and later groups are untouched, where
// j* is the first group whose cumulative surplus sum_{g<=j}(c_g - 1) reaches k and
// X = k + j*.
//
// Overflow.  Algorithm 1 keeps the T largest groups (stable over the short-to-long list,
// so equal sizes favour the later-formed group).  With sigma = the largest size such
// that at least T groups have size >= sigma, every group larger than sigma is kept and
// the remaining places go to the size-sigma groups with the highest formation index.
#include <algorithm>
#include <climits>
#include <cstring>
#include <vector>

#include "odb_internal.h"

namespace odb {

// A pair of int64 sums, scanned together by the generic scan (its shuffles are found by
// argument-dependent lookup, next to the scalar ones).  Trivially default-constructible, so
// it can live in LDS.
struct I64Pair {
    int64_t a, b;
    I64Pair() = default;
    __host__ __device__ constexpr I64Pair(int z) : a(z), b(z) {}
    __host__ __device__ constexpr I64Pair(int64_t x, int64_t y) : a(x), b(y) {}
};
__device__ __forceinline__ I64Pair operator+(I64Pair x, I64Pair y) { return I64Pair{x.a + y.a, x.b + y.b}; }
__device__ __forceinline__ I64Pair operator-(I64Pair x, I64Pair y) { return I64Pair{x.a - y.a, x.b - y.b}; }
__device__ __forceinline__ I64Pair& operator+=(I64Pair& x, I64Pair y) {
    x.a += y.a;
    x.b += y.b;
    return x;
}
__device__ __forceinline__ I64Pair __shfl_up(I64Pair v, unsigned int d, int width) {
    return I64Pair{::__shfl_up(v.a, d, width), ::__shfl_up(v.b, d, width)};
}
__device__ __forceinline__ I64Pair __shfl_xor(I64Pair v, int m, int width) {
    return I64Pair{::__shfl_xor(v.a, m, width), ::__shfl_xor(v.b, m, width)};
}

namespace {

template <typename T, typename Op>
__device__ __forceinline__ T block_reduce(T v, Op op) {
    __shared__ T buf[kBlock];
    buf[threadIdx.x] = v;
    __syncthreads();
    for (unsigned s = kBlock / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) buf[threadIdx.x] = op(buf[threadIdx.x], buf[threadIdx.x + s]);
        __syncthreads();
    }
    T r = buf[0];
    __syncthreads();
    return r;
}

struct MaxOp {
    __device__ int64_t operator()(int64_t a, int64_t b) const { return a > b ? a : b; }
};
struct MinOp {
    __device__ int64_t operator()(int64_t a, int64_t b) const { return a < b ? a : b; }
};
struct SumOp {
    __device__ int64_t operator()(int64_t a, int64_t b) const { return a + b; }
};

__global__ void init_align_kernel(RoundState* rs, DevInfo* info) {
    if (threadIdx.x == 0) {
        *rs = RoundState{};
        *info = DevInfo{};
    }
}

__global__ void clear_view_counters_kernel(DevInfo* info, int with_ids) {
    if (threadIdx.x == 0) {
        info->bad_views = 0;
        if (with_ids) {
            info->missing_ids = 0;
            info->duplicate_ids = 0;
        }
    }
}

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = v;
}


// ---------------------------------------------------------------- round 0 inputs
// Rank state from the stage-1 group counts; G_r must be 0 exactly for empty ranks and
// at most S_r.  One block.
__global__ void __launch_bounds__(kBlock) round0_ranks_kernel(const int64_t* __restrict__ off,
                                                              const int32_t* __restrict__ groups, int W,
                                                              RankState* ranks, int64_t* __restrict__ gbase,
                                                              DevStatus* st, RoundState* rs, DevInfo* info) {
    __shared__ int64_t carry;
    if (threadIdx.x == 0) {
        carry = 0;
        *rs = RoundState{};
        *info = DevInfo{};
    }
    __syncthreads();
    for (int b = 0; b < W; b += kBlock) {
        const int r = b + threadIdx.x;
        int64_t G = 0, cnt = 0;
        if (r < W) {
            G = groups[r];
            cnt = off[r + 1] - off[r];
            if (G < 0 || G > cnt || ((cnt == 0) != (G == 0))) {
                atomicOr(&st->err, kErrGroupIndex);
                G = 0;
            }
        }
        int64_t tot;
        const int64_t ex = block_excl_sum(G, &tot);
        const int64_t c = carry;
        if (r < W) {
            RankState z = {};
            z.cnt = cnt;
            z.G = G;
            z.gbase = c + ex;
            ranks[r] = z;
            gbase[r] = c + ex;
        }
        __syncthreads();
        if (threadIdx.x == 0) carry = c + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) gbase[W] = carry;
}

// Checks that stage-1 arrays describe this window: order[p] is a sample of p's rank,
// sorted_len[p] >= 1, the order strictly (length desc, id asc) -- so each rank's segment
// is a permutation of its ids -- and the group indices run 0, 0|+1, ..., G_r - 1.
// Records every group start.  That sorted_len[p] is the CSR length of order[p] is
// checked once the plan is built (row_check_kernel, leftover_kernel), where the CSR
// offsets of every emitted sample are gathered anyway for the row records.
__global__ void __launch_bounds__(kBlock) round0_check_kernel(
    const int64_t* __restrict__ off, const RankState* __restrict__ ranks,
    int W, int64_t n, const int32_t* __restrict__ order, const int32_t* __restrict__ slen,
    const int32_t* __restrict__ gidx, int32_t* __restrict__ gstart, DevStatus* st) {
    __shared__ int64_t s_off[kLdsRanks + 1];
    off = stage_ranks(off, W, s_off);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        const int r = rank_of(off, W, p);
        const int64_t base = off[r];
        const int64_t q = p - base, nr = ranks[r].cnt;
        const int64_t G = ranks[r].G;
        const int32_t id = order[p];
        const int32_t l = slen[p];
        bool ok = id >= base && id < base + nr && l >= 1;
        const int32_t g = gidx[p];
        bool gok = g >= 0 && g < G;
        if (q == 0) {
            gok = gok && g == 0;
        } else {
            const int32_t pl = slen[p - 1], pid = order[p - 1];
            ok = ok && (pl > l || (pl == l && pid < id));
            const int32_t d = g - gidx[p - 1];
            gok = gok && (d == 0 || d == 1);
        }
        if (q == nr - 1) gok = gok && g == G - 1;
        if (!ok) {
            atomicOr(&st->err, kErrOrder);
            atomicMin((unsigned long long*)&st->first_bad, (unsigned long long)p);
        }
        if (!gok) {
            atomicOr(&st->err, kErrGroupIndex);
            atomicMin((unsigned long long*)&st->first_bad, (unsigned long long)p);
        } else if (q == 0 || g != gidx[p - 1]) {
            gstart[ranks[r].gbase + g] = (int32_t)p;
        }
    }
}

// ---------------------------------------------------------------- one round
struct LiveLen {
    const int32_t* len;
    const int64_t* off;
    const RankState* ranks;
    int W;
    int gaps;
    __device__ int64_t operator()(int64_t i) const {
        if (!gaps) return len[i];
        const int r = rank_of(off, W, i);
        return (i - off[r] < ranks[r].cnt) ? (int64_t)len[i] : 0;
    }
};
struct LiveLenIncl {
    LiveLen ld;
    int64_t* cs;
    __device__ void operator()(int64_t i, int64_t ex) const { cs[i] = ex + ld(i); }
};

// Stage-1 arrays that round0_check_kernel found inconsistent: the round's kernels that
// index through group starts do nothing (the host reports the error at the round's
// synchronisation).
__device__ __forceinline__ bool stage1_bad(const DevStatus* st) {
    return (*(volatile const int32_t*)&st->err & (kErrOrder | kErrGroupIndex)) != 0;
}

__global__ void __launch_bounds__(kBlock) group_sizes_kernel(const int32_t* __restrict__ gstart,
                                                             const int64_t* __restrict__ gbase,
                                                             const int64_t* __restrict__ off,
                                                             const RankState* __restrict__ ranks, int W,
                                                             int32_t* __restrict__ gsize, int64_t* __restrict__ steps,
                                                             int64_t nsteps, const DevStatus* st) {
    if (stage1_bad(st)) return;
    const int64_t total = gbase[W];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    // the round's per-step sample counts, summed by slot_records_kernel
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < nsteps; j += stride) steps[j] = 0;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += stride) {
        const int r = rank_of(gbase, W, g);
        const int64_t lg = g - gbase[r];
        const int64_t start = gstart[g];
        const int64_t end = (lg + 1 < ranks[r].G) ? (int64_t)gstart[g + 1] : off[r] + ranks[r].cnt;
        gsize[g] = (int32_t)(end - start);
    }
}

// Per rank (one block each): the simulated all_gather of (G_r, S_r, C_r) and Eq. 3's
// target T over the active ranks (every block computes it; block 0 also records the round's
// statistics), then this rank's action: split position or overflow selection.
__global__ void __launch_bounds__(kBlock) adjust_kernel(RankState* ranks, const int64_t* __restrict__ cap,
                                                        int has_cap, int W, RoundState* rs,
                                                        const int32_t* __restrict__ gsize,
                                                        int32_t* __restrict__ ov_slot, int32_t* __restrict__ kept,
                                                        DevStatus* st) {
    if (stage1_bad(st)) return;
    int64_t maxG = 0, minC = LLONG_MAX, minS = LLONG_MAX;
    for (int q = threadIdx.x; q < W; q += kBlock) {
        const int64_t Gq = ranks[q].G;
        if (Gq <= 0) continue;
        maxG = Gq > maxG ? Gq : maxG;
        const int64_t S = ranks[q].cnt;
        if (S > 0 && S < minS) minS = S;
        if (has_cap && cap[q] > 0 && cap[q] < minC) minC = cap[q];
    }
    maxG = block_reduce(maxG, MaxOp{});
    minC = block_reduce(minC, MinOp{});
    minS = block_reduce(minS, MinOp{});
    int64_t T = maxG;
    if (minC != LLONG_MAX && minC < T) T = minC;
    if (minS != LLONG_MAX && minS < T) T = minS;
    if (T < 1) T = 1;
    if (blockIdx.x == 0) {
        int64_t active = 0, totalG = 0, splits = 0, over = 0, changed = 0;
        for (int q = threadIdx.x; q < W; q += kBlock) {
            const int64_t Gq = ranks[q].G;
            totalG += Gq;
            if (Gq <= 0) continue;
            active += 1;
            if (Gq < T) {
                splits += T - Gq;
                changed += 1;
            } else if (Gq > T) {
                over += Gq - T;
                changed += 1;
            }
        }
        active = block_reduce(active, SumOp{});
        totalG = block_reduce(totalG, SumOp{});
        splits = block_reduce(splits, SumOp{});
        over = block_reduce(over, SumOp{});
        changed = block_reduce(changed, SumOp{});
        if (threadIdx.x == 0) {
            // App. B: the pre-alignment counts of the first exchange are exact only if no
            // active rank's groups changed; otherwise exact token weights need a second one
            rs->second_gather += changed > 0 ? 1 : 0;
            rs->T = T;
            rs->active = active;
            rs->total_groups = totalG;
            rs->splits += splits;
            rs->overflow += over;
            rs->cut = 0;
        }
    }
    const int r = blockIdx.x;
    const int64_t G = ranks[r].G;
    const int32_t action = G <= 0 ? kActInactive : (G < T ? kActSplit : (G > T ? kActOverflow : kActKeep));
    if (threadIdx.x == 0) {
        ranks[r].X = 0;
        ranks[r].jstar = 0;
        ranks[r].qcut = 0;
        ranks[r].action = action;
    }
    if (action != kActSplit && action != kActOverflow) return;
    const int64_t gb = ranks[r].gbase;
    __shared__ int64_t s_found;
    if (action == kActSplit) {
        const int64_t k = T - G;
        if (threadIdx.x == 0) s_found = -1;
        __syncthreads();
        int64_t carry = 0;
        for (int64_t b = 0; b < G; b += kBlock) {
            const int64_t j = b + threadIdx.x;
            const int64_t v = j < G ? (int64_t)gsize[gb + j] - 1 : 0;
            int64_t tot;
            const int64_t ex = block_excl_sum(v, &tot);
            if (j < G && carry + ex < k && carry + ex + v >= k) s_found = j;
            __syncthreads();
            if (s_found >= 0) break;
            carry += tot;
        }
        if (threadIdx.x == 0) {
            const int64_t js = s_found;
            if (js < 1) {
                // the group sizes do not add up to the buffer: drop the rank from this round
                // (nothing is indexed through the split) and report an internal error
                atomicOr(&st->err, kErrInternal);
                ranks[r].action = kActInactive;
            } else {
                ranks[r].jstar = js;
                ranks[r].X = k + js;
            }
        }
        return;
    }
    // overflow: sigma = largest size with at least T groups of size >= sigma
    int64_t mx = 0;
    for (int64_t j = threadIdx.x; j < G; j += kBlock) {
        const int64_t s = gsize[gb + j];
        mx = s > mx ? s : mx;
    }
    mx = block_reduce(mx, MaxOp{});
    int64_t lo = 1, hi = mx;
    while (lo < hi) {
        const int64_t mid = lo + (hi - lo + 1) / 2;
        int64_t c = 0;
        for (int64_t j = threadIdx.x; j < G; j += kBlock) c += gsize[gb + j] >= mid ? 1 : 0;
        c = block_reduce(c, SumOp{});
        if (c >= T) lo = mid; else hi = mid - 1;
    }
    const int64_t sigma = lo;
    int64_t above = 0;
    for (int64_t j = threadIdx.x; j < G; j += kBlock) above += gsize[gb + j] > sigma ? 1 : 0;
    above = block_reduce(above, SumOp{});
    const int64_t need = T - above;
    // walk groups from the highest formation index down
    int64_t ceq = 0, ckept = 0;
    for (int64_t b = 0; b < G; b += kBlock) {
        const int64_t i = b + threadIdx.x;
        const bool valid = i < G;
        const int64_t g = G - 1 - i;
        const int64_t s = valid ? gsize[gb + g] : 0;
        const int64_t eq = (valid && s == sigma) ? 1 : 0;
        int64_t teq;
        const int64_t xeq = block_excl_sum(eq, &teq);
        const int64_t keep = (valid && (s > sigma || (eq && ceq + xeq < need))) ? 1 : 0;
        int64_t tk;
        const int64_t xk = block_excl_sum(keep, &tk);
        if (valid) {
            if (keep) {
                ov_slot[gb + g] = (int32_t)(ckept + xk);
                kept[gb + ckept + xk] = (int32_t)g;
            } else {
                ov_slot[gb + g] = -1;
            }
        }
        ceq += teq;
        ckept += tk;
    }
}

// First formation position and one-past-last of adjusted group a (formation order) of a
// keep / split rank.
__device__ __forceinline__ void adjusted_range(const RankState& R, int64_t base, int64_t a,
                                               const int32_t* __restrict__ gstart,
                                               const int32_t* __restrict__ gsize, int64_t* start, int64_t* end) {
    if (a < R.X) {
        *start = base + a;
        *end = base + a + 1;
    } else if (a == R.X) {
        const int64_t g = R.gbase + R.jstar;
        *start = base + R.X;
        *end = (int64_t)gstart[g] + gsize[g];
    } else {
        const int64_t g = R.gbase + R.jstar + (a - R.X);
        *start = gstart[g];
        *end = *start + gsize[g];
    }
}

// Step j of every active rank: adjusted group T-1-j (emission runs short to long).
// Besides rows, longest length and real tokens, each record carries the approximate
// token count of App. B: rows times the mean length of the rank's buffer at the start of
// this round (the counts a rank can advertise before alignment).
__global__ void __launch_bounds__(kBlock) slot_records_kernel(
    const RankState* __restrict__ ranks, const RoundState* __restrict__ rs, const int64_t* __restrict__ off, int W,
    const int32_t* __restrict__ gstart, const int32_t* __restrict__ gsize, const int32_t* __restrict__ kept,
    const int32_t* __restrict__ cur_len, const int64_t* __restrict__ cs, int32_t* __restrict__ srows,
    int32_t* __restrict__ smax, int64_t* __restrict__ stok, double* __restrict__ sadj,
    int64_t* __restrict__ steps, const DevStatus* st) {
#pragma clang fp contract(off)
    if (stage1_bad(st)) return;
    const int64_t T = rs->T;
    const int64_t total = (int64_t)W * T;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < total; idx += stride) {
        const int r = (int)(idx / T);
        const int64_t j = idx - (int64_t)r * T;
        const RankState R = ranks[r];
        if (R.action == kActInactive) continue;
        const int64_t base = off[r];
        int64_t start, end;
        if (R.action == kActOverflow) {
            const int64_t g = R.gbase + kept[R.gbase + j];
            start = gstart[g];
            end = start + gsize[g];
        } else {
            adjusted_range(R, base, T - 1 - j, gstart, gsize, &start, &end);
        }
        const int64_t rows = end - start;
        const int64_t dst = base + R.slots + j;
        srows[dst] = (int32_t)rows;
        smax[dst] = cur_len[start];
        stok[dst] = cs[end - 1] - (start > 0 ? cs[start - 1] : 0);
        // live positions of the rank are [base, base + cnt); cs is inclusive over all n
        const int64_t buf_tok = cs[base + R.cnt - 1] - (base > 0 ? cs[base - 1] : 0);
        const double mean = (double)buf_tok / (double)R.cnt;
        sadj[dst] = (double)rows * mean;
        atomicAdd((unsigned long long*)&steps[j], (unsigned long long)rows);
    }
}

// Steps of this round that are emitted: join, all T; non-join, up to the first step at
// which the cumulative global emitted count reaches the quota (Theorem 2).  Block-uniform;
// *sum and *mx receive the emitted steps' sample total and largest step.
__device__ int64_t round_cut(const int64_t* __restrict__ steps, int64_t T, int64_t before, int nonjoin,
                             int64_t quota, int64_t* sum_out, int64_t* mx_out) {
    __shared__ int64_t s_cut;
    if (threadIdx.x == 0) s_cut = T;
    __syncthreads();
    if (nonjoin) {
        int64_t carry = 0;
        for (int64_t b = 0; b < T; b += kBlock) {
            const int64_t j = b + threadIdx.x;
            const int64_t v = j < T ? steps[j] : 0;
            int64_t tot;
            const int64_t ex = block_excl_sum(v, &tot);
            if (j < T && before + carry + ex < quota && before + carry + ex + v >= quota) s_cut = j + 1;
            __syncthreads();
            if (s_cut < T) break;
            carry += tot;
        }
    }
    const int64_t cut = s_cut;
    int64_t sum = 0, mx = 0;
    for (int64_t j = threadIdx.x; j < cut; j += kBlock) {
        const int64_t v = steps[j];
        sum += v;
        mx = v > mx ? v : mx;
    }
    *sum_out = block_reduce(sum, SumOp{});
    *mx_out = block_reduce(mx, MaxOp{});
    return cut;
}

// Per rank (one block each): the round's cut (every block computes it; block 0 records it
// and the running totals, which advance_kernel makes current), then the rank's emitted
// positions and the layout of its next buffer.
__global__ void __launch_bounds__(kBlock) finalize_kernel(RankState* ranks, RoundState* rs,
                                                          const int64_t* __restrict__ steps, int nonjoin,
                                                          int64_t quota, const int64_t* __restrict__ off,
                                                          const int32_t* __restrict__ gstart,
                                                          const int32_t* __restrict__ gsize,
                                                          const int32_t* __restrict__ ov_slot,
                                                          const int32_t* __restrict__ kept,
                                                          int32_t* __restrict__ ov_lo, const DevStatus* st) {
    if (stage1_bad(st)) return;
    const int r = blockIdx.x;
    RankState& R = ranks[r];
    const int64_t T = rs->T;
    const int64_t before = rs->emitted_total;
    int64_t step_sum, step_mx;
    const int64_t cut = round_cut(steps, T, before, nonjoin, quota, &step_sum, &step_mx);
    if (r == 0 && threadIdx.x == 0) {
        rs->cut = cut;
        rs->emitted_next = before + step_sum;
        if (step_mx > rs->step_max) rs->step_max = step_mx;
        if (nonjoin && before + step_sum >= quota) rs->quota_hit = 1;
    }
    if (threadIdx.x == 0) R.ebase = R.emitted;
    if (R.action == kActInactive) {
        if (threadIdx.x == 0) R.next_cnt = 0;
        return;
    }
    const int64_t base = off[r];
    if (R.action != kActOverflow) {
        if (threadIdx.x == 0) {
            int64_t q = 0;
            if (cut < T) {
                int64_t s, e;
                adjusted_range(R, base, T - cut, gstart, gsize, &s, &e);
                q = s - base;
            }
            R.qcut = q;
            R.next_cnt = q;
            R.emitted += R.cnt - q;
            R.slots += cut;
        }
        return;
    }
    const int64_t G = R.G, gb = R.gbase;
    // emitted groups, slot order: consecutive emission offsets
    int64_t carry = 0;
    for (int64_t b = 0; b < cut; b += kBlock) {
        const int64_t j = b + threadIdx.x;
        const int64_t g = j < cut ? gb + kept[gb + j] : 0;
        const int64_t v = j < cut ? gsize[g] : 0;
        int64_t tot;
        const int64_t ex = block_excl_sum(v, &tot);
        if (j < cut) ov_lo[g] = (int32_t)(carry + ex);
        carry += tot;
    }
    const int64_t emitted_now = carry;
    // everything else, formation order: offsets in the next buffer
    carry = 0;
    for (int64_t b = 0; b < G; b += kBlock) {
        const int64_t j = b + threadIdx.x;
        const int32_t sl = j < G ? ov_slot[gb + j] : 0;
        const bool stay = j < G && (sl < 0 || sl >= cut);
        const int64_t v = stay ? gsize[gb + j] : 0;
        int64_t tot;
        const int64_t ex = block_excl_sum(v, &tot);
        if (stay) ov_lo[gb + j] = (int32_t)(carry + ex);
        carry += tot;
    }
    if (threadIdx.x == 0) {
        R.next_cnt = carry;
        R.emitted += emitted_now;
        R.slots += cut;
    }
}

__global__ void __launch_bounds__(kBlock) emit_kernel(
    const RankState* __restrict__ ranks, const RoundState* __restrict__ rs, const int64_t* __restrict__ off, int W,
    int64_t n, const int32_t* __restrict__ cur_ids, const int32_t* __restrict__ cur_len,
    const int32_t* __restrict__ gidx, const int32_t* __restrict__ gstart, const int32_t* __restrict__ gsize,
    const int32_t* __restrict__ ov_slot, const int32_t* __restrict__ ov_lo, int32_t* __restrict__ dst,
    int32_t* __restrict__ dst_len, int32_t* __restrict__ next_ids, int32_t* __restrict__ next_len,
    const DevStatus* st) {
    if (stage1_bad(st)) return;
    __shared__ int64_t s_off[kLdsRanks + 1];
    off = stage_ranks(off, W, s_off);
    const int64_t cut = rs->cut;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        const int r = rank_of(off, W, p);
        const int64_t base = off[r];
        const int64_t q = p - base;
        const RankState& R = ranks[r];
        const int64_t cnt = R.cnt;
        if (q >= cnt) continue;
        const int32_t id = cur_ids[p];
        if (R.action != kActOverflow) {
            if (q >= R.qcut) {
                const int64_t o = base + R.ebase + (cnt - 1 - q);
                dst[o] = id;
                dst_len[o] = cur_len[p];
            } else {
                next_ids[base + q] = id;
                next_len[base + q] = cur_len[p];
            }
        } else {
            const int64_t g = R.gbase + gidx[p];
            const int32_t sl = ov_slot[g];
            const int64_t st = (int64_t)gstart[g] - base;
            if (sl >= 0 && sl < cut) {
                const int64_t o = base + R.ebase + ov_lo[g] + (st + gsize[g] - 1 - q);
                dst[o] = id;
                dst_len[o] = cur_len[p];
            } else {
                const int64_t o = ov_lo[g] + (q - st);
                next_ids[base + o] = id;
                next_len[base + o] = cur_len[p];
            }
        }
    }
}

// End of a round: the next buffers' counts and the running emitted total become current.
__global__ void advance_kernel(RankState* ranks, int W, RoundState* rs) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) rs->emitted_total = rs->emitted_next;
    for (int r = i; r < W; r += gridDim.x * blockDim.x) ranks[r].cnt = ranks[r].next_cnt;
}

// ---------------------------------------------------------------- final plan
__global__ void __launch_bounds__(kBlock) plan_slots_kernel(const RankState* __restrict__ ranks,
                                                            const int64_t* __restrict__ off, int W, int64_t S,
                                                            const int32_t* __restrict__ srows,
                                                            const int32_t* __restrict__ smax,
                                                            const int64_t* __restrict__ stok,
                                                            const double* __restrict__ sadj,
                                                            int32_t* __restrict__ rows, int32_t* __restrict__ maxlen,
                                                            int64_t* __restrict__ tokens, double* __restrict__ approx,
                                                            DevInfo* info) {
    const int64_t K = (int64_t)W * S;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    int64_t real = 0;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < K; k += stride) {
        const int r = (int)(k / S);
        const int64_t j = k - (int64_t)r * S;
        if (j < ranks[r].slots) {
            const int64_t src = off[r] + j;
            rows[k] = srows[src];
            maxlen[k] = smax[src];
            tokens[k] = stok[src];
            real += stok[src];
            if (approx) approx[k] = sadj[src];
        } else {
            rows[k] = 0;
            maxlen[k] = 0;
            tokens[k] = 0;
            if (approx) approx[k] = 0.0;
        }
    }
    // the plan's real tokens (Sec. 2.1 / App. I padding fraction)
    real = block_sum(real);
    if (threadIdx.x == 0 && real) atomicAdd((unsigned long long*)&info->real_tokens, (unsigned long long)real);
}

// The row and tile offsets of the slots in one scan: a slot contributes (rows, rows *
// maxlen).
struct RowsTilesLoad {
    const int32_t* rows;
    const int32_t* mx;
    int64_t K;
    __device__ I64Pair operator()(int64_t i) const {
        return i < K ? I64Pair{(int64_t)rows[i], (int64_t)rows[i] * mx[i]} : I64Pair{0, 0};
    }
};
struct RowsTilesStore {
    int64_t* row_off;
    int64_t* tile_off;
    __device__ void operator()(int64_t i, I64Pair v) const {
        row_off[i] = v.a;
        tile_off[i] = v.b;
    }
};

__global__ void __launch_bounds__(kBlock) compact_emit_kernel(const int32_t* __restrict__ stage,
                                                              const int32_t* __restrict__ stage_len,
                                                              const int64_t* __restrict__ off,
                                                              const RankState* __restrict__ ranks, int W, int64_t n,
                                                              const int64_t* __restrict__ row_off, int64_t S,
                                                              int32_t* __restrict__ emit, int32_t* __restrict__ len) {
    __shared__ int64_t s_off[kLdsRanks + 1];
    off = stage_ranks(off, W, s_off);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        const int r = rank_of(off, W, p);
        const int64_t e = p - off[r];
        if (e < ranks[r].emitted) {
            const int64_t o = row_off[(int64_t)r * S] + e;
            emit[o] = stage[p];
            len[o] = stage_len[p];
        }
    }
}

// Row records of the emitted rows: the CSR token start of each row's sample (written
// when `ts` is not NULL) and the check that the length the plan carried for it (from
// the stage-1 sorted lengths) is the sample's CSR length.  Ids are in range here:
// round0_check_kernel verified that every rank's order is a permutation of its ids.
//
// The offsets are gathered in random order, one 128-byte line per 8-byte read unless the
// line is still cached.  A rank's rows hold only that rank's ids, whose offsets span
// 8 B per sample (2 MB at 262,144 samples), so with `xcd_ranks` set, rank r is gathered
// only by the blocks of group r mod kXcds (workgroups are dealt to the XCDs round
// robin, so block b runs on XCD b mod kXcds): each rank's offsets then stay in one XCD's
// L2 and are read from HBM about once.
constexpr int kXcds = 8;

// The CSR length of sample s against the length its plan row carries: a length outside
// [1, 2^31) or a negative offset is invalid data (grouping took such a sample as length
// 1); any other difference means the stage-1 arrays are not this window's.
__device__ __forceinline__ void check_csr_length(int32_t s, int64_t a, int64_t b, int32_t carried, DevStatus* st) {
    const int64_t l = b - a;
    if (l < 1 || l > INT_MAX || a < 0) {
        atomicOr(&st->err, kErrLength);
        atomicMin((unsigned long long*)&st->first_bad_len, (unsigned long long)s);
    } else if (l != (int64_t)carried) {
        atomicOr(&st->err, kErrSortedLen);
        atomicMin((unsigned long long*)&st->first_bad, (unsigned long long)s);
    }
}

__global__ void __launch_bounds__(kBlock) row_check_kernel(const int64_t* __restrict__ tok_off,
                                                           const int32_t* __restrict__ emit,
                                                           const int32_t* __restrict__ len,
                                                           const int64_t* __restrict__ row_off, int64_t S, int W,
                                                           int xcd_ranks, int64_t* __restrict__ ts, DevStatus* st) {
    const int group = xcd_ranks ? (int)(blockIdx.x % kXcds) : 0;
    const int groups = xcd_ranks ? kXcds : 1;
    const int64_t gb = xcd_ranks ? blockIdx.x / kXcds : blockIdx.x;   // block within its group
    const int64_t nb = xcd_ranks ? gridDim.x / kXcds : gridDim.x;
    const int64_t stride = nb * blockDim.x;
    for (int r = group; r < W; r += groups) {
        // all ranks at once in the plain mode: the rows of ranks group .. W-1 are contiguous
        const int64_t lo = row_off[(int64_t)r * S];
        const int64_t hi = row_off[(int64_t)(xcd_ranks ? r + 1 : W) * S];
        for (int64_t k = lo + gb * blockDim.x + threadIdx.x; k < hi; k += stride) {
            const int32_t s = emit[k];
            const int64_t a = tok_off[s];
            check_csr_length(s, a, tok_off[s + 1], len[k], st);
            if (ts) ts[k] = a;
        }
        if (!xcd_ranks) break;
    }
}

__global__ void __launch_bounds__(kBlock) leftover_off_kernel(const RankState* __restrict__ ranks, int W,
                                                              int64_t* __restrict__ loff) {
    __shared__ int64_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int b = 0; b < W; b += kBlock) {
        const int r = b + threadIdx.x;
        const int64_t v = r < W ? ranks[r].cnt : 0;
        int64_t tot;
        const int64_t ex = block_excl_sum(v, &tot);
        const int64_t c = carry;
        if (r < W) loff[r] = c + ex;
        __syncthreads();
        if (threadIdx.x == 0) carry = c + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) loff[W] = carry;
}

// Left-over ids, and the length check of row_check_kernel for them.
__global__ void __launch_bounds__(kBlock) leftover_kernel(const int32_t* __restrict__ cur_ids,
                                                          const int32_t* __restrict__ cur_len,
                                                          const int64_t* __restrict__ tok_off,
                                                          const int64_t* __restrict__ off,
                                                          const RankState* __restrict__ ranks, int W, int64_t n,
                                                          const int64_t* __restrict__ loff,
                                                          int32_t* __restrict__ left, DevStatus* st) {
    __shared__ int64_t s_off[kLdsRanks + 1];
    off = stage_ranks(off, W, s_off);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n; p += stride) {
        const int r = rank_of(off, W, p);
        const int64_t q = p - off[r];
        if (q < ranks[r].cnt) {
            const int32_t s = cur_ids[p];
            left[loff[r] + q] = s;
            check_csr_length(s, tok_off[s], tok_off[s + 1], cur_len[p], st);
        }
    }
}

// ---------------------------------------------------------------- coverage
// cnt[v] += 1 for every view id (or its identity) in ids[0, m).
__global__ void __launch_bounds__(kBlock) count_kernel(const int32_t* __restrict__ ids, int64_t m, int64_t n,
                                                       const int64_t* __restrict__ identity, int64_t range,
                                                       int32_t* cnt, DevStatus* st) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        int64_t v = ids[i];
        if (v < 0 || v >= n) {
            atomicOr(&st->err, kErrInternal);
            continue;
        }
        if (identity) v = identity[v];
        if (v < 0 || v >= range) {
            atomicOr(&st->err, kErrIdentity);
            continue;
        }
        atomicAdd(&cnt[v], 1);
    }
}

// bad = #(cnt != 1) (views); missing = #(cnt == 0); dup = sum max(cnt - 1, 0).
__global__ void __launch_bounds__(kBlock) coverage_reduce_kernel(const int32_t* __restrict__ cnt, int64_t m,
                                                                 int want_bad, int want_ids, DevInfo* info) {
    int64_t bad = 0, miss = 0, dup = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const int32_t c = cnt[i];
        bad += c != 1 ? 1 : 0;
        miss += c == 0 ? 1 : 0;
        dup += c > 1 ? c - 1 : 0;
    }
    bad = block_sum(bad);
    miss = block_sum(miss);
    dup = block_sum(dup);
    if (threadIdx.x == 0) {
        if (want_bad && bad) atomicAdd((unsigned long long*)&info->bad_views, (unsigned long long)bad);
        if (want_ids && miss) atomicAdd((unsigned long long*)&info->missing_ids, (unsigned long long)miss);
        if (want_ids && dup) atomicAdd((unsigned long long*)&info->duplicate_ids, (unsigned long long)dup);
    }
}

// Sets bit v of `bits` for every view id v in ids[0, m) (ids outside [0, n) are errors).
__global__ void __launch_bounds__(kBlock) mark_views_kernel(const int32_t* __restrict__ ids, int64_t m, int64_t n,
                                                            uint32_t* bits, DevStatus* st) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += stride) {
        const int32_t v = ids[i];
        if (v < 0 || v >= n) {
            atomicOr(&st->err, kErrInternal);
            continue;
        }
        atomicOr(&bits[v >> 5], 1u << (v & 31));
    }
}

__global__ void __launch_bounds__(kBlock) popcount_kernel(const uint32_t* __restrict__ bits, int64_t words,
                                                          DevInfo* info) {
    int64_t c = 0;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) c += __popc(bits[i]);
    c = block_sum(c);
    if (threadIdx.x == 0 && c) atomicAdd((unsigned long long*)&info->distinct_views, (unsigned long long)c);
}

// Missing and duplicate identities of an identity map over the listed views.
int count_identities(const odb_window_t* w, const Layout& L, void* ws, const int32_t* emit, int64_t ne,
                     const int32_t* left, int64_t nl, hipStream_t s) {
    int32_t* cover = ws_at<int32_t>(ws, L.cover);
    DevStatus* st = ws_at<DevStatus>(ws, L.status);
    const int64_t n = w->num_samples, nid = w->num_identities;
    const int64_t cap = (int64_t)num_cus() * kPlanBlocksPerCU;
    hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(nid, kBlock, cap)), dim3(kBlock), 0, s, cover, nid, 0);
    ODB_LAUNCHED();
    if (ne > 0) {
        hipLaunchKernelGGL(count_kernel, dim3(grid_for(ne, kBlock, cap)), dim3(kBlock), 0, s, emit, ne, n,
                           w->d_identity, nid, cover, st);
        ODB_LAUNCHED();
    }
    if (nl > 0) {
        hipLaunchKernelGGL(count_kernel, dim3(grid_for(nl, kBlock, cap)), dim3(kBlock), 0, s, left, nl, n,
                           w->d_identity, nid, cover, st);
        ODB_LAUNCHED();
    }
    hipLaunchKernelGGL(coverage_reduce_kernel, dim3(grid_for(nid, kBlock, cap)), dim3(kBlock), 0, s,
                       (const int32_t*)cover, nid, 0, 1, ws_at<DevInfo>(ws, L.info));
    ODB_LAUNCHED();
    return ODB_OK;
}

// Coverage (App. C): a bitset over the sampler views proves "every view exactly once"
// when it holds n distinct views and n ids were listed; the exact per-view counters run
// only when it does not (run_coverage_exact).  Identities of an identity map are always
// counted exactly (duplicates are expected there: sampler padding).
int run_coverage(const odb_window_t* w, const Layout& L, void* ws, const int32_t* emitted, int64_t ne,
                 const int32_t* left, int64_t nl, hipStream_t s) {
    const int64_t n = w->num_samples;
    int32_t* cover = ws_at<int32_t>(ws, L.cover);
    DevStatus* st = ws_at<DevStatus>(ws, L.status);
    DevInfo* info = ws_at<DevInfo>(ws, L.info);
    const int64_t cap = (int64_t)num_cus() * kPlanBlocksPerCU;
    if (n > 0) {
        uint32_t* bits = reinterpret_cast<uint32_t*>(cover);
        const int64_t words = (n + 31) / 32;
        hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(words, kBlock, cap)), dim3(kBlock), 0, s, cover, words, 0);
        ODB_LAUNCHED();
        if (ne > 0) {
            hipLaunchKernelGGL(mark_views_kernel, dim3(grid_for(ne, kBlock, cap)), dim3(kBlock), 0, s, emitted, ne, n,
                               bits, st);
            ODB_LAUNCHED();
        }
        if (nl > 0) {
            hipLaunchKernelGGL(mark_views_kernel, dim3(grid_for(nl, kBlock, cap)), dim3(kBlock), 0, s, left, nl, n,
                               bits, st);
            ODB_LAUNCHED();
        }
        hipLaunchKernelGGL(popcount_kernel, dim3(grid_for(words, kBlock, cap)), dim3(kBlock), 0, s,
                           (const uint32_t*)bits, words, info);
        ODB_LAUNCHED();
    }
    // the identity counters reuse the bitset's memory: the popcount above has consumed it
    if (w->d_identity && n > 0) ODB_TRY(count_identities(w, L, ws, emitted, ne, left, nl, s));
    return ODB_OK;
}

// Exact per-view counts: bad_views (and missing / duplicates without an identity map).
// Needed only when the bitset pass found fewer than n distinct views or n != ne + nl.
int run_coverage_exact(const odb_window_t* w, const Layout& L, void* ws, const int32_t* emitted, int64_t ne,
                       const int32_t* left, int64_t nl, hipStream_t s) {
    const int64_t n = w->num_samples;
    int32_t* cover = ws_at<int32_t>(ws, L.cover);
    DevStatus* st = ws_at<DevStatus>(ws, L.status);
    DevInfo* info = ws_at<DevInfo>(ws, L.info);
    const int64_t cap = (int64_t)num_cus() * kPlanBlocksPerCU;
    hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(n, kBlock, cap)), dim3(kBlock), 0, s, cover, n, 0);
    ODB_LAUNCHED();
    if (ne > 0) {
        hipLaunchKernelGGL(count_kernel, dim3(grid_for(ne, kBlock, cap)), dim3(kBlock), 0, s, emitted, ne, n,
                           (const int64_t*)nullptr, n, cover, st);
        ODB_LAUNCHED();
    }
    if (nl > 0) {
        hipLaunchKernelGGL(count_kernel, dim3(grid_for(nl, kBlock, cap)), dim3(kBlock), 0, s, left, nl, n,
                           (const int64_t*)nullptr, n, cover, st);
        ODB_LAUNCHED();
    }
    hipLaunchKernelGGL(coverage_reduce_kernel, dim3(grid_for(n, kBlock, cap)), dim3(kBlock), 0, s,
                       (const int32_t*)cover, n, 1, w->d_identity ? 0 : 1, info);
    ODB_LAUNCHED();
    return ODB_OK;
}

// Coverage of one rank's views, one id chunk per block, in LDS.  The views of rank r are
// its ids [off[r], off[r+1]); they may appear only in rank r's emitted rows
// (emit[row_off[r*S] .. row_off[(r+1)*S])) and leftovers (left[loff[r] .. loff[r+1])).
// Block b covers ids [lo, hi) of one rank: it scans both lists, sets bit v in `once`,
// and in `twice` if it was already set.  missing = (hi - lo) - |once|, views listed
// more than once = |twice|, extra listings = dup.  An id of another rank in these lists
// is an internal error.
constexpr int kCovBlock = 1024;

// The chunk's view of one listed id.  Ids, ranks and chunks stay below 2^31, so the
// range tests are single unsigned compares: (uint32)(x - base) < nr holds exactly for
// base <= x < base + nr, negative x included.
struct CovChunk {
    uint32_t* once;
    uint32_t* twice;
    uint32_t base, nr;  // the rank's views [base, base + nr)
    uint32_t lo, span;  // this chunk's views [lo, lo + span)
    int32_t dup, foreign;
    int first;          // chunk 0 of its rank counts the foreign ids

    __device__ __forceinline__ void add(int32_t x) {
        if ((uint32_t)x - base >= nr) {
            foreign += first;
            return;
        }
        const uint32_t d = (uint32_t)x - lo;
        if (d >= span) return;
        const uint32_t bit = 1u << (d & 31);
        if (atomicOr(&once[d >> 5], bit) & bit) {
            atomicOr(&twice[d >> 5], bit);
            dup += 1;
        }
    }
};

typedef int v4i_cov __attribute__((ext_vector_type(4)));

// Feeds ids[a, b) to the chunk: a scalar head up to the first 16-byte aligned address,
// two 16-byte loads per thread and iteration, a scalar tail.
__device__ __forceinline__ void cov_scan(CovChunk& c, const int32_t* __restrict__ ids, int64_t a, int64_t b) {
    if (b <= a) return;
    int64_t a4 = a + ((4 - ((reinterpret_cast<uintptr_t>(ids + a) >> 2) & 3)) & 3);
    if (a4 > b) a4 = b;
    const int64_t b4 = a4 + ((b - a4) & ~(int64_t)3);
    if (a + threadIdx.x < a4) c.add(ids[a + threadIdx.x]);
    if (b4 + threadIdx.x < b) c.add(ids[b4 + threadIdx.x]);
    const v4i_cov* v = reinterpret_cast<const v4i_cov*>(ids + a4);
    const int32_t nv = (int32_t)((b4 - a4) >> 2);
    for (int32_t q = threadIdx.x; q < nv; q += 2 * kCovBlock) {
        const v4i_cov x = __builtin_nontemporal_load(v + q);
        const bool two = q + kCovBlock < nv;
        const v4i_cov y = __builtin_nontemporal_load(v + (two ? q + kCovBlock : q));
#pragma unroll
        for (int k = 0; k < 4; ++k) c.add(x[k]);
        if (two) {
#pragma unroll
            for (int k = 0; k < 4; ++k) c.add(y[k]);
        }
    }
}

__global__ void __launch_bounds__(kCovBlock) coverage_lds_kernel(
    const int64_t* __restrict__ off, int W, const int64_t* __restrict__ chunk_first, int64_t C,
    const int32_t* __restrict__ emit, const int64_t* __restrict__ row_off, int64_t S,
    const int32_t* __restrict__ left, const int64_t* __restrict__ loff, int want_ids, DevInfo* info,
    DevStatus* st) {
    extern __shared__ uint32_t lds[];
    const int64_t words = C / 32;
    const int64_t b = blockIdx.x;
    const int r = rank_of(chunk_first, W, b);
    const int64_t j = b - chunk_first[r];
    const int64_t base = off[r], end = off[r + 1];
    const int64_t lo = base + j * C;
    const int64_t hi = lo + C < end ? lo + C : end;
    CovChunk c{lds, lds + words, (uint32_t)base, (uint32_t)(end - base), (uint32_t)lo, (uint32_t)(hi - lo), 0, 0,
               j == 0 ? 1 : 0};
    for (int64_t i = threadIdx.x; i < 2 * words; i += kCovBlock) lds[i] = 0;
    __syncthreads();
    cov_scan(c, emit, row_off[(int64_t)r * S], row_off[(int64_t)(r + 1) * S]);
    cov_scan(c, left, loff[r], loff[r + 1]);
    __syncthreads();
    int32_t distinct = 0, multi = 0;
    const int32_t nw = (int32_t)((hi - lo + 31) / 32);
    for (int32_t i = threadIdx.x; i < nw; i += kCovBlock) {
        distinct += __popc(c.once[i]);
        multi += __popc(c.twice[i]);
    }
    // block sums of the four counters: per-wave partials in LDS, summed by wave 0
    __shared__ int64_t part[kCovBlock / kWave][4];
    const int64_t v0 = wave_sum((int64_t)distinct), v1 = wave_sum((int64_t)multi);
    const int64_t v2 = wave_sum((int64_t)c.dup), v3 = wave_sum((int64_t)c.foreign);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        int64_t* q = part[threadIdx.x / kWave];
        q[0] = v0;
        q[1] = v1;
        q[2] = v2;
        q[3] = v3;
    }
    __syncthreads();
    if (threadIdx.x < kWave) {
        const int i = threadIdx.x;
        const bool has = i < kCovBlock / kWave;
        const int64_t d_sum = wave_sum(has ? part[i][0] : (int64_t)0);
        const int64_t m_sum = wave_sum(has ? part[i][1] : (int64_t)0);
        const int64_t dup = wave_sum(has ? part[i][2] : (int64_t)0);
        const int64_t foreign = wave_sum(has ? part[i][3] : (int64_t)0);
        if (i != 0) return;
        const int64_t missing = (hi - lo) - d_sum;
        const int64_t bad = missing + m_sum;
        if (bad) atomicAdd((unsigned long long*)&info->bad_views, (unsigned long long)bad);
        if (want_ids && missing) atomicAdd((unsigned long long*)&info->missing_ids, (unsigned long long)missing);
        if (want_ids && dup) atomicAdd((unsigned long long*)&info->duplicate_ids, (unsigned long long)dup);
        if (foreign) atomicOr(&st->err, kErrInternal);
    }
}

// The plan's totals (padded elements, emitted rows, pad fraction) and the coverage chunks:
// chunk_first[r] = sum_{r' < r} ceil(n_r' / C).  One block.
__global__ void __launch_bounds__(kBlock) finish_plan_kernel(const int64_t* __restrict__ row_off,
                                                             const int64_t* __restrict__ tile_off, int64_t K,
                                                             DevInfo* info, const int64_t* __restrict__ off, int W,
                                                             int64_t C, int64_t* __restrict__ chunk_first) {
    __shared__ int64_t carry;
    if (threadIdx.x == 0) {
        carry = 0;
        info->padded_elems = K > 0 ? tile_off[K] : 0;
        info->emitted = K > 0 ? row_off[K] : 0;
        info->pad_fraction =
            info->padded_elems > 0 ? 1.0 - (double)info->real_tokens / (double)info->padded_elems : 0.0;
    }
    __syncthreads();
    for (int b = 0; b < W; b += kBlock) {
        const int r = b + threadIdx.x;
        const int64_t v = r < W ? (off[r + 1] - off[r] + C - 1) / C : 0;
        int64_t tot;
        const int64_t ex = block_excl_sum(v, &tot);
        const int64_t c = carry;
        if (r < W) chunk_first[r] = c + ex;
        __syncthreads();
        if (threadIdx.x == 0) carry = c + tot;
        __syncthreads();
    }
    if (threadIdx.x == 0) chunk_first[W] = carry;
}

// Coverage of an aligned plan: per-rank LDS bitsets for the views, global counters for
// the identities of an identity map.
int run_plan_coverage(const odb_window_t* w, const Layout& L, void* ws, const int32_t* emit,
                      const int64_t* row_off, const int64_t* tile_off, int64_t S, const int32_t* left,
                      const int64_t* loff, int64_t ne, int64_t nl, hipStream_t s) {
    const int W = w->num_ranks;
    const int64_t n = w->num_samples;
    int64_t max_nr = 0, chunks = 0;
    for (int r = 0; r < W; ++r) {
        const int64_t nr = w->rank_offsets[r + 1] - w->rank_offsets[r];
        max_nr = nr > max_nr ? nr : max_nr;
    }
    // one chunk per rank up to 131072 views (two 16 KB bitsets); larger ranks are split
    int64_t C = ((max_nr + 4095) / 4096) * 4096;
    C = C < 4096 ? 4096 : (C > 131072 ? 131072 : C);
    for (int r = 0; r < W; ++r) chunks += (w->rank_offsets[r + 1] - w->rank_offsets[r] + C - 1) / C;
    int64_t* chunk_first = ws_at<int64_t>(ws, L.tile_first);
    const int64_t* d_off = ws_at<int64_t>(ws, L.rank_off);
    hipLaunchKernelGGL(finish_plan_kernel, dim3(1), dim3(kBlock), 0, s, row_off, tile_off, (int64_t)W * S,
                       ws_at<DevInfo>(ws, L.info), d_off, W, C, chunk_first);
    ODB_LAUNCHED();
    if (n == 0) return ODB_OK;
    hipLaunchKernelGGL(coverage_lds_kernel, dim3((unsigned)chunks), dim3(kCovBlock), (size_t)(C / 4), s, d_off, W,
                       (const int64_t*)chunk_first, C, emit, row_off, S, left, loff, w->d_identity ? 0 : 1,
                       ws_at<DevInfo>(ws, L.info), ws_at<DevStatus>(ws, L.status));
    ODB_LAUNCHED();
    if (w->d_identity) ODB_TRY(count_identities(w, L, ws, emit, ne, left, nl, s));
    return ODB_OK;
}

// Reads the coverage counters after run_coverage; runs the exact view count when the
// bitset pass did not prove that every view was listed exactly once.
int finish_coverage(const odb_window_t* w, const Layout& L, void* ws, const int32_t* emitted, int64_t ne,
                    const int32_t* left, int64_t nl, DevInfo* hi, hipStream_t s) {
    const int64_t n = w->num_samples;
    if (hi->distinct_views == n && ne + nl == n) {
        hi->bad_views = 0;
        if (!w->d_identity) {
            hi->missing_ids = 0;
            hi->duplicate_ids = 0;
        }
        return ODB_OK;
    }
    DevInfo* info = ws_at<DevInfo>(ws, L.info);
    hipLaunchKernelGGL(clear_view_counters_kernel, dim3(1), dim3(64), 0, s, info, w->d_identity ? 0 : 1);
    ODB_LAUNCHED();
    ODB_TRY(run_coverage_exact(w, L, ws, emitted, ne, left, nl, s));
    ODB_TRY(read_device(hi, info, sizeof(*hi), s));
    return ODB_OK;
}

// ---------------------------------------------------------------- windows aligned in one round
// Without overflow (T = the largest group count: no active rank buffers fewer samples and
// no smaller positive capacity) the first round empties every buffer.  A rank's emitted rows
// are then its formation order reversed, whatever the split, and everything else has a
// closed form: the singletons of a split end at X = k + j*, where j* is the first group with
// start(j* + 1) - (j* + 1) >= k = T - G (the surplus of groups 0 .. j* is their samples less
// their number).  Five launches in place of a round's nine and the final plan's seven:
//
//   rows_kernel       checks the stage-1 arrays, records the group starts and writes every
//                     rank's reversed order with its row records
//   rank_tiles_kernel tokens before every tile of a rank
//   cut_steps_kernel, cut_kernel (sample quota only)
//                     step sizes, the first step that reaches the quota, each rank's share
//   slots_kernel      T, and rows, longest length, tokens and row offset of every slot
//   tiles_kernel      tile offsets, the largest step, the totals
//   share_kernel      (sample quota only) rows and left-overs moved to their final place
//
// S is known on the device only, so slots_kernel and tiles_kernel run a grid that does not
// depend on it: block b takes the b-th of gridDim.x equal ranges of slots, and the ranges'
// sums are scanned by every block of the second launch.
//
// The stage-1 check also proves coverage: a rank's order holds ids of the rank only, strictly
// ordered by (length desc, id asc) under lengths that equal each id's CSR length, so no id
// comes twice, and it has as many places as the rank has ids.
struct OneArgs {
    int W;
    int64_t n;
    int nonjoin;
    int64_t quota;
    int64_t slot_capacity;
    const int64_t* tok_off;
    const int64_t* off;        // [W + 1] rank offsets
    const int32_t* order;
    const int32_t* slen;
    const int32_t* gidx;
    const int32_t* groups;     // [W] G_r
    int32_t* gs;               // [n] rank-local start of group g of rank r at off[r] + g
    int64_t* gpre;             // [n] tokens before that start within its tile of the rank
    int64_t* tpre;             // [W * per_rank] tokens of each of the rank's tiles, or before it
    int per_rank;              // tiles (kRowTile positions) of the largest rank
    int64_t min_nr;            // samples of the smallest rank that has any
    int64_t* lo;               // [W + 1] first row of every rank (the rank offsets in join mode)
    int64_t* steps;            // [max n_r] samples per step (sample quota only)
    I64Pair* part;             // [gridDim.x] (padded elements, real tokens) per range of slots
    RoundState* rs;
    DevInfo* info;
    DevStatus* st;
    // rows: the final arrays in join mode, else staged at the rank's own positions
    int32_t* emit;
    int32_t* len;
    int64_t* ts;               // may be null
};

constexpr int kRowItems = 4;                       // consecutive positions per thread
constexpr int64_t kRowTile = kBlock * kRowItems;   // positions of one rank per block
constexpr int kMaxRanges = 1024;                   // blocks of slots_kernel / tiles_kernel
typedef int32_t I4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int64_t L2 __attribute__((ext_vector_type(2), aligned(8)));

// Group counts a rank may have: 0 exactly for an empty rank, at most its samples.
__device__ __forceinline__ bool groups_ok(int64_t G, int64_t cnt) {
    return G >= 0 && G <= cnt && ((cnt == 0) == (G == 0));
}

// Blocks `per_rank` tiles of every rank.  With xcd set, rank r's blocks run on XCD r mod 8
// (blocks are dealt to the XCDs round robin), whose L2 then holds the rank's CSR offsets for
// the random reads: 16.7 M rows of 64 ranks gather from 134 MB of offsets.
//
// Bound by those reads (one 16-byte load per row, each in its own cache line) and, beside
// them, 12 B read and 16 B written per row in 16-byte accesses.  64 x 262,144 rows: 0.58 ms as
// five kernels (check, length prefix, emit, row records, coverage), 0.19 ms here (0.08 ms of it the
// streams; the 16.7 M reads fill a 128-byte line of the first-level cache each, 64 B a clock).
__global__ void __launch_bounds__(kBlock) rows_kernel(OneArgs a, int xcd) {
    const int64_t b = blockIdx.x;
    int r;
    int64_t tile;
    if (xcd) {
        const int64_t g = b / kXcds;
        r = (int)(g / a.per_rank) * kXcds + (int)(b % kXcds);
        tile = g % a.per_rank;
    } else {
        r = (int)(b / a.per_rank);
        tile = b % a.per_rank;
    }
    if (b == 0) {   // ranks without samples have no block of their own
        for (int k = threadIdx.x; k < a.W; k += kBlock) {
            if (!groups_ok(a.groups[k], a.off[k + 1] - a.off[k])) atomicOr(&a.st->err, kErrGroupIndex);
            if (a.groups[k] > a.min_nr) a.rs->overflowed = 1;
        }
    }
    if (r >= a.W) return;
    const int64_t base = a.off[r], nr = a.off[r + 1] - base;
    if (tile * kRowTile >= nr) return;
    const int64_t q0 = tile * kRowTile + (int64_t)threadIdx.x * kRowItems;
    if (a.groups[r] > a.min_nr) return;   // this rank overflows: the window goes round by round
    const int64_t G = groups_ok(a.groups[r], nr) ? a.groups[r] : 0;
    const int64_t p0 = base + q0;
    const int m = nr - q0 < kRowItems ? (int)(nr - q0) : kRowItems;   // live positions, <= 0 past the rank
    int32_t id[kRowItems], l[kRowItems], g[kRowItems];
    if (m == kRowItems) {
        // streamed past the caches, which hold the offsets
        const I4 x = __builtin_nontemporal_load(reinterpret_cast<const I4*>(a.order + p0));
        const I4 y = __builtin_nontemporal_load(reinterpret_cast<const I4*>(a.slen + p0));
        const I4 z = __builtin_nontemporal_load(reinterpret_cast<const I4*>(a.gidx + p0));
#pragma unroll
        for (int i = 0; i < kRowItems; ++i) {
            id[i] = x[i];
            l[i] = y[i];
            g[i] = z[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < kRowItems; ++i) {
            const int64_t p = i < m ? p0 + i : base;
            id[i] = a.order[p];
            l[i] = a.slen[p];
            g[i] = a.gidx[p];
        }
    }
    // the position before the thread's first: the lane below's last (full by then), or a load
    int32_t pid = ::__shfl_up(id[kRowItems - 1], 1, kWave), pl = ::__shfl_up(l[kRowItems - 1], 1, kWave),
            pg = ::__shfl_up(g[kRowItems - 1], 1, kWave);
    if ((threadIdx.x & (kWave - 1)) == 0 && q0 > 0 && m > 0) {
        pid = a.order[p0 - 1];
        pl = a.slen[p0 - 1];
        pg = a.gidx[p0 - 1];
    }
    int64_t t0[kRowItems], t1[kRowItems];
#pragma unroll
    for (int i = 0; i < kRowItems; ++i) {
        const bool in = id[i] >= base && id[i] < base + nr;
        const L2 o = *reinterpret_cast<const L2*>(a.tok_off + (in ? (int64_t)id[i] : base));
        t0[i] = o[0];
        t1[i] = o[1];
    }
    // tokens of the tile before each position
    int64_t pre;
    {
        int64_t sum = 0, tot;
#pragma unroll
        for (int i = 0; i < kRowItems; ++i) sum += i < m ? l[i] : 0;
        const int64_t inc = wave_scan_dpp<OpAdd>(sum);
        __shared__ int64_t s_w[kBlock / kWave];
        const int w = threadIdx.x / kWave;
        if ((threadIdx.x & (kWave - 1)) == kWave - 1) s_w[w] = inc;
        __syncthreads();
        pre = inc - sum;
        tot = 0;
#pragma unroll
        for (int i = 0; i < kBlock / kWave; ++i) {
            pre += i < w ? s_w[i] : 0;
            tot += s_w[i];
        }
        if (threadIdx.x == 0) a.tpre[(int64_t)r * a.per_rank + tile] = tot;   // rank_tiles_kernel: prefix
    }
    if (m <= 0) return;
    bool bad_order = false, bad_group = false;
    int64_t first = LLONG_MAX;
#pragma unroll
    for (int i = 0; i < kRowItems; ++i) {
        if (i < m) {
            const int64_t q = q0 + i;
            const bool in = id[i] >= base && id[i] < base + nr;
            bool ok = in && l[i] >= 1;
            bool gok = g[i] >= 0 && g[i] < G;
            if (q == 0) {
                gok = gok && g[i] == 0;
            } else {
                ok = ok && (pl > l[i] || (pl == l[i] && pid < id[i]));
                const int32_t d = g[i] - pg;
                gok = gok && (d == 0 || d == 1);
            }
            if (q == nr - 1) gok = gok && g[i] == G - 1;
            if (gok && (q == 0 || g[i] != pg)) {
                a.gs[base + g[i]] = (int32_t)q;
                a.gpre[base + g[i]] = pre;
            }
            if (!ok || !gok) {
                bad_order |= !ok;
                bad_group |= !gok;
                first = first < base + q ? first : base + q;
            }
            if (in) {
                const int64_t w = t1[i] - t0[i];
                if (w < 1 || w > INT_MAX || t0[i] < 0) {
                    atomicOr(&a.st->err, kErrLength);
                    atomicMin((unsigned long long*)&a.st->first_bad_len, (unsigned long long)id[i]);
                } else if (w != (int64_t)l[i]) {
                    atomicOr(&a.st->err, kErrSortedLen);
                    atomicMin((unsigned long long*)&a.st->first_bad_csr, (unsigned long long)id[i]);
                }
            }
        }
        pre += l[i];
        pid = id[i];
        pl = l[i];
        pg = g[i];
    }
    if (bad_order || bad_group) {
        atomicOr(&a.st->err, (bad_order ? kErrOrder : 0) | (bad_group ? kErrGroupIndex : 0));
        atomicMin((unsigned long long*)&a.st->first_bad, (unsigned long long)first);
    }
    // position q goes to row nr - 1 - q of the rank
    const int64_t o = base + nr - q0 - m;
    if (m == kRowItems) {
        __builtin_nontemporal_store(I4{id[3], id[2], id[1], id[0]}, reinterpret_cast<I4*>(a.emit + o));
        __builtin_nontemporal_store(I4{l[3], l[2], l[1], l[0]}, reinterpret_cast<I4*>(a.len + o));
        if (a.ts) {
            __builtin_nontemporal_store(L2{t0[3], t0[2]}, reinterpret_cast<L2*>(a.ts + o));
            __builtin_nontemporal_store(L2{t0[1], t0[0]}, reinterpret_cast<L2*>(a.ts + o + 2));
        }
    } else {
#pragma unroll
        for (int i = 0; i < kRowItems; ++i) {
            if (i >= m) break;
            a.emit[o + m - 1 - i] = id[i];
            a.len[o + m - 1 - i] = l[i];
            if (a.ts) a.ts[o + m - 1 - i] = t0[i];
        }
    }
}

// Ranks of at most this many tiles leave tpre as the tiles' own tokens: a slot sums the few it
// needs, which saves the launch that turns them into prefixes.
constexpr int kTilesSummed = 16;

// One block per rank: the tokens of the rank's tiles become the tokens before each tile.
__global__ void __launch_bounds__(kBlock) rank_tiles_kernel(OneArgs a) {
    if (a.rs->overflowed) return;
    const int r = blockIdx.x;
    const int64_t tiles = (a.off[r + 1] - a.off[r] + kRowTile - 1) / kRowTile;
    int64_t* t = a.tpre + (int64_t)r * a.per_rank;
    int64_t carry = 0;
    for (int64_t b = 0; b < tiles; b += kBlock) {
        const int64_t i = b + threadIdx.x;
        const int64_t v = i < tiles ? t[i] : 0;
        int64_t tot;
        const int64_t ex = block_excl_sum(v, &tot);
        if (i < tiles) t[i] = carry + ex;
        carry += tot;
    }
}

// The target over the active ranks, and whether a rank would overflow (Eq. 3's S+_min below
// the largest group count).  Block-uniform.
struct OneTarget {
    int64_t T;
    bool overflow;
};

__device__ __forceinline__ OneTarget one_target(const OneArgs& a) {
    int64_t mx = 0;
    for (int r = threadIdx.x; r < a.W; r += blockDim.x) mx = a.groups[r] > mx ? a.groups[r] : mx;
    __shared__ int64_t s_mx[kBlock / kWave];
    mx = wave_last(wave_scan_dpp<OpMax>(mx));
    if ((threadIdx.x & (kWave - 1)) == 0) s_mx[threadIdx.x / kWave] = mx;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kBlock / kWave; ++i) mx = s_mx[i] > mx ? s_mx[i] : mx;
    __syncthreads();
    return OneTarget{mx > 1 ? mx : 1, mx > a.min_nr};
}

// Where a rank of G > 0 groups (starts gs[0 .. G)) aligned to T >= G is split: adjusted groups
// [0, X) are singletons, the X-th ends with group j*; X = -1 without a split.
struct OneSplit {
    int64_t js, X;
};

__device__ __forceinline__ OneSplit one_split(const int32_t* __restrict__ gs, int64_t G, int64_t T) {
    const int64_t k = T - G;
    if (k <= 0) return OneSplit{0, -1};
    int64_t lo = -1, hi = G - 1;   // surplus(lo) < k <= surplus(hi) = cnt - G
    while (hi - lo > 1) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)gs[mid + 1] - (mid + 1) >= k) hi = mid; else lo = mid;
    }
    return OneSplit{hi, k + hi};
}

// The same for a rank that a whole wave asks for: 64 places at a time, so 1,000 groups take two
// trips to memory, not ten.
__device__ __forceinline__ OneSplit wave_split(const int32_t* __restrict__ gs, int64_t G, int64_t T) {
    const int64_t k = T - G;
    if (k <= 0) return OneSplit{0, -1};
    const int lane = threadIdx.x & (kWave - 1);
    int64_t lo = -1, hi = G - 1;
    while (hi - lo > 1) {
        const int64_t w = (hi - lo + kWave) / (kWave + 1), x = lo + (lane + 1) * w;
        const bool low = x < hi && (int64_t)gs[(x < hi ? x : lo) + 1] - (x + 1) < k;
        const int64_t c = __popcll(__ballot(low));
        const int64_t end = lo + (c + 1) * w;
        lo += c * w;
        hi = end < hi ? end : hi;
    }
    return OneSplit{hi, k + hi};
}

// Positions [*a0, *a1) of adjusted group t of a rank with cnt > 0 samples in G groups (starts
// gs[0 .. G)), split at sp.  Returns the formation group they are, or -1 for a piece of one (a
// split's singletons and what is left of group j*).
__device__ __forceinline__ int64_t one_group(const int32_t* __restrict__ gs, int64_t G, int64_t cnt, OneSplit sp,
                                             int64_t t, int64_t* a0, int64_t* a1) {
    if (t < sp.X) {
        *a0 = t;
        *a1 = t + 1;
        return -1;
    }
    const int64_t g = sp.X >= 0 ? sp.js + (t - sp.X) : t;
    *a0 = t == sp.X ? sp.X : (int64_t)gs[g];
    *a1 = g + 1 < G ? (int64_t)gs[g + 1] : cnt;
    return t == sp.X ? -1 : g;
}

// Samples per step over the ranks, for the sample quota: a block takes 64 steps, its waves
// every fourth rank.  Bound by the trips to memory of a rank's search for its split (16 x 65,536
// samples: 12.7 us lane by lane, 7.8 by the whole wave; for the slots below, whose waves may
// hold several ranks, it gains nothing).  Beyond kCutSlice ranks, blockIdx.y takes a slice of them
// and adds to the steps, cleared before: the one block of the few steps of 8,192 ranks x 100 samples went
// through all of them, 2.2 ms (the quota plan 3.2 ms, now 0.88; 1,024 x 1,000 samples 500 and 214 us, 96 x
// 4,000 121 and 110, 65 x 16,384 168 and 169).
constexpr int kCutSlice = 64;

__global__ void __launch_bounds__(kBlock) cut_steps_kernel(OneArgs a) {
    if (stage1_bad(a.st)) return;
    const OneTarget tg = one_target(a);
    if (tg.overflow) return;
    __shared__ int64_t s_n[kBlock / kWave][kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int r0 = blockIdx.y * kCutSlice;
    const int r1 = gridDim.y > 1 && r0 + kCutSlice < a.W ? r0 + kCutSlice : a.W;
    for (int64_t j0 = (int64_t)blockIdx.x * kWave; j0 < tg.T; j0 += (int64_t)gridDim.x * kWave) {
        const int64_t j = j0 + lane;
        int64_t n = 0;
        for (int r = r0 + w; r < r1; r += kBlock / kWave) {
            const int64_t cnt = a.off[r + 1] - a.off[r];
            if (cnt == 0) continue;
            const int32_t* gs = a.gs + a.off[r];
            const OneSplit sp = wave_split(gs, a.groups[r], tg.T);
            int64_t a0 = 0, a1 = 0;
            if (j < tg.T) one_group(gs, a.groups[r], cnt, sp, tg.T - 1 - j, &a0, &a1);
            n += a1 - a0;
        }
        s_n[w][lane] = n;
        __syncthreads();
        if (w == 0 && j < tg.T) {
#pragma unroll
            for (int i = 1; i < kBlock / kWave; ++i) n += s_n[i][lane];
            if (gridDim.y > 1)
                atomicAdd((unsigned long long*)&a.steps[j], (unsigned long long)n);
            else
                a.steps[j] = n;
        }
        __syncthreads();
    }
}

int cut_steps(const OneArgs& a, int64_t max_nr, hipStream_t s) {
    const int64_t slices = (a.W + kCutSlice - 1) / kCutSlice;
    if (slices > 1) {   // no more steps than samples of a rank
        hipLaunchKernelGGL(fill_i32_kernel, dim3(grid_for(2 * max_nr, kBlock, kMaxRanges)), dim3(kBlock), 0, s,
                           reinterpret_cast<int32_t*>(a.steps), 2 * max_nr, 0);
        ODB_LAUNCHED();
    }
    // at most 65,535 slices a launch; more ranks than those hold go in one
    hipLaunchKernelGGL(cut_steps_kernel, dim3(grid_for(max_nr, kWave, kMaxRanges), slices <= 65535 ? (unsigned)slices : 1u),
                       dim3(kBlock), 0, s, a);
    ODB_LAUNCHED();
    return ODB_OK;
}

// The first step at which the emitted samples reach the quota, every rank's emitted rows
// (lo: running sum over the ranks) and left-overs.  One block.
__global__ void __launch_bounds__(kBlock) cut_kernel(OneArgs a, int64_t* __restrict__ left_off) {
    if (stage1_bad(a.st)) return;
    const OneTarget tg = one_target(a);
    if (tg.overflow) return;
    __shared__ int64_t s_cut;
    if (threadIdx.x == 0) s_cut = tg.T;
    __syncthreads();
    int64_t carry = 0;
    for (int64_t b = 0; b < tg.T; b += kBlock) {
        const int64_t j = b + threadIdx.x;
        const int64_t v = j < tg.T ? a.steps[j] : 0;
        int64_t tot;
        const int64_t ex = carry + block_excl_sum(v, &tot);
        if (j < tg.T && ex < a.quota && ex + v >= a.quota) s_cut = j + 1;
        carry += tot;
        if (carry >= a.quota) break;   // uniform
    }
    __syncthreads();
    const int64_t cut = s_cut;
    I64Pair at{0, 0};
    for (int b = 0; b < a.W; b += kBlock) {
        const int r = b + threadIdx.x;
        I64Pair v{0, 0};
        if (r < a.W) {
            const int64_t cnt = a.off[r + 1] - a.off[r];
            int64_t q = 0, e;   // formation positions that stay
            if (cut < tg.T && cnt > 0) {
                const int32_t* gs = a.gs + a.off[r];
                one_group(gs, a.groups[r], cnt, one_split(gs, a.groups[r], tg.T), tg.T - cut, &q, &e);
            }
            v = I64Pair{cnt - q, q};
        }
        I64Pair tot;
        const I64Pair ex = block_excl_sum(v, &tot);
        if (r < a.W) {
            a.lo[r] = at.a + ex.a;
            left_off[r] = at.b + ex.b;
        }
        at += tot;
    }
    if (threadIdx.x == 0) {
        a.lo[a.W] = at.a;
        left_off[a.W] = at.b;
        a.rs->cut = cut;
        a.rs->quota_hit = at.a >= a.quota ? 1 : 0;
    }
}

// Rows, longest length, tokens and row offset of every slot, one thread each.  A slot that is
// a whole group takes its tokens from the prefixes at its start and at the next group's; a
// piece of a split group longer than one row (one slot of a split rank) is summed by its
// wave.  (Summing every slot's lengths, 64 lanes a slot, took 229 us on 64 x 262,144 samples:
// the first slots of a rank hold thousands of its shortest samples, so a few waves read
// half the lengths.)
__global__ void __launch_bounds__(kBlock) slots_kernel(OneArgs a, int32_t* __restrict__ rows,
                                                       int32_t* __restrict__ maxlen, int64_t* __restrict__ row_off,
                                                       int64_t* __restrict__ tokens, double* __restrict__ approx) {
#pragma clang fp contract(off)
    if (stage1_bad(a.st)) return;
    const OneTarget tg = one_target(a);
    const int64_t S = a.nonjoin && !tg.overflow ? a.rs->cut : tg.T;
    const int64_t K = (int64_t)a.W * S;
    if (blockIdx.x == 0) {
        int64_t splits = 0, changed = 0;
        for (int r = threadIdx.x; r < a.W; r += kBlock) {
            const int64_t G = a.groups[r];
            if (G <= 0) continue;
            splits += tg.T - G;
            changed += G != tg.T;
        }
        splits = block_sum(splits);
        changed = block_sum(changed);
        if (threadIdx.x == 0) {
            a.rs->T = tg.T;
            a.rs->overflowed = tg.overflow ? 1 : 0;   // the host goes round by round
            a.rs->splits = splits;
            a.rs->second_gather = changed > 0 ? 1 : 0;
            if (!a.nonjoin) a.rs->cut = S;
        }
    }
    if (tg.overflow || K > a.slot_capacity) return;
    const int64_t per = (K + gridDim.x - 1) / gridDim.x;
    const int64_t k0 = (int64_t)blockIdx.x * per, k1 = k0 + per < K ? k0 + per : K;
    const int lane = threadIdx.x & (kWave - 1);
    int64_t cells = 0, real = 0;
    for (int64_t b = k0; b < k1; b += kBlock) {   // uniform
        const int64_t k = b + threadIdx.x;
        const bool on = k < k1;
        int64_t a0 = 0, a1 = 0, base = 0, cnt = 0, sum = 0;
        int32_t ml = 0;
        int r = 0;
        bool piece = false;
        if (on) {
            r = (int)(k / S);
            base = a.off[r];
            cnt = a.off[r + 1] - base;
        }
        if (on && cnt > 0) {
            const int64_t G = a.groups[r];
            const OneSplit sp = one_split(a.gs + base, G, tg.T);
            const int64_t g = one_group(a.gs + base, G, cnt, sp, tg.T - 1 - (k - (int64_t)r * S), &a0, &a1);
            ml = a.slen[base + a0];
            const int64_t* tp = a.tpre + (int64_t)r * a.per_rank;
            if (g >= 0) {
                if (a1 < cnt)
                    sum = a.gpre[base + g + 1] - a.gpre[base + g];
                else
                    sum = a.tok_off[base + cnt] - a.tok_off[base] - a.gpre[base + g];
                const int x0 = (int)(a0 / kRowTile), x1 = a1 < cnt ? (int)(a1 / kRowTile) : 0;
                if (a.per_rank > kTilesSummed) {
                    sum += (a1 < cnt ? tp[x1] : 0) - tp[x0];
                } else if (a1 < cnt) {
                    for (int i = x0; i < x1; ++i) sum += tp[i];
                } else {
                    for (int i = 0; i < x0; ++i) sum -= tp[i];
                }
            } else if (a1 - a0 == 1) {
                sum = ml;
            } else {
                piece = true;
            }
        }
        uint64_t need = __ballot(piece);
        while (need) {   // uniform in the wave
            const int src = __builtin_ctzll(need);
            need &= need - 1;
            const int64_t from = ::__shfl(base + a0, src, kWave), to = ::__shfl(base + a1, src, kWave);
            int64_t part = 0;
            for (int64_t q = from + lane; q < to; q += kWave) part += a.slen[q];
            part = wave_last(wave_scan_dpp<OpAdd>(part));
            if (lane == src) sum = part;
        }
        if (on) {
            rows[k] = (int32_t)(a1 - a0);
            maxlen[k] = ml;
            tokens[k] = sum;
            row_off[k] = a.lo[r] + (cnt - a1);
            if (approx) {
                double v = 0.0;
                if (cnt > 0) {
                    const double mean = (double)(a.tok_off[base + cnt] - a.tok_off[base]) / (double)cnt;
                    v = (double)(a1 - a0) * mean;
                }
                approx[k] = v;
            }
            cells += (a1 - a0) * ml;
            real += sum;
        }
    }
    cells = block_sum(cells);
    real = block_sum(real);
    if (threadIdx.x == 0) a.part[blockIdx.x] = I64Pair{cells, real};
}

// Tile offsets of a range of slots after the ranges before it; the largest step; the totals
// and, in join mode, the (empty) left-over offsets.
__global__ void __launch_bounds__(kBlock) tiles_kernel(OneArgs a, const int32_t* __restrict__ rows,
                                                       const int32_t* __restrict__ maxlen,
                                                       int64_t* __restrict__ row_off, int64_t* __restrict__ tile_off,
                                                       int64_t* __restrict__ left_off) {
    if (stage1_bad(a.st) || a.rs->overflowed) return;
    const int64_t S = a.rs->cut, K = (int64_t)a.W * S;
    if (K > a.slot_capacity) return;
    const int64_t per = (K + gridDim.x - 1) / gridDim.x;
    const int64_t k0 = (int64_t)blockIdx.x * per, k1 = k0 + per < K ? k0 + per : K;
    // the ranges before this block's, and all of them
    I64Pair before{0, 0}, all{0, 0};
    for (unsigned i = threadIdx.x; i < gridDim.x; i += kBlock) {
        const I64Pair p = a.part[i];
        all += p;
        if (i < blockIdx.x) before += p;
    }
    before.a = block_sum(before.a);
    all.a = block_sum(all.a);
    all.b = block_sum(all.b);
    int64_t carry = before.a;
    for (int64_t b = k0; b < k1; b += kBlock) {
        const int64_t k = b + threadIdx.x;
        const int64_t v = k < k1 ? (int64_t)rows[k] * maxlen[k] : 0;
        int64_t tot;
        const int64_t ex = block_excl_sum(v, &tot);
        if (k < k1) tile_off[k] = carry + ex;
        carry += tot;
    }
    if (blockIdx.x == 0) {
        const int64_t emitted = a.lo[a.W];
        if (!a.nonjoin)
            for (int r = threadIdx.x; r <= a.W; r += kBlock) left_off[r] = 0;
        if (threadIdx.x == 0) {
            tile_off[K] = all.a;
            row_off[K] = emitted;
            a.rs->emitted_total = emitted;
            a.info->emitted = emitted;
            a.info->padded_elems = all.a;
            a.info->real_tokens = all.b;
            a.info->pad_fraction = all.a > 0 ? 1.0 - (double)all.b / (double)all.a : 0.0;
        }
    }
    // 64 steps at a time, a wave taking every fourth rank
    __shared__ int64_t s_n[kBlock / kWave][kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    int64_t mx = 0;
    for (int64_t j0 = (int64_t)blockIdx.x * kWave; j0 < S; j0 += (int64_t)gridDim.x * kWave) {
        const int64_t j = j0 + lane;
        int64_t n = 0;
        if (j < S) {
#pragma unroll 8
            for (int r = w; r < a.W; r += kBlock / kWave) n += rows[(int64_t)r * S + j];
        }
        s_n[w][lane] = n;
        __syncthreads();
        if (w == 0) {
#pragma unroll
            for (int i = 1; i < kBlock / kWave; ++i) n += s_n[i][lane];
            mx = n > mx ? n : mx;
        }
        __syncthreads();
    }
    if (w == 0) {
        mx = wave_last(wave_scan_dpp<OpMax>(mx));
        if (lane == 0 && mx) atomicMax((unsigned long long*)&a.rs->step_max, (unsigned long long)mx);
    }
}

// Sample quota: the staged rows of rank r up to its share go to lo[r] on, its first formation
// positions (the rows past the share) to the left-overs.  Blocks as in rows_kernel.
__global__ void __launch_bounds__(kBlock) share_kernel(OneArgs a, const int64_t* __restrict__ left_off,
                                                       int32_t* __restrict__ emit, int32_t* __restrict__ len,
                                                       int64_t* __restrict__ ts, int32_t* __restrict__ left) {
    if (stage1_bad(a.st) || a.rs->overflowed) return;
    const int r = (int)(blockIdx.x / a.per_rank);
    const int64_t base = a.off[r], nr = a.off[r + 1] - base;
    const int64_t lo = a.lo[r], share = a.lo[r + 1] - lo, l0 = left_off[r];
    const int64_t i0 = (int64_t)(blockIdx.x % a.per_rank) * kRowTile;
#pragma unroll
    for (int c = 0; c < kRowItems; ++c) {
        const int64_t i = i0 + c * kBlock + threadIdx.x;
        if (i < share) {
            emit[lo + i] = a.emit[base + i];
            len[lo + i] = a.len[base + i];
            if (ts) ts[lo + i] = a.ts[base + i];
        } else if (i < nr) {
            left[l0 + (nr - 1 - i)] = a.emit[base + i];   // row i is formation position nr - 1 - i
        }
    }
}

// ---------------------------------------------------------------- rounds of short ranks
// Join-mode windows whose ranks hold at most kRankBlockMax samples and overflow (an
// output-slot capacity, as a rule) run a round in two launches of one block per rank, with no
// wait for the host between rounds: short_round_kernel aligns and emits, group_short_ranks
// groups what it returned.  A round of the general path is twelve launches and one
// synchronisation (~95 us on 8 x 4,096 samples; 20 us here).
//
// Overflow in closed form.  Along a rank the groups' sizes never decrease (the step B(l)
// grows as the lengths fall), except for the last group, which the buffer's end clips.  The T
// largest, ties to the later-formed, are therefore T consecutive groups: the last T, unless T
// of the others are larger than the last group, then the T before it.  So what a round emits
// is one range of positions, reversed, and what it returns the positions before it and after
// it.  Stage-1 groups that are not sized like this (arrays that odb_form_groups did not
// write) are left to the general path.
struct ShortArgs {
    int W;
    int has_cap;
    const int64_t* cap;
    const int64_t* off;
    RankState* ranks;
    RoundState* rs;
    DevStatus* st;
    int32_t* dst;        // emitted ids and lengths, rank r from off[r] on
    int32_t* dst_len;
    // staged slot records, rank r's slots from off[r] on
    int32_t* srows;
    int32_t* smax;
    int64_t* stok;
    double* sadj;
    int64_t* sroff;      // first row of the slot among the rank's
};

// 512 threads: 53 registers and two waves per SIMD, which fit beside the three collate waves of 84
// (88 allocated) there (1,024 threads took 101 registers, so that a round waited for the collate of the step
// before).
constexpr int kShortThreads = 512;

template <typename T, typename Op>
__device__ __forceinline__ T short_reduce(T v, Op op) {
    __shared__ T s_v[kShortThreads / kWave];
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v = op(v, ::__shfl_xor(v, d, kWave));
    if ((threadIdx.x & (kWave - 1)) == 0) s_v[threadIdx.x / kWave] = v;
    __syncthreads();
    T r = s_v[0];
#pragma unroll
    for (int i = 1; i < kShortThreads / kWave; ++i) r = op(r, s_v[i]);
    __syncthreads();
    return r;
}

__global__ void __launch_bounds__(kShortThreads) short_round_kernel(ShortArgs a, const int32_t* __restrict__ cur_ids,
                                                                    const int32_t* __restrict__ cur_len,
                                                                    const int32_t* __restrict__ gidx,
                                                                    int32_t* __restrict__ next_ids,
                                                                    int32_t* __restrict__ next_len) {
#pragma clang fp contract(off)
    __shared__ int32_t s_len[kRankBlockMax];
    __shared__ uint16_t s_gs[kRankBlockMax + 2];
    __shared__ int64_t s_pre[kShortThreads];   // tokens before position t << sh
    __shared__ int64_t s_w[kShortThreads / kWave];
    if (stage1_bad(a.st)) return;
    const int t = threadIdx.x, r = blockIdx.x;
    // Eq. 3 over the active ranks
    int64_t maxG = 0, minC = LLONG_MAX, minS = LLONG_MAX;
    for (int q = t; q < a.W; q += kShortThreads) {
        const int64_t Gq = a.ranks[q].G, Sq = a.ranks[q].cnt;
        if (Gq <= 0) continue;
        maxG = Gq > maxG ? Gq : maxG;
        minS = Sq < minS ? Sq : minS;
        if (a.has_cap && a.cap[q] > 0 && a.cap[q] < minC) minC = a.cap[q];
    }
    maxG = short_reduce(maxG, MaxOp{});
    minC = short_reduce(minC, MinOp{});
    minS = short_reduce(minS, MinOp{});
    RankState& R = a.ranks[r];
    const int cnt = (int)R.cnt;
    if (maxG == 0) {   // every buffer is empty
        if (t == 0) R.next_cnt = 0;
        return;
    }
    int64_t T64 = maxG;
    T64 = minC < T64 ? minC : T64;
    T64 = minS < T64 ? minS : T64;
    const int T = (int)(T64 < 1 ? 1 : T64);
    if (r == 0) {
        int64_t splits = 0, over = 0, changed = 0;
        for (int q = t; q < a.W; q += kShortThreads) {
            const int64_t Gq = a.ranks[q].G;
            if (Gq <= 0) continue;
            splits += Gq < T ? T - Gq : 0;
            over += Gq > T ? Gq - T : 0;
            changed += Gq != T;
        }
        splits = short_reduce(splits, SumOp{});
        over = short_reduce(over, SumOp{});
        changed = short_reduce(changed, SumOp{});
        if (t == 0) {
            a.rs->T = T;
            a.rs->splits += splits;
            a.rs->overflow += over;
            a.rs->second_gather += changed > 0 ? 1 : 0;
            a.rs->rounds += 1;
            a.rs->cut += T;   // steps so far
        }
    }
    if (cnt == 0) {
        if (t == 0) R.next_cnt = 0;
        return;
    }
    const int64_t base = a.off[r];
    const int G = (int)R.G;
    for (int q = t; q < cnt; q += kShortThreads) {
        s_len[q] = cur_len[base + q];
        const int32_t g = gidx[base + q];
        if (q == 0 || g != gidx[base + q - 1]) s_gs[g] = (uint16_t)q;
    }
    if (t == 0) s_gs[G] = (uint16_t)cnt;
    __syncthreads();
    // tokens before every (1 << sh)-th position, the fewest a thread that cover the buffer: 16 each
    // left all but a few waves of a small buffer idle, their reads 16 words apart on 4 LDS banks
    // (8 x 4,096 samples: 12.8 us a round, now 11.9)
    int sh = 0;
    while (kShortThreads << sh < cnt) ++sh;
    int64_t tok;
    {
        int64_t v = 0;
        const int q0 = t << sh, q1 = q0 + (1 << sh) < cnt ? q0 + (1 << sh) : cnt;
        for (int q = q0; q < q1; ++q) v += s_len[q];
        const int64_t inc = wave_scan_dpp<OpAdd>(v);
        if ((t & (kWave - 1)) == kWave - 1) s_w[t / kWave] = inc;
        // sizes must not decrease up to the last group but one
        bool odd = false;
        for (int g = t; g + 2 < G; g += kShortThreads)
            odd |= s_gs[g + 2] - s_gs[g + 1] < s_gs[g + 1] - s_gs[g] && g + 2 < G;
        __syncthreads();
        int64_t pre = inc - v;
        tok = 0;
#pragma unroll
        for (int i = 0; i < kShortThreads / kWave; ++i) {
            pre += i < t / kWave ? s_w[i] : 0;
            tok += s_w[i];
        }
        s_pre[t] = pre;
        if (G > T && odd) a.rs->irregular = 1;
    }
    __syncthreads();
    auto tokens_before = [&](int p) {
        const int c = p >> sh;
        if (c >= kShortThreads) return tok;
        int64_t v = s_pre[c];
        for (int q = c << sh; q < p; ++q) v += s_len[q];
        return v;
    };
    // what is emitted: positions [A, B)
    int A = 0, B = cnt, g0 = 0, js = 0, X = -1;
    if (G < T) {
        const int k = T - G;
        int lo = -1, hi = G - 1;   // surplus(lo) < k <= surplus(hi)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (s_gs[mid + 1] - (mid + 1) >= k) hi = mid; else lo = mid;
        }
        js = hi;
        X = k + js;
    } else if (G > T) {
        // groups 0 .. G-2 larger than the last one: from index `lo` on
        const int size_last = cnt - s_gs[G - 1];
        int lo = 0, hi = G - 1;
        while (lo < hi) {
            const int mid = (lo + hi) >> 1;
            if (s_gs[mid + 1] - s_gs[mid] > size_last) hi = mid; else lo = mid + 1;
        }
        g0 = G - 1 - lo < T ? G - T : G - 1 - T;
        A = s_gs[g0];
        B = s_gs[g0 + T];
    }
    const int64_t emitted = R.emitted, slots = R.slots;
    const double mean = (double)tok / (double)cnt;
    for (int j = t; j < T; j += kShortThreads) {
        const int u = T - 1 - j;   // emission runs short to long
        int a0, a1;
        if (u < X) {
            a0 = u;
            a1 = u + 1;
        } else {
            const int g = X >= 0 ? js + (u - X) : g0 + u;
            a0 = u == X ? X : s_gs[g];
            a1 = s_gs[g + 1];
        }
        const int64_t o = base + slots + j;
        a.srows[o] = a1 - a0;
        a.smax[o] = s_len[a0];
        a.stok[o] = tokens_before(a1) - tokens_before(a0);
        a.sadj[o] = (double)(a1 - a0) * mean;
        a.sroff[o] = emitted + (B - a1);
    }
    for (int q = t; q < cnt; q += kShortThreads) {
        const int32_t id = cur_ids[base + q];
        if (q >= A && q < B) {
            const int64_t o = base + emitted + (B - 1 - q);
            a.dst[o] = id;
            a.dst_len[o] = s_len[q];
        } else {
            const int64_t o = base + (q < A ? q : A + q - B);
            next_ids[o] = id;
            next_len[o] = s_len[q];
        }
    }
    __syncthreads();
    if (t == 0) {
        R.emitted = emitted + (B - A);
        R.slots = slots + T;
        R.next_cnt = A + (cnt - B);
    }
}

// Whether the rounds have emptied every buffer; *S receives the steps.
__device__ __forceinline__ bool short_done(const ShortArgs& a, int64_t* S) {
    int64_t left = 0;
    for (int q = threadIdx.x; q < a.W; q += blockDim.x) left += a.ranks[q].cnt;
    *S = a.rs->cut;
    return __syncthreads_or(left != 0) == 0 && !a.rs->irregular;
}

// The staged slots in the plan's layout, in equal ranges as tiles_kernel takes them.
__global__ void __launch_bounds__(kBlock) short_slots_kernel(ShortArgs a, I64Pair* __restrict__ part,
                                                             int64_t slot_capacity, int32_t* __restrict__ rows,
                                                             int32_t* __restrict__ maxlen,
                                                             int64_t* __restrict__ row_off,
                                                             int64_t* __restrict__ tokens, double* __restrict__ approx) {
    if (stage1_bad(a.st)) return;
    int64_t S;
    const bool done = short_done(a, &S);
    const int64_t K = (int64_t)a.W * S;
    if (blockIdx.x == 0 && threadIdx.x == 0) a.rs->overflowed = done ? 0 : 1;   // tiles_kernel: nothing to do yet
    if (!done || K > slot_capacity) return;
    const int64_t per = (K + gridDim.x - 1) / gridDim.x;
    const int64_t k0 = (int64_t)blockIdx.x * per, k1 = k0 + per < K ? k0 + per : K;
    int64_t cells = 0, real = 0;
    for (int64_t k = k0 + threadIdx.x; k < k1; k += kBlock) {
        const int r = (int)(k / S);
        const int64_t j = k - (int64_t)r * S, base = a.off[r];
        const bool live = j < a.ranks[r].slots;   // past them: IDLE
        const int32_t n = live ? a.srows[base + j] : 0, m = live ? a.smax[base + j] : 0;
        const int64_t tk = live ? a.stok[base + j] : 0;
        rows[k] = n;
        maxlen[k] = m;
        tokens[k] = tk;
        row_off[k] = live ? base + a.sroff[base + j] : a.off[r + 1];
        if (approx) approx[k] = live ? a.sadj[base + j] : 0.0;
        cells += (int64_t)n * m;
        real += tk;
    }
    cells = block_sum(cells);
    real = block_sum(real);
    if (threadIdx.x == 0) part[blockIdx.x] = I64Pair{cells, real};
}

// Row records of rank r = blockIdx.x, the check of the carried lengths against the CSR
// offsets, and coverage: the rank's rows are its ids, each once (one bit per id).
__global__ void __launch_bounds__(kShortThreads) short_rows_kernel(ShortArgs a, const int64_t* __restrict__ tok_off,
                                                                   int64_t* __restrict__ ts, int want_ids,
                                                                   DevInfo* info) {
    __shared__ uint32_t s_bit[kRankBlockMax / 32];
    if (stage1_bad(a.st)) return;
    int64_t S;
    if (!short_done(a, &S)) return;
    const int r = blockIdx.x, t = threadIdx.x;
    const int64_t base = a.off[r];
    const int nr = (int)(a.off[r + 1] - base);
    for (int i = t; i < (int)(kRankBlockMax / 32); i += kShortThreads) s_bit[i] = 0;
    __syncthreads();
    int64_t fresh = 0;
    for (int k = t; k < nr; k += kShortThreads) {
        const int32_t id = a.dst[base + k];
        const uint32_t v = (uint32_t)(id - (int32_t)base);
        if (v >= (uint32_t)nr) {
            atomicOr(&a.st->err, kErrInternal);
            continue;
        }
        const uint32_t bit = 1u << (v & 31);
        fresh += (atomicOr(&s_bit[v >> 5], bit) & bit) == 0;
        const int64_t t0 = tok_off[id], w = tok_off[id + 1] - t0;
        if (w < 1 || w > INT_MAX || t0 < 0) {
            atomicOr(&a.st->err, kErrLength);
            atomicMin((unsigned long long*)&a.st->first_bad_len, (unsigned long long)id);
        } else if (w != (int64_t)a.dst_len[base + k]) {
            atomicOr(&a.st->err, kErrSortedLen);
            atomicMin((unsigned long long*)&a.st->first_bad_csr, (unsigned long long)id);
        }
        if (ts) ts[base + k] = t0;
    }
    fresh = short_reduce(fresh, SumOp{});
    if (t == 0 && fresh != nr) {   // nr - fresh ids are missing, as many listings come again
        atomicAdd((unsigned long long*)&info->bad_views, (unsigned long long)(nr - fresh));
        if (want_ids) {
            atomicAdd((unsigned long long*)&info->missing_ids, (unsigned long long)(nr - fresh));
            atomicAdd((unsigned long long*)&info->duplicate_ids, (unsigned long long)(nr - fresh));
        }
    }
}

// Rounds enqueued before the host first looks (twice as many each further time): windows with
// capacities take two to six rounds as a rule, and a launch past the last one returns at once.
constexpr int64_t kShortChunk = 4;

// Samples per step over the ranks of the staged slots.
__global__ void __launch_bounds__(kBlock) short_steps_kernel(ShortArgs a, int64_t* __restrict__ steps) {
    const int64_t S = a.rs->cut, stride = (int64_t)gridDim.x * kBlock;
    for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < S; j += stride) {
        int64_t n = 0;
        for (int r = 0; r < a.W; ++r)
            if (j < a.ranks[r].slots) n += a.srows[a.off[r] + j];
        steps[j] = n;
    }
}

// The largest step from the samples per step.  One block.
__global__ void __launch_bounds__(kBlock) step_max_kernel(const int64_t* __restrict__ steps, RoundState* rs) {
    int64_t mx = 0;
    for (int64_t j = threadIdx.x; j < rs->cut; j += kBlock) mx = steps[j] > mx ? steps[j] : mx;
    mx = block_reduce(mx, MaxOp{});
    if (threadIdx.x == 0) rs->step_max = mx;
}

// A plan that does not fit the slot arrays has no slots to take its largest step from, and reports it all
// the same: from the samples per step, in the workspace.
int step_max_without_slots(const int64_t* steps, RoundState* d_rs, RoundState* rs, hipStream_t s) {
    hipLaunchKernelGGL(step_max_kernel, dim3(1), dim3(kBlock), 0, s, steps, d_rs);
    ODB_LAUNCHED();
    return read_device(rs, d_rs, sizeof(*rs), s);
}

// The plan summary of a device-side alignment, and what it reports.
int finish_short(const HostState& h, int W, int64_t n, int64_t slot_capacity, int stop, odb_plan_info_t* out) {
    const int64_t S = h.rs.cut, K = (int64_t)W * S;
    out->steps = S;
    out->rounds = (int32_t)h.rs.rounds;
    out->stop_reason = stop;
    out->splits = h.rs.splits;
    out->overflow_groups = h.rs.overflow;
    out->second_gather_rounds = h.rs.second_gather;
    out->max_step_samples = h.rs.step_max;
    out->required_slot_capacity = K;
    if (K > slot_capacity)
        return set_error(ODB_E_CAPACITY, "plan needs %lld slots, capacity is %lld", (long long)K,
                         (long long)slot_capacity);
    out->emitted_samples = h.info.emitted;
    out->leftover_samples = n - h.info.emitted;
    out->real_tokens = h.info.real_tokens;
    out->padded_elems = h.info.padded_elems;
    out->missing_ids = h.info.missing_ids;
    out->duplicate_ids = h.info.duplicate_ids;
    out->bad_views = h.info.bad_views;
    out->pad_fraction = h.info.pad_fraction;
    if (h.st.err & kErrLength)
        return set_error(ODB_E_INVALID_DATA, "sample %lld has a length outside [1, 2^31) or a negative token offset",
                         (long long)h.st.first_bad_len);
    if (h.st.err & kErrSortedLen)
        return set_error(ODB_E_INVALID_DATA,
                         "stage-1 arrays do not describe this window (sorted length of sample %lld is not its CSR "
                         "length)", (long long)h.st.first_bad_csr);
    if (h.st.err & kErrIdentity)
        return set_error(ODB_E_INVALID_DATA, "identity map holds a value outside [0, num_identities)");
    if (h.st.err & kErrInternal) return set_error(ODB_E_INTERNAL, "internal inconsistency in the aligned plan");
    if (out->bad_views != 0)
        return set_error(ODB_E_COVERAGE, "%lld sampler views are not emitted (or left over) exactly once",
                         (long long)out->bad_views);
    return ODB_OK;
}

struct RoundBuffers {
    const int32_t* ids;
    const int32_t* len;
    const int32_t* gidx;
};

}  // namespace

}  // namespace odb

using namespace odb;

extern "C" int odb_align_groups(const odb_window_t* w, int64_t budget, const odb_align_params_t* params,
                                const int32_t* d_order, const int32_t* d_sorted_len, const int32_t* d_group_index,
                                const int32_t* d_groups_per_rank, int64_t slot_capacity, int32_t* d_emit_order,
                                int64_t* d_row_token_start, int32_t* d_row_len, int32_t* d_slot_rows, int32_t* d_slot_maxlen, int64_t* d_slot_row_off,
                                int64_t* d_slot_tile_off, int64_t* d_slot_tokens, double* d_slot_tokens_approx,
                                int32_t* d_leftover, int64_t* d_leftover_off, odb_plan_info_t* h_info, void* d_ws,
                                size_t ws_bytes, void* stream) {
    Layout L;
    ODB_TRY(check_workspace(w, d_ws, ws_bytes, &L));
    if (budget < 1) return set_error(ODB_E_INVALID_ARG, "budget must be >= 1");
    if (!params) return set_error(ODB_E_INVALID_ARG, "params is NULL");
    if (params->mode != ODB_MODE_JOIN && params->mode != ODB_MODE_NONJOIN_QUOTA)
        return set_error(ODB_E_INVALID_ARG, "unknown mode %d", params->mode);
    if (params->reserved0 != 0) return set_error(ODB_E_INVALID_ARG, "params.reserved0 must be 0");
    const bool nonjoin = params->mode == ODB_MODE_NONJOIN_QUOTA;
    if (nonjoin && params->quota < 1) return set_error(ODB_E_INVALID_ARG, "quota must be >= 1 in non-join mode");
    if (!h_info) return set_error(ODB_E_INVALID_ARG, "h_info is NULL");
    if (slot_capacity < 0) return set_error(ODB_E_INVALID_ARG, "slot_capacity must be >= 0");
    if ((d_row_token_start == nullptr) != (d_row_len == nullptr))
        return set_error(ODB_E_INVALID_ARG, "d_row_token_start and d_row_len are given together or not at all");
    const int W = w->num_ranks;
    const int64_t n = w->num_samples;
    if (n > 0 && (!d_order || !d_sorted_len || !d_group_index || !d_emit_order || !d_leftover))
        return set_error(ODB_E_INVALID_ARG, "sample arrays must not be NULL");
    if (!d_groups_per_rank || !d_slot_row_off || !d_slot_tile_off || !d_leftover_off)
        return set_error(ODB_E_INVALID_ARG, "offset arrays must not be NULL");
    if (slot_capacity > 0 && (!d_slot_rows || !d_slot_maxlen || !d_slot_tokens))
        return set_error(ODB_E_INVALID_ARG, "slot arrays must not be NULL");
    const int64_t* cap = params->slot_capacity;
    if (cap)
        for (int r = 0; r < W; ++r)
            if (cap[r] < 0) return set_error(ODB_E_INVALID_ARG, "slot_capacity[%d] must be >= 0", r);
    memset(h_info, 0, sizeof(*h_info));

    hipStream_t s = static_cast<hipStream_t>(stream);
    ODB_TRY(upload_small(w, L, d_ws, cap, s, true));
    const int64_t* d_off = ws_at<int64_t>(d_ws, L.rank_off);
    const int64_t* d_cap = ws_at<int64_t>(d_ws, L.cap);
    RankState* d_ranks = ws_at<RankState>(d_ws, L.ranks);
    RoundState* d_rs = ws_at<RoundState>(d_ws, L.round);
    DevStatus* st = ws_at<DevStatus>(d_ws, L.status);
    DevInfo* d_info = ws_at<DevInfo>(d_ws, L.info);
    int64_t* d_gbase = ws_at<int64_t>(d_ws, L.gbase);
    int32_t* gstart = ws_at<int32_t>(d_ws, L.gstart);
    int32_t* gsize = ws_at<int32_t>(d_ws, L.gsize);
    int64_t* cs = ws_at<int64_t>(d_ws, L.cs);
    int32_t* ov_slot = ws_at<int32_t>(d_ws, L.ov_slot);
    int32_t* ov_lo = ws_at<int32_t>(d_ws, L.ov_lo);
    int32_t* kept = ws_at<int32_t>(d_ws, L.kept);
    int32_t* srows = ws_at<int32_t>(d_ws, L.srows);
    int32_t* smax = ws_at<int32_t>(d_ws, L.smax);
    int64_t* stok = ws_at<int64_t>(d_ws, L.stok);
    double* sadj = ws_at<double>(d_ws, L.sadj);
    int64_t* steps = ws_at<int64_t>(d_ws, L.steps);
    int32_t* bids[2] = {ws_at<int32_t>(d_ws, L.buf_ids0), ws_at<int32_t>(d_ws, L.buf_ids1)};
    int32_t* blen[2] = {ws_at<int32_t>(d_ws, L.buf_len0), ws_at<int32_t>(d_ws, L.buf_len1)};
    int32_t* wgidx = ws_at<int32_t>(d_ws, L.gidx);
    int32_t* dst = nonjoin ? ws_at<int32_t>(d_ws, L.stage) : d_emit_order;
    // the length each emitted row carries (from the stage-1 sorted lengths): the row
    // records' lengths, checked against the CSR offsets once the plan is built
    int32_t* row_len = d_row_len ? d_row_len : ws_at<int32_t>(d_ws, L.row_len);
    int32_t* dst_len = nonjoin ? ws_at<int32_t>(d_ws, L.stage_len) : row_len;
    const int64_t gcap = (int64_t)num_cus() * kPlanBlocksPerCU;
    const unsigned gridn = grid_for(n, kBlock, gcap);

    // ---- a window that aligns in one round
    int64_t max_nr = 0, min_nr = LLONG_MAX, empty_ranks = 0, min_cap = LLONG_MAX;
    for (int r = 0; r < W; ++r) {
        const int64_t nr = w->rank_offsets[r + 1] - w->rank_offsets[r];
        max_nr = std::max(max_nr, nr);
        if (nr > 0) min_nr = std::min(min_nr, nr);
        empty_ranks += nr == 0;
        if (cap && cap[r] > 0) min_cap = std::min(min_cap, cap[r]);
    }
    const int64_t per_rank = (max_nr + kRowTile - 1) / kRowTile;
    // XCD-affine random reads pay off when every XCD has a rank and a rank's offsets fit in its
    // L2 with room to spare
    const int xcd = W >= kXcds && max_nr * 8 <= (int64_t)2 << 20;
    const int64_t row_blocks = (xcd ? (W + kXcds - 1) / kXcds * kXcds : W) * per_rank;
    // a positive capacity below a rank's samples makes overflow likely, a sample-quota window
    // with an empty rank stops before its first round, and ranks of very unequal sizes would
    // leave most of the per-rank blocks without work (tpre has room for n of them): these go
    // round by round
    if (n > 0 && min_cap >= max_nr && !(nonjoin && empty_ranks > 0) && W * per_rank <= n &&
        row_blocks <= 32 * ((n + kRowTile - 1) / kRowTile + W) && row_blocks < (1 << 23)) {
        OneArgs a{};
        a.W = W;
        a.n = n;
        a.nonjoin = nonjoin ? 1 : 0;
        a.quota = params->quota;
        a.slot_capacity = slot_capacity;
        a.tok_off = w->d_token_offsets;
        a.off = d_off;
        a.order = d_order;
        a.slen = d_sorted_len;
        a.gidx = d_group_index;
        a.groups = d_groups_per_rank;
        a.gs = gstart;
        a.gpre = stok;
        a.tpre = reinterpret_cast<int64_t*>(sadj);
        a.per_rank = (int)per_rank;
        a.min_nr = min_nr;
        a.lo = nonjoin ? d_gbase : const_cast<int64_t*>(d_off);
        a.steps = steps;
        a.part = ws_at<I64Pair>(d_ws, L.cs);
        a.rs = d_rs;
        a.info = d_info;
        a.st = st;
        a.emit = dst;
        a.len = dst_len;
        a.ts = nonjoin && d_row_token_start ? ws_at<int64_t>(d_ws, L.row_ts) : d_row_token_start;
        // one wave of slots each, up to kMaxRanges blocks (part holds n + 1 words, two a block)
        const unsigned ranges = grid_for(n, 64, kMaxRanges);
        hipLaunchKernelGGL(rows_kernel, dim3((unsigned)row_blocks), dim3(kBlock), 0, s, a, xcd);
        ODB_LAUNCHED();
        if (per_rank > kTilesSummed) {
            hipLaunchKernelGGL(rank_tiles_kernel, dim3(W), dim3(kBlock), 0, s, a);
            ODB_LAUNCHED();
        }
        if (nonjoin) {
            ODB_TRY(cut_steps(a, max_nr, s));
            hipLaunchKernelGGL(cut_kernel, dim3(1), dim3(kBlock), 0, s, a, d_leftover_off);
            ODB_LAUNCHED();
        }
        hipLaunchKernelGGL(slots_kernel, dim3(ranges), dim3(kBlock), 0, s, a, d_slot_rows, d_slot_maxlen, d_slot_row_off,
                           d_slot_tokens, d_slot_tokens_approx);
        ODB_LAUNCHED();
        hipLaunchKernelGGL(tiles_kernel, dim3(ranges), dim3(kBlock), 0, s, a, (const int32_t*)d_slot_rows,
                           (const int32_t*)d_slot_maxlen, d_slot_row_off, d_slot_tile_off, d_leftover_off);
        ODB_LAUNCHED();
        if (nonjoin) {
            hipLaunchKernelGGL(share_kernel, dim3((unsigned)(W * per_rank)), dim3(kBlock), 0, s, a,
                               (const int64_t*)d_leftover_off, d_emit_order, row_len, d_row_token_start, d_leftover);
            ODB_LAUNCHED();
        }
        // every view is emitted or left over once, so the identities count over all views
        if (w->d_identity) ODB_TRY(count_identities(w, L, d_ws, d_order, n, nullptr, 0, s));
        HostState h;
        ODB_TRY(read_state(L, d_ws, 0, &h, s));
        if (!h.rs.overflowed) {
            if (h.st.err & (kErrOrder | kErrGroupIndex))
                return set_error(ODB_E_INVALID_DATA,
                                 "stage-1 arrays do not describe this window (first inconsistent position %lld)",
                                 (long long)h.st.first_bad);
            if ((int64_t)W * h.rs.cut > slot_capacity) {
                if (!nonjoin) ODB_TRY(cut_steps(a, max_nr, s));   // else the cut has counted them
                ODB_TRY(step_max_without_slots(steps, d_rs, &h.rs, s));
            }
            h.rs.rounds = 1;
            return finish_short(h, W, n, slot_capacity, nonjoin && h.rs.quota_hit ? ODB_STOP_QUOTA : ODB_STOP_DRAINED,
                                h_info);
        }
        // some rank overflows: start over, round by round, which also checks the ranks left out here
        if (h.st.err) ODB_TRY(upload_small(w, L, d_ws, cap, s));
    }

    hipLaunchKernelGGL(round0_ranks_kernel, dim3(1), dim3(kBlock), 0, s, d_off, d_groups_per_rank, W, d_ranks,
                       d_gbase, st, d_rs, d_info);
    ODB_LAUNCHED();
    if (n > 0) {
        hipLaunchKernelGGL(round0_check_kernel, dim3(gridn), dim3(kBlock), 0, s, d_off, (const RankState*)d_ranks, W,
                           n, d_order, d_sorted_len, d_group_index, gstart, st);
        ODB_LAUNCHED();
    }

    // ---- rounds of short ranks
    if (n > 0 && !nonjoin && max_nr <= kRankBlockMax && chain_fits(budget, max_nr)) {
        ShortArgs a{};
        a.W = W;
        a.has_cap = cap ? 1 : 0;
        a.cap = d_cap;
        a.off = d_off;
        a.ranks = d_ranks;
        a.rs = d_rs;
        a.st = st;
        a.dst = d_emit_order;
        a.dst_len = row_len;
        a.srows = srows;
        a.smax = smax;
        a.stok = stok;
        a.sadj = sadj;
        a.sroff = ws_at<int64_t>(d_ws, L.row_ts);
        OneArgs tl{};   // what tiles_kernel reads
        tl.W = W;
        tl.slot_capacity = slot_capacity;
        tl.lo = const_cast<int64_t*>(d_off);
        tl.part = ws_at<I64Pair>(d_ws, L.cs);
        tl.rs = d_rs;
        tl.info = d_info;
        tl.st = st;
        const unsigned ranges = grid_for(n, 64, kMaxRanges);
        const int32_t *ids = d_order, *len = d_sorted_len, *gix = d_group_index;
        int f = 0;
        HostState h;
        bool redo = false;
        // join mode emits every view, so the identities count over all of them
        if (w->d_identity) ODB_TRY(count_identities(w, L, d_ws, d_order, n, nullptr, 0, s));
        for (int64_t more = kShortChunk;; more *= 2) {
            for (int64_t k = 0; k < more; ++k) {
                hipLaunchKernelGGL(short_round_kernel, dim3(W), dim3(kShortThreads), 0, s, a, ids, len, gix, bids[f],
                                   blen[f]);
                ODB_LAUNCHED();
                ODB_TRY(group_short_ranks(W, budget, max_nr, d_off, blen[f], wgidx, d_ranks, st, s));
                ids = bids[f];
                len = blen[f];
                gix = wgidx;
                f ^= 1;
            }
            // the final plan, if these rounds were enough
            hipLaunchKernelGGL(short_slots_kernel, dim3(ranges), dim3(kBlock), 0, s, a, tl.part, slot_capacity, d_slot_rows,
                               d_slot_maxlen, d_slot_row_off, d_slot_tokens, d_slot_tokens_approx);
            ODB_LAUNCHED();
            hipLaunchKernelGGL(tiles_kernel, dim3(ranges), dim3(kBlock), 0, s, tl, (const int32_t*)d_slot_rows,
                               (const int32_t*)d_slot_maxlen, d_slot_row_off, d_slot_tile_off, d_leftover_off);
            ODB_LAUNCHED();
            hipLaunchKernelGGL(short_rows_kernel, dim3(W), dim3(kShortThreads), 0, s, a, w->d_token_offsets,
                               d_row_token_start, w->d_identity ? 0 : 1, d_info);
            ODB_LAUNCHED();
            ODB_TRY(read_state(L, d_ws, 0, &h, s));
            if (h.st.err & (kErrOrder | kErrGroupIndex))
                return set_error(ODB_E_INVALID_DATA,
                                 "stage-1 arrays do not describe this window (first inconsistent position %lld)",
                                 (long long)h.st.first_bad);
            redo = h.rs.irregular != 0;
            if (redo || !h.rs.overflowed) break;
            if (h.rs.rounds > n) return set_error(ODB_E_INTERNAL, "alignment does not end");
        }
        if (!redo && (int64_t)W * h.rs.cut > slot_capacity) {
            hipLaunchKernelGGL(short_steps_kernel, dim3(grid_for(h.rs.cut, kBlock, gcap)), dim3(kBlock), 0, s, a, steps);
            ODB_LAUNCHED();
            ODB_TRY(step_max_without_slots(steps, d_rs, &h.rs, s));
        }
        if (!redo) return finish_short(h, W, n, slot_capacity, ODB_STOP_DRAINED, h_info);
        ODB_TRY(upload_small(w, L, d_ws, cap, s, true));
        hipLaunchKernelGGL(round0_ranks_kernel, dim3(1), dim3(kBlock), 0, s, d_off, d_groups_per_rank, W, d_ranks,
                           d_gbase, st, d_rs, d_info);
        ODB_LAUNCHED();
        hipLaunchKernelGGL(round0_check_kernel, dim3(gridn), dim3(kBlock), 0, s, d_off, (const RankState*)d_ranks, W,
                           n, d_order, d_sorted_len, d_group_index, gstart, st);
        ODB_LAUNCHED();
    }

    std::vector<int64_t> cnt(W);
    for (int r = 0; r < W; ++r) cnt[r] = w->rank_offsets[r + 1] - w->rank_offsets[r];
    RoundBuffers cur{d_order, d_sorted_len, d_group_index};
    int flip = 0;
    int64_t S = 0;
    int32_t rounds = 0;
    int32_t stop = ODB_STOP_DRAINED;
    RoundState hrs{};
    HostState hstate;
    for (;;) {
        int nonempty = 0;
        int64_t max_cnt = 0;
        for (int r = 0; r < W; ++r) {
            nonempty += cnt[r] > 0;
            if (cnt[r] > max_cnt) max_cnt = cnt[r];
        }
        if (nonempty == 0) {
            stop = ODB_STOP_DRAINED;
            break;
        }
        // non-join: a rank that is empty while others are not advertises "finished"
        if (nonjoin && nonempty < W) {
            stop = ODB_STOP_RANK_FINISHED;
            break;
        }
        if (rounds > 0) {
            ODB_TRY(group_sequences(L, d_ws, W, n, budget, d_off, max_cnt, 0, false, cur.len, wgidx, nullptr, d_ranks,
                                    s));
            cur.gidx = wgidx;
        }
        rounds += 1;
        // real tokens prefix over the live positions
        ODB_TRY((device_excl_scan<int64_t>(LiveLen{cur.len, d_off, d_ranks, W, rounds > 1 ? 1 : 0},
                                           LiveLenIncl{LiveLen{cur.len, d_off, d_ranks, W, rounds > 1 ? 1 : 0}, cs},
                                           n, ws_at<int64_t>(d_ws, L.partials), s)));
        hipLaunchKernelGGL(group_sizes_kernel, dim3(gridn), dim3(kBlock), 0, s, (const int32_t*)gstart,
                           (const int64_t*)d_gbase, d_off, (const RankState*)d_ranks, W, gsize, steps, max_cnt,
                           (const DevStatus*)st);
        ODB_LAUNCHED();
        hipLaunchKernelGGL(adjust_kernel, dim3(W), dim3(kBlock), 0, s, d_ranks, d_cap, cap ? 1 : 0, W, d_rs,
                           (const int32_t*)gsize, ov_slot, kept, st);
        ODB_LAUNCHED();
        hipLaunchKernelGGL(slot_records_kernel, dim3(gridn), dim3(kBlock), 0, s, (const RankState*)d_ranks,
                           (const RoundState*)d_rs, d_off, W, (const int32_t*)gstart, (const int32_t*)gsize,
                           (const int32_t*)kept, cur.len, (const int64_t*)cs, srows, smax, stok, sadj, steps,
                           (const DevStatus*)st);
        ODB_LAUNCHED();
        hipLaunchKernelGGL(finalize_kernel, dim3(W), dim3(kBlock), 0, s, d_ranks, d_rs, (const int64_t*)steps,
                           nonjoin ? 1 : 0, params->quota, d_off,
                           (const int32_t*)gstart, (const int32_t*)gsize, (const int32_t*)ov_slot,
                           (const int32_t*)kept, ov_lo, (const DevStatus*)st);
        ODB_LAUNCHED();
        hipLaunchKernelGGL(emit_kernel, dim3(gridn), dim3(kBlock), 0, s, (const RankState*)d_ranks,
                           (const RoundState*)d_rs, d_off, W, n, cur.ids, cur.len, cur.gidx, (const int32_t*)gstart,
                           (const int32_t*)gsize, (const int32_t*)ov_slot, (const int32_t*)ov_lo, dst, dst_len,
                           bids[flip], blen[flip], (const DevStatus*)st);
        ODB_LAUNCHED();
        hipLaunchKernelGGL(advance_kernel, dim3(grid_for(W, kBlock)), dim3(kBlock), 0, s, d_ranks, W, d_rs);
        ODB_LAUNCHED();
        ODB_TRY(read_state(L, d_ws, W, &hstate, s));
        hrs = hstate.rs;
        const DevStatus& hst = hstate.st;
        const std::vector<RankState>& hranks = hstate.ranks;
        if (hst.err & (kErrOrder | kErrGroupIndex))
            return set_error(ODB_E_INVALID_DATA,
                             "stage-1 arrays do not describe this window (first inconsistent position %lld)",
                             (long long)hst.first_bad);
        if (hst.err & kErrInternal)
            return set_error(ODB_E_INTERNAL, "alignment round %d: group sizes inconsistent", rounds);
        // every round empties part of some buffer (T >= 1 steps of >= 1 sample for each
        // active rank) and never grows one; anything else is device state this call did
        // not write, and the loop stops rather than run on it
        int64_t left_before = 0, left_after = 0;
        for (int r = 0; r < W; ++r) {
            if (hranks[r].cnt < 0 || hranks[r].cnt > cnt[r])
                return set_error(ODB_E_INTERNAL, "alignment round %d: rank %d's buffer grew", rounds, r);
            left_before += cnt[r];
            left_after += hranks[r].cnt;
        }
        if (left_after == left_before && !(nonjoin && hrs.quota_hit))
            return set_error(ODB_E_INTERNAL, "alignment round %d emitted nothing", rounds);
        S += hrs.cut;
        for (int r = 0; r < W; ++r) cnt[r] = hranks[r].cnt;
        cur = RoundBuffers{bids[flip], blen[flip], nullptr};
        flip ^= 1;
        if (nonjoin && hrs.quota_hit) {
            stop = ODB_STOP_QUOTA;
            break;
        }
    }

    const int64_t K = (int64_t)W * S;
    h_info->steps = S;
    h_info->rounds = rounds;
    h_info->stop_reason = stop;
    h_info->splits = hrs.splits;
    h_info->overflow_groups = hrs.overflow;
    h_info->max_step_samples = hrs.step_max;
    h_info->second_gather_rounds = hrs.second_gather;
    h_info->required_slot_capacity = K;
    if (K > slot_capacity)
        return set_error(ODB_E_CAPACITY, "plan needs %lld slots, capacity is %lld", (long long)K,
                         (long long)slot_capacity);

    if (K > 0) {
        hipLaunchKernelGGL(plan_slots_kernel, dim3(grid_for(K, kBlock, gcap)), dim3(kBlock), 0, s,
                           (const RankState*)d_ranks, d_off, W, S, (const int32_t*)srows, (const int32_t*)smax,
                           (const int64_t*)stok, (const double*)sadj, d_slot_rows, d_slot_maxlen, d_slot_tokens,
                           d_slot_tokens_approx, d_info);
        ODB_LAUNCHED();
    }
    ODB_TRY((device_excl_scan<I64Pair>(RowsTilesLoad{d_slot_rows, d_slot_maxlen, K},
                                       RowsTilesStore{d_slot_row_off, d_slot_tile_off}, K + 1,
                                       ws_at<I64Pair>(d_ws, L.partials), s)));
    if (nonjoin && n > 0) {
        hipLaunchKernelGGL(compact_emit_kernel, dim3(gridn), dim3(kBlock), 0, s, (const int32_t*)dst,
                           (const int32_t*)dst_len, d_off, (const RankState*)d_ranks, W, n,
                           (const int64_t*)d_slot_row_off, S, d_emit_order, row_len);
        ODB_LAUNCHED();
    }
    const int64_t nemit = hrs.emitted_total;
    if (nemit > 0 && K > 0) {
        const unsigned grid = xcd ? (unsigned)(kXcds * std::max<int64_t>(1, std::min<int64_t>(
                                        (int64_t)num_cus() * 2 / kXcds, (max_nr + kBlock - 1) / kBlock)))
                                  : grid_for(nemit, kBlock, gcap);
        hipLaunchKernelGGL(row_check_kernel, dim3(grid), dim3(kBlock), 0, s, w->d_token_offsets,
                           (const int32_t*)d_emit_order, (const int32_t*)row_len, (const int64_t*)d_slot_row_off, S,
                           W, xcd, d_row_token_start, st);
        ODB_LAUNCHED();
    }
    hipLaunchKernelGGL(leftover_off_kernel, dim3(1), dim3(kBlock), 0, s, (const RankState*)d_ranks, W,
                       d_leftover_off);
    ODB_LAUNCHED();
    int64_t nleft = 0;
    for (int r = 0; r < W; ++r) nleft += cnt[r];
    if (nleft > 0) {
        hipLaunchKernelGGL(leftover_kernel, dim3(gridn), dim3(kBlock), 0, s, cur.ids, cur.len, w->d_token_offsets,
                           d_off, (const RankState*)d_ranks, W, n, (const int64_t*)d_leftover_off, d_leftover, st);
        ODB_LAUNCHED();
    }
    // stats (Sec. 2.1 / App. I padding fraction) and coverage (App. C)
    ODB_TRY(run_plan_coverage(w, L, d_ws, d_emit_order, d_slot_row_off, d_slot_tile_off, S, d_leftover,
                              d_leftover_off, nemit, nleft, s));

    ODB_TRY(read_state(L, d_ws, W, &hstate, s));
    const DevInfo& hi = hstate.info;
    const DevStatus& hs = hstate.st;
    h_info->emitted_samples = hi.emitted;
    h_info->leftover_samples = nleft;
    h_info->real_tokens = hi.real_tokens;
    h_info->padded_elems = hi.padded_elems;
    h_info->missing_ids = hi.missing_ids;
    h_info->duplicate_ids = hi.duplicate_ids;
    h_info->bad_views = hi.bad_views;
    h_info->pad_fraction = hi.pad_fraction;
    if (hs.err & kErrLength)
        return set_error(ODB_E_INVALID_DATA,
                         "sample %lld has a length outside [1, 2^31) or a negative token offset",
                         (long long)hs.first_bad_len);
    if (hs.err & kErrSortedLen)
        return set_error(ODB_E_INVALID_DATA,
                         "stage-1 arrays do not describe this window (sorted length of sample %lld is not its CSR "
                         "length)", (long long)hs.first_bad);
    if (hs.err & kErrIdentity)
        return set_error(ODB_E_INVALID_DATA, "identity map holds a value outside [0, num_identities)");
    if ((hs.err & kErrInternal) || hi.emitted != nemit)
        return set_error(ODB_E_INTERNAL, "internal inconsistency in the aligned plan");
    if (hi.bad_views != 0)
        return set_error(ODB_E_COVERAGE, "%lld sampler views are not emitted (or left over) exactly once",
                         (long long)hi.bad_views);
    return ODB_OK;
}

extern "C" int odb_check_coverage(const odb_window_t* w, const int32_t* d_emitted, int64_t num_emitted,
                                  const int32_t* d_leftover, int64_t num_leftover, odb_plan_info_t* h_info,
                                  void* d_ws, size_t ws_bytes, void* stream) {
    Layout L;
    ODB_TRY(check_workspace(w, d_ws, ws_bytes, &L));
    if (!h_info) return set_error(ODB_E_INVALID_ARG, "h_info is NULL");
    if (num_emitted < 0 || num_leftover < 0) return set_error(ODB_E_INVALID_ARG, "negative counts");
    if ((num_emitted > 0 && !d_emitted) || (num_leftover > 0 && !d_leftover))
        return set_error(ODB_E_INVALID_ARG, "id arrays must not be NULL");
    hipStream_t s = static_cast<hipStream_t>(stream);
    ODB_TRY(upload_small(w, L, d_ws, nullptr, s));
    hipLaunchKernelGGL(init_align_kernel, dim3(1), dim3(64), 0, s, ws_at<RoundState>(d_ws, L.round),
                       ws_at<DevInfo>(d_ws, L.info));
    ODB_LAUNCHED();
    ODB_TRY(run_coverage(w, L, d_ws, d_emitted, num_emitted, d_leftover, num_leftover, s));
    HostState h;
    ODB_TRY(read_state(L, d_ws, 0, &h, s));
    DevInfo& hi = h.info;
    const DevStatus& hs = h.st;
    ODB_TRY(finish_coverage(w, L, d_ws, d_emitted, num_emitted, d_leftover, num_leftover, &hi, s));
    h_info->bad_views = hi.bad_views;
    h_info->missing_ids = hi.missing_ids;
    h_info->duplicate_ids = hi.duplicate_ids;
    if (hs.err & (kErrIdentity | kErrInternal))
        return set_error(ODB_E_INVALID_DATA, "an id lies outside the window or its identity outside the map");
    return ODB_OK;
}
