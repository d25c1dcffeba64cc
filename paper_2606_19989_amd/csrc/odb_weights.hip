// Loss-scaling weights of an aligned plan (Sec. 2.3 "Loss scaling", Eq. 2, App. B, and
// the three scaling modes of the loss-scaling ablation in App. N).
//
// At step j every rank r trains on its slot (r, j).  DDP averages the ranks' per-token
// mean losses, so rank r pre-scales its mean by W * w_{r,j}; the exact token-level weight
// w = t_{r,j} / sum_r t_{r,j} makes the result the per-token mean over the whole step.
// The sample-level weight uses the slot's rows instead of its tokens, the approximate
// token-level weight the approximate token counts that alignment records per slot.
//
// Slots are rank-major (k = r * S + j): a block takes 64 consecutive steps, one per lane, and
// its four waves every fourth rank, so that a few hundred steps already spread over several
// compute units and a thread's loads over ranks are in flight together.  One thread per step
// with a loop over the ranks left the loads in a chain: 35 us for 974 steps of 64 ranks,
// 8.7 us now.  The integer sums may run in any order; the sum of the approximate counts runs
// over the ranks in rank order (from LDS) and each fp64 operation is rounded on its own
// (contraction off), which makes the weights reproducible bit for bit on any device or host
// that follows the same order.
#include "odb_internal.h"

namespace odb {

namespace {

constexpr int kWeightWaves = kBlock / kWave;
constexpr int kWeightRanks = 64;                             // ranks per pass of a block
constexpr int kWeightItems = kWeightRanks / kWeightWaves;    // of them per thread

__global__ void __launch_bounds__(kBlock) loss_weights_kernel(int W, int64_t S, int mode,
                                                              const int32_t* __restrict__ rows,
                                                              const int64_t* __restrict__ tokens,
                                                              const double* __restrict__ approx,
                                                              double* __restrict__ weight,
                                                              int64_t* __restrict__ step_tokens,
                                                              int64_t* __restrict__ step_samples) {
#pragma clang fp contract(off)
    __shared__ double s_a[kWeightRanks][kWave];
    __shared__ int64_t s_t[kWeightWaves][kWave], s_n[kWeightWaves][kWave];
    __shared__ double s_sum[kWave];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    for (int64_t j0 = (int64_t)blockIdx.x * kWave; j0 < S; j0 += (int64_t)gridDim.x * kWave) {
        const int64_t j = j0 + lane;
        const bool on = j < S;
        int64_t t = 0, n = 0;
        double a = 0.0;
        for (int r0 = 0; r0 < W; r0 += kWeightRanks) {   // uniform
#pragma unroll
            for (int i = 0; i < kWeightItems; ++i) {
                const int r = r0 + i * kWeightWaves + w;
                const bool live = on && r < W;
                const int64_t k = live ? (int64_t)r * S + j : 0;
                const int64_t tk = tokens[k];
                const int32_t nk = rows[k];
                t += live ? tk : 0;
                n += live ? nk : 0;
                if (mode == ODB_WEIGHT_TOKEN_APPROX) s_a[i * kWeightWaves + w][lane] = live ? approx[k] : 0.0;
            }
            if (mode == ODB_WEIGHT_TOKEN_APPROX) {
                __syncthreads();
                if (w == 0) {
                    const int m = W - r0 < kWeightRanks ? W - r0 : kWeightRanks;
#pragma unroll 8
                    for (int i = 0; i < m; ++i) a = a + s_a[i][lane];
                }
                __syncthreads();
            }
        }
        s_t[w][lane] = t;
        s_n[w][lane] = n;
        if (w == 0) s_sum[lane] = a;
        __syncthreads();
        t = n = 0;
#pragma unroll
        for (int i = 0; i < kWeightWaves; ++i) {
            t += s_t[i][lane];
            n += s_n[i][lane];
        }
        a = s_sum[lane];
        if (on) {
#pragma unroll 4
            for (int r = w; r < W; r += kWeightWaves) {
                const int64_t k = (int64_t)r * S + j;
                double v = 0.0;
                if (mode == ODB_WEIGHT_SAMPLE) {
                    if (n > 0) v = (double)rows[k] / (double)n;
                } else if (mode == ODB_WEIGHT_TOKEN_APPROX) {
                    if (a > 0.0) v = approx[k] / a;
                } else {
                    if (t > 0) v = (double)tokens[k] / (double)t;
                }
                weight[k] = v;
            }
            if (w == 0) {
                if (step_tokens) step_tokens[j] = t;
                if (step_samples) step_samples[j] = n;
            }
        }
        __syncthreads();
    }
}

// Few ranks and many steps: one thread per step.  The steps alone fill the chip, a load over 64 steps is
// as wide, and no wave waits for another or loads for ranks that are not there.  us per call, the waves
// over the ranks / one thread per step, sample and approximate mode: 1 x 1,048,576 steps 67 / 21 and
// 86 / 21, 4 x 100,000 21 / 17 and 24 / 17, 8 x 30,000 17.8 / 17.3 and 18.6 / 18.2, 12 x 100,000
// 24 / 22 and 27 / 26, 16 x 100,000 24.4 / 25.0 and 28 / 30, 16 x 400,000 46 / 40 and 70 / 49,
// 24 x 200,000 36 / 37 and 53 / 46, 32 x 200,000 40 / 45 and 63 / 56, 64 x 100,000 43 / 55 and 54 / 68;
// below 30,000 steps equal for up to 8 ranks.  So the line lies at 32,768 steps for up to 10 ranks and
// 16,384 more for each rank after them, up to 24; the approximate mode, whose waves wait for each other,
// takes up to 32 ranks from 196,608 steps on.
constexpr int kFewItems = 4;

inline bool few_ranks(int W, int64_t S, int mode) {
    if (mode == ODB_WEIGHT_TOKEN_APPROX && W <= 32 && S >= 196608) return true;
    return W <= 24 && S >= 16384 * (int64_t)(W > 10 ? W - 8 : 2);
}

__global__ void __launch_bounds__(kBlock) loss_weights_few_kernel(int W, int64_t S, int mode,
                                                                  const int32_t* __restrict__ rows,
                                                                  const int64_t* __restrict__ tokens,
                                                                  const double* __restrict__ approx,
                                                                  double* __restrict__ weight,
                                                                  int64_t* __restrict__ step_tokens,
                                                                  int64_t* __restrict__ step_samples) {
#pragma clang fp contract(off)
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < S; j += stride) {
        int64_t t = 0, n = 0;
        double a = 0.0;
#pragma unroll kFewItems
        for (int r = 0; r < W; ++r) {
            const int64_t k = (int64_t)r * S + j;
            t += tokens[k];
            n += rows[k];
            if (mode == ODB_WEIGHT_TOKEN_APPROX) a = a + approx[k];
        }
#pragma unroll kFewItems
        for (int r = 0; r < W; ++r) {
            const int64_t k = (int64_t)r * S + j;
            double v = 0.0;
            if (mode == ODB_WEIGHT_SAMPLE) {
                if (n > 0) v = (double)rows[k] / (double)n;
            } else if (mode == ODB_WEIGHT_TOKEN_APPROX) {
                if (a > 0.0) v = approx[k] / a;
            } else {
                if (t > 0) v = (double)tokens[k] / (double)t;
            }
            weight[k] = v;
        }
        if (step_tokens) step_tokens[j] = t;
        if (step_samples) step_samples[j] = n;
    }
}

}  // namespace

}  // namespace odb

using namespace odb;

extern "C" int odb_loss_weights(int32_t num_ranks, int64_t steps, int32_t mode, const int32_t* d_slot_rows,
                                const int64_t* d_slot_tokens, const double* d_slot_tokens_approx, double* d_weight,
                                int64_t* d_step_tokens, int64_t* d_step_samples, void* stream) {
    if (num_ranks < 1) return set_error(ODB_E_INVALID_ARG, "num_ranks must be >= 1");
    if (steps < 0) return set_error(ODB_E_INVALID_ARG, "steps must be >= 0");
    if (steps > INT64_MAX / num_ranks) return set_error(ODB_E_INVALID_ARG, "num_ranks * steps overflows");
    if (mode != ODB_WEIGHT_SAMPLE && mode != ODB_WEIGHT_TOKEN_APPROX && mode != ODB_WEIGHT_TOKEN_EXACT)
        return set_error(ODB_E_INVALID_ARG, "unknown loss-weight mode %d", mode);
    if (steps == 0) return ODB_OK;
    if (!d_slot_rows || !d_slot_tokens || !d_weight)
        return set_error(ODB_E_INVALID_ARG, "slot arrays and d_weight must not be NULL");
    if (mode == ODB_WEIGHT_TOKEN_APPROX && !d_slot_tokens_approx)
        return set_error(ODB_E_INVALID_ARG, "the approximate mode needs d_slot_tokens_approx");
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool few = few_ranks(num_ranks, steps, mode);
    hipLaunchKernelGGL(few ? loss_weights_few_kernel : loss_weights_kernel,
                       dim3(grid_for(steps, few ? kBlock : kWave, (int64_t)num_cus() * 8)), dim3(kBlock), 0, s,
                       (int)num_ranks, steps, (int)mode, d_slot_rows, d_slot_tokens, d_slot_tokens_approx, d_weight,
                       d_step_tokens, d_step_samples);
    ODB_LAUNCHED();
    return ODB_OK;
}
