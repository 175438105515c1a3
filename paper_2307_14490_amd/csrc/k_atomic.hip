// The atomicAdd variant of the step, and the forward-only loss evaluation.
//
// Atomic variant: three kernels keep the step synchronous without grouping
// rows.  (a) gathers every row and computes the coefficients and the source
// gradient; (b) adds -lr coef S[u] into the context rows with fp32 atomics
// (S still holds pre-step values); (c) adds -lr dS into the source rows.
// The result equals the sorted variant's up to the order of the additions.
// It works on float tables only (bf16 has no native atomic add of the
// precision the step needs); the loss evaluation reads either element type.
#include "common.hpp"
#include "device.hpp"
#include "dispatch.hpp"

namespace huge {

__device__ __forceinline__ void block_loss_a(float loss, double* __restrict__ out) {
    __shared__ double s_w[kBlock / 64];
    double v = (double)loss;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    if ((threadIdx.x & 63) == 0) s_w[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double acc = 0.0;
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) acc += s_w[w];
        out[blockIdx.x] = acc;
    }
}

// Forward for one positive: the loss, the (1 + K) coefficients and the source
// gradient.
template <int G, int C>
__device__ __forceinline__ float forward_positive(const TableArgs& t, int64_t i, int32_t u,
                                                  int32_t v, float c,
                                                  const int32_t* __restrict__ neg, int lane,
                                                  float* __restrict__ coef,
                                                  float* __restrict__ gsrc) {
    using IO = RowIO<G, C>;
    const float* __restrict__ S = static_cast<const float*>(t.S);
    const float* __restrict__ T = static_cast<const float*>(t.T);
    const int K = t.K;
    const int32_t D = t.D;
    float4 s[C], t0[C], dS[C];
    IO::load(s, S, u, D, lane);
    IO::load(t0, T, v, D, lane);
    const float x = group_sum<G>(IO::dot(s, t0));
    const float g = coef_pos(c, x);
    float lsum = softplus_f(-x);
    if (lane == 0) coef[i * (int64_t)(1 + K)] = g;
#pragma unroll
    for (int q = 0; q < C; ++q) dS[q] = scale4(g, t0[q]);
    for (int kb = 0; kb < K; kb += kNegBlock) {
        const int cnt = (K - kb) < kNegBlock ? (K - kb) : kNegBlock;
        float4 tk[kNegBlock][C];
        int32_t mk[kNegBlock];
#pragma unroll
        for (int j = 0; j < kNegBlock; ++j)
            if (j < cnt) mk[j] = neg[i * (int64_t)K + kb + j];
#pragma unroll
        for (int j = 0; j < kNegBlock; ++j)
            if (j < cnt) IO::load(tk[j], T, mk[j], D, lane);
        float y[kNegBlock];
#pragma unroll
        for (int j = 0; j < kNegBlock; ++j) y[j] = (j < cnt) ? IO::dot(s, tk[j]) : 0.f;
#pragma unroll
        for (int j = 0; j < kNegBlock; ++j) y[j] = group_sum<G>(y[j]);
#pragma unroll
        for (int j = 0; j < kNegBlock; ++j) {
            if (j < cnt) {
                lsum += softplus_f(y[j]);
                const float h = coef_neg(c, y[j]);
                if (lane == 0) coef[i * (int64_t)(1 + K) + 1 + kb + j] = h;
#pragma unroll
                for (int q = 0; q < C; ++q) dS[q] = axpy4(h, tk[j][q], dS[q]);
            }
        }
    }
    IO::store(gsrc, i, D, lane, dS);
    return c * lsum;
}

template <int G, int C>
__global__ __launch_bounds__(kBlock) void k_atomic_gather(TableArgs t, Control* __restrict__ ctl,
                                                          StepArgs a,
                                                          const int32_t* __restrict__ neg,
                                                          float* __restrict__ gsrc,
                                                          float* __restrict__ coef,
                                                          double* __restrict__ lossp) {
    if (ctl->step_bad) return;
    constexpr int PPB = kBlock / G;
    const int lane = threadIdx.x % G;
    const int64_t i = (int64_t)blockIdx.x * PPB + threadIdx.x / G;
    float loss = 0.f;
    if (i < a.n) {
        // validated when the batch was grouped; checked again so that a batch
        // changed before its apply is reported instead of read out of bounds
        const int32_t u = a.src[i], v = a.dst[i];
        if (u >= 0 && (int64_t)u < t.N && v >= 0 && (int64_t)v < t.N) {
            const float l =
                forward_positive<G, C>(t, i, u, v, positive_weight(a, i), neg, lane, coef, gsrc);
            if (lane == 0) loss = l;
        } else if (lane == 0) {
            raise_internal(ctl, kSiteAtomicIds);
        }
    }
    block_loss_a(loss, lossp);
}

// A row of D floats over the G lanes of a group, lane l owning the elements
// l, l + G, ...: an atomic instruction of the group then adds to consecutive
// words, and the atomic unit takes a cache line's words together (with four
// consecutive words per lane each instruction touched every line of the row
// with a quarter of its words: a step of 65,536 positives, K = 5, 4e6 x 128,
// 878 us before and 290 now).
template <int G, int C>
__device__ __forceinline__ void load_lanes(float (&x)[4 * C], const float* __restrict__ row,
                                           int32_t D, int lane) {
#pragma unroll
    for (int q = 0; q < 4 * C; ++q) x[q] = lane + q * G < D ? row[lane + q * G] : 0.f;
}

template <int G, int C>
__device__ __forceinline__ void add_lanes(float* __restrict__ row, float w,
                                          const float (&x)[4 * C], int32_t D, int lane) {
#pragma unroll
    for (int q = 0; q < 4 * C; ++q)
        if (lane + q * G < D) unsafeAtomicAdd(row + lane + q * G, w * x[q]);
}

template <int G, int C>
__global__ __launch_bounds__(kBlock) void k_atomic_scatter_T(TableArgs t,
                                                             const Control* __restrict__ ctl,
                                                             StepArgs a,
                                                             const int32_t* __restrict__ neg,
                                                             const float* __restrict__ coef) {
    if (ctl->step_bad) return;
    constexpr int PPB = kBlock / G;
    const int lane = threadIdx.x % G;
    const int64_t i = (int64_t)blockIdx.x * PPB + threadIdx.x / G;
    if (i >= a.n) return;
    const int32_t u = a.src[i], v = a.dst[i];
    if (u < 0 || (int64_t)u >= t.N || v < 0 || (int64_t)v >= t.N) return;
    const int K = t.K;
    const int32_t D = t.D;
    float s[4 * C];
    load_lanes<G, C>(s, static_cast<const float*>(t.S) + u * (int64_t)D, D, lane);
    for (int j = 0; j <= K; ++j) {
        const int64_t row = j == 0 ? (int64_t)v : (int64_t)neg[i * (int64_t)K + j - 1];
        const float w = -a.lr * coef[i * (int64_t)(1 + K) + j];
        float* p = static_cast<float*>(t.T) + row * (int64_t)D;
        add_lanes<G, C>(p, w, s, D, lane);
    }
}

template <int G, int C>
__global__ __launch_bounds__(kBlock) void k_atomic_scatter_S(TableArgs t,
                                                             const Control* __restrict__ ctl,
                                                             StepArgs a,
                                                             const float* __restrict__ gsrc) {
    if (ctl->step_bad) return;
    constexpr int PPB = kBlock / G;
    const int lane = threadIdx.x % G;
    const int64_t i = (int64_t)blockIdx.x * PPB + threadIdx.x / G;
    if (i >= a.n) return;
    const int32_t u = a.src[i];
    if (u < 0 || (int64_t)u >= t.N) return;
    const int32_t D = t.D;
    float g[4 * C];
    load_lanes<G, C>(g, gsrc + i * (int64_t)D, D, lane);
    add_lanes<G, C>(static_cast<float*>(t.S) + (int64_t)u * D, -a.lr, g, D, lane);
}

// Loss of a batch at the current tables; validates ids and counts itself and
// draws the negatives inline (no workspace for them).
// The rows are random reads, so the kernel lives on rows in flight and on few
// instructions between them: a negative is drawn by one lane of the group and
// read by the others (every lane drawing every negative, K Philox blocks each,
// kept the vector units busy for longer than the rows take to arrive), the
// rows stay packed, in blocks of NB, and lane q evaluates the loss term of
// value q.  262,144 positives, K = 5, 1e7 x 128 fp32: 235 -> 158 us (5.9 TB/s);
// 100,000 positives, K = 31, 4e6 x 128 bf16: 501 -> 150.
template <int G, int NB, typename IO>
__global__ __launch_bounds__(kBlock) void k_eval(TableArgs t, Control* __restrict__ ctl, StepArgs a,
                                                 double* __restrict__ lossp) {
    using E = typename IO::Elem;
    using Reg = typename IO::Reg;
    constexpr int C = IO::C, R = IO::R;
    constexpr int PPB = kBlock / G;
    constexpr int kDraws = (NB + G - 1) / G;  // draws of a lane per block
    const int lane = threadIdx.x % G;
    const int first = (int)(threadIdx.x & 63u) - lane;  // the group's first lane in the wave
    const int64_t i = (int64_t)blockIdx.x * PPB + threadIdx.x / G;
    const E* __restrict__ S = static_cast<const E*>(t.S);
    const E* __restrict__ T = static_cast<const E*>(t.T);
    const int K = t.K;
    const int32_t D = t.D;
    float loss = 0.f;
    // groups of one wave shuffle together: a group without a positive, or with
    // an invalid one, takes part in the draws but reads no rows
    bool active = i < a.n;
    int32_t u = 0, v = 0;
    float c = 0.f;
    if (active) {
        u = a.src[i];
        v = a.dst[i];
        const bool ok_id = u >= 0 && (int64_t)u < t.N && v >= 0 && (int64_t)v < t.N;
        const bool ok_c = weight_valid(a, i);
        c = positive_weight(a, i);
        if (!ok_id || !ok_c) {
            if (lane == 0) raise_error(ctl, ok_id ? kBadCount : kBadId);
            active = false;
        }
    }
    float4 s[C];
    Reg t0[R];
    if (active) {
        IO::load(s, S, u, D, lane);
        IO::load_packed(t0, T, v, D, lane);
    }
    float lsum = 0.f;
    for (int kb = 0; kb < K; kb += NB) {
        const int cnt = (K - kb) < NB ? (K - kb) : NB;
        int32_t drawn[kDraws];
#pragma unroll
        for (int q = 0; q < kDraws; ++q) {
            const int j = q * G + lane;
            drawn[q] = active && j < cnt
                           ? draw_negative(t.seed, a.first_pos + (uint64_t)i, (uint32_t)(kb + j),
                                           (uint64_t)t.N, t.thr, t.alias)
                           : 0;
        }
        int32_t mk[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) mk[j] = __shfl(drawn[j / G], first + j % G, 64);
        if (!active) continue;
        Reg tk[NB][R];
#pragma unroll
        for (int j = 0; j < NB; ++j)
            if (j < cnt) IO::load_packed(tk[j], T, mk[j], D, lane);
        if (kb == 0) {
            const float x = group_sum<G>(IO::dotp(s, t0));
            if (lane == 0) lsum += softplus_f(-x);
        }
        float y[NB];
#pragma unroll
        for (int j = 0; j < NB; ++j) y[j] = (j < cnt) ? IO::dotp(s, tk[j]) : 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j) y[j] = group_sum<G>(y[j]);
        if constexpr (G >= NB) {
            float z = y[0];
#pragma unroll
            for (int j = 1; j < NB; ++j) z = lane == j ? y[j] : z;
            if (lane < cnt) lsum += softplus_f(z);
        } else if (lane == 0) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
                if (j < cnt) lsum += softplus_f(y[j]);
        }
    }
    if (active) loss = c * lsum;
    block_loss_a(loss, lossp);
}

static int64_t blocks_for(int dim, int64_t n) {
    const RowShape rs = row_shape(dim);
    const int64_t ppb = kBlock / rs.G;
    return (n + ppb - 1) / ppb;
}

hipError_t launch_atomic_gather(const TableArgs& t, Control* ctl, const StepArgs& a,
                                const int32_t* neg, float* gsrc, float* coef, double* lossp,
                                int64_t* blocks_out, hipStream_t s) {
    const RowShape rs = row_shape(t.D);
    const int64_t blocks = blocks_for(t.D, a.n);
    *blocks_out = blocks;
    if (blocks == 0) return hipSuccess;
    HUGE_ROW_DISPATCH(rs, {
        hipLaunchKernelGGL((k_atomic_gather<G_, C_>), dim3((unsigned)blocks), dim3(kBlock), 0, s,
                           t, ctl, a, neg, gsrc, coef, lossp);
    });
    return hipGetLastError();
}

hipError_t launch_atomic_scatter_T(const TableArgs& t, Control* ctl, const StepArgs& a,
                                   const int32_t* neg, const float* coef, hipStream_t s) {
    const RowShape rs = row_shape(t.D);
    const int64_t blocks = blocks_for(t.D, a.n);
    if (blocks == 0) return hipSuccess;
    HUGE_ROW_DISPATCH(rs, {
        hipLaunchKernelGGL((k_atomic_scatter_T<G_, C_>), dim3((unsigned)blocks), dim3(kBlock), 0,
                           s, t, ctl, a, neg, coef);
    });
    return hipGetLastError();
}

hipError_t launch_atomic_scatter_S(const TableArgs& t, Control* ctl, const StepArgs& a,
                                   const float* gsrc, hipStream_t s) {
    const RowShape rs = row_shape(t.D);
    const int64_t blocks = blocks_for(t.D, a.n);
    if (blocks == 0) return hipSuccess;
    HUGE_ROW_DISPATCH(rs, {
        hipLaunchKernelGGL((k_atomic_scatter_S<G_, C_>), dim3((unsigned)blocks), dim3(kBlock), 0,
                           s, t, ctl, a, gsrc);
    });
    return hipGetLastError();
}

hipError_t launch_eval(const TableArgs& t, Control* ctl, const StepArgs& a, double* lossp,
                       int64_t* blocks_out, hipStream_t s) {
    const bool pairs = uses_pairs(t.dtype, t.D);
    const int64_t ppb = kBlock / (pairs ? pair_shape(t.D).G : row_shape(t.D).G);
    const int64_t blocks = (a.n + ppb - 1) / ppb;
    *blocks_out = blocks;
    if (blocks == 0) return hipSuccess;
    if (pairs) {
        HUGE_PAIR_DISPATCH(pair_shape(t.D), {
            HUGE_NEG_DISPATCH(neg_block(t.K), {
                hipLaunchKernelGGL((k_eval<G_, NB_, PairIO<G_, U_, bf16_t>>),
                                   dim3((unsigned)blocks), dim3(kBlock), 0, s, t, ctl, a, lossp);
            });
        });
    } else {
        HUGE_ROW_DISPATCH(row_shape(t.D), {
            HUGE_NEG_DISPATCH(neg_block(t.K), {
                HUGE_ELEM_DISPATCH(t.dtype, {
                    hipLaunchKernelGGL((k_eval<G_, NB_, RowIO<G_, C_, E_>>),
                                       dim3((unsigned)blocks), dim3(kBlock), 0, s, t, ctl, a,
                                       lossp);
                });
            });
        });
    }
    return hipGetLastError();
}

}  // namespace huge
