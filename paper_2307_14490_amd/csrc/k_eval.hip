// Unsupervised evaluation of an embedding table (HUGE Sec. 4): the rows are
// L2-normalised and compared by Euclidean distance;
//   - edge SNR: mean distance over a random sample of non-edges divided by the
//     mean over a sample of edges, with the distribution of both (percentiles);
//   - sampled edge recall: for a few query nodes u, the k rows nearest to u
//     form S, and recall@k(u) = |N(u) & S| / k.
// Kernels:
//   k_eval_pairs    edge and non-edge pairs from counter-based Philox draws
//   k_eval_dist     distances of normalised rows, G lanes per pair
//   k_sum_*         the summary: means, SNR and percentiles (a radix selection
//                   of the order statistics on the float bit patterns);
//   k_knn_queries   the normalised query rows;
//   k_knn_tiles_h   distances of every row to every query (32 queries x 32 rows
//                   per tile) for dim <= 128: rows and queries split into two
//                   fp16 parts on the fp16 matrix cores; per-wave top-k lists;
//   k_knn_tiles     the same for wider rows: fp32 matrix cores, queries in LDS;
//   k_knn_scan      threshold scans for dim <= 128, k_knn_wide_* for wider rows;
//   k_knn_select    the candidates of a scan, sorted: the next scan's bound;
//   k_knn_merge     the k nearest of each query over all lists (bitonic sort);
//   k_eval_recall   recall@k from the nearest rows and the sorted CSR lists.
#include "common.hpp"
#include "device.hpp"
#include "dispatch.hpp"

namespace huge {

__device__ __forceinline__ void eval_fail(int32_t* status, int32_t code) {
    atomicCAS(status, 0, code);
}

// The row whose list holds edge e: the last row r with off[r] <= e, by
// bisection over the offsets (off[0] = 0 <= e < off[N] = E): first over every
// `step`-th of them, `have` entries in LDS, then from a linear guess between
// two of those outwards, by doubling distances, until e is enclosed (the
// lists of one range have about the same length, so most searches touch a cache
// line or two there instead of six).
constexpr int kEdgeIndex = 2048;

__device__ __forceinline__ int64_t edge_row(const int64_t* __restrict__ off, int64_t N,
                                            const int64_t* s_off, int have, int64_t step,
                                            int64_t E, int64_t e) {
    int a = 0, b = have;
    while (b - a > 1) {
        const int mid = a + (b - a) / 2;
        if (s_off[mid] <= e)
            a = mid;
        else
            b = mid;
    }
    int64_t lo = a * step, hi = lo + step < N ? lo + step : N;
    const int64_t o0 = s_off[a], o1 = b < have ? s_off[b] : E;
    if (hi - lo > 8) {
        int64_t g = lo + (int64_t)((float)(e - o0) / (float)(o1 - o0) * (float)(hi - lo));
        g = g < lo ? lo : g < hi ? g : hi - 1;
        if (off[g] <= e) {
            lo = g;
            for (int64_t w = 4; g + w < hi; w *= 2) {
                if (off[g + w] > e) {
                    hi = g + w;
                    break;
                }
                lo = g + w;
            }
        } else {
            hi = g;
            for (int64_t w = 4; g - w > lo; w *= 2) {
                if (off[g - w] <= e) {
                    lo = g - w;
                    break;
                }
                hi = g - w;
            }
        }
    }
    while (hi - lo > 1) {
        const int64_t mid = lo + (hi - lo) / 2;
        if (off[mid] <= e)
            lo = mid;
        else
            hi = mid;
    }
    return lo;
}

// Whether v is in the ascending list nbr[b, e).
__device__ __forceinline__ bool in_sorted_list(const int32_t* __restrict__ nbr, int64_t b,
                                               int64_t e, int32_t v) {
    while (b < e) {
        const int64_t mid = b + (e - b) / 2;
        const int32_t x = nbr[mid];
        if (x == v) return true;
        if (x < v)
            b = mid + 1;
        else
            e = mid;
    }
    return false;
}

// ---------------------------------------------------------------------------
// Pairs.  Edge pair j: Philox counter (lo32 j, hi32 j, 0, kEdgeWord), edge
// index floor(x E / 2^64) with x = (r1 << 32) | r0, the pair (its row, its
// neighbour).  Non-edge pair j: tries a = 0 .. max_tries - 1 with counter
// (lo32 j, hi32 j, a, kNonEdgeWord), u = floor(x0 N / 2^64), v =
// floor(x1 N / 2^64) (x0 = (r1 << 32) | r0, x1 = (r3 << 32) | r2); the first
// try with u != v and v not in u's list, else (-1, -1).
// ---------------------------------------------------------------------------
constexpr uint32_t kEdgeWord = 0x80000001u;
constexpr uint32_t kNonEdgeWord = 0x80000002u;

// Workgroups 0 .. edge_blocks - 1 take the edge pairs, with the upper levels of
// the bisection in LDS (11 of 20 dependent reads for 1e6 nodes), the others
// the non-edge pairs.  1e6 + 1e6 pairs over 1e6 nodes, 2.2e7 edges: 180 us with
// every level read from memory, 152 us now (random lines of the offsets and the
// lists, which no L2 holds).
__global__ __launch_bounds__(kBlock) void k_eval_pairs(
    const int64_t* __restrict__ off, const int32_t* __restrict__ nbr, int64_t N, int64_t E,
    uint64_t seed, int64_t n_edge, int64_t n_non, int32_t max_tries, int edge_blocks,
    int32_t* __restrict__ u_out, int32_t* __restrict__ v_out, int32_t* __restrict__ status) {
    __shared__ int64_t s_off[kEdgeIndex];
    const uint32_t klo = (uint32_t)seed, khi = (uint32_t)(seed >> 32);
    if ((int)blockIdx.x < edge_blocks) {
        const int64_t step = (N + kEdgeIndex - 1) / kEdgeIndex;
        const int have = (int)((N + step - 1) / step);
        for (int j = threadIdx.x; j < have; j += kBlock) s_off[j] = off[j * step];
        __syncthreads();
        const int64_t stride = (int64_t)edge_blocks * kBlock;
        for (int64_t j = (int64_t)blockIdx.x * kBlock + threadIdx.x; j < n_edge; j += stride) {
            const uint4 r = philox4x32_10(make_uint4((uint32_t)j, (uint32_t)((uint64_t)j >> 32),
                                                     0u, kEdgeWord), klo, khi);
            const uint64_t x = ((uint64_t)r.y << 32) | r.x;
            const int64_t e = (int64_t)__umul64hi(x, (uint64_t)E);
            const int32_t v = nbr[e];
            const int64_t row = edge_row(off, N, s_off, have, step, E, e);
            const bool ok = off[row] <= e && e < off[row + 1] && v >= 0 && (int64_t)v < N;
            if (!ok) eval_fail(status, -2);
            u_out[j] = ok ? (int32_t)row : -1;
            v_out[j] = ok ? v : -1;
        }
        return;
    }
    const int64_t jj = (int64_t)((int)blockIdx.x - edge_blocks) * kBlock + threadIdx.x;
    if (jj >= n_non) return;
    int32_t pu = -1, pv = -1;
    for (int32_t a = 0; a < max_tries; ++a) {
        const uint4 r = philox4x32_10(
            make_uint4((uint32_t)jj, (uint32_t)((uint64_t)jj >> 32), (uint32_t)a, kNonEdgeWord),
            klo, khi);
        const int64_t u = (int64_t)__umul64hi(((uint64_t)r.y << 32) | r.x, (uint64_t)N);
        const int64_t v = (int64_t)__umul64hi(((uint64_t)r.w << 32) | r.z, (uint64_t)N);
        if (u == v) continue;
        const int64_t b = off[u], e = off[u + 1];
        if (b < 0 || e < b || e > E) {
            eval_fail(status, -2);
            break;
        }
        if (in_sorted_list(nbr, b, e, (int32_t)v)) continue;
        pu = (int32_t)u;
        pv = (int32_t)v;
        break;
    }
    u_out[n_edge + jj] = pu;
    v_out[n_edge + jj] = pv;
}

hipError_t launch_eval_pairs(const int64_t* off, const int32_t* nbr, int64_t N, int64_t E,
                             uint64_t seed, int64_t n_edge, int64_t n_non, int32_t max_tries,
                             int32_t* u, int32_t* v, int32_t* status, hipStream_t s) {
    const int64_t eb = (n_edge + kBlock - 1) / kBlock, nb = (n_non + kBlock - 1) / kBlock;
    // eight edge workgroups per CU at most: the table is loaded once for each
    const int64_t edge_blocks = eb < 2048 ? eb : 2048;
    if (edge_blocks + nb == 0) return hipSuccess;
    hipLaunchKernelGGL(k_eval_pairs, dim3((unsigned)(edge_blocks + nb)), dim3(kBlock), 0, s, off,
                       nbr, N, E, seed, n_edge, n_non, max_tries, (int)edge_blocks, u, v, status);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Distances: |x_u / |x_u| - x_v / |x_v||, G lanes per pair and C float4 per
// lane (a zero row stays zero); NaN for a pair with a negative id.
// ---------------------------------------------------------------------------
template <int G, int C>
__global__ __launch_bounds__(kBlock) void k_eval_dist(const float* __restrict__ T, int64_t N,
                                                      int32_t D, const int32_t* __restrict__ u,
                                                      const int32_t* __restrict__ v, int64_t n,
                                                      float* __restrict__ out,
                                                      int32_t* __restrict__ status) {
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t p = t / G;  // groups are aligned in the wave and exit together
    const int g = (int)(t % G);
    if (p >= n) return;
    const int32_t a = u[p], b = v[p];
    if (a < 0 || b < 0) {
        if (g == 0) out[p] = __builtin_nanf("");
        return;
    }
    if ((int64_t)a >= N || (int64_t)b >= N) {
        if (g == 0) {
            out[p] = __builtin_nanf("");
            eval_fail(status, -2);
        }
        return;
    }
    const int q4 = D / 4;
    const float4* xa = reinterpret_cast<const float4*>(T + (int64_t)a * D);
    const float4* xb = reinterpret_cast<const float4*>(T + (int64_t)b * D);
    float4 ra[C], rb[C];
    float na = 0.f, nb = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int idx = g + G * c;
        ra[c] = idx < q4 ? xa[idx] : make_float4(0.f, 0.f, 0.f, 0.f);
        rb[c] = idx < q4 ? xb[idx] : make_float4(0.f, 0.f, 0.f, 0.f);
        na += ra[c].x * ra[c].x + ra[c].y * ra[c].y + ra[c].z * ra[c].z + ra[c].w * ra[c].w;
        nb += rb[c].x * rb[c].x + rb[c].y * rb[c].y + rb[c].z * rb[c].z + rb[c].w * rb[c].w;
    }
    na = group_sum<G>(na);
    nb = group_sum<G>(nb);
    const float ia = na > 0.f ? 1.0f / sqrtf(na) : 0.f;
    const float ib = nb > 0.f ? 1.0f / sqrtf(nb) : 0.f;
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const float dx = ra[c].x * ia - rb[c].x * ib, dy = ra[c].y * ia - rb[c].y * ib;
        const float dz = ra[c].z * ia - rb[c].z * ib, dw = ra[c].w * ia - rb[c].w * ib;
        s += dx * dx + dy * dy + dz * dz + dw * dw;
    }
    s = group_sum<G>(s);
    if (g == 0) out[p] = sqrtf(s);
}

hipError_t launch_eval_dist(const float* T, int64_t N, int32_t D, const int32_t* u,
                            const int32_t* v, int64_t n, float* out, int32_t* status,
                            hipStream_t s) {
    if (n == 0) return hipSuccess;
    const RowShape rs = row_shape(D);
    const int64_t threads = n * rs.G;
    const dim3 grid((unsigned)((threads + kBlock - 1) / kBlock));
    HUGE_ROW_DISPATCH(rs, hipLaunchKernelGGL((k_eval_dist<G_, C_>), grid, dim3(kBlock), 0, s, T,
                                             N, D, u, v, n, out, status));
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Summary of n_edge edge distances followed by n_non non-edge distances (set
// 0 and set 1): out[0..4] = count_edge, count_non, mean_edge, mean_non,
// mean_non / mean_edge over the values that are numbers, then the percentiles
// of each set: position h = (count - 1) q / 100 of the ascending values,
// linear between the order statistics around h.  Values are ordered by their
// bit patterns (non-negative floats order as unsigned integers).
//
// Only the 2 nq order statistics of a set are needed, so the values are not
// sorted: they are counted by their upper 16 bits; the bins that hold wanted
// ranks get a slot each, whose values are counted by the next 8 bits, and
// those of the wanted bins there by the last 8.  Three passes over the values
// (a bin of 16 bits is 1/128 of an octave: the wanted ones hold about a tenth
// of them), where the radix sort of each set took eight, with 26 launches of
// at most 122 workgroups: 1e6 + 1e6 distances and 11 percentiles 410 us before,
// 95 us now.
//   k_sum_clear  zeroes the counters;
//   k_sum_hist   sums and 16-bit counts: a workgroup's share of a set in LDS
//                (two 16-bit counters per word, flushed every 32768 values);
//   k_sum_bins   the totals, the wanted ranks and their bins (a workgroup per
//                set);
//   k_sum_count, k_sum_pick  the next 8 bits of the wanted bins, twice; the
//                last pick forms the percentiles.
// ---------------------------------------------------------------------------
constexpr int kSumThreads = 1024;
constexpr int kSumChunk = 32768;  // values per flush of the 16-bit counters
constexpr uint32_t kNoSlot = 0xFFFFu;
// Slots of the counters of 8 bits: 4 per percentile at most; fewer percentiles
// leave room for copies, over which the workgroups are spread (2e6 values of
// 22 wanted bins queued on 180 cache lines: 81 us; with 11 copies 25 us).
constexpr int kSumSlots = 4 * kEvalMaxQuantiles;

inline int sum_copies(int nq) {
    const int c = kSumSlots / (4 * nq);
    return c < 16 ? c : 16;
}

struct Quantiles {
    double q[kEvalMaxQuantiles];
};

// The order statistics around percentile q of count > 0 values.
__device__ __forceinline__ void quantile_place(double q, int64_t count, int64_t* lo, int64_t* hi,
                                               double* frac) {
    const double h = (double)(count - 1) * (q / 100.0);
    int64_t l = (int64_t)floor(h);
    if (l < 0) l = 0;
    if (l > count - 1) l = count - 1;
    *lo = l;
    *hi = l + 1 < count ? l + 1 : count - 1;
    *frac = h - (double)l;
}

__global__ __launch_bounds__(kBlock) void k_sum_clear(uint32_t* __restrict__ bins,
                                                      uint32_t* __restrict__ mid,
                                                      uint32_t* __restrict__ low) {
    const int64_t n1 = 2 * 65536, n2 = (int64_t)kSumSlots * 256;
    const int64_t step = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n1 + 2 * n2; i += step) {
        if (i < n1)
            bins[i] = 0u;
        else if (i < n1 + n2)
            mid[i - n1] = 0u;
        else
            low[i - n1 - n2] = 0u;
    }
}

// Workgroups 0 .. edge_blocks - 1 share set 0, the others set 1.  part[2 b] =
// the sum of workgroup b's values (fixed order), part[2 b + 1] = their number.
__global__ __launch_bounds__(kSumThreads) void k_sum_hist(const float* __restrict__ d,
                                                          int64_t n_edge, int64_t n,
                                                          int edge_blocks,
                                                          uint32_t* __restrict__ bins,
                                                          double* __restrict__ part) {
    extern __shared__ uint32_t s_bin[];  // [32768]: bins 2 j and 2 j + 1
    __shared__ double s_w[2][kSumThreads / 64];
    const int tid = threadIdx.x;
    const bool non = (int)blockIdx.x >= edge_blocks;
    const int b = non ? (int)blockIdx.x - edge_blocks : (int)blockIdx.x;
    const int nb = non ? (int)gridDim.x - edge_blocks : edge_blocks;
    const int64_t first = non ? n_edge : 0, cnt = non ? n - n_edge : n_edge;
    const int64_t per = (cnt + nb - 1) / nb;
    const int64_t i0 = first + b * per;
    const int64_t i1 = b * per + per < cnt ? i0 + per : first + cnt;
    uint32_t* const out = bins + (non ? 65536 : 0);
    double sum = 0.0, num = 0.0;
    for (int64_t c0 = i0; c0 < i1; c0 += kSumChunk) {
        const int64_t c1 = c0 + kSumChunk < i1 ? c0 + kSumChunk : i1;
        for (int j = tid; j < 32768; j += kSumThreads) s_bin[j] = 0u;
        __syncthreads();
        for (int64_t i = c0 + tid; i < c1; i += kSumThreads) {
            const float x = d[i];
            if (x != x) continue;
            sum += (double)x;
            num += 1.0;
            const uint32_t bin = __float_as_uint(x) >> 16;
            atomicAdd(&s_bin[bin >> 1], 1u << (16u * (bin & 1u)));
        }
        __syncthreads();
        for (int j = tid; j < 32768; j += kSumThreads) {
            const uint32_t w = s_bin[j];
            if (w & 0xFFFFu) atomicAdd(&out[2 * j], w & 0xFFFFu);
            if (w >> 16) atomicAdd(&out[2 * j + 1], w >> 16);
        }
        __syncthreads();
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        sum += __shfl_xor(sum, off, 64);
        num += __shfl_xor(num, off, 64);
    }
    if ((tid & 63) == 0) {
        s_w[0][tid >> 6] = sum;
        s_w[1][tid >> 6] = num;
    }
    __syncthreads();
    if (tid < 2) {
        double t = 0.0;
        for (int w = 0; w < kSumThreads / 64; ++w) t += s_w[tid][w];
        part[2 * blockIdx.x + tid] = t;
    }
}

// out[0..4] from the sets' sums and counts.
__device__ __forceinline__ void write_means(double* __restrict__ out, double se, double sn,
                                            double ce, double cn) {
    const double nan = __builtin_nan("");
    const double me = ce > 0.0 ? se / ce : nan, mn = cn > 0.0 ? sn / cn : nan;
    out[0] = ce;
    out[1] = cn;
    out[2] = me;
    out[3] = mn;
    out[4] = (ce > 0.0 && cn > 0.0) ? mn / me : nan;
}

// Workgroup s: set s's totals (workgroup 0 writes out[0..4]), the ranks its
// percentiles need and the bins that hold them.  Rank r of the set is state
// entry s 2 nq + r (r even: the lower statistic of percentile r / 2); a bin's
// slot is the entry of the first rank in it.
__global__ __launch_bounds__(kSumThreads) void k_sum_bins(const uint32_t* __restrict__ bins,
                                                          const double* __restrict__ part,
                                                          int blocks, int edge_blocks,
                                                          Quantiles Q, int nq,
                                                          uint16_t* __restrict__ map,
                                                          SumState st,
                                                          double* __restrict__ out) {
    __shared__ double s_t[4][kEvalSumBlocks];
    __shared__ uint32_t s_wave[kSumThreads / 64];
    __shared__ uint32_t s_rank[2 * kEvalMaxQuantiles], s_found[2 * kEvalMaxQuantiles],
        s_rest[2 * kEvalMaxQuantiles];
    const int tid = threadIdx.x, set = blockIdx.x, nr = 2 * nq;
    if (tid < kEvalSumBlocks) {
        const bool have = tid < blocks, non = tid >= edge_blocks;
        const double a = have ? part[2 * tid] : 0.0, c = have ? part[2 * tid + 1] : 0.0;
        s_t[0][tid] = non ? 0.0 : a;
        s_t[1][tid] = non ? a : 0.0;
        s_t[2][tid] = non ? 0.0 : c;
        s_t[3][tid] = non ? c : 0.0;
    }
    __syncthreads();
    for (int w = kEvalSumBlocks / 2; w > 0; w >>= 1) {
        if (tid < 4 * w) s_t[tid / w][tid % w] += s_t[tid / w][tid % w + w];
        __syncthreads();
    }
    const double se = s_t[0][0], sn = s_t[1][0], ce = s_t[2][0], cn = s_t[3][0];
    if (set == 0 && tid == 0) write_means(out, se, sn, ce, cn);
    const int64_t count = (int64_t)(set ? cn : ce);
    if (tid < nr) {
        int64_t lo = 0, hi = 0;
        double frac;
        if (count > 0) quantile_place(Q.q[tid >> 1], count, &lo, &hi, &frac);
        s_rank[tid] = (uint32_t)(tid & 1 ? hi : lo);
        s_found[tid] = 0u;
        s_rest[tid] = 0u;
    }
    // this thread's 64 bins, and the values before them
    const uint4* mine = reinterpret_cast<const uint4*>(bins + set * 65536 + tid * 64);
    uint32_t sum = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
        const uint4 v = mine[j];
        sum += v.x + v.y + v.z + v.w;
    }
    const int lane = tid & 63, wave = tid >> 6;
    uint32_t incl = sum;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, 64);
        if (lane >= off) incl += t;
    }
    if (lane == 63) s_wave[wave] = incl;
    // the map of this set: no slots
    uint4* mw = reinterpret_cast<uint4*>(map + set * 65536);
#pragma unroll
    for (int j = 0; j < 8; ++j)
        mw[j * kSumThreads + tid] = make_uint4(~0u, ~0u, ~0u, ~0u);
    __threadfence_block();
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += s_wave[w];
    const uint32_t base = incl - sum;
    // the 64 bins that hold a rank, then a wave finds the bin among them
    if (sum > 0u) {
        for (int r = 0; r < nr; ++r) {
            const uint32_t rank = s_rank[r];
            if (rank < base || rank - base >= sum) continue;
            s_found[r] = (uint32_t)tid;
            s_rest[r] = rank - base;
        }
    }
    __syncthreads();
    for (int r = wave; r < nr; r += kSumThreads / 64) {
        const uint32_t owner = s_found[r], rest = s_rest[r];
        const uint32_t c = bins[set * 65536 + owner * 64u + (uint32_t)lane];
        uint32_t end = c;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t t = __shfl_up(end, off, 64);
            if (lane >= off) end += t;
        }
        if (rest < end && rest >= end - c) {
            s_found[r] = owner * 64u + (uint32_t)lane;
            s_rest[r] = rest - (end - c);
        }
    }
    __syncthreads();
    if (tid < nr) {
        const int e = set * nr + tid;
        int first = 0;
        while (s_found[first] != s_found[tid]) ++first;  // ends at tid
        st.slot[e] = count > 0 ? (uint32_t)(set * nr + first) : kNoSlot;
        st.rest[e] = s_rest[tid];
        st.prefix[e] = s_found[tid];
        if (count > 0 && first == tid) map[set * 65536 + s_found[tid]] = (uint16_t)e;
    }
}

// Count value key at counters[at] for the lanes with `want` (the whole wave
// calls it): equal counters of a wave are added once, twice over, so that sets
// of few distinct values do not queue on one counter.
__device__ __forceinline__ void count_wave(uint32_t* __restrict__ counters, uint32_t at,
                                           bool want) {
#pragma unroll
    for (int round = 0; round < 2; ++round) {
        const uint64_t left = __ballot(want);
        if (left == 0ull) return;  // uniform
        const int lead = __ffsll((long long)left) - 1;
        const bool same = want && at == (uint32_t)__shfl((int)at, lead, 64);
        const uint64_t all = __ballot(same);
        if ((int)(threadIdx.x & 63u) == lead) atomicAdd(&counters[at], (uint32_t)__popcll(all));
        want = want && !same;
    }
    if (want) atomicAdd(&counters[at], 1u);
}

// Level 1: the values of the wanted 16-bit bins by their next 8 bits; level 2:
// those of the wanted bins there by their last 8.
template <int LEVEL>
__global__ __launch_bounds__(kBlock) void k_sum_count(const float* __restrict__ d, int64_t n_edge,
                                                      int64_t n,
                                                      const uint16_t* __restrict__ map,
                                                      const uint16_t* __restrict__ map2,
                                                      uint32_t* __restrict__ counters, int slots,
                                                      int copies) {
    counters += (size_t)(blockIdx.x % (unsigned)copies) * slots * 256;
    const int64_t step = (int64_t)gridDim.x * kBlock;
    for (int64_t i0 = (int64_t)blockIdx.x * kBlock; i0 < n; i0 += step) {  // uniform
        const int64_t i = i0 + threadIdx.x;
        const float x = i < n ? d[i] : __builtin_nanf("");
        const uint32_t key = __float_as_uint(x);
        uint32_t slot = kNoSlot;
        if (x == x) slot = map[(i < n_edge ? 0u : 65536u) + (key >> 16)];
        uint32_t digit = key >> 8 & 255u;
        if (LEVEL == 2 && slot != kNoSlot) {
            slot = map2[slot * 256u + digit];
            digit = key & 255u;
        }
        count_wave(counters, slot * 256u + digit, slot != kNoSlot);
    }
}

// The digit of every wanted rank among its slot's counters, a wave per rank.
// Level 1: the ranks' slots of the next level and their map; level 2: the
// order statistics, from which the percentiles.
template <int LEVEL>
__global__ __launch_bounds__(kSumThreads) void k_sum_pick(const uint32_t* __restrict__ counters,
                                                          Quantiles Q, int nq,
                                                          int copies,
                                                          uint16_t* __restrict__ map2,
                                                          SumState st,
                                                          double* __restrict__ out) {
    __shared__ uint32_t s_slot[kSumSlots], s_digit[kSumSlots];
    __shared__ float s_val[kSumSlots];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nr = 4 * nq;
    for (int r = wave; r < nr; r += kSumThreads / 64) {
        const uint32_t slot = st.slot[r];
        if (lane == 0) s_slot[r] = slot;
        if (slot == kNoSlot) continue;  // an empty set
        const uint32_t rest = st.rest[r];
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        for (int k = 0; k < copies; ++k) {
            const uint4 a = reinterpret_cast<const uint4*>(
                counters + ((uint32_t)(k * nr) + slot) * 256u)[lane];
            v = make_uint4(v.x + a.x, v.y + a.y, v.z + a.z, v.w + a.w);
        }
        const uint32_t c[4] = {v.x, v.y, v.z, v.w};
        uint32_t incl = v.x + v.y + v.z + v.w;
        const uint32_t sum = incl;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t t = __shfl_up(incl, off, 64);
            if (lane >= off) incl += t;
        }
        const uint32_t base = incl - sum;
        if (rest >= base && rest - base < sum) {
            uint32_t left = rest - base, j = 0;
#pragma unroll
            for (int e = 0; e < 3; ++e) {
                if (j == (uint32_t)e && left >= c[e]) {
                    left -= c[e];
                    ++j;
                }
            }
            const uint32_t digit = (uint32_t)lane * 4u + j;
            s_digit[r] = digit;
            const uint32_t prefix = st.prefix[r] << 8 | digit;
            if (LEVEL == 1) {
                st.rest[r] = left;
                st.prefix[r] = prefix;
            } else {
                s_val[r] = __uint_as_float(prefix);
            }
        }
        if (LEVEL == 1 && slot == (uint32_t)r)  // the slot's map: no slots
            reinterpret_cast<uint2*>(map2 + slot * 256u)[lane] = make_uint2(~0u, ~0u);
    }
    __threadfence_block();
    __syncthreads();
    if (LEVEL == 1) {
        if (tid < nr && s_slot[tid] != kNoSlot) {
            int first = 0;
            while (s_slot[first] != s_slot[tid] || s_digit[first] != s_digit[tid]) ++first;
            st.slot[tid] = (uint32_t)first;
            if (first == tid) map2[s_slot[tid] * 256u + s_digit[tid]] = (uint16_t)tid;
        }
    } else if (tid < 2 * nq) {
        const int set = tid / nq, i = tid - set * nq;
        const int64_t count = (int64_t)out[set];
        double v = __builtin_nan("");
        if (count > 0) {
            int64_t lo, hi;
            double frac;
            quantile_place(Q.q[i], count, &lo, &hi, &frac);
            const double a = (double)s_val[2 * tid], b = (double)s_val[2 * tid + 1];
            v = a + frac * (b - a);
        }
        out[5 + tid] = v;
    }
}

// The same for a workspace that does not hold the counters (below about 233,000
// distances the size asked for is less than they take): one workgroup per set,
// the selection in LDS, eight bits at a time from the top, and no workspace.
// The values are read once per level and 128 slots, so it takes the longer the
// more there are (1,000, 10,000, 100,000, 230,000 distances and 11 percentiles: 23,
// 32, 148, 331 us; with the counters 63 to 64).  The sums are formed in k_sum_hist's and
// k_sum_bins's order: the same bits.
//   s_bin    [128][256] counters of a level's slots, 128 slots at a time
//   s_order  the ranks in ascending order, so that the values found so far
//            (s_pre, their upper bits) ascend too and a value's slot among the
//            distinct ones (s_uniq) is found by bisection
constexpr int kSmallSlots = 128;
constexpr int kSmallLoads = 8;  // values of a thread in flight

// fn(value) for every value that is a number in d[i0 .. i1), thread by thread
// in strides of the workgroup.
template <typename Fn>
__device__ __forceinline__ void small_values(const float* __restrict__ d, int64_t i0, int64_t i1,
                                             Fn fn) {
    for (int64_t c = i0 + threadIdx.x; c < i1; c += kSmallLoads * kSumThreads) {
        float x[kSmallLoads];
#pragma unroll
        for (int j = 0; j < kSmallLoads; ++j) {
            const int64_t i = c + j * kSumThreads;
            x[j] = i < i1 ? d[i] : __builtin_nanf("");
        }
#pragma unroll
        for (int j = 0; j < kSmallLoads; ++j)
            if (x[j] == x[j]) fn(x[j]);
    }
}

__global__ __launch_bounds__(kSumThreads) void k_sum_small(const float* __restrict__ d,
                                                           int64_t n_edge, int64_t n,
                                                           int edge_blocks, int blocks,
                                                           Quantiles Q, int nq,
                                                           double* __restrict__ out) {
    extern __shared__ uint32_t s_bin[];  // [kSmallSlots][256]
    __shared__ double s_t[4][kEvalSumBlocks];
    __shared__ double s_w[2][kSumThreads / 64];
    constexpr int kRanks = 2 * kEvalMaxQuantiles;
    __shared__ uint32_t s_rank[kRanks], s_rest[kRanks], s_pre[kRanks], s_uniq[kRanks];
    __shared__ uint16_t s_order[kRanks], s_slot[kRanks];
    __shared__ int s_slots;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int set = blockIdx.x, nr = 2 * nq;
    // the sums of both sets, part by part as k_sum_hist's workgroups form them
    if (tid < kEvalSumBlocks)
        for (int c = 0; c < 4; ++c) s_t[c][tid] = 0.0;
    __syncthreads();
    for (int p = 0; p < blocks; ++p) {
        const bool non = p >= edge_blocks;
        const int b = non ? p - edge_blocks : p, nb = non ? blocks - edge_blocks : edge_blocks;
        const int64_t first = non ? n_edge : 0, cnt = non ? n - n_edge : n_edge;
        const int64_t per = (cnt + nb - 1) / nb;
        const int64_t i0 = first + b * per;
        const int64_t i1 = b * per + per < cnt ? i0 + per : first + cnt;
        double sum = 0.0, num = 0.0;
        small_values(d, i0, i1, [&](float x) {
            sum += (double)x;
            num += 1.0;
        });
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            sum += __shfl_xor(sum, off, 64);
            num += __shfl_xor(num, off, 64);
        }
        if (lane == 0) {
            s_w[0][wave] = sum;
            s_w[1][wave] = num;
        }
        __syncthreads();
        if (tid < 2) {
            double t = 0.0;
            for (int w = 0; w < kSumThreads / 64; ++w) t += s_w[tid][w];
            s_t[2 * tid + (non ? 1 : 0)][p] = t;
        }
        __syncthreads();
    }
    for (int w = kEvalSumBlocks / 2; w > 0; w >>= 1) {
        if (tid < 4 * w) s_t[tid / w][tid % w] += s_t[tid / w][tid % w + w];
        __syncthreads();
    }
    const double se = s_t[0][0], sn = s_t[1][0], ce = s_t[2][0], cn = s_t[3][0];
    if (set == 0 && tid == 0) write_means(out, se, sn, ce, cn);
    const int64_t count = (int64_t)(set ? cn : ce);
    if (count == 0 || nq == 0) {  // uniform
        if (tid < nq) out[5 + set * nq + tid] = __builtin_nan("");
        return;
    }
    // the wanted ranks, ascending
    if (tid < nr) {
        int64_t lo, hi;
        double frac;
        quantile_place(Q.q[tid >> 1], count, &lo, &hi, &frac);
        s_rank[tid] = (uint32_t)(tid & 1 ? hi : lo);
    }
    __syncthreads();
    if (tid < nr) {
        const uint32_t mine = s_rank[tid];
        int at = 0;
        for (int j = 0; j < nr; ++j)
            at += s_rank[j] < mine || (s_rank[j] == mine && j < tid) ? 1 : 0;
        s_order[at] = (uint16_t)tid;
        s_rest[at] = mine;
        s_pre[at] = 0u;
    }
    __syncthreads();
    const int64_t i0 = set ? n_edge : 0, i1 = set ? n : n_edge;
    for (int shift = 24; shift >= 0; shift -= 8) {
        // the distinct values of the bits above, ascending: the level's slots
        if (tid < nr) {
            int slot = 0;
            for (int j = 1; j <= tid; ++j) slot += s_pre[j] != s_pre[j - 1] ? 1 : 0;
            s_slot[tid] = (uint16_t)slot;
            s_uniq[slot] = s_pre[tid];
            if (tid == nr - 1) s_slots = slot + 1;
        }
        __syncthreads();
        const int slots = s_slots;
        for (int g0 = 0; g0 < slots; g0 += kSmallSlots) {
            const int g1 = g0 + kSmallSlots < slots ? g0 + kSmallSlots : slots;
            for (int j = tid; j < kSmallSlots * 256; j += kSumThreads) s_bin[j] = 0u;
            __syncthreads();
            small_values(d, i0, i1, [&](float x) {
                const uint32_t key = __float_as_uint(x);
                // (all of the value, shifted out, at the first level)
                const uint32_t above = shift == 24 ? 0u : key >> (shift + 8);
                int lo = g0, hi = g1;  // the first slot not below
                while (lo < hi) {
                    const int mid = (lo + hi) / 2;
                    if (s_uniq[mid] < above)
                        lo = mid + 1;
                    else
                        hi = mid;
                }
                if (lo < g1 && s_uniq[lo] == above)
                    atomicAdd(&s_bin[(lo - g0) * 256 + (int)(key >> shift & 255u)], 1u);
            });
            __syncthreads();
            // a wave per rank: its digit among the slot's counters
            for (int r = wave; r < nr; r += kSumThreads / 64) {
                const int slot = s_slot[r];
                if (slot < g0 || slot >= g1) continue;
                const uint32_t* const bin = s_bin + (slot - g0) * 256 + lane * 4;
                const uint32_t c[4] = {bin[0], bin[1], bin[2], bin[3]};
                const uint32_t sum = c[0] + c[1] + c[2] + c[3], rest = s_rest[r];
                uint32_t incl = sum;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) {
                    const uint32_t t = __shfl_up(incl, off, 64);
                    if (lane >= off) incl += t;
                }
                const uint32_t base = incl - sum;
                if (rest >= base && rest - base < sum) {
                    uint32_t left = rest - base, j = 0;
                    while (j < 3u && left >= c[j]) left -= c[j++];
                    s_rest[r] = left;
                    s_pre[r] = s_pre[r] << 8 | ((uint32_t)lane * 4u + j);
                }
            }
            __syncthreads();
        }
    }
    // s_pre holds the order statistics' bits: back to the percentiles' order
    if (tid < nr) s_rank[s_order[tid]] = s_pre[tid];
    __syncthreads();
    if (tid < nq) {
        int64_t lo, hi;
        double frac;
        quantile_place(Q.q[tid], count, &lo, &hi, &frac);
        const double a = (double)__uint_as_float(s_rank[2 * tid]);
        const double b = (double)__uint_as_float(s_rank[2 * tid + 1]);
        out[5 + set * nq + tid] = a + frac * (b - a);
    }
}

hipError_t launch_eval_summary(const float* d, int64_t n_edge, int64_t n_non, const double* q,
                               int nq, const SumBuffers& B, bool have_counters, double* out,
                               hipStream_t s) {
    if (nq < 0 || nq > kEvalMaxQuantiles) return hipErrorInvalidValue;
    const int64_t n = n_edge + n_non;
    Quantiles Q;
    for (int i = 0; i < nq; ++i) Q.q[i] = q[i];
    // workgroups of each set: 8192 values each, at most half of kEvalSumBlocks
    auto blocks_of = [](int64_t m) {
        const int64_t b = (m + 8191) / 8192;
        return (int)(b < kEvalSumBlocks / 2 ? b : kEvalSumBlocks / 2);
    };
    const int eb = blocks_of(n_edge), blocks = eb + blocks_of(n_non);
    if (!have_counters) {
        constexpr size_t kLds = sizeof(uint32_t) * kSmallSlots * 256;
        const hipError_t e = allow_lds<&k_sum_small>(kLds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_sum_small, dim3(2), dim3(kSumThreads), kLds, s, d, n_edge, n, eb,
                           blocks, Q, nq, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_sum_clear, dim3(128), dim3(kBlock), 0, s, B.bins, B.mid, B.low);
    if (blocks > 0) {
        constexpr size_t kLds = sizeof(uint32_t) * 32768;
        const hipError_t e = allow_lds<&k_sum_hist>(kLds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_sum_hist, dim3((unsigned)blocks), dim3(kSumThreads), kLds, s, d,
                           n_edge, n, eb, B.bins, B.part);
    }
    hipLaunchKernelGGL(k_sum_bins, dim3(2), dim3(kSumThreads), 0, s, B.bins, B.part, blocks, eb,
                       Q, nq, B.map, B.state, out);
    if (nq > 0) {
        const int copies = sum_copies(nq);
        if (n > 0) {
            int64_t grid = (n + kBlock - 1) / kBlock;
            grid = grid < 2048 ? grid : 2048;
            hipLaunchKernelGGL(k_sum_count<1>, dim3((unsigned)grid), dim3(kBlock), 0, s, d,
                               n_edge, n, B.map, B.map2, B.mid, 4 * nq, copies);
            hipLaunchKernelGGL(k_sum_pick<1>, dim3(1), dim3(kSumThreads), 0, s, B.mid, Q, nq,
                               copies, B.map2, B.state, out);
            hipLaunchKernelGGL(k_sum_count<2>, dim3((unsigned)grid), dim3(kBlock), 0, s, d,
                               n_edge, n, B.map, B.map2, B.low, 4 * nq, copies);
        }
        hipLaunchKernelGGL(k_sum_pick<2>, dim3(1), dim3(kSumThreads), 0, s, B.low, Q, nq, copies,
                           B.map2, B.state, out);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Nearest rows of up to kKnnPass queries per pass over the table.
// ---------------------------------------------------------------------------
// Normalised query rows qn[j * D ..] (zero for a zero row or a padding slot)
// and qn2[j] = |qn_j|^2 in {0, 1}; with the threshold scans, their state: no
// candidates, the bound +inf (-inf for a padding slot: nothing passes it) and
// the fallback gate closed.  A query row whose squared norm is no normal
// number (not finite, or so small that its sum has lost bits) is not of
// length 1 after the scaling, which the screens' bounds take for granted: its
// bound is -inf too, and k_knn_select opens the gate for it.  qh (if not null)
// receives the queries' fp16 parts as matrix operands.
constexpr float kKnnSplitScale = 1024.0f;  // 2^10: the scale of the fp16 parts
// Squared norms between these have kept their precision: squares below 2^-149
// are lost, at most dim 2^-150 in all, 2^-40 of the smallest.
constexpr float kKnnNormMin = 1e-30f, kKnnNormMax = 1e38f;

__global__ __launch_bounds__(kBlock) void k_knn_queries(const float* __restrict__ T, int64_t N,
                                                        int32_t D, const int32_t* __restrict__ q,
                                                        int32_t nq, int32_t nqp,
                                                        float* __restrict__ qn,
                                                        float* __restrict__ qn2,
                                                        int32_t* __restrict__ qid,
                                                        float* __restrict__ tau,
                                                        uint32_t* __restrict__ cnt,
                                                        int32_t cnt_stride,
                                                        int32_t* __restrict__ gate,
                                                        _Float16* __restrict__ qh,
                                                        int32_t* __restrict__ status) {
    __shared__ float s_red[kBlock];
    const int j = blockIdx.x;
    if (j >= nqp) return;
    int32_t id = j < nq ? q[j] : -1;
    if (id >= 0 && (int64_t)id >= N) {
        if (threadIdx.x == 0) eval_fail(status, -2);
        id = -1;
    }
    if (j < nq && id < 0 && q[j] < 0 && threadIdx.x == 0) eval_fail(status, -2);
    float part = 0.f;
    for (int c = threadIdx.x; c < D; c += kBlock) {
        const float x = id >= 0 ? T[(int64_t)id * D + c] : 0.f;
        part += x * x;
    }
    s_red[threadIdx.x] = part;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) s_red[threadIdx.x] += s_red[threadIdx.x + w];
        __syncthreads();
    }
    const float n2 = s_red[0];
    const float inv = n2 > 0.f ? 1.0f / sqrtf(n2) : 0.f;
    for (int c = threadIdx.x; c < D; c += kBlock)
        qn[(int64_t)j * D + c] = id >= 0 ? T[(int64_t)id * D + c] * inv : 0.f;
    if (qh != nullptr) {
        // matrix operands: element e of lane x + 32 h of chunk c of query
        // block j / 32 is dimension 16 c + 8 h + e of query j = 32 (j / 32) + x
        const int nc = (D + 15) / 16, x = j & 31;
        for (int d = threadIdx.x; d < 16 * nc; d += kBlock) {
            const float v = id >= 0 && d < D ? T[(int64_t)id * D + d] * inv : 0.f;
            const int lane = x + 32 * ((d >> 3) & 1);
            qh[(((size_t)(j >> 5) * nc + (d >> 4)) * 64 + lane) * 8 + (d & 7)] =
                (_Float16)(v * kKnnSplitScale);
        }
    }
    if (threadIdx.x == 0) {
        qn2[j] = n2 > 0.f ? 1.f : 0.f;
        qid[j] = id;
        if (cnt) {
            cnt[j * cnt_stride] = 0u;
            const bool screened = n2 == 0.f || (n2 >= kKnnNormMin && n2 <= kKnnNormMax);
            tau[j] = id >= 0 && screened ? __builtin_inff() : -__builtin_inff();
        }
        if (gate && j == 0) *gate = 0;
    }
}

typedef float knn_acc16 __attribute__((ext_vector_type(16)));

// The exact products of the search for wide rows (dim > 128): lane (x, h)
// holds dimensions c 128 + h 64 + 4 m .. + 3 (m < 16) of its row of the A and
// of the B operand, from a(dim) and b(dim) (float4; past dim, zeros); chunk by
// chunk, v_mfma_f32_32x32x2f32 per component, even m in one accumulation
// chain, odd m in another.  The row's squared norm (its B operand) is one
// fixed sequence of fused multiply-adds per lane, added to the other half's.
// Every kernel of this search forms a pair's distance this way, so all give
// the same bits.
template <typename LoadA, typename LoadB>
__device__ __forceinline__ void knn_exact_products(int D, int h, LoadA a, LoadB b,
                                                   knn_acc16& acc, float& nr) {
    constexpr int kQ4 = kKnnDimChunk / 8;  // float4 of a lane's half row
    knn_acc16 acc1;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = acc1[r] = 0.f;
    nr = 0.f;
    for (int c = 0; c < D; c += kKnnDimChunk) {
        const int d0 = c + h * (kKnnDimChunk / 2);
        float4 bv[kQ4];
#pragma unroll
        for (int m = 0; m < kQ4; ++m)
            bv[m] = d0 + 4 * m < D ? b(d0 + 4 * m) : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int m = 0; m < kQ4; ++m) {
            float t = bv[m].x * bv[m].x;
            t = fmaf(bv[m].y, bv[m].y, t);
            t = fmaf(bv[m].z, bv[m].z, t);
            t = fmaf(bv[m].w, bv[m].w, t);
            nr += t;
            const float4 av = d0 + 4 * m < D ? a(d0 + 4 * m) : make_float4(0.f, 0.f, 0.f, 0.f);
            knn_acc16& s = m % 2 == 0 ? acc : acc1;
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(av.x, bv[m].x, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(av.y, bv[m].y, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(av.z, bv[m].z, s, 0, 0, 0);
            s = __builtin_amdgcn_mfma_f32_32x32x2f32(av.w, bv[m].w, s, 0, 0, 0);
        }
    }
    acc += acc1;
    nr += __shfl_xor(nr, 32, 64);
}

// d^2 = |q|^2 + [row != 0] - 2 <q, row> / |row|, clamped at 0 (also where it
// is not a number).
__device__ __forceinline__ float knn_exact_d2(float q2, float nr, float dot) {
    const float inv = nr > 0.f ? 1.0f / sqrtf(nr) : 0.f;
    const float nx = nr > 0.f ? 1.f : 0.f;
    const float d2 = fmaf(-2.f * dot, inv, q2 + nx);
    return d2 > 0.f ? d2 : 0.f;
}

// The list search for wide rows.  One workgroup of kKnnWaves waves, the
// queries of a sub-pass (32 QB of them) in LDS; wave w serves query block
// w % QB over tiles t = S, S + NS, ... of 32 rows, S = its list slot.  Keys
// (bits of d^2) << 32 | row below the query's current k-th best are staged per
// query (at most 32 per tile) and inserted by the query's own lane into its
// sorted list of k.  Sub-pass p's lists go to
// partial[((p NS + S) * 32 QB + q) * k + t].
struct KnnArgs {
    const float* T;
    int64_t N;
    int32_t D;
    int32_t k;
    int32_t nqp;   // queries in this pass (wide rows: sub-pass), padded to 32 * QB
    int32_t QB;    // query blocks: 1, 2 or 4
    int32_t subs;  // wide rows: sub-passes of nqp queries each
    int32_t stride;  // LDS floats per query row (D + 4)
    int64_t tiles;
    const float* qn;
    const float* qn2;
    const int32_t* qid;
    uint64_t* partial;
    const int32_t* gate;  // null: always run; else run only where *gate != 0
};

constexpr uint64_t kNoKey = ~0ull;

__global__ __launch_bounds__(kKnnWaves * 64) void k_knn_tiles(KnnArgs A) {
    __shared__ __align__(16) float s_q[kKnnQueryFloats];
    __shared__ uint64_t s_list[kKnnWaves][32][kKnnMaxK];
    __shared__ uint64_t s_stage[kKnnWaves][32][32];
    __shared__ uint64_t s_thr[kKnnWaves][32];
    __shared__ uint32_t s_cnt[kKnnWaves][32];
    __shared__ uint32_t s_len[kKnnWaves][32];
    __shared__ float s_qn2[kKnnPass];
    __shared__ int32_t s_qid[kKnnPass];

    if (A.gate && *A.gate == 0) return;  // the threshold scans answered every query
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int x = lane & 31, h = lane >> 5;
    const int D = A.D, k = A.k, stride = A.stride;
    const int qb = w % A.QB;
    const int wpb = kKnnWaves / A.QB;  // waves per query block
    const int64_t S = (int64_t)blockIdx.x * wpb + w / A.QB;
    const int64_t NS = (int64_t)gridDim.x * wpb;
    for (int sub = 0; sub < A.subs; ++sub) {
    const int q0 = sub * A.nqp;  // the sub-pass's first query
    __syncthreads();  // LDS of the previous sub-pass
    for (int64_t i = tid; i < (int64_t)A.nqp * D; i += kKnnWaves * 64)
        s_q[(i / D) * stride + (i % D)] = A.qn[(int64_t)q0 * D + i];
    for (int i = tid; i < A.nqp; i += kKnnWaves * 64) {
        s_qn2[i] = A.qn2[q0 + i];
        s_qid[i] = A.qid[q0 + i];
    }
    if (lane < 32) {
        s_thr[w][lane] = kNoKey;
        s_cnt[w][lane] = 0u;
        s_len[w][lane] = 0u;
    }
    __syncthreads();
    const float* qrow = s_q + (qb * 32 + x) * stride;
    for (int64_t t = S; t < A.tiles; t += NS) {
        const int64_t row = t * 32 + x;
        const bool row_ok = row < A.N;
        const float* src = A.T + (row_ok ? row : 0) * (int64_t)D;
        knn_acc16 acc;
        float nr;
        knn_exact_products(
            D, h, [&](int d) { return *reinterpret_cast<const float4*>(qrow + d); },
            [&](int d) { return *reinterpret_cast<const float4*>(src + d); }, acc, nr);
        // lane (x, h) holds query i = 8 (r / 4) + 4 h + r % 4 against row x
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = 8 * (r / 4) + 4 * h + (r % 4);
            const int q = qb * 32 + i;
            const float d2 = knn_exact_d2(s_qn2[q], nr, acc[r]);
            const bool ok = row_ok && s_qid[q] >= 0 && row != (int64_t)s_qid[q];
            const uint64_t key =
                ok ? (((uint64_t)__float_as_uint(d2) << 32) | (uint64_t)row) : kNoKey;
            if (key < s_thr[w][i]) {
                const uint32_t pos = atomicAdd(&s_cnt[w][i], 1u);
                s_stage[w][i][pos] = key;  // pos < 32: one row per lane x
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
        if (h == 0) {
            const uint32_t c = s_cnt[w][x];
            if (c > 0u) {
                uint64_t* L = s_list[w][x];
                uint32_t len = s_len[w][x];
                for (uint32_t e = 0; e < c; ++e) {
                    const uint64_t key = s_stage[w][x][e];
                    if (len == (uint32_t)k && key >= L[k - 1]) continue;
                    int p = len < (uint32_t)k ? (int)len : k - 1;
                    while (p > 0 && L[p - 1] > key) {
                        L[p] = L[p - 1];
                        --p;
                    }
                    L[p] = key;
                    if (len < (uint32_t)k) ++len;
                }
                s_len[w][x] = len;
                s_cnt[w][x] = 0u;
                s_thr[w][x] = len == (uint32_t)k ? L[k - 1] : kNoKey;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
    }
    if (h == 0) {
        const uint32_t len = s_len[w][x];
        uint64_t* dst =
            A.partial + (((size_t)sub * NS + S) * A.nqp + qb * 32 + x) * k;
        for (int t = 0; t < k; ++t) dst[t] = (uint32_t)t < len ? s_list[w][x][t] : kNoKey;
    }
    }  // sub-passes
}

// The k smallest keys of query q over all NS lists: running best k plus a
// chunk of candidates, bitonic-sorted together in LDS.
__global__ __launch_bounds__(kBlock) void k_knn_merge(const uint64_t* __restrict__ partial,
                                                      int64_t NS, int32_t nqp, int32_t k,
                                                      int32_t q_first, int32_t* __restrict__ ids,
                                                      float* __restrict__ dist,
                                                      const int32_t* __restrict__ gate) {
    __shared__ uint64_t s_buf[kKnnMergeCap];
    if (gate && *gate == 0) return;
    // query q of the pass is query q % nqp of sub-pass q / nqp
    const int q = blockIdx.x % nqp;
    partial += (size_t)(blockIdx.x / nqp) * NS * nqp * k;
    const int64_t total = NS * k;
    for (int i = threadIdx.x; i < k; i += kBlock) s_buf[i] = kNoKey;
    for (int64_t base = 0; base < total; base += kKnnMergeCap - k) {
        const int64_t chunk =
            total - base < kKnnMergeCap - k ? total - base : (int64_t)(kKnnMergeCap - k);
        for (int i = threadIdx.x; i < kKnnMergeCap - k; i += kBlock) {
            uint64_t v = kNoKey;
            if (i < chunk) {
                const int64_t c = base + i;
                v = partial[((c / k) * nqp + q) * k + (c % k)];
            }
            s_buf[k + i] = v;
        }
        __syncthreads();
        for (int size = 2; size <= kKnnMergeCap; size <<= 1) {
            for (int st = size >> 1; st > 0; st >>= 1) {
                for (int i = threadIdx.x; i < kKnnMergeCap / 2; i += kBlock) {
                    const int lo = 2 * i - (i & (st - 1));
                    const int hi = lo + st;
                    const bool up = (lo & size) == 0;
                    const uint64_t a = s_buf[lo], b = s_buf[hi];
                    if ((a > b) == up) {
                        s_buf[lo] = b;
                        s_buf[hi] = a;
                    }
                }
                __syncthreads();
            }
        }
    }
    for (int t = threadIdx.x; t < k; t += kBlock) {
        const uint64_t key = s_buf[t];
        const int64_t o = (int64_t)(q_first + (int)blockIdx.x) * k + t;
        ids[o] = key == kNoKey ? -1 : (int32_t)(uint32_t)key;
        dist[o] = key == kNoKey ? __builtin_nanf("") : sqrtf(__uint_as_float((uint32_t)(key >> 32)));
    }
}

// The same search for dim <= 128 on the fp16 matrix cores.  Queries and rows
// are normalised and scaled by 2^10 (|x| <= 1024), and each value is split
// into two fp16 parts, x = hi + lo + e with |e| <= 2^-22 |x| (hi the nearest
// fp16 of x, lo that of the exact remainder x - hi); the three products
// hi.hi + hi.lo + lo.hi (v_mfma_f32_32x32x16_f16, exact fp16 products summed
// in fp32) leave out lo.lo and e, about 2^-21 of each term, against the 2^-24
// of fp32 products: well inside the search's distance bound.  A 16-dimension
// chunk takes three matrix instructions here against eight in fp32.
// Operand layout (checked on the GPU): A[i][c] comes from element c % 8 of
// lane i + 32 (c / 8), B[c][j] from element c % 8 of lane j + 32 (c / 8); the
// accumulators are laid out as for the fp32 instruction.
typedef _Float16 knn_h8 __attribute__((ext_vector_type(8)));
constexpr float kKnnSplitUnscale = 1.0f / (1024.0f * 1024.0f);  // 2^-20, exact

// The split of 8 values scaled by sc.  Each product v is pinned as one fp32
// value (an empty asm statement that the compiler must assume redefines it),
// so the multiplication cannot be fused into the conversions: hi is the fp16
// of v and the remainder v - hi is exact, so hi + lo equals v up to the
// rounding of lo.  Left to the default contraction, the product was rounded
// once for hi and once, differently, for lo, and at an exact fp16 tie hi + lo
// missed v by one fp16 step; the pinned form also measured faster than
// placing hi on the fp16 grid with integer operations on the bits of v.
__device__ __forceinline__ void knn_split8(float4 a, float4 b, float sc, knn_h8& hi,
                                           knn_h8& lo) {
    float v[8] = {a.x * sc, a.y * sc, a.z * sc, a.w * sc, b.x * sc, b.y * sc, b.z * sc,
                  b.w * sc};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        asm volatile("" : "+v"(v[e]));
        const _Float16 h = (_Float16)v[e];
        hi[e] = h;
        lo[e] = (_Float16)(v[e] - (float)h);
    }
}

// The hi parts alone of knn_split8 (the same pinned products, the same
// conversions): hi[e] equals knn_split8's hi[e] bit for bit.
__device__ __forceinline__ knn_h8 knn_hi8(float4 a, float4 b, float sc) {
    float v[8] = {a.x * sc, a.y * sc, a.z * sc, a.w * sc, b.x * sc, b.y * sc, b.z * sc,
                  b.w * sc};
    knn_h8 hi;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        asm volatile("" : "+v"(v[e]));
        hi[e] = (_Float16)v[e];
    }
    return hi;
}

// Squared norm of the 16 values v[0 .. 3] in a fixed order of explicit fused
// multiply-adds, and that of a row held by a lane pair (x, 0), (x, 1) as
// 16 float4 each: four such sums per lane, each added to its partner's, then
// (P0 + P1) + (P2 + P3).  Every fp16 search forms a row's norm this way (the
// four-block search from partial sums that its four waves exchange), so all of
// them compute the same scale and the same distances for a row.
__device__ __forceinline__ float knn_sq4(const float4* v) {
    float p = 0.f;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        float t = v[m].x * v[m].x;
        t = fmaf(v[m].y, v[m].y, t);
        t = fmaf(v[m].z, v[m].z, t);
        t = fmaf(v[m].w, v[m].w, t);
        p += t;
    }
    return p;
}

__device__ __forceinline__ float knn_row_norm(const float4 (&v)[16]) {
    float P[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        P[i] = knn_sq4(v + 4 * i);
        P[i] += __shfl_xor(P[i], 32, 64);
    }
    return (P[0] + P[1]) + (P[2] + P[3]);
}

__global__ __launch_bounds__(kKnnWavesR * 64) void k_knn_tiles_h(KnnArgs A) {
    __shared__ uint64_t s_list[kKnnWavesR][32][kKnnMaxK];
    __shared__ uint64_t s_stage[kKnnWavesR][32][32];
    __shared__ uint64_t s_thr[kKnnWavesR][32];
    __shared__ uint32_t s_cnt[kKnnWavesR][32];
    __shared__ uint32_t s_len[kKnnWavesR][32];

    if (A.gate && *A.gate == 0) return;  // the threshold scans answered every query
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int x = lane & 31, h = lane >> 5;
    const int D = A.D, k = A.k;
    const int qb = w % A.QB;
    const int wpb = kKnnWavesR / A.QB;
    const int64_t S = (int64_t)blockIdx.x * wpb + w / A.QB;
    const int64_t NS = (int64_t)gridDim.x * wpb;
    constexpr int kCh = kKnnDimChunk / 16;  // 16-dimension chunks
    // lane (x, h) holds dimensions 16 s + 8 h .. 16 s + 8 h + 7 of chunk s
    const int d0 = 8 * h;

    // operands of query qb * 32 + x (already normalised)
    knn_h8 qh[kCh], ql[kCh];
    {
        const float* qrow = A.qn + (int64_t)(qb * 32 + x) * D;
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            const int d = 16 * c + d0;
            const float4 a = d + 4 <= D ? *reinterpret_cast<const float4*>(qrow + d)
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 b = d + 8 <= D ? *reinterpret_cast<const float4*>(qrow + d + 4)
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
            knn_split8(a, b, kKnnSplitScale, qh[c], ql[c]);
        }
    }
    // this lane's 16 score slots: query i = 8 (r / 4) + 4 h + r % 4; the
    // squared norm of a normalised query is 1 (0 for a zero query): one bit.
    // A padding slot (no query) keeps the threshold -inf: nothing passes it.
    float thr[16];
    int32_t qid[16];
    uint32_t qone = 0u;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int q = qb * 32 + 8 * (r / 4) + 4 * h + (r % 4);
        qone |= A.qn2[q] > 0.f ? 1u << r : 0u;
        qid[r] = A.qid[q];
        thr[r] = qid[r] >= 0 ? __builtin_inff() : -__builtin_inff();
    }
    if (lane < 32) {
        s_thr[w][lane] = kNoKey;
        s_cnt[w][lane] = 0u;
        s_len[w][lane] = 0u;
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
    __builtin_amdgcn_wave_barrier();

    for (int64_t t = S; t < A.tiles; t += NS) {
        const int64_t row = t * 32 + x;
        const bool ok = row < A.N;
        const float* src = A.T + (ok ? row : 0) * (int64_t)D;
        float4 bv[2 * kCh];
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            const int d = 16 * c + d0;
            bv[2 * c] = (ok && d + 4 <= D) ? *reinterpret_cast<const float4*>(src + d)
                                           : make_float4(0.f, 0.f, 0.f, 0.f);
            bv[2 * c + 1] = (ok && d + 8 <= D) ? *reinterpret_cast<const float4*>(src + d + 4)
                                               : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        const float nr = knn_row_norm(bv);
        const float sc = nr > 0.f ? kKnnSplitScale / sqrtf(nr) : 0.f;
        const float nx = nr > 0.f ? 1.f : 0.f;
        knn_acc16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            knn_h8 bh, bl;
            knn_split8(bv[2 * c], bv[2 * c + 1], sc, bh, bl);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(qh[c], bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(qh[c], bl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ql[c], bh, acc, 0, 0, 0);
        }
        bool staged = false;
        const float nx1 = nx + 1.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            // d^2 = |q|^2 + [r != 0] - 2 <q, r>, clamped at 0
            const float base = (qone >> r) & 1u ? nx1 : nx;
            float d2 = fmaf(-2.f * kKnnSplitUnscale, acc[r], base);
            d2 = d2 > 0.f ? d2 : 0.f;
            if (d2 <= thr[r] && ok && row != (int64_t)qid[r]) {
                const int i = 8 * (r / 4) + 4 * h + (r % 4);
                const uint64_t key = ((uint64_t)__float_as_uint(d2) << 32) | (uint64_t)row;
                if (key < s_thr[w][i]) {
                    const uint32_t pos = atomicAdd(&s_cnt[w][i], 1u);
                    s_stage[w][i][pos] = key;  // pos < 32: one row per lane x
                    staged = true;
                }
            }
        }
        if (__ballot(staged) == 0ull) continue;  // wave-uniform: nothing to merge
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
        if (h == 0) {
            const uint32_t c = s_cnt[w][x];
            if (c > 0u) {
                uint64_t* L = s_list[w][x];
                uint32_t len = s_len[w][x];
                for (uint32_t e = 0; e < c; ++e) {
                    const uint64_t key = s_stage[w][x][e];
                    if (len == (uint32_t)k && key >= L[k - 1]) continue;
                    int p = len < (uint32_t)k ? (int)len : k - 1;
                    while (p > 0 && L[p - 1] > key) {
                        L[p] = L[p - 1];
                        --p;
                    }
                    L[p] = key;
                    if (len < (uint32_t)k) ++len;
                }
                s_len[w][x] = len;
                s_cnt[w][x] = 0u;
                s_thr[w][x] = len == (uint32_t)k ? L[k - 1] : kNoKey;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = 8 * (r / 4) + 4 * h + (r % 4);
            const uint64_t tk = s_thr[w][i];
            const float tv = tk == kNoKey ? __builtin_inff() : __uint_as_float((uint32_t)(tk >> 32));
            thr[r] = qid[r] >= 0 ? tv : -__builtin_inff();
        }
    }
    if (h == 0) {
        const uint32_t len = s_len[w][x];
        uint64_t* dst = A.partial + ((size_t)S * A.nqp + qb * 32 + x) * k;
        for (int t = 0; t < k; ++t) dst[t] = (uint32_t)t < len ? s_list[w][x][t] : kNoKey;
    }
}

// The same search when a pass holds four query blocks (97-128 queries): the
// four waves of a row tile (one per query block) share its load, norm and
// split instead of each doing all of it.  Wave qb loads chunks 2 qb and
// 2 qb + 1 (16-dimension chunks) of the tile's rows and publishes their
// partial squared norms; after a barrier each wave forms the row scales,
// splits its two chunks and publishes the fp16 parts; after a second barrier
// every wave reads all eight chunks' parts from LDS for its products.  Every
// wave of the workgroup runs the same number of iterations (that of the
// workgroup's first tile stream; a stream past its last tile loads nothing
// and offers no candidates), so all of them reach both barriers each time.
// Candidates are staged as (d^2, row in tile) to leave LDS for the parts.
__global__ __launch_bounds__(kKnnWavesR * 64) void k_knn_tiles_h4(KnnArgs A) {
    constexpr int kQB = 4;
    constexpr int kStreams = kKnnWavesR / kQB;  // tile streams per workgroup
    constexpr int kCh = kKnnDimChunk / 16;      // 16-dimension chunks
    __shared__ uint64_t s_list[kKnnWavesR][32][kKnnMaxK];
    __shared__ float s_sd[kKnnWavesR][32][32];    // staged d^2
    __shared__ uint8_t s_sx[kKnnWavesR][32][32];  // staged row within the tile
    __shared__ uint64_t s_thr[kKnnWavesR][32];
    __shared__ uint32_t s_cnt[kKnnWavesR][32];
    __shared__ uint32_t s_len[kKnnWavesR][32];
    __shared__ float s_nr[kStreams][kQB][32];     // partial squared norms of the rows
    // fp16 parts of the tile: [stream][chunk][row][h] = {hi, lo} of 8 dimensions
    __shared__ knn_h8 s_part[kStreams][kCh][32][2][2];

    if (A.gate && *A.gate == 0) return;  // the threshold scans answered every query
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int x = lane & 31, h = lane >> 5;
    const int D = A.D, k = A.k;
    const int qb = w % kQB;
    const int st = w / kQB;
    const int64_t S0 = (int64_t)blockIdx.x * kStreams;
    const int64_t S = S0 + st;
    const int64_t NS = (int64_t)gridDim.x * kStreams;
    const int d0 = 8 * h;
    // iterations of every wave: those of the workgroup's first stream
    const int64_t iters = A.tiles > S0 ? (A.tiles - S0 + NS - 1) / NS : 0;

    // operands of query qb * 32 + x (already normalised)
    knn_h8 qh[kCh], ql[kCh];
    {
        const float* qrow = A.qn + (int64_t)(qb * 32 + x) * D;
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            const int d = 16 * c + d0;
            const float4 a = d + 4 <= D ? *reinterpret_cast<const float4*>(qrow + d)
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
            const float4 b = d + 8 <= D ? *reinterpret_cast<const float4*>(qrow + d + 4)
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
            knn_split8(a, b, kKnnSplitScale, qh[c], ql[c]);
        }
    }
    float thr[16];
    int32_t qid[16];
    uint32_t qone = 0u;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int q = qb * 32 + 8 * (r / 4) + 4 * h + (r % 4);
        qone |= A.qn2[q] > 0.f ? 1u << r : 0u;
        qid[r] = A.qid[q];
        thr[r] = qid[r] >= 0 ? __builtin_inff() : -__builtin_inff();
    }
    if (lane < 32) {
        s_thr[w][lane] = kNoKey;
        s_cnt[w][lane] = 0u;
        s_len[w][lane] = 0u;
    }

    // this wave's two chunks of row x of its stream's tile of iteration it2
    // (zeros past the table)
    auto load_chunks = [&](int64_t it2, float4 (&dst)[4]) {
        const int64_t t2 = S + it2 * NS;
        const int64_t row2 = t2 * 32 + x;
        const bool ok2 = it2 < iters && t2 < A.tiles && row2 < A.N;
        const float* src = A.T + (ok2 ? row2 : 0) * (int64_t)D;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int d = 16 * (2 * qb + j) + d0;
            dst[2 * j] = (ok2 && d + 4 <= D) ? *reinterpret_cast<const float4*>(src + d)
                                             : make_float4(0.f, 0.f, 0.f, 0.f);
            dst[2 * j + 1] = (ok2 && d + 8 <= D) ? *reinterpret_cast<const float4*>(src + d + 4)
                                                 : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    // The chunks are loaded one iteration ahead: the next tile's loads are in
    // flight during the products and the candidate merge of the current one
    // (the barriers wait for LDS accesses only; loading two tiles ahead, in
    // two register buffers, measured no faster).
    float4 nb[4];
    load_chunks(0, nb);

    for (int64_t it = 0; it < iters; ++it) {
        const int64_t t = S + it * NS;
        const int64_t row = t * 32 + x;
        const bool ok = t < A.tiles && row < A.N;
        float4 bv[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) bv[m] = nb[m];
        float pn = knn_sq4(bv);
        pn += __shfl_xor(pn, 32, 64);
        if (h == 0) s_nr[st][qb][x] = pn;
        __syncthreads();
        const float nr = (s_nr[st][0][x] + s_nr[st][1][x]) + (s_nr[st][2][x] + s_nr[st][3][x]);
        const float sc = nr > 0.f ? kKnnSplitScale / sqrtf(nr) : 0.f;
        const float nx = nr > 0.f ? 1.f : 0.f;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            knn_h8 bh, bl;
            knn_split8(bv[2 * j], bv[2 * j + 1], sc, bh, bl);
            s_part[st][2 * qb + j][x][h][0] = bh;
            s_part[st][2 * qb + j][x][h][1] = bl;
        }
        load_chunks(it + 1, nb);
        __syncthreads();
        knn_acc16 acc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                         0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            const knn_h8 bh = s_part[st][c][x][h][0];
            const knn_h8 bl = s_part[st][c][x][h][1];
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(qh[c], bh, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(qh[c], bl, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ql[c], bh, acc, 0, 0, 0);
        }
        bool staged = false;
        const float nx1 = nx + 1.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            // d^2 = |q|^2 + [r != 0] - 2 <q, r>, clamped at 0
            const float base = (qone >> r) & 1u ? nx1 : nx;
            float d2 = fmaf(-2.f * kKnnSplitUnscale, acc[r], base);
            d2 = d2 > 0.f ? d2 : 0.f;
            if (d2 <= thr[r] && ok && row != (int64_t)qid[r]) {
                const int i = 8 * (r / 4) + 4 * h + (r % 4);
                const uint64_t key = ((uint64_t)__float_as_uint(d2) << 32) | (uint64_t)row;
                if (key < s_thr[w][i]) {
                    const uint32_t pos = atomicAdd(&s_cnt[w][i], 1u);
                    s_sd[w][i][pos] = d2;  // pos < 32: one row per lane x
                    s_sx[w][i][pos] = (uint8_t)x;
                    staged = true;
                }
            }
        }
        if (__ballot(staged) == 0ull) continue;  // wave-uniform: nothing to merge
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
        if (h == 0) {
            const uint32_t c = s_cnt[w][x];
            if (c > 0u) {
                uint64_t* L = s_list[w][x];
                uint32_t len = s_len[w][x];
                for (uint32_t e = 0; e < c; ++e) {
                    const uint64_t key = ((uint64_t)__float_as_uint(s_sd[w][x][e]) << 32) |
                                         (uint64_t)(t * 32 + s_sx[w][x][e]);
                    if (len == (uint32_t)k && key >= L[k - 1]) continue;
                    int p = len < (uint32_t)k ? (int)len : k - 1;
                    while (p > 0 && L[p - 1] > key) {
                        L[p] = L[p - 1];
                        --p;
                    }
                    L[p] = key;
                    if (len < (uint32_t)k) ++len;
                }
                s_len[w][x] = len;
                s_cnt[w][x] = 0u;
                s_thr[w][x] = len == (uint32_t)k ? L[k - 1] : kNoKey;
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int i = 8 * (r / 4) + 4 * h + (r % 4);
            const uint64_t tk = s_thr[w][i];
            const float tv = tk == kNoKey ? __builtin_inff() : __uint_as_float((uint32_t)(tk >> 32));
            thr[r] = qid[r] >= 0 ? tv : -__builtin_inff();
        }
    }
    if (h == 0) {
        const uint32_t len = s_len[w][x];
        uint64_t* dst = A.partial + ((size_t)S * A.nqp + qb * 32 + x) * k;
        for (int t = 0; t < k; ++t) dst[t] = (uint32_t)t < len ? s_list[w][x][t] : kNoKey;
    }
}

// ---------------------------------------------------------------------------
// Threshold scans (dim <= 128): the default search.  A scan visits the row
// tiles i * step (0 <= i < count); every wave takes whole 32-row tiles, loads
// the next one while it works on the current one, and forms the distances of
// its tile to every query of the pass with the fp16 parts of the queries in
// LDS.  Row x's norm, scale and split, the products and d^2 are those of the
// list-merging kernels above, bit for bit (the matrix instruction takes the
// row parts as its first operand here, the same products in the same order).
// A (row, query) pair whose d^2 is at most the query's bound tau is appended
// to the query's candidate list; only the count of a list that overflows its
// capacity keeps growing.  Between scans a selection sorts each list: its
// k-th key bounds the k-th distance over the whole table (any k rows do), so
// the next, denser scan keeps every row of the true answer.  The scans are
// nested (each one's tiles are among the next one's), so each finds at least
// the k rows that set its bound; the last one visits every tile and its k
// smallest keys are the answer.
// A tile is screened first by the hi.hi products alone (one matrix
// instruction per chunk instead of three, no lo parts): they differ from the
// full products hi.hi + hi.lo + lo.hi by at most the dropped terms,
// sum |hi_q lo_r| + |lo_q hi_r| <= 2^-10 (1 + 2^-10) 2^20 with |q|, |r| <= 2^10
// after scaling, plus the accumulations' roundings (at most 384 of 2^-4
// each) and fp16 subnormal steps: below 1100 units of the product.  For a
// present, nonzero row, d^2 <= tau needs acc >= (|q|^2 + 1 - tau) 2^19 - 2
// (the bound is computed within 2^-3 and d^2's one rounding moves it by at
// most 2^-21, a quarter of a unit of acc), so a screened product below that
// less kKnnScreenMargin = 1536 clears the pair.  A query block with any pair
// left, or a tile with a zero or missing row, gets the full products of the
// list search (bit for bit) and the exact test.  So does a tile with a row
// whose squared norm lies outside [kKnnNormMin, kKnnNormMax] (its scaled norm
// may not be 2^10, or its scaled values are no numbers), and a pair whose
// screened product is no number.
// ---------------------------------------------------------------------------
struct KnnScanArgs {
    const float* T;
    int64_t N;
    int32_t D;
    int32_t cap;    // keys kept per list
    int32_t cnt_stride;  // words between the counts of two queries
    int64_t step;   // tiles i * step, 0 <= i < count
    int64_t count;
    const float* qn;
    const float* qn2;
    const int32_t* qid;
    const float* tau;
    uint32_t* cnt;
    uint64_t* cand;  // [query slot][cap]
};

constexpr float kKnnAccPerD2 = 524288.0f;  // 2^19: a unit of d^2 in the product's units
constexpr float kKnnScreenMargin = 1536.0f;  // product units: hi.hi against the full products

// The exact test of a tile's pairs with query block qb and the append of the
// passing ones (a tile with a candidate, a zero or a missing row).
template <int QB>
__device__ __forceinline__ void knn_scan_append(const KnnScanArgs& A, int qb, int x, int h,
                                                int64_t t, uint64_t live,
                                                const knn_acc16& acc) {
    const int q = qb * 32 + x;
    const float tau = A.tau[q];
    const int64_t qid = A.qid[q];
    const bool q1 = A.qn2[q] > 0.f;
    const int64_t rows = A.N - t * 32;  // rows of the tile present
    uint32_t pass = 0u;
    float d2v[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        // d^2 = |q|^2 + [row != 0] - 2 <q, row>, clamped at 0
        const int m = 8 * (r / 4) + 4 * h + (r % 4);
        const float nx = (live >> m) & 1ull ? 1.f : 0.f;
        const float base = q1 ? nx + 1.f : nx;
        float d2 = fmaf(-2.f * kKnnSplitUnscale, acc[r], base);
        d2 = d2 > 0.f ? d2 : 0.f;
        d2v[r] = d2;
        if (d2 <= tau && m < rows && t * 32 + m != qid) pass |= 1u << r;
    }
    if (pass == 0u) return;
    uint32_t pos = atomicAdd(&A.cnt[q * A.cnt_stride], (uint32_t)__popc(pass));
    uint64_t* dst = A.cand + (size_t)q * A.cap;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if (!((pass >> r) & 1u)) continue;
        const int m = 8 * (r / 4) + 4 * h + (r % 4);
        if (pos < (uint32_t)A.cap)
            dst[pos] = ((uint64_t)__float_as_uint(d2v[r]) << 32) | (uint64_t)(t * 32 + m);
        ++pos;
    }
}

// FULL: dim is 128, so no dimension of a chunk lies past the row.
template <int QB, bool FULL>
__global__ __launch_bounds__(kKnnScanWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_knn_scan(KnnScanArgs A) {
    constexpr int kCh = kKnnDimChunk / 16;  // 16-dimension chunks
    // B operands: lane (x, h) of s_q[qb][c][p] holds the fp16 part p (0 hi,
    // 1 lo) of query qb * 32 + x's dimensions 16 c + 8 h .. 16 c + 8 h + 7
    __shared__ knn_h8 s_q[QB][kCh][2][64];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int x = lane & 31, h = lane >> 5;
    const int D = A.D;
    const int d0 = 8 * h;
    for (int j = w; j < QB * kCh; j += kKnnScanWaves) {
        const int qb = j / kCh, c = j % kCh;
        const float* qrow = A.qn + (int64_t)(qb * 32 + x) * D;
        const int d = 16 * c + d0;
        const float4 a = d + 4 <= D ? *reinterpret_cast<const float4*>(qrow + d)
                                    : make_float4(0.f, 0.f, 0.f, 0.f);
        const float4 b = d + 8 <= D ? *reinterpret_cast<const float4*>(qrow + d + 4)
                                    : make_float4(0.f, 0.f, 0.f, 0.f);
        knn_h8 hi, lo;
        knn_split8(a, b, kKnnSplitScale, hi, lo);
        s_q[qb][c][0][lane] = hi;
        s_q[qb][c][1][lane] = lo;
    }
    // lane (x, h) holds query qb * 32 + x of every block against rows
    // 8 (r / 4) + 4 h + r % 4 of the tile (accumulator r); a screened
    // product below athr[qb] is no candidate for a present, nonzero row
    float athr[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        const int q = qb * 32 + x;
        const float q1 = A.qn2[q] > 0.f ? 1.f : 0.f;
        athr[qb] = ((q1 + 1.f) - A.tau[q]) * kKnnAccPerD2 - 2.f - kKnnScreenMargin;
    }
    __syncthreads();

    const int64_t W = (int64_t)gridDim.x * kKnnScanWaves;
    const int64_t i0 = (int64_t)blockIdx.x * kKnnScanWaves + w;
    // Row x of tile i * step: lane (x, h) loads dimensions 16 c + 8 h .. + 7
    // of every chunk c.  Past the scan's last tile or the table a lane loads
    // row 0 instead (its rows are marked missing below); past dim, zeros.
    auto load_tile = [&](int64_t i, float4 (&dst)[2 * kCh]) {
        const int64_t row = i * A.step * 32 + x;
        const bool ok = i < A.count && row < A.N;
        const float* src = A.T + (ok ? row : 0) * (int64_t)D;
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            const int d = 16 * c + d0;
            if (FULL) {
                dst[2 * c] = *reinterpret_cast<const float4*>(src + d);
                dst[2 * c + 1] = *reinterpret_cast<const float4*>(src + d + 4);
            } else {
                dst[2 * c] = d + 4 <= D ? *reinterpret_cast<const float4*>(src + d)
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
                dst[2 * c + 1] = d + 8 <= D ? *reinterpret_cast<const float4*>(src + d + 4)
                                            : make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
    };
    auto scan_tile = [&](int64_t i, const float4 (&bv)[2 * kCh]) {
        const int64_t t = i * A.step;
        const float nr = knn_row_norm(bv);
        const float sc = nr > 0.f ? kKnnSplitScale / sqrtf(nr) : 0.f;
        // bit m (and m + 32): row m of the tile is present and nonzero
        const uint64_t live = __ballot(nr > 0.f && t * 32 + x < A.N);
        // every row is one that the screen's bound holds for
        const bool sure =
            __ballot(nr >= kKnnNormMin && nr <= kKnnNormMax && t * 32 + x < A.N) == ~0ull;
        // the screen: hi.hi products of every query block
        knn_acc16 acc[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[qb][r] = 0.f;
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            const knn_h8 bh = knn_hi8(bv[2 * c], bv[2 * c + 1], sc);
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
                acc[qb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, s_q[qb][c][0][lane],
                                                                 acc[qb], 0, 0, 0);
        }
        // bit qb: the block has a pair left (wave-uniform)
        uint32_t need = 0u;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            bool look = !sure;
#pragma unroll
            for (int r = 0; r < 16; ++r) look |= !(acc[qb][r] < athr[qb]);
            need |= __ballot(look) != 0ull ? 1u << qb : 0u;
        }
        // the full products of the list search for those blocks, then the exact test
#pragma unroll 1
        for (; need != 0u; need &= need - 1u) {
            const int qb = __builtin_ctz(need);
            knn_acc16 ex = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f,
                            0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < kCh; ++c) {
                knn_h8 bh, bl;
                knn_split8(bv[2 * c], bv[2 * c + 1], sc, bh, bl);
                const knn_h8 qh = s_q[qb][c][0][lane];
                const knn_h8 ql = s_q[qb][c][1][lane];
                ex = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, qh, ex, 0, 0, 0);
                ex = __builtin_amdgcn_mfma_f32_32x32x16_f16(bl, qh, ex, 0, 0, 0);
                ex = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, ql, ex, 0, 0, 0);
            }
            knn_scan_append<QB>(A, qb, x, h, t, live, ex);
        }
    };
    // two register buffers in turn: a tile's rows load during the previous
    // tile's products
    float4 ba[2 * kCh], bb[2 * kCh];
    load_tile(i0, ba);
    for (int64_t i = i0; i < A.count; i += 2 * W) {
        load_tile(i + W, bb);
        scan_tile(i, ba);
        if (i + W >= A.count) break;
        load_tile(i + 2 * W, ba);
        scan_tile(i + W, bb);
    }
}

// Candidate selection, one workgroup per query slot: the k smallest of the
// list's kept keys (at most cap, a power of two).  After a sample scan the
// k-th key's d^2 becomes the query's bound (fewer than k keys leave it); after
// the last scan the k smallest keys are the answer, written as the
// list-merging search writes it, and a list that overflowed, or a query whose
// bound is -inf (no screen holds for it), opens the gate for that search.  The
// count is reset for the next scan.
// The keys' distances are counted in kKnnSelectBins equal ranges of their bit
// patterns between the smallest and the largest; only the keys up to the range
// that holds the k-th are sorted (a bitonic network in LDS).  Sorting all of
// 8192 keys took 75 us, of 1024 20; counting and sorting those left
// 14 and 13.
struct KnnSelectArgs {
    uint32_t* cnt;
    const uint64_t* cand;
    int32_t cap;
    int32_t cnt_stride;  // words between the counts of two queries
    int32_t k;
    int32_t last;      // 1: the last scan
    int32_t m;         // queries of the pass (slots beyond are padding)
    int32_t q_first;   // the pass's first query
    const int32_t* qid;
    float* tau;
    int32_t* ids;
    float* dist;
    int32_t* gate;
};

constexpr int kKnnSelectBins = 1024;

__global__ __launch_bounds__(kKnnSelectThreads) void k_knn_select(KnnSelectArgs S) {
    extern __shared__ uint64_t s_key[];  // [cap]
    __shared__ uint32_t s_bin[kKnnSelectBins];
    __shared__ uint32_t s_wave[kKnnSelectThreads / 64];
    __shared__ uint32_t s_min, s_max, s_last, s_kept;
    static_assert(kKnnSelectBins == kKnnSelectThreads, "a bin per thread");
    static_assert(kKnnCandCap % kKnnSelectThreads == 0, "whole keys per thread");
    const int q = blockIdx.x, tid = threadIdx.x;
    const uint32_t c = S.cnt[q * S.cnt_stride];
    const uint32_t n = c < (uint32_t)S.cap ? c : (uint32_t)S.cap;
    constexpr int kPer = kKnnCandCap / kKnnSelectThreads;
    s_bin[tid] = 0u;
    if (tid == 0) {
        s_min = ~0u;
        s_max = 0u;
        s_last = (uint32_t)kKnnSelectBins;  // no bin: every key is kept
        s_kept = 0u;
    }
    __syncthreads();
    // the range of the distances (a missing pair's key, ~0, is none)
    uint64_t key[kPer];
    uint32_t lo = ~0u, hi = 0u;
#pragma unroll
    for (int e = 0; e < kPer; ++e) {
        const uint32_t i = (uint32_t)(e * kKnnSelectThreads + tid);
        key[e] = i < n ? S.cand[(size_t)q * S.cap + i] : kNoKey;
        if (key[e] != kNoKey) {
            const uint32_t d = (uint32_t)(key[e] >> 32);
            lo = d < lo ? d : lo;
            hi = d > hi ? d : hi;
        }
    }
    if (lo <= hi) {
        atomicMin(&s_min, lo);
        atomicMax(&s_max, hi);
    }
    __syncthreads();
    const uint32_t base = s_min;
    const uint32_t span = s_max >= base ? s_max - base : 0u;
    // d - base <= span < 2^32: range (d - base) 2^-shift, shift such that the
    // largest is below kKnnSelectBins
    int shift = 0;
    while ((span >> shift) >= (uint32_t)kKnnSelectBins) ++shift;
#pragma unroll
    for (int e = 0; e < kPer; ++e)
        if (key[e] != kNoKey) atomicAdd(&s_bin[((uint32_t)(key[e] >> 32) - base) >> shift], 1u);
    __syncthreads();
    {
        const int lane = tid & 63, wave = tid >> 6;
        const uint32_t mine = s_bin[tid];
        uint32_t incl = mine;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const uint32_t t = __shfl_up(incl, off, 64);
            if (lane >= off) incl += t;
        }
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        for (int w = 0; w < wave; ++w) incl += s_wave[w];
        // the range that holds the k-th key
        if (incl >= (uint32_t)S.k && incl - mine < (uint32_t)S.k) s_last = (uint32_t)tid;
    }
    __syncthreads();
    const uint32_t last = s_last;
#pragma unroll
    for (int e = 0; e < kPer; ++e)
        if (key[e] != kNoKey && ((uint32_t)(key[e] >> 32) - base) >> shift <= last)
            s_key[atomicAdd(&s_kept, 1u)] = key[e];
    __syncthreads();
    const uint32_t kept = s_kept;
    uint32_t P = 2u;
    while (P < kept || P < (uint32_t)S.k) P <<= 1;
    for (uint32_t i = kept + tid; i < P; i += kKnnSelectThreads) s_key[i] = kNoKey;
    __syncthreads();
    for (uint32_t size = 2; size <= P; size <<= 1) {
        for (uint32_t st = size >> 1; st > 0; st >>= 1) {
            for (uint32_t i = tid; i < P / 2; i += kKnnSelectThreads) {
                const uint32_t lo_i = 2 * i - (i & (st - 1));
                const uint32_t hi_i = lo_i + st;
                const bool up = (lo_i & size) == 0;
                const uint64_t a = s_key[lo_i], b = s_key[hi_i];
                if ((a > b) == up) {
                    s_key[lo_i] = b;
                    s_key[hi_i] = a;
                }
            }
            __syncthreads();
        }
    }
    if (S.last) {
        if (q < S.m) {
            for (int t = tid; t < S.k; t += kKnnSelectThreads) {
                const uint64_t key = s_key[t];  // k <= P
                const int64_t o = (int64_t)(S.q_first + q) * S.k + t;
                S.ids[o] = key == kNoKey ? -1 : (int32_t)(uint32_t)key;
                S.dist[o] = key == kNoKey ? __builtin_nanf("")
                                          : sqrtf(__uint_as_float((uint32_t)(key >> 32)));
            }
        }
        // a list that overflowed, or a query that the scans do not answer
        if (tid == 0 &&
            (c > (uint32_t)S.cap || (S.qid[q] >= 0 && S.tau[q] == -__builtin_inff())))
            *S.gate = 1;
    } else if (tid == 0 && s_key[S.k - 1] != kNoKey && S.tau[q] != -__builtin_inff()) {
        S.tau[q] = __uint_as_float((uint32_t)(s_key[S.k - 1] >> 32));
    }
    if (tid == 0) S.cnt[q * S.cnt_stride] = 0u;
}

// ---------------------------------------------------------------------------
// Threshold scans of wide rows (128 < dim): the exact products cost dim / 2
// fp32 matrix instructions of 64 cycles per 32 x 32 pairs, so they are formed
// for few pairs only.
//   k_knn_wide_dense    the first scan, no bound yet: every pair of at most
//                       kKnnStageTiles tiles, exactly, each key at its place;
//   k_knn_wide_scan     the others screen every tile of theirs with fp16
//                       products and append the rows left to the queries'
//                       lists;
//   k_knn_wide_rescore  replaces those rows by their exact keys.
// Between scans k_knn_select sorts the lists, as for narrower rows.  A scan of
// stride s after one of stride g s keeps about k g rows per query, so
// fewer, coarser scans cost exact products and more, finer ones launches:
// g is at most kKnnWideGrowth.
//
// The screen.  A tile's rows are taken in slabs of 128 dimensions, the next
// slab's loads in flight during the current one's products.  A row is scaled
// by sc = 64 / |its first slab| before its fp16 rounding, since its own norm
// is known only after the last slab (where a slab takes the scaled norm past
// 2^14, by 64 / |the slabs so far|, and the products so far with it, one more
// rounding each); with f = sc |row| / 2^10, the product of
// the fp16 parts is f times that of the normalised parts scaled by 2^20, up to
//   the roundings: 2^-11 of each operand's norm, 2^10 (1 + 2^-11) units in all
//     (a unit is f times one of a product of size 2^20); parts below 2^-14
//     round by 2^-25 instead, under 1 unit while sc |row| >= 1;
//   dim / 16 units for the sums here, as many for those of the exact
//     products, 16 for f and 3 for the bound:
// below 1150 units for dim <= 528.  A pair can pass d^2 <= tau only if its
// product is at least f ((|q|^2 + 1 - tau) 2^19) less those (a zero row:
// |q|^2 - tau); kKnnScreenMargin = 1536 units are left.  A row whose scaled
// norm leaves [1, 2^14], or whose norm is tiny or not finite, is no subject of
// the screen: it is appended to every list that has not overflowed.  Should a
// list overflow, the pass is computed by the list search.
// 500,000 x 256 rows, 100 queries, k = 10: the list search alone, in two passes
// over the table, took 1349 us, the scans take 274 us (dense 19, scan
// 123, rescore 49, selections 14 each; the table once at the copy rate: 106).
// With the first 128 dimensions zero, or 1e-4 of the others: 1322 us in the list
// search, 11,980 while such rows went to every list, 241 now; a table of rows
// that are no numbers: 1052, 11,840 and 1071.
// ---------------------------------------------------------------------------
struct KnnWideArgs {
    const float* T;
    int64_t N;
    int32_t D;
    int32_t cap;
    int32_t cnt_stride;  // words between the counts of two queries
    int64_t step;   // tiles i * step, 0 <= i < count
    int64_t count;
    const float* qn;
    const float* qn2;
    const int32_t* qid;
    const _Float16* qh;
    const float* tau;
    uint32_t* cnt;
    uint64_t* cand;
};

// Wave (tile i, query block qb): the keys of their pairs at cand[q][32 i + row]
// (no pair: kNoKey); the first tile's waves set the counts.
template <int QB>
__global__ __launch_bounds__(256) void k_knn_wide_dense(KnnWideArgs A) {
    const int lane = threadIdx.x & 63;
    const int x = lane & 31, h = lane >> 5;
    const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int64_t i = w / QB;
    const int qb = (int)(w % QB);
    if (i >= A.count) return;  // no barrier below
    const int64_t row = i * A.step * 32 + x;
    const bool ok = row < A.N;
    const float* src = A.T + (ok ? row : 0) * (int64_t)A.D;
    const float* qrow = A.qn + (int64_t)(qb * 32 + x) * A.D;
    knn_acc16 acc;
    float nr;
    knn_exact_products(
        A.D, h, [&](int d) { return *reinterpret_cast<const float4*>(qrow + d); },
        [&](int d) { return *reinterpret_cast<const float4*>(src + d); }, acc, nr);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int q = qb * 32 + 8 * (r / 4) + 4 * h + (r % 4);
        const float d2 = knn_exact_d2(A.qn2[q], nr, acc[r]);
        const int32_t id = A.qid[q];
        const bool pair = ok && id >= 0 && row != (int64_t)id;
        A.cand[(size_t)q * A.cap + (size_t)i * 32 + x] =
            pair ? ((uint64_t)__float_as_uint(d2) << 32) | (uint64_t)row : kNoKey;
        if (i == 0 && x == 0) A.cnt[q * A.cnt_stride] = (uint32_t)(A.count * 32);
    }
}

// The listed rows of query blockIdx.x, 32 per wave and round: their exact keys
// in their places.  The A operand holds the query in every row, so each lane
// finds its row's product in accumulator 0.
__global__ __launch_bounds__(256) void k_knn_wide_rescore(KnnWideArgs A) {
    extern __shared__ __align__(16) float s_query[];  // [dim]
    const int lane = threadIdx.x & 63;
    const int x = lane & 31, h = lane >> 5;
    const int q = blockIdx.x;
    const uint32_t c = A.cnt[q * A.cnt_stride];
    const uint32_t n = c < (uint32_t)A.cap ? c : (uint32_t)A.cap;
    if (32u * 4u * blockIdx.y >= n) return;  // uniform
    for (int d = threadIdx.x; d < A.D; d += 256) s_query[d] = A.qn[(int64_t)q * A.D + d];
    __syncthreads();
    const float q2 = A.qn2[q];
    const int32_t id = A.qid[q];
    uint64_t* list = A.cand + (size_t)q * A.cap;
    const uint32_t first = 32u * (blockIdx.y * 4u + (threadIdx.x >> 6));
    for (uint32_t j0 = first; j0 < n; j0 += 128u * gridDim.y) {
        const uint32_t j = j0 + (uint32_t)x;
        const bool ok = j < n;
        const int64_t row = ok ? (int64_t)(uint32_t)list[j] : 0;
        const float* src = A.T + row * (int64_t)A.D;
        knn_acc16 acc;
        float nr;
        knn_exact_products(
            A.D, h, [&](int d) { return *reinterpret_cast<const float4*>(s_query + d); },
            [&](int d) { return *reinterpret_cast<const float4*>(src + d); }, acc, nr);
        const float d2 = knn_exact_d2(q2, nr, acc[0]);
        if (ok && h == 0)
            list[j] = id >= 0 && row != (int64_t)id
                          ? ((uint64_t)__float_as_uint(d2) << 32) | (uint64_t)row
                          : kNoKey;
    }
}

// LDS: the queries' operands, [QB][chunks][64 lanes], then the bounds
// ((|q|^2 + 1 - tau) 2^19 less the margin), 32 per query block.
template <int QB>
__global__ __launch_bounds__(kKnnWideWaves * 64) __attribute__((amdgpu_waves_per_eu(2, 2)))
void k_knn_wide_scan(KnnWideArgs A) {
    constexpr int kCh = kKnnDimChunk / 16;  // chunks of a slab
    extern __shared__ __align__(16) uint8_t s_wide[];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int x = lane & 31, h = lane >> 5;
    const int D = A.D, nc = (D + 15) / 16;
    const int slabs = (nc + kCh - 1) / kCh;
    knn_h8* const s_q = reinterpret_cast<knn_h8*>(s_wide);
    float* const s_thr = reinterpret_cast<float*>(s_wide + sizeof(knn_h8) * 64 * QB * nc);
    for (int j = tid; j < QB * nc * 64; j += kKnnWideWaves * 64)
        s_q[j] = reinterpret_cast<const knn_h8*>(A.qh)[j];
    for (int q = tid; q < 32 * QB; q += kKnnWideWaves * 64) {
        const float q1 = A.qn2[q] > 0.f ? 1.f : 0.f;
        s_thr[q] = A.qid[q] >= 0
                       ? ((q1 + 1.f) - A.tau[q]) * kKnnAccPerD2 - 3.f - kKnnScreenMargin
                       : __builtin_inff();
    }
    __syncthreads();

    const int64_t W = (int64_t)gridDim.x * kKnnWideWaves;
    const int d0 = 8 * h;
    // slab sl of row x of tile i * step; past the scan or the table, row 0
    auto load_slab = [&](int64_t i, int sl, float4 (&dst)[2 * kCh]) {
        const int64_t row = i * A.step * 32 + x;
        const bool ok = i < A.count && row < A.N;
        const float* src = A.T + (ok ? row : 0) * (int64_t)D;
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            const int d = sl * kKnnDimChunk + 16 * c + d0;
            dst[2 * c] = d + 4 <= D ? *reinterpret_cast<const float4*>(src + d)
                                    : make_float4(0.f, 0.f, 0.f, 0.f);
            dst[2 * c + 1] = d + 8 <= D ? *reinterpret_cast<const float4*>(src + d + 4)
                                        : make_float4(0.f, 0.f, 0.f, 0.f);
        }
    };
    knn_acc16 acc[QB];
    float nr = 0.f, sc = 0.f;
    auto take_slab = [&](int64_t i, int sl, const float4 (&bv)[2 * kCh]) {
        float p = (knn_sq4(bv) + knn_sq4(bv + 4)) + (knn_sq4(bv + 8) + knn_sq4(bv + 12));
        p += __shfl_xor(p, 32, 64);
        if (sl == 0) {
            nr = p;
            sc = p > 0.f ? 64.f / sqrtf(p) : 0.f;
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[qb][r] = 0.f;
        } else {
            nr += p;
            // this slab would take the scaled norm past 2^14 (or is the first
            // that is not zero): the row is scaled anew, and its products with it
            const bool anew = sc * sc * nr > 268435456.f || (sc == 0.f && p > 0.f);
            if (__ballot(anew) != 0ull) {
                const float to = anew ? 64.f / sqrtf(nr) : sc;
                const float by = anew ? (sc > 0.f ? to / sc : 0.f) : 1.f;
                sc = to;
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[qb][r] *= by;
            }
        }
#pragma unroll
        for (int c = 0; c < kCh; ++c) {
            const int ch = sl * kCh + c;
            if (ch < nc) {
                const knn_h8 bh = knn_hi8(bv[2 * c], bv[2 * c + 1], sc);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb)
                    acc[qb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(
                        s_q[(qb * nc + ch) * 64 + lane], bh, acc[qb], 0, 0, 0);
            }
        }
        if (sl + 1 < slabs) return;
        // the tile is done: lane (x, h) holds row x against the queries
        // 8 (r / 4) + 4 h + r % 4 of every block
        const int64_t row = i * A.step * 32 + x;
        const float norm = sc * sqrtf(nr);
        const bool zero = nr == 0.f;
        const bool fits = nr >= kKnnNormMin && nr <= kKnnNormMax && norm >= 1.f && norm <= 16384.f;
        const bool there = row < A.N;
        const float f = zero ? 1.f : norm * (1.f / 1024.f);
        const float off = zero ? -kKnnAccPerD2 : 0.f;
        const bool force = there && !zero && !fits;
        uint32_t mask[QB];
        bool any = false;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            mask[qb] = 0u;
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const float4 th = *reinterpret_cast<const float4*>(s_thr + qb * 32 + 8 * r4 + 4 * h);
                const float t4[4] = {th.x, th.y, th.z, th.w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    // not below the bound (nor a number at all)
                    const bool left = !(acc[qb][4 * r4 + e] < fmaf(t4[e], f, off));
                    mask[qb] |= (left || force) && there ? 1u << (4 * r4 + e) : 0u;
                }
            }
            any |= mask[qb] != 0u;
        }
        if (__ballot(any) == 0ull) return;
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            for (uint32_t m = mask[qb]; m != 0u; m &= m - 1u) {
                const int r = __builtin_ctz(m);
                const int q = qb * 32 + 8 * (r / 4) + 4 * h + (r % 4);
                // a padding slot, or a query that the scans do not answer
                if (A.tau[q] == -__builtin_inff()) continue;
                // (an append is an atomic: not for rows in their thousands)
                if (force && __hip_atomic_load(&A.cnt[q * A.cnt_stride], __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT) > (uint32_t)A.cap)
                    continue;
                const uint32_t pos = atomicAdd(&A.cnt[q * A.cnt_stride], 1u);
                if (pos < (uint32_t)A.cap) A.cand[(size_t)q * A.cap + pos] = (uint64_t)row;
            }
        }
    };
    // slabs one after the other, in two register buffers
    float4 ba[2 * kCh], bb[2 * kCh];
    int64_t i = (int64_t)blockIdx.x * kKnnWideWaves + w;
    int sl = 0;
    if (i >= A.count) return;
    load_slab(i, 0, ba);
    while (true) {
        int64_t ni = i;
        int ns = sl + 1;
        if (ns == slabs) {
            ns = 0;
            ni += W;
        }
        load_slab(ni, ns, bb);
        take_slab(i, sl, ba);
        i = ni;
        sl = ns;
        if (i >= A.count) break;
        ns = sl + 1;
        if (ns == slabs) {
            ns = 0;
            ni += W;
        }
        load_slab(ni, ns, ba);
        take_slab(i, sl, bb);
        i = ni;
        sl = ns;
        if (i >= A.count) break;
    }
}

template <int QB>
static hipError_t launch_knn_wide_scan(const KnnWideArgs& A, hipStream_t s) {
    auto lds_bytes = [](int D) {
        return sizeof(knn_h8) * 64 * QB * (size_t)((D + 15) / 16) + sizeof(float) * 32 * QB;
    };
    const size_t lds = lds_bytes(A.D);
    // the widest rows taken: 32 queries of them fill kKnnQueryFloats
    const hipError_t e = allow_lds<&k_knn_wide_scan<QB>>(lds_bytes(kKnnQueryFloats / 32));
    if (e != hipSuccess) return e;
    int64_t grid = (A.count + kKnnWideWaves - 1) / kKnnWideWaves;
    grid = grid < kKnnGrid ? grid : kKnnGrid;
    hipLaunchKernelGGL(k_knn_wide_scan<QB>, dim3((unsigned)grid), dim3(kKnnWideWaves * 64), lds,
                       s, A);
    return hipGetLastError();
}

int knn_pass_queries(int D) {
    int qp = kKnnQueryFloats / (D + 4);
    qp = qp > kKnnPass ? kKnnPass : qp;
    return (qp / 32) * 32;
}

// Query blocks of a sub-pass of the list search for wide rows: as many (1 or 2)
// as its LDS holds and as the pass needs.
static int knn_wide_blocks(int D, int blocks) {
    return blocks >= 2 && knn_pass_queries(D) >= 64 ? 2 : 1;
}

// Tile strides of the scans of wide rows, coarsest first: the first visits at
// most kKnnStageTiles tiles (whose keys fit the lists), each next one is finer
// by one factor of at most kKnnWideGrowth, the last visits every tile.
// Returns the number of scans.
int knn_wide_steps(int64_t tiles, int64_t* steps) {
    int n = 1;
    for (int64_t reach = kKnnStageTiles; reach < tiles; reach *= kKnnWideGrowth) ++n;
    int64_t g = 1;  // the smallest factor that reaches every tile in n scans
    for (;; ++g) {
        int64_t reach = kKnnStageTiles;
        for (int j = 1; j < n && reach < tiles; ++j) reach *= g;
        if (reach >= tiles) break;
    }
    int64_t s = 1;
    for (int j = n - 1; j >= 0; --j, s *= g) steps[j] = s;
    return n;
}

// Lists of one pass: (workgroups) x (waves per query block).
int64_t knn_lists(int64_t N, int D, int QB) {
    const int64_t tiles = (N + 31) / 32;
    const int waves = D <= kKnnDimChunk ? kKnnWavesR : kKnnWaves;
    const int wpb = waves / QB;
    int64_t grid = (tiles + wpb - 1) / wpb;
    grid = grid < kKnnGrid ? grid : kKnnGrid;
    return grid * wpb;
}

template <int QB>
static void launch_knn_scan(const KnnScanArgs& A, hipStream_t s) {
    int64_t grid = (A.count + kKnnScanWaves - 1) / kKnnScanWaves;
    grid = grid < kKnnScanGrid ? grid : kKnnScanGrid;
    if (A.D == kKnnDimChunk)
        hipLaunchKernelGGL((k_knn_scan<QB, true>), dim3((unsigned)grid),
                           dim3(kKnnScanWaves * 64), 0, s, A);
    else
        hipLaunchKernelGGL((k_knn_scan<QB, false>), dim3((unsigned)grid),
                           dim3(kKnnScanWaves * 64), 0, s, A);
}

// Tile strides of the threshold scans, coarsest first: the first visits at
// most kKnnStageTiles tiles with no bound (so its lists cannot overflow), each
// next one a stride kKnnStageGrowth times finer, the last every tile.  Returns
// the number of scans.
int knn_scan_steps(int64_t tiles, int64_t* steps) {
    int64_t s = 1;
    while ((tiles + s - 1) / s > kKnnStageTiles) s *= kKnnStageGrowth;
    int n = 0;
    for (; s >= 1; s /= kKnnStageGrowth) steps[n++] = s;
    return n;
}

hipError_t launch_knn(const float* T, int64_t N, int32_t D, const int32_t* q, int32_t nq,
                      int32_t k, int32_t* ids, float* dist, const KnnBuffers& B,
                      bool lists_only, int32_t* status, hipStream_t s) {
    if (knn_pass_queries(D) < 32 || k < 1 || k > kKnnMaxK || N < 1) return hipErrorInvalidValue;
    const bool wide = D > kKnnDimChunk;
    const bool scans = !lists_only;
    const int64_t tiles = (N + 31) / 32;
    for (int32_t q0 = 0; q0 < nq; q0 += kKnnPass) {
        const int32_t m = nq - q0 < kKnnPass ? nq - q0 : kKnnPass;
        int QB = (m + 31) / 32;
        if (QB == 3) QB = 4;
        const int32_t nqp = 32 * QB;
        hipLaunchKernelGGL(k_knn_queries, dim3((unsigned)nqp), dim3(kBlock), 0, s, T, N, D,
                           q + q0, m, nqp, B.qn, B.qn2, B.qid, scans ? B.tau : nullptr,
                           scans ? B.cnt : nullptr, B.cnt_stride, scans ? B.gate : nullptr,
                           scans && wide && tiles > kKnnStageTiles ? B.qh : nullptr, status);
        KnnSelectArgs SS;
        SS.cnt = B.cnt;
        SS.cand = B.cand;
        SS.cap = kKnnCandCap;
        SS.cnt_stride = B.cnt_stride;
        SS.k = k;
        SS.m = m;
        SS.q_first = q0;
        SS.qid = B.qid;
        SS.tau = B.tau;
        SS.ids = ids;
        SS.dist = dist;
        SS.gate = B.gate;
        int64_t steps[16];
        if (scans && wide) {
            KnnWideArgs WA;
            WA.T = T;
            WA.N = N;
            WA.D = D;
            WA.cap = kKnnCandCap;
            WA.cnt_stride = B.cnt_stride;
            WA.qn = B.qn;
            WA.qn2 = B.qn2;
            WA.qid = B.qid;
            WA.qh = B.qh;
            WA.tau = B.tau;
            WA.cnt = B.cnt;
            WA.cand = B.cand;
            const int ns = knn_wide_steps(tiles, steps);
            for (int j = 0; j < ns; ++j) {
                WA.step = steps[j];
                WA.count = (tiles + steps[j] - 1) / steps[j];
                if (j == 0) {
                    const dim3 grid((unsigned)((WA.count * QB + 3) / 4));
                    if (QB == 4)
                        hipLaunchKernelGGL(k_knn_wide_dense<4>, grid, dim3(256), 0, s, WA);
                    else if (QB == 2)
                        hipLaunchKernelGGL(k_knn_wide_dense<2>, grid, dim3(256), 0, s, WA);
                    else
                        hipLaunchKernelGGL(k_knn_wide_dense<1>, grid, dim3(256), 0, s, WA);
                } else {
                    const hipError_t e = QB == 4   ? launch_knn_wide_scan<4>(WA, s)
                                         : QB == 2 ? launch_knn_wide_scan<2>(WA, s)
                                                   : launch_knn_wide_scan<1>(WA, s);
                    if (e != hipSuccess) return e;
                    // k g rows per query and those within the screen's margin: a
                    // round or two of 32 rows for each of 32 waves
                    hipLaunchKernelGGL(k_knn_wide_rescore, dim3((unsigned)nqp, 8), dim3(256),
                                       sizeof(float) * (size_t)D, s, WA);
                }
                SS.last = j == ns - 1;
                hipLaunchKernelGGL(k_knn_select, dim3((unsigned)nqp), dim3(kKnnSelectThreads),
                                   sizeof(uint64_t) * kKnnCandCap, s, SS);
            }
        } else if (scans) {
            KnnScanArgs SA;
            SA.T = T;
            SA.N = N;
            SA.D = D;
            SA.cap = kKnnCandCap;
            SA.cnt_stride = B.cnt_stride;
            SA.qn = B.qn;
            SA.qn2 = B.qn2;
            SA.qid = B.qid;
            SA.tau = B.tau;
            SA.cnt = B.cnt;
            SA.cand = B.cand;
            const int ns = knn_scan_steps(tiles, steps);
            for (int j = 0; j < ns; ++j) {
                SA.step = steps[j];
                SA.count = (tiles + steps[j] - 1) / steps[j];
                if (QB == 4)
                    launch_knn_scan<4>(SA, s);
                else if (QB == 2)
                    launch_knn_scan<2>(SA, s);
                else
                    launch_knn_scan<1>(SA, s);
                SS.last = j == ns - 1;
                hipLaunchKernelGGL(k_knn_select, dim3((unsigned)nqp), dim3(kKnnSelectThreads),
                                   sizeof(uint64_t) * kKnnCandCap, s, SS);
            }
        }
        // the list-merging search: asked for, or where a final candidate list
        // overflowed (the gate; otherwise its kernels return at once)
        KnnArgs A;
        A.T = T;
        A.N = N;
        A.D = D;
        A.k = k;
        A.QB = wide ? knn_wide_blocks(D, QB) : QB;
        A.nqp = 32 * A.QB;
        A.subs = nqp / A.nqp;
        A.stride = D + 4;
        A.tiles = tiles;
        A.qn = B.qn;
        A.qn2 = B.qn2;
        A.qid = B.qid;
        A.partial = B.partial;
        A.gate = scans ? B.gate : nullptr;
        const int64_t NS = knn_lists(N, D, A.QB);
        if (!wide) {
            const int64_t grid = NS / (kKnnWavesR / QB);
            if (QB == 4)
                hipLaunchKernelGGL(k_knn_tiles_h4, dim3((unsigned)grid), dim3(kKnnWavesR * 64), 0,
                                   s, A);
            else
                hipLaunchKernelGGL(k_knn_tiles_h, dim3((unsigned)grid), dim3(kKnnWavesR * 64), 0,
                                   s, A);
        } else {
            const int64_t grid = NS / (kKnnWaves / A.QB);
            hipLaunchKernelGGL(k_knn_tiles, dim3((unsigned)grid), dim3(kKnnWaves * 64), 0, s, A);
        }
        hipLaunchKernelGGL(k_knn_merge, dim3((unsigned)m), dim3(kBlock), 0, s, B.partial, NS,
                           A.nqp, k, q0, ids, dist, A.gate);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// recall@k(u) = |N(u) & S| / k, S = the query's k nearest rows (ids[q k ..]),
// N(u) = the ids of u's ascending list other than u.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_eval_recall(const int64_t* __restrict__ off,
                                                    const int32_t* __restrict__ nbr, int64_t N,
                                                    int64_t E, const int32_t* __restrict__ q,
                                                    const int32_t* __restrict__ ids, int32_t k,
                                                    double* __restrict__ out,
                                                    int32_t* __restrict__ status) {
    const int qi = blockIdx.x;
    const int t = threadIdx.x;
    const int32_t u = q[qi];
    bool found = false;
    bool bad = u < 0 || (int64_t)u >= N;
    int64_t b = 0, e = 0;
    if (!bad) {
        b = off[u];
        e = off[u + 1];
        bad = b < 0 || e < b || e > E;
    }
    if (!bad && t < k) {
        const int32_t id = ids[(int64_t)qi * k + t];
        found = id >= 0 && id != u && in_sorted_list(nbr, b, e, id);
    }
    const uint64_t m = __ballot(found);
    if (t == 0) {
        if (bad) eval_fail(status, -2);
        out[qi] = bad ? __builtin_nan("") : (double)__popcll(m) / (double)k;
    }
}

hipError_t launch_eval_recall(const int64_t* off, const int32_t* nbr, int64_t N, int64_t E,
                              const int32_t* q, int32_t nq, const int32_t* ids, int32_t k,
                              double* out, int32_t* status, hipStream_t s) {
    if (nq == 0) return hipSuccess;
    if (k < 1 || k > 64) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_eval_recall, dim3((unsigned)nq), dim3(64), 0, s, off, nbr, N, E, q, ids,
                       k, out, status);
    return hipGetLastError();
}

__global__ void k_eval_status_clear(int32_t* status) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *status = 0;
}

hipError_t launch_eval_status_clear(int32_t* status, hipStream_t s) {
    hipLaunchKernelGGL(k_eval_status_clear, dim3(1), dim3(64), 0, s, status);
    return hipGetLastError();
}

}  // namespace huge
