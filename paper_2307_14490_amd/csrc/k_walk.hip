// Co-occurrence triples from uniform random walks on a CSR graph in device
// memory: the sampler that produces the training step's input (HUGE
// Sec. 3.2, Alg. 1), on the GPU.
//
// Every seed node s is repeated gamma times; walk r of s takes k uniform
// steps: w_0 = s, and w_t is neighbour floor(x deg / 2^64) of w_{t-1}, with x
// the first 64 bits of Philox4x32-10 on counter (lo32 s, hi32 s, r, 4 + t); a
// node without neighbours ends the walk.  The walks of one seed are grouped
// and their co-occurrences combined (Alg. 1, GroupByKey and CombineValues):
// the pairs (s, w_t) for t <= window, or -- DeepWalk's window -- every ordered
// pair (w_a, w_b) of a walk with 1 <= |a - b| <= window; pairs of a node with
// itself are dropped.  One triple per distinct (source, destination) of a
// seed: cc = its co-occurrences, hist[d - 1] = those at distance d.  Seeds are
// emitted in ascending order and, within a seed, (source, destination)
// ascending, so the output is bitwise reproducible.
//
//   k_walk_nodes  one thread per walk takes it and writes its nodes to the
//                 workspace;
//   k_walk_group  one wave per seed: the seed's pairs as 32-bit keys, sorted
//                 in registers, equal keys adjacent.  A first pass counts the
//                 seed's triples;
//   k_walk_sums,  the triples' places: sums of ranges of the counts, then
//   k_walk_scan   their exclusive scan;
//   k_walk_group  a second pass repeats the sort and writes them.  (Keeping the
//                 sorted keys was not tried: a walk of 20 steps in windows of 3
//                 has 456 bytes of them, written and read, for 80 of nodes.)
// The nodes of the walks fill kWalkNodeBytesMax at most (or what the workspace
// holds): more seeds are taken in chunks, whose walks are taken once for each
// pass.
#include "common.hpp"
#include "device.hpp"

namespace huge {

// Order a wave's LDS accesses: a wave's LDS instructions execute in order, so
// the compiler keeping them in order is all that is needed.
__device__ __forceinline__ void wave_lds_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// ---------------------------------------------------------------------------
// Walk r of seed s (thread w = g walks + r of the chunk) into
// nodes[w steps .. + steps): its nodes w_1 ..; -1 past its end, and for the
// whole of a walk on a malformed graph (reported).  The kernel waits for the
// dependent reads of the CSR arrays (two offsets, one neighbour per hop): one
// thread per walk keeps up to 2048 walks per CU in flight.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void k_walk_nodes(WalkArgs A, int64_t g0, uint32_t nw,
                                                       const int64_t* __restrict__ total,
                                                       int64_t capacity, int again,
                                                       int32_t* __restrict__ nodes,
                                                       int32_t* __restrict__ status) {
    // the second pass of a call that writes nothing
    if (again && (*status != 0 || *total > capacity)) return;
    const uint32_t w = blockIdx.x * (uint32_t)kBlock + threadIdx.x;
    if (w >= nw) return;
    const uint32_t g = w / (uint32_t)A.walks, r = w - g * (uint32_t)A.walks;
    const int64_t s = A.first_seed + g0 + g;
    int32_t* __restrict__ out = nodes + (int64_t)w * A.steps;
    const uint32_t key_lo = (uint32_t)A.seed, key_hi = (uint32_t)(A.seed >> 32);
    const bool vec = (A.steps & 3) == 0;
    int64_t cur = s;  // -1: the walk has ended
    bool bad = false;
    for (int32_t t0 = 0; t0 < A.steps; t0 += 4) {
        int32_t v[4] = {-1, -1, -1, -1};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int32_t t = t0 + j;
            if (t >= A.steps || cur < 0) continue;
            const uint4 rr = philox4x32_10(make_uint4((uint32_t)s, (uint32_t)((uint64_t)s >> 32),
                                                      r, 5u + (uint32_t)t), key_lo, key_hi);
            const int64_t b = A.off[cur], e = A.off[cur + 1];
            if (b < 0 || e < b || e > A.num_edges) {
                bad = true;
                cur = -1;
                continue;
            }
            const uint64_t deg = (uint64_t)(e - b);
            if (deg == 0) {
                cur = -1;
                continue;
            }
            const uint64_t x = ((uint64_t)rr.y << 32) | (uint64_t)rr.x;
            const int64_t next = A.nbr[b + (int64_t)__umul64hi(x, deg)];
            if (next < 0 || next >= A.num_nodes) {
                bad = true;
                cur = -1;
                continue;
            }
            v[j] = (int32_t)next;
            cur = next;
        }
        if (vec) {
            *reinterpret_cast<int4*>(out + t0) = make_int4(v[0], v[1], v[2], v[3]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (t0 + j < A.steps) out[t0 + j] = v[j];
        }
    }
    if (bad) {
        atomicCAS(status, 0, -2);
        for (int32_t t = 0; t < A.steps; ++t) out[t] = -1;
    }
}

// ---------------------------------------------------------------------------
// Bitonic sort of 64 R keys over a wave, ascending, element l R + i in lane
// l's register i.  Strides below R are compare-exchanges of a lane's own
// registers; the others meet the lane l XOR (stride / R) by DPP and row swaps.
// A direction that depends on the lane costs nothing: the median of (a, b, 0)
// is their minimum, that of (a, b, ~0) their maximum.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t med3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t d;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// min (sel = 0) or max (sel = ~0) of x and of lane (lane XOR D)'s x.
template <int D>
__device__ __forceinline__ uint32_t xor_pick(uint32_t x, uint32_t sel) {
    const int v = (int)x;
    if constexpr (D == 1) {
        return med3(x, (uint32_t)__builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false), sel);
    } else if constexpr (D == 2) {
        return med3(x, (uint32_t)__builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false), sel);
    } else if constexpr (D == 4) {  // mirror within 8 (XOR 7), then within 4 (XOR 3)
        const int m = __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);
        return med3(x, (uint32_t)__builtin_amdgcn_update_dpp(0, m, 0x1B, 0xF, 0xF, false), sel);
    } else if constexpr (D == 8) {  // rotation by 8 within 16
        return med3(x, (uint32_t)__builtin_amdgcn_update_dpp(0, v, 0x128, 0xF, 0xF, false), sel);
    } else if constexpr (D == 16) {  // both results: the lane's own and its partner's
        const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return med3(p[0], p[1], sel);
    } else {
        static_assert(D == 32, "a power of two below 64");
        const auto p = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return med3(p[0], p[1], sel);
    }
}

// One stride of the merge of runs of SIZE elements.
template <int R, int SIZE, int STRIDE>
__device__ __forceinline__ void sort_stride(uint32_t (&v)[R], uint32_t lane) {
    if constexpr (STRIDE >= R) {
        constexpr int D = STRIDE / R;
        const bool asc = SIZE >= 64 * R || (lane & (uint32_t)(SIZE / R)) == 0u;
        const uint32_t sel = ((lane & (uint32_t)D) == 0u) == asc ? 0u : ~0u;
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = xor_pick<D>(v[i], sel);
    } else if constexpr (SIZE < R) {  // the direction is the register's
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (i & STRIDE) continue;
            const uint32_t a = v[i], b = v[i | STRIDE];
            const uint32_t lo = a < b ? a : b, hi = a < b ? b : a;
            v[i] = (i & SIZE) ? hi : lo;
            v[i | STRIDE] = (i & SIZE) ? lo : hi;
        }
    } else {
        const bool asc = SIZE >= 64 * R || (lane & (uint32_t)(SIZE / R)) == 0u;
        const uint32_t sel = asc ? 0u : ~0u;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            if (i & STRIDE) continue;
            const uint32_t a = v[i], b = v[i | STRIDE];
            v[i] = med3(a, b, sel);
            v[i | STRIDE] = med3(a, b, ~sel);
        }
    }
}

template <int R, int SIZE, int STRIDE>
__device__ __forceinline__ void sort_merge(uint32_t (&v)[R], uint32_t lane) {
    sort_stride<R, SIZE, STRIDE>(v, lane);
    if constexpr (STRIDE > 1) sort_merge<R, SIZE, STRIDE / 2>(v, lane);
}

template <int R, int SIZE = 2>
__device__ __forceinline__ void wave_sort(uint32_t (&v)[R], uint32_t lane) {
    sort_merge<R, SIZE, SIZE / 2>(v, lane);
    if constexpr (SIZE < 64 * R) wave_sort<R, 2 * SIZE>(v, lane);
}

// Store a lane's registers at s[lane R ..] (their sorted places).
template <int R>
__device__ __forceinline__ void store_blocked(uint32_t* s, const uint32_t (&v)[R],
                                              uint32_t lane) {
    if constexpr (R >= 4) {
#pragma unroll
        for (int i = 0; i < R; i += 4)
            *reinterpret_cast<uint4*>(s + lane * R + i) =
                make_uint4(v[i], v[i + 1], v[i + 2], v[i + 3]);
    } else {
#pragma unroll
        for (int i = 0; i < R; ++i) s[lane * R + i] = v[i];
    }
}

// Sort the n values of s (n <= 64 R) in place; places n .. 64 R - 1 receive ~0.
template <int R>
__device__ __forceinline__ void sort_lds(uint32_t* s, uint32_t n, uint32_t lane) {
    uint32_t v[R];
#pragma unroll
    for (int i = 0; i < R; ++i) v[i] = lane + 64u * i < n ? s[lane + 64u * i] : ~0u;
    wave_lds_order();
    wave_sort<R>(v, lane);
    store_blocked<R>(s, v, lane);
    wave_lds_order();
}

// Index of the first of the n ascending values not below x.
__device__ __forceinline__ uint32_t lower_bound(const uint32_t* s, uint32_t n, uint32_t x) {
    uint32_t lo = 0;
    for (uint32_t len = n; len > 0;) {
        const uint32_t half = len >> 1;
        const bool below = s[lo + half] < x;
        lo = below ? lo + half + 1u : lo;
        len = below ? len - half - 1u : half;
    }
    return lo;
}

// Registers per lane of the node sort of a RANK variant with R per lane for
// the pairs: R, or the small size where the nodes fit in it.
template <int R>
constexpr int small_sort() {
    return R >= 4 ? R / 4 : 1;
}

// ---------------------------------------------------------------------------
// The triples of seed g0 + (the wave's index), from its walks' nodes:
//   pair keys: seed pairs are (destination << 5 | distance - 1) where ids
//     have at most 27 bits; otherwise (RANK) the seed's nodes are sorted
//     first and a key holds the nodes' places in that order, at most 13 bits
//     each (source << 18 | destination << 5 | distance - 1), so every key has
//     32 bits and their order is that of (source, destination, distance).  A
//     pair that does not exist (a walk that ended, a node with itself) is ~0;
//   sort: 64 R keys in registers;
//   runs: a key whose pair differs from the one before starts a triple.
// WRITE = false stores the number of triples in counts[g]; WRITE = true
// writes them from offsets[g]: the run starts go to LDS by rank, then lane i
// takes runs i, i + 64, ..., so that the triples' stores are contiguous.
// LDS per wave: 64 R keys, 64 R run starts (16 bits) and, with RANK, the
// sorted nodes and the places (16 bits) of the walks' nodes.
// The wave has no barrier to wait for; against one workgroup per seed with a
// bitonic sort in LDS (73 KB: two workgroups per CU), 65,536 seeds of 128
// walks x 3 steps took 5.07 ms before and 0.56 ms now (nodes 0.29, counting 0.09,
// writing 0.19), 500,000 seeds of one walk x 20 steps in windows of 3 took
// 91.7 ms and 1.04 ms (0.29, 0.36, 0.45).
// ---------------------------------------------------------------------------
constexpr uint32_t kNoPair = ~0u;
constexpr uint32_t kNoPlace = 0xFFFFu;
constexpr int64_t kDirectNodes = (int64_t)1 << 27;  // ids below it fit a key directly
constexpr int64_t kWalkMostSeeds = (int64_t)1 << 25;  // seeds of a launch

template <int R, bool RANK, bool WRITE>
__global__ __launch_bounds__(kBlock) void k_walk_group(
    WalkArgs A, int64_t g0, int64_t ng, int32_t pairs, const int32_t* __restrict__ nodes,
    uint32_t* __restrict__ counts, const uint64_t* __restrict__ offsets,
    const int64_t* __restrict__ total, int64_t capacity, int32_t* __restrict__ src,
    int32_t* __restrict__ dst, int32_t* __restrict__ cc, int32_t* __restrict__ hist,
    const int32_t* __restrict__ status, uint32_t wave_words) {
    extern __shared__ __align__(16) uint32_t s_dyn[];
    if (WRITE && (*status != 0 || *total > capacity)) return;  // nothing is written
    const uint32_t lane = threadIdx.x & 63u;
    const int64_t i = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
    if (i >= ng) return;  // no barrier below
    uint32_t* const s_key = s_dyn + (threadIdx.x >> 6) * wave_words;      // [64 R]
    uint16_t* const s_start = reinterpret_cast<uint16_t*>(s_key + 64 * R);  // [64 R]
    uint32_t* const s_node = s_key + 96 * R;                              // with RANK
    const int64_t g = g0 + i;
    const int32_t s = (int32_t)(A.first_seed + g);
    const int32_t* __restrict__ nd = nodes + i * (int64_t)(A.walks * A.steps);
    const uint32_t P = (uint32_t)pairs, window = (uint32_t)A.window, steps = (uint32_t)A.steps;

    // slots of seed pairs: slot q is walk q / window, distance q % window + 1
    auto seed_slots = [&](auto&& take) {
        const uint32_t dr = 64u / window, dt = 64u - dr * window;
        uint32_t r = lane / window, t = lane - r * window;
        for (uint32_t q = lane; q < P; q += 64u) {
            take(q, nd[r * steps + t], t);
            r += dr;
            t += dt;
            if (t >= window) {
                t -= window;
                ++r;
            }
        }
    };
    uint32_t v[R];
    if constexpr (!RANK) {
        seed_slots([&](uint32_t q, int32_t node, uint32_t t) {
            s_key[q] = node >= 0 && node != s ? (uint32_t)node << 5 | t : kNoPair;
        });
        wave_lds_order();
    } else {
        // the walks' nodes: those of the seed pairs' slots, or every position
        // (walk p / (steps + 1), node p % (steps + 1), node 0 the seed)
        const uint32_t L1 = steps + 1u;
        const uint32_t L = A.seed_only ? P : (uint32_t)A.walks * L1;
        const bool small = L <= 64u * small_sort<R>();
        const uint32_t Lp = 64u * (small ? small_sort<R>() : R);
        uint16_t* const s_place = reinterpret_cast<uint16_t*>(s_node + Lp);
        if (A.seed_only) {
            seed_slots([&](uint32_t q, int32_t node, uint32_t) { s_node[q] = (uint32_t)node; });
        } else {
            for (uint32_t p = lane; p < L; p += 64u) {
                const uint32_t r = p / L1, t = p - r * L1;
                s_node[p] = t == 0u ? (uint32_t)s : (uint32_t)nd[r * steps + t - 1u];
            }
        }
        wave_lds_order();
        // a position's node, then the nodes in order, then its place there
        // (a missing node is -1, the largest value)
        uint32_t own[R];
#pragma unroll
        for (int c = 0; c < R; ++c) own[c] = lane + 64u * c < L ? s_node[lane + 64u * c] : ~0u;
        if (small)
            sort_lds<small_sort<R>()>(s_node, L, lane);
        else
            sort_lds<R>(s_node, L, lane);
#pragma unroll
        for (int c = 0; c < R; ++c) {
            const uint32_t p = lane + 64u * c;
            if (p < L)
                s_place[p] = (uint16_t)(own[c] == ~0u ? kNoPlace
                                                      : lower_bound(s_node, L, own[c]));
        }
        wave_lds_order();
        if (A.seed_only) {
            const uint32_t dt = 64u - 64u / window * window;
            uint32_t t = lane % window;
            for (uint32_t q = lane; q < P; q += 64u) {
                const uint32_t b = s_place[q];
                s_key[q] = b != kNoPlace && s_node[b] != (uint32_t)s ? b << 5 | t : kNoPair;
                t += dt;
                if (t >= window) t -= window;
            }
        } else {
            // slots of one walk: distance by distance, its 2 (steps + 1 - d)
            // ordered pairs (a, a + d), (a + d, a)
            const uint32_t per = P / (uint32_t)A.walks;
            for (uint32_t q = lane; q < P; q += 64u) {
                const uint32_t r = q / per;
                uint32_t k = q - r * per, d = 1u, n = 2u * (L1 - 1u);
                while (k >= n) {
                    k -= n;
                    n -= 2u;
                    ++d;
                }
                const uint32_t a = r * L1 + (k >> 1);
                const uint32_t x = s_place[a], y = s_place[a + d];
                const uint32_t from = k & 1u ? y : x, to = k & 1u ? x : y;
                s_key[q] = x != kNoPlace && y != kNoPlace && x != y
                               ? from << 18 | to << 5 | (d - 1u)
                               : kNoPair;
            }
        }
        wave_lds_order();
    }
#pragma unroll
    for (int c = 0; c < R; ++c) v[c] = lane + 64u * c < P ? s_key[lane + 64u * c] : kNoPair;
    wave_lds_order();
    wave_sort<R>(v, lane);

    // runs: element lane R + c starts one if its pair differs from the one
    // before (the missing pairs sort last)
    const uint32_t before = __shfl_up(v[R - 1], 1, 64);
    uint32_t runs = 0, mine = 0, valid = 0;
    uint64_t starts = 0;  // bit c: register c starts a run
#pragma unroll
    for (int c = 0; c < R; ++c) {
        const uint32_t prev = c > 0 ? v[c > 0 ? c - 1 : 0] : before;
        const bool pair = v[c] != kNoPair;
        const bool st = pair && ((lane == 0u && c == 0) || (v[c] >> 5) != (prev >> 5));
        runs += (uint32_t)__popcll(__ballot(st));
        if constexpr (WRITE) {
            valid += (uint32_t)__popcll(__ballot(pair));
            starts |= st ? 1ull << c : 0ull;
            mine += st ? 1u : 0u;
        }
    }
    if constexpr (!WRITE) {
        if (lane == 0u) counts[g] = runs;
        return;
    }
    uint32_t incl = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, 64);
        if (lane >= (uint32_t)off) incl += t;
    }
    uint32_t rank = incl - mine;
    store_blocked<R>(s_key, v, lane);
#pragma unroll
    for (int c = 0; c < R; ++c)
        if (starts >> c & 1ull) s_start[rank++] = (uint16_t)(lane * R + c);
    wave_lds_order();
    const int64_t base = (int64_t)offsets[g];
    for (uint32_t q = lane; q < runs; q += 64u) {
        const int64_t o = base + q;
        if (o >= capacity) break;  // cannot happen: the total fits
        uint32_t e = s_start[q];
        const uint32_t end = q + 1u < runs ? s_start[q + 1u] : valid;
        const uint32_t key = s_key[e];
        if constexpr (RANK) {
            src[o] = A.seed_only ? s : (int32_t)s_node[key >> 18];
            dst[o] = (int32_t)s_node[key >> 5 & 0x1FFFu];
        } else {
            src[o] = s;
            dst[o] = (int32_t)(key >> 5);
        }
        cc[o] = (int32_t)(end - e);
        if (hist != nullptr) {
            for (uint32_t d = 0; d < window; ++d) {
                uint32_t n = 0;
                while (e < end && (s_key[e] & 31u) == d) {
                    ++e;
                    ++n;
                }
                hist[o * (int64_t)window + d] = (int32_t)n;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Exclusive scan of the per-seed counts into 64-bit offsets, by the sums of at
// most kWalkRanges ranges of `len` counts (a multiple of kWalkStep): every
// workgroup of k_walk_scan adds the sums before its range itself, so the two
// kernels read the counts twice and nothing waits.  (One workgroup for the
// whole scan took 550 us of 500,000 seeds; these two take 11 us.)
// ---------------------------------------------------------------------------
constexpr int kWalkPer = 8;                       // counts per thread and step
constexpr int64_t kWalkStep = kBlock * kWalkPer;

// Sum over the workgroup (kBlock threads) of one value per thread: returns
// the exclusive prefix of this thread, *total gets the sum.  Synchronises;
// s_tmp may be reused after the next barrier.
__device__ __forceinline__ uint64_t walk_block_excl(uint64_t v, uint64_t* s_tmp,
                                                    uint64_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint64_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t t = __shfl_up((unsigned long long)incl, off, 64);
        if (lane >= off) incl += t;
    }
    if (lane == 63) s_tmp[wave] = incl;
    __syncthreads();
    uint64_t add = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        const uint64_t x = s_tmp[w];
        if (w < wave) add += x;
        all += x;
    }
    *total = all;
    return add + incl - v;
}

__global__ __launch_bounds__(kBlock) void k_walk_sums(const uint32_t* __restrict__ counts,
                                                      int64_t n, int64_t len,
                                                      uint64_t* __restrict__ sums) {
    __shared__ uint64_t s_tmp[kBlock / 64];
    const int64_t a = (int64_t)blockIdx.x * len;
    const int64_t b = a + len < n ? a + len : n;
    uint64_t sum = 0;
    for (int64_t i = a + threadIdx.x; i < b; i += kBlock) sum += counts[i];
    uint64_t total;
    walk_block_excl(sum, s_tmp, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// The last workgroup writes the number of triples; one above the capacity is
// reported (nothing is written then).
__global__ __launch_bounds__(kBlock) void k_walk_scan(const uint32_t* __restrict__ counts,
                                                      const uint64_t* __restrict__ sums,
                                                      uint64_t* __restrict__ offsets, int64_t n,
                                                      int64_t len, int64_t* __restrict__ total,
                                                      int64_t capacity,
                                                      int32_t* __restrict__ status) {
    __shared__ uint64_t s_tmp[2][kBlock / 64];
    uint64_t before = 0;
    for (uint32_t j = threadIdx.x; j < blockIdx.x; j += kBlock) before += sums[j];
    uint64_t carry;
    walk_block_excl(before, s_tmp[0], &carry);
    const int64_t a = (int64_t)blockIdx.x * len;
    const int64_t b = a + len < n ? a + len : n;
    int turn = 1;  // the two halves of s_tmp in turn: one barrier per step
    for (int64_t c0 = a; c0 < b; c0 += kWalkStep, turn ^= 1) {
        uint32_t v[kWalkPer];
        uint64_t sum = 0;
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) {
            const int64_t i = c0 + (int64_t)threadIdx.x * kWalkPer + q;
            v[q] = i < b ? counts[i] : 0u;
            sum += v[q];
        }
        uint64_t step;
        uint64_t run = carry + walk_block_excl(sum, s_tmp[turn], &step);
#pragma unroll
        for (int q = 0; q < kWalkPer; ++q) {
            const int64_t i = c0 + (int64_t)threadIdx.x * kWalkPer + q;
            if (i < b) offsets[i] = run;
            run += v[q];
        }
        carry += step;
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        *total = (int64_t)carry;
        if (*status == 0 && (int64_t)carry > capacity) *status = -4;
    }
}

// Clears the status word; with no seeds, the number of triples too.
__global__ void k_walk_begin(int32_t* status, int64_t* total, int none) {
    if (threadIdx.x == 0) {
        *status = 0;
        if (none) *total = 0;
    }
}

namespace {

// LDS words of one wave of k_walk_group<R, RANK> for nl nodes.
uint32_t walk_wave_words(int R, bool rank, int64_t nl) {
    uint32_t w = 96u * (uint32_t)R;
    if (rank) {
        const int rs = R >= 4 ? R / 4 : 1;
        w += 96u * (uint32_t)(nl <= 64 * rs ? rs : R);  // the nodes, their places
    }
    return w;
}

template <int R, bool RANK>
void launch_walk_group(const WalkArgs& A, int64_t g0, int64_t ng, int32_t pairs, bool write,
                       const WalkBuffers& B, const WalkOut& O, hipStream_t s) {
    const int64_t nl = A.seed_only ? pairs : (int64_t)A.walks * (A.steps + 1);
    const uint32_t words = walk_wave_words(R, RANK, nl);
    // four waves per workgroup while their LDS stays within 64 KB
    const int waves = words * 4u * sizeof(uint32_t) <= 65536u ? 4 : 1;
    const dim3 grid((unsigned)((ng + waves - 1) / waves)), block((unsigned)(64 * waves));
    const size_t lds = sizeof(uint32_t) * words * (size_t)waves;
    if (write)
        hipLaunchKernelGGL((k_walk_group<R, RANK, true>), grid, block, lds, s, A, g0, ng, pairs,
                           B.nodes, B.counts, B.offsets, O.count, O.capacity, O.src, O.dst, O.cc,
                           O.hist, O.status, words);
    else
        hipLaunchKernelGGL((k_walk_group<R, RANK, false>), grid, block, lds, s, A, g0, ng, pairs,
                           B.nodes, B.counts, B.offsets, O.count, O.capacity, O.src, O.dst, O.cc,
                           O.hist, O.status, words);
}

template <bool RANK>
hipError_t launch_walk_pass(const WalkArgs& A, int64_t g0, int64_t ng, int32_t pairs, bool write,
                            const WalkBuffers& B, const WalkOut& O, hipStream_t s) {
    int R = 1;
    while (64 * R < pairs) R <<= 1;
    switch (R) {
        case 1: launch_walk_group<1, RANK>(A, g0, ng, pairs, write, B, O, s); break;
        case 2: launch_walk_group<2, RANK>(A, g0, ng, pairs, write, B, O, s); break;
        case 4: launch_walk_group<4, RANK>(A, g0, ng, pairs, write, B, O, s); break;
        case 8: launch_walk_group<8, RANK>(A, g0, ng, pairs, write, B, O, s); break;
        case 16: launch_walk_group<16, RANK>(A, g0, ng, pairs, write, B, O, s); break;
        case 32: launch_walk_group<32, RANK>(A, g0, ng, pairs, write, B, O, s); break;
        case 64: launch_walk_group<64, RANK>(A, g0, ng, pairs, write, B, O, s); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_walks(const WalkArgs& A, int32_t pairs, const WalkBuffers& B, const WalkOut& O,
                        hipStream_t s) {
    const int64_t n = A.num_seeds;
    hipLaunchKernelGGL(k_walk_begin, dim3(1), dim3(64), 0, s, O.status, O.count,
                       n == 0 ? 1 : 0);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || n == 0) return e;
    if (pairs < 1 || pairs > kWalkMaxPairs || (int64_t)A.walks * A.steps > kWalkMaxNodes)
        return hipErrorInvalidValue;
    // seeds whose nodes fit the buffer at a time
    const int64_t per_seed = (int64_t)A.walks * A.steps;
    int64_t fit = B.node_cap / per_seed;
    if (fit < 1) return hipErrorInvalidValue;
    // a wave per seed and fewer than 2^32 threads in a launch: 2^26 seeds of one
    // walk of one step, whose nodes fit, are 2^32
    if (fit > kWalkMostSeeds) fit = kWalkMostSeeds;
    const int64_t chunk = n < fit ? n : fit;
    const bool direct = A.seed_only && A.num_nodes < kDirectNodes;
    for (int pass = 0; pass < 2; ++pass) {
        const bool write = pass == 1;
        for (int64_t g0 = 0; g0 < n; g0 += chunk) {
            const int64_t ng = n - g0 < chunk ? n - g0 : chunk;
            if (!write || chunk < n) {  // one chunk: its nodes are still there
                const uint32_t nw = (uint32_t)(ng * A.walks);
                hipLaunchKernelGGL(k_walk_nodes, dim3((nw + kBlock - 1) / kBlock), dim3(kBlock),
                                   0, s, A, g0, nw, O.count, O.capacity, write ? 1 : 0, B.nodes,
                                   O.status);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
            e = direct ? launch_walk_pass<false>(A, g0, ng, pairs, write, B, O, s)
                       : launch_walk_pass<true>(A, g0, ng, pairs, write, B, O, s);
            if (e != hipSuccess) return e;
        }
        if (!write) {
            int64_t len = (n + kWalkRanges - 1) / kWalkRanges;
            len = (len + kWalkStep - 1) / kWalkStep * kWalkStep;
            const unsigned ranges = (unsigned)((n + len - 1) / len);
            // one range (at most kWalkStep seeds): the scan reads no sums
            if (ranges > 1)
                hipLaunchKernelGGL(k_walk_sums, dim3(ranges), dim3(kBlock), 0, s, B.counts, n,
                                   len, B.sums);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            hipLaunchKernelGGL(k_walk_scan, dim3(ranges), dim3(kBlock), 0, s, B.counts, B.sums,
                               B.offsets, n, len, O.count, O.capacity, O.status);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
    }
    return hipSuccess;
}

}  // namespace huge
