// Grouping of the rows a batch touches (the de-duplication of HUGE Sec. 3.3.2):
// which rows occur once -- those are updated in place by the step -- and, for
// every row that occurs several times, the list of its occurrences in
// occurrence order, which is the order in which its contributions are summed.
//
// Occurrence o = i (2 + K) + slot of positive i carries key N + src (slot 0,
// source table) or the context row id (destination, negatives).
//   1. the occurrences of each digit (lowest 8-10 key bits) per tile, counted
//      by the sampler as it writes the keys, a tile being one sampler
//      workgroup's keys (at most kSortTile); k_tile_scan: their sums over
//      earlier tiles, and the bucket sizes;
//   2. k_radix_pass: one stable scatter of the occurrences into bucket
//      (digit) order, each bucket in occurrence order; no tile waits for
//      another;
//   3. k_group: one workgroup per bucket finds the bucket's repeated keys,
//      gives every repeated row a contiguous range of duplicate-buffer slots
//      (inside the bucket's own range of positions), writes the slot of each
//      of its occurrences, in occurrence order, to info[o], and lists the
//      repeated rows, and by slot their occurrences, for the finish kernel.
// Beside the previous batch's fused step they run in 256-thread workgroups
// whose waves hold few registers (one item per thread at a time, loads issued in
// small groups, uniform values as scalars) and work mostly in LDS; a step that
// waits for its own grouping runs 2 and 3 with 512 threads.
#include <math.h>

#include "common.hpp"
#include "device.hpp"

namespace huge {

// A value that every lane of the wave holds alike: beside a fused step
// (workgroups of kBlock threads) as a scalar, so that what follows from it
// (counts, table sizes, levels) takes no vector registers; alone, where
// registers are free, as it is (a scalar has to be waited for: the step of 1024
// positives took 41.3 us with vector values and 42.0 with scalars).
template <int THREADS>
__device__ __forceinline__ uint32_t uniform(uint32_t v) {
    if constexpr (THREADS == kBlock) return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
    return v;
}

// Exclusive sum of one value per thread over the workgroup (THREADS threads);
// *total receives the sum.  Synchronises; s_tmp holds THREADS / 64 words and
// may be reused after the next barrier.
template <int THREADS = kBlock>
__device__ __forceinline__ uint32_t block_excl(uint32_t v, uint32_t* s_tmp, uint32_t* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t t = __shfl_up(incl, off, 64);
        if (lane >= off) incl += t;
    }
    if (lane == 63) s_tmp[wave] = incl;
    __syncthreads();
    uint32_t add = 0, all = 0;
    const int me = (int)uniform<THREADS>((uint32_t)wave);
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        const uint32_t x = uniform<THREADS>(s_tmp[w]);
        if (w < me) add += x;
        all += x;
    }
    *total = all;
    return add + incl - v;
}

// Lanes of the wave whose `bits`-bit value equals this lane's, among the
// lanes in `mask`.
__device__ __forceinline__ uint64_t match_peers(uint32_t value, int bits, uint64_t mask) {
    uint64_t peers = mask;
    for (int b = 0; b < bits; ++b) {
        const bool bit = (value >> b) & 1u;
        const uint64_t ones = __ballot(bit);
        peers &= bit ? ones : ~ones;
    }
    return peers;
}

__device__ __forceinline__ uint64_t lanes_below() {
    const int lane = threadIdx.x & 63;
    return lane == 0 ? 0ull : (~0ull >> (64 - lane));
}

// ---------------------------------------------------------------------------
// Per digit d: tprefix[t * bins + d] = sum of tcount[u * bins + d] over tiles
// u < t, and hist[d] = the sum over all tiles.  A workgroup takes
// kScanDigits digits; its kBlock / kScanDigits thread groups each sum a
// contiguous range of tiles, and the ranges are combined through LDS.
// ---------------------------------------------------------------------------
constexpr int kScanGroups = kBlock / kScanDigits;

__global__ __launch_bounds__(kBlock) HUGE_BESIDE void k_tile_scan(const Control* __restrict__ ctl,
                                                      const uint32_t* __restrict__ tcount,
                                                      int64_t tiles, int bits,
                                                      uint32_t* __restrict__ tprefix,
                                                      uint32_t* __restrict__ hist) {
    __shared__ uint32_t s_part[kScanGroups][kScanDigits];
    if (ctl->step_bad) return;  // uniform
    const int bins = 1 << bits;
    const int dl = threadIdx.x % kScanDigits, g = threadIdx.x / kScanDigits;
    const int d = blockIdx.x * kScanDigits + dl;
    const int64_t per = (tiles + kScanGroups - 1) / kScanGroups;
    const int64_t t0 = (int64_t)g * per;
    const int64_t t1 = t0 + per < tiles ? t0 + per : tiles;
    uint32_t sum = 0;
#pragma unroll 4
    for (int64_t t = t0; t < t1; ++t) sum += tcount[t * bins + d];
    s_part[g][dl] = sum;
    __syncthreads();
    uint32_t run = 0, total = 0;
#pragma unroll 8
    for (int h = 0; h < kScanGroups; ++h) {
        const uint32_t v = s_part[h][dl];
        run += h < g ? v : 0u;
        total += v;
    }
    if (g == 0) hist[d] = total;
#pragma unroll 1
    for (int64_t t = t0; t < t1; ++t) {
        const uint32_t v = tcount[t * bins + d];
        tprefix[t * bins + d] = run;
        run += v;
    }
}

hipError_t launch_tile_scan(Control* ctl, const uint32_t* tcount, int64_t m, int64_t tile,
                            int bits, uint32_t* tprefix, uint32_t* hist, hipStream_t s) {
    if (tile < 1 || tile > kSortTile) return hipErrorInvalidValue;
    const int64_t tiles = (m + tile - 1) / tile;
    if (tiles == 0) return hipSuccess;
    if (bits < kMinDigitBits || bits > kMaxDigitBits) return hipErrorInvalidValue;
    static_assert((1 << kMinDigitBits) % kScanDigits == 0, "whole digit groups");
    hipLaunchKernelGGL(k_tile_scan, dim3((unsigned)((1 << bits) / kScanDigits)), dim3(kBlock), 0,
                       s, ctl, tcount, tiles, bits, tprefix, hist);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Stable scatter by the lowest BITS bits over a tile of tile_keys <=
// kSortTile consecutive items; wave w owns the w-th share of the tile's
// items, in rounds of 64.
//   count: lanes of a round holding the same digit are found with BITS
//          ballots; the lowest of them adds the round's count to the wave's
//          LDS counter of that digit (one writer per digit and round);
//   order: per digit (kBins / kBlock digits per thread) the tile-local start,
//          the wave offsets, and the shift to the global position: bucket
//          start + the digit's count in earlier tiles - tile-local start;
//   place: the rounds again; a lane's position is its wave's running offset
//          of the digit plus the lanes of its round before it; the items go
//          to LDS in digit order (stable);
//   write: LDS position p goes to global position p + shift of its digit:
//          runs of equal digits are contiguous, so the writes coalesce.
// vals_out receives the position of each key in keys_in; bstart the first
// position of each bucket.
// ---------------------------------------------------------------------------
// THREADS = kBlock runs beside another batch's fused step, within the
// HUGE_BESIDE registers; a step that waits for its own grouping runs
// kRadixAlone threads (its 134 KB of LDS leave one workgroup per CU either
// way): K = 31, 4.3M keys,
// 125 -> 91 us; 2.2M 83 -> 60; medium 13.7 -> 11.3.
constexpr int kRadixAlone = 512;

template <int BITS, int THREADS>
__global__ __launch_bounds__(THREADS)
__attribute__((amdgpu_waves_per_eu(THREADS == kBlock ? 8 : 2, 8))) void k_radix_pass(
    Control* __restrict__ ctl, const uint32_t* __restrict__ keys_in,
    uint32_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out, int64_t m,
    int64_t tile_keys, const uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ tprefix, uint32_t* __restrict__ bstart) {
    constexpr int kBins = 1 << BITS;
    constexpr int kWaves = THREADS / 64;
    constexpr int kDpt = kBins > THREADS ? kBins / THREADS : 1;  // digits per thread
    static_assert(kBins % kDpt == 0, "whole digits per thread");
    // dynamic LDS (radix_lds_bytes<BITS, THREADS>()): with a static size this large
    // the compiler, seeing one wave per SIMD at most, would not keep to the
    // HUGE_BESIDE register budget
    extern __shared__ uint32_t s_dyn[];
    uint32_t(*const s_wave)[kBins] = reinterpret_cast<uint32_t(*)[kBins]>(s_dyn);
    int32_t* const s_delta = reinterpret_cast<int32_t*>(s_dyn + kWaves * kBins);
    uint32_t* const s_in = s_dyn + (kWaves + 1) * kBins;  // the tile's keys in input order
    uint32_t* const s_keys = s_in + kSortTile;            // ... in digit order
    uint32_t* const s_vals = s_keys + kSortTile;          // and their input positions
    __shared__ uint32_t s_tmp[2][kWaves];

    if (ctl->step_bad) return;  // uniform: the call is a no-op

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int64_t tile = blockIdx.x;
    const int64_t tile_base = tile * tile_keys;  // tile_keys <= kSortTile
    const int64_t valid_n = (m - tile_base) < tile_keys ? (m - tile_base) : tile_keys;
    // wave w owns the w-th share of the tile (a multiple of 64 items), in
    // order, so the scatter stays stable
    const int rounds = (int)((valid_n + kWaves * 64 - 1) / (kWaves * 64));
    const int wbase = wave * rounds * 64;

    for (int j = tid; j < kWaves * kBins; j += THREADS) (&s_wave[0][0])[j] = 0u;
    for (int p = tid; p < valid_n; p += THREADS) s_in[p] = keys_in[tile_base + p];
    __syncthreads();

    // count
    for (int r = 0; r < rounds; ++r) {
        const int p = wbase + r * 64 + lane;
        const bool valid = p < valid_n;
        const uint32_t dg = valid ? s_in[p] & (kBins - 1) : 0u;
        const uint64_t peers = match_peers(dg, BITS, __ballot(valid));
        if (valid && (peers & lanes_below()) == 0)
            s_wave[wave][dg] += (uint32_t)__popcll(peers);
    }
    __syncthreads();

    // order
    uint32_t cnt_sum = 0, hist_sum = 0;
    const bool digits = tid * kDpt < kBins;  // this thread has digits
#pragma unroll
    for (int j = 0; j < kDpt; ++j) {
        const int d = tid * kDpt + j;
        if (!digits) break;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) cnt_sum += s_wave[w][d];
        hist_sum += hist[d];
    }
    uint32_t total;
    uint32_t local = block_excl<THREADS>(cnt_sum, s_tmp[0], &total);
    uint32_t gstart = block_excl<THREADS>(hist_sum, s_tmp[1], &total);
#pragma unroll
    for (int j = 0; j < kDpt; ++j) {
        const int d = tid * kDpt + j;
        if (!digits) break;
        uint32_t run = local;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) {
            const uint32_t c = s_wave[w][d];
            s_wave[w][d] = run;
            run += c;
        }
        s_delta[d] = (int32_t)(gstart + tprefix[tile * kBins + d]) - (int32_t)local;
        if (tile == 0) bstart[d] = gstart;
        gstart += hist[d];
        local = run;
    }
    __syncthreads();

    // place
    for (int r = 0; r < rounds; ++r) {
        const int p = wbase + r * 64 + lane;
        const bool valid = p < valid_n;
        const uint32_t key = valid ? s_in[p] : 0u;
        const uint32_t dg = key & (kBins - 1);
        const uint64_t peers = match_peers(dg, BITS, __ballot(valid));
        const uint32_t before = (uint32_t)__popcll(peers & lanes_below());
        uint32_t off = 0;
        if (valid) off = s_wave[wave][dg];  // every lane reads before the first lane adds
        if (valid && before == 0) s_wave[wave][dg] = off + (uint32_t)__popcll(peers);
        if (valid && off + before < (uint32_t)kSortTile) {
            s_keys[off + before] = key;
            s_vals[off + before] = (uint32_t)(tile_base + p);
        } else if (valid) {
            raise_internal(ctl, kSiteRadixDest);
        }
    }
    __syncthreads();

    // write
    for (int p = tid; p < valid_n; p += THREADS) {
        const uint32_t k = s_keys[p];
        const int64_t dest = (int64_t)s_delta[k & (kBins - 1)] + p;
        if (dest >= 0 && dest < m) {
            keys_out[dest] = k;
            vals_out[dest] = s_vals[p];
        } else {
            raise_internal(ctl, kSiteRadixDest);
        }
    }
}

// Dynamic LDS bytes of k_radix_pass<BITS, THREADS>.
template <int BITS, int THREADS>
constexpr size_t radix_lds_bytes() {
    return sizeof(uint32_t) * ((size_t)(THREADS / 64 + 1) * (1 << BITS) + 3 * (size_t)kSortTile);
}

template <int BITS, int THREADS>
hipError_t launch_radix_bits(Control* ctl, const uint32_t* keys_in, uint32_t* keys_out,
                             uint32_t* vals_out, int64_t m, int64_t tile,
                             const uint32_t* hist, const uint32_t* tprefix, uint32_t* bstart,
                             int64_t tiles, hipStream_t s) {
    constexpr size_t kLds = radix_lds_bytes<BITS, THREADS>();
    const hipError_t e = allow_lds<&k_radix_pass<BITS, THREADS>>(kLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_radix_pass<BITS, THREADS>), dim3((unsigned)tiles), dim3(THREADS),
                       kLds, s, ctl, keys_in, keys_out, vals_out, m, tile,
                       hist, tprefix, bstart);
    return hipGetLastError();
}

hipError_t launch_radix_pass(Control* ctl, const uint32_t* keys_in, uint32_t* keys_out,
                             uint32_t* vals_out, int64_t m, int64_t tile, int bits,
                             const uint32_t* hist, const uint32_t* tprefix, uint32_t* bstart,
                             bool beside, hipStream_t s) {
    if (tile < 1 || tile > kSortTile) return hipErrorInvalidValue;
    const int64_t tiles = (m + tile - 1) / tile;
    if (tiles == 0) return hipSuccess;
#define HUGE_RADIX_LAUNCH(B)                                                                  \
    return beside                                                                             \
               ? launch_radix_bits<B, kBlock>(ctl, keys_in, keys_out, vals_out, m, tile,   \
                                                 hist, tprefix, bstart, tiles, s)             \
                  : launch_radix_bits<B, kRadixAlone>(ctl, keys_in, keys_out, vals_out, m,    \
                                                      tile, hist, tprefix, bstart, tiles, s)
    switch (bits) {
        case 8: HUGE_RADIX_LAUNCH(8);
        case 9: HUGE_RADIX_LAUNCH(9);
        case 10: HUGE_RADIX_LAUNCH(10);
        default: return hipErrorInvalidValue;
    }
#undef HUGE_RADIX_LAUNCH
}

// ---------------------------------------------------------------------------
// Grouping of one bucket (its items are in occurrence order).
//
// A first pass copies the keys and occurrence indices of a bucket of at most
// `cap` items to LDS, in one round of loads.
// With BM (the bucket's keys differ in at most kBitmapBits bits above the
// bucket digit) the same pass sets, per item, the key's bit in an LDS bitmap
// and, where it was set already, the key's bit in a second bitmap of
// repeated keys; it also counts the bucket's distinct source and destination
// rows.  Only keys marked repeated take part in what follows.
//
// The (repeated) keys are counted in an LDS hash table of 2^most_tbits slots
// (linear probing).  A bucket with more than 3/4 of the slots in distinct
// keys is split into key ranges by further hash bits, each range counted and
// placed in turn (depth first over the binary tree of ranges); at depth 32 a
// range holds one key value, so the split ends.  A count that overflows
// stops at the first chunk that would load the table past 7/8, and the
// number of distinct keys seen so far, scaled to the whole bucket, sets how
// many levels the split descends at once (later sibling ranges start at
// that depth).  Per range:
//   count:  every item of the range inserts its key and counts it;
//   emit:   rows counted more than once get consecutive duplicate-buffer
//           slots (positions of the bucket, after those of earlier ranges),
//           and a work record: a short run or a piece appended to the
//           batch's lists, or pieces plus a combine record (in the bucket's
//           own region) for a run longer than kPiece;
//   place:  the repeated items, taken in occurrence order (chunk by chunk,
//           compacted, then ranked by one wave 64 at a time), receive their
//           row's next slot: info[o] = slot, occ[slot] = o.
// No step waits for another workgroup; the only device-scope atomics reserve a range's places
// in the batch's record lists.  Where a row's range lands
// depends on the order of the hash insertions, the order of its occurrences
// does not: every sum is taken in occurrence order.  Items that occur once
// keep info = -1.
// ---------------------------------------------------------------------------
constexpr uint32_t kEmptyKey = 0xFFFFFFFFu;   // keys are below 2N <= 2^32 - 2
constexpr uint32_t kRepFlag = 0x80000000u;    // table count word: a repeated row, next slot
constexpr int kMaxProbe = 512;                // a longer probe also splits the range

// Slot of a key in a table of 2^tbits slots.
__device__ __forceinline__ uint32_t slot_hash(uint32_t key, int tbits) {
    return (key * 0x85EBCA6Bu) >> (32 - tbits);
}

__device__ __forceinline__ bool in_range(uint32_t key, int level, uint32_t idx) {
    return level == 0 || ((key * 0xC2B2AE35u) >> (32 - level)) == idx;
}

// LDS of a grouping workgroup, chosen per batch: `cap` keys and occurrence
// indices of a bucket in LDS, a table of 2^tbits slots, the bitmaps as wide as
// the keys need.  A bucket's steps are short and full of barriers, so the
// kernel alone lives on several workgroups per CU: the most (4 .. 1) for which
// the LDS left holds the batch's average bucket with six standard deviations
// of an even spread to spare.  Beside a fused step whose waves stay resident one
// workgroup per CU fits by its registers (more settle as those waves end), but
// what it takes of the LDS the finish kernel's 10 KB workgroups lack, so 48 KB
// are left to them where the bucket still fits (1e8 rows, fp32: finish 27 us
// beside 148 KB and a loss sum with 8 loads in flight, 17 beside 112 KB and 16
// loads; the two were not timed apart).  A skewed batch's largest buckets are
// read from memory: steps of 3,000, 8,000, 20,000 and 40,000 positives of a
// power-law graph (5e4 to 1e6 nodes) took 57.0, 74.1, 113.9 and 215 us when
// every bucket of 4096 keys was copied, 54.5, 74.2, 105.8 and 202 now.

// And never all of it: a fused step's workgroup needs some LDS too, so a CU whose
// LDS a grouping workgroup has filled takes none of them (1e8 rows, K = 31,
// 262,144 positives, buckets of 8448 keys that no share holds: grouping 1873 us
// with 159 KB, 1023 with 147; the pipelined step 2618 and 2344).
constexpr int kGroupBesideLds = kLdsBytes - 12 * 1024;

struct GroupShape {
    int cap;    // keys and indices cached, a multiple of 64
    int tbits;  // table slots: enough for the repeated keys of an average
                // bucket (half its items) at a load of 3/4
    size_t words;  // dynamic LDS
};

inline GroupShape group_shape(int64_t m, int bins, int sub_bits, bool beside) {
    const bool bm = sub_bits <= kBitmapBits;
    const size_t bits = bm ? 2 * (size_t)(sub_bits > 5 ? 1 << (sub_bits - 5) : 1) : 0;
    const double avg = (double)m / bins;
    const double want = avg + 6.0 * sqrt(avg) + 64.0;
    int tb = kMinTableBits;
    while (tb < kGroupTableBits && (double)(1 << tb) < 0.75 * want) ++tb;
    const size_t fixed = 2 * ((size_t)1 << tb) + kGroupChunk + bits;
    GroupShape g{64, tb, 0};
    // a quarter, a third, half, 112 KB or all of a CU's LDS (beside: all but 12 KB)
    const int most = beside ? kGroupBesideLds : kLdsBytes;
    for (const int share : {kLdsBytes / 4, kLdsBytes / 3, kLdsBytes / 2, 112 * 1024, most}) {
        // the statically allocated LDS of the kernel is below 1 KB
        const size_t budget = (size_t)(share - 1024) / sizeof(uint32_t);
        if (budget < fixed + 2 * 64) continue;
        size_t cap = (budget - fixed) / 2 / 64 * 64;
        if (cap > (size_t)kGroupCacheMost) cap = kGroupCacheMost;
        g.cap = (int)cap;
        if ((double)cap >= want) break;
    }
    g.words = fixed + 2 * (size_t)g.cap;
    return g;
}

// THREADS = kBlock runs beside another batch's fused step; a step that waits
// for its own grouping runs it alone with kGroupAlone threads.  Beside, the
// kernel is held to 72 VGPRs (it takes 66 to 69, with every value that is the
// same for a workgroup in scalar registers), the most that fits beside five
// waves of a float step; with vector values it took 93, so that a wave of the
// step had to end first, and the preparation became longer than the update (1e8
// rows, 200 pipelined steps: 470 us a step, 459 now; the grouping beside a
// fused kernel 267 and 175).  Alone it takes the registers it needs, 109.  With
// 148 KB of LDS, 256 threads and 72 VGPRs (a few of them spilled) for all, then
// with this split: sequential steps of 1,024 positives 43.5 -> 40.9 us, 65,536
// (medium) 192 -> 183, 131,072 with K = 31 1548 -> 1436 (buckets of 4200 keys
// found no room for their indices), 100,003 of a power-law graph with K = 20
// 1373 -> 1318; six pipelined steps of 262,144 fp32 3102 -> 3055, bf16 2179 ->
// 1985.  256 and 1024 threads alone: 42.3, 189, 1481, 1346 and 47.4, 191, 1455,
// 1358; 512 beside: 3108 and 2073.
constexpr int kGroupAlone = 512;

template <bool BM, int THREADS>
__global__ __launch_bounds__(THREADS)
__attribute__((amdgpu_waves_per_eu(THREADS == kBlock ? 7 : 4, THREADS == kBlock ? 7 : 4)))
void k_group(
    Control* __restrict__ ctl, const uint32_t* __restrict__ keys,
    const uint32_t* __restrict__ vals, int64_t m, int64_t N, const uint32_t* __restrict__ hist,
    const uint32_t* __restrict__ bstart, int32_t* __restrict__ info,
    uint32_t* __restrict__ occ, uint4* __restrict__ shorts, uint4* __restrict__ pieces,
    uint4* __restrict__ combs, uint32_t* __restrict__ ccount, ListCaps caps,
    uint32_t* __restrict__ wstats, int bins, int shift, int sub_bits, int cap, int most_tbits) {
    constexpr int ITEMS = kGroupChunk / THREADS;  // consecutive keys of a thread
    static_assert(ITEMS * THREADS == kGroupChunk, "whole keys per thread");
    // words of one bitmap
    const uint32_t bit_words = sub_bits > 5 ? 1u << (sub_bits - 5) : 1u;
    // The large arrays live in dynamic LDS (group_shape): the compiler then
    // keeps to the register budget, which a static size above a fifth of the
    // LDS would let it exceed.
    extern __shared__ uint32_t s_dyn[];
    uint32_t* const s_key = s_dyn;                          // [2^most_tbits]
    uint32_t* const s_cnt = s_key + (1 << most_tbits);      // count; after emit, kRepFlag | next slot
    uint32_t* const s_ckey = s_cnt + (1 << most_tbits);     // [cap]
    uint32_t* const s_cval = s_ckey + cap;                  // [cap]
    // repeated items of a chunk in order: their table slot, then their
    // duplicate slot
    uint32_t* const s_rep = s_cval + cap;                   // [kGroupChunk]
    uint32_t* const s_seen = s_rep + kGroupChunk;           // [bit_words] with BM
    uint32_t* const s_dup = s_seen + bit_words;             // [bit_words] with BM
    __shared__ uint32_t s_tmp[6][THREADS / 64];
    __shared__ uint32_t s_distinct, s_fail, s_nrep;
    __shared__ uint32_t s_stat[3];
    __shared__ uint32_t s_rbase[2];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // the first failed internal check of this thread, raised once at the end
    // (one atomic site keeps its operands out of the registers of the loops)
    uint32_t bad = 0u;
#define HUGE_FAIL(site) (bad = bad ? bad : (uint32_t)(site))
    for (int b = blockIdx.x; b < bins; b += gridDim.x) {
    __syncthreads();  // LDS of the previous bucket
    if (tid < 3) s_stat[tid] = 0u;
    if (tid == 0) s_nrep = 0u;
    const uint32_t n = ctl->step_bad ? 0u : hist[b];
    const int64_t s0 = n ? (int64_t)bstart[b] : 0;
    if (n == 0u || s0 + (int64_t)n > m) {
        if (n != 0u && tid == 0) HUGE_FAIL(kSiteGroupBucket);
        if (tid < 3) wstats[b * 3 + tid] = 0u;
        continue;
    }
    const bool cached = n <= (uint32_t)cap;
    // the ITEMS keys of this thread in chunk c0
    // (after the compaction: of the first nw items)
    auto load_keys = [&](uint32_t c0, uint32_t nlim, uint32_t (&k)[ITEMS]) {
        const uint32_t e0 = c0 + (uint32_t)(tid * ITEMS);
        if (cached) {
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) k[r] = e0 + r < nlim ? s_ckey[e0 + r] : 0u;
        } else {
            const uint32_t* kp = keys + s0 + e0;
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) k[r] = e0 + r < nlim ? kp[r] : 0u;
        }
    };

    // ---- copy to LDS; repeated keys (BM) ----
    // the bit of key k is bit (k >> shift) of the bucket's bitmap; a key
    // beyond the bitmap cannot occur (sub_bits <= kBitmapBits)
    auto repeated = [&](uint32_t k) -> bool {
        if (!BM) return true;
        const uint32_t sub = k >> shift;
        return sub >> 5 < bit_words && ((s_dup[sub >> 5] >> (sub & 31u)) & 1u);
    };
    if (BM) {
        for (uint32_t j = tid; j < bit_words; j += THREADS) {
            s_seen[j] = 0u;
            s_dup[j] = 0u;
        }
    }
    if (cached) {  // coalesced: item j + q THREADS by thread j
        for (uint32_t e0 = 0; e0 < n; e0 += 4 * THREADS) {
            uint32_t kk[4], vv[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t e = e0 + (uint32_t)(q * THREADS + tid);
                kk[q] = e < n ? keys[s0 + e] : 0u;
                vv[q] = e < n ? vals[s0 + e] : 0u;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t e = e0 + (uint32_t)(q * THREADS + tid);
                if (e < n) {
                    s_ckey[e] = kk[q];
                    s_cval[e] = vv[q];
                }
            }
        }
    }
    __syncthreads();
    if (BM) {
        uint32_t nS = 0, nT = 0, nR = 0;
        for (uint32_t c0 = 0; c0 < n; c0 += kGroupChunk) {
            uint32_t k[ITEMS];
            load_keys(c0, n, k);
#pragma unroll 1
            for (int r = 0; r < ITEMS; ++r) {
                const uint32_t e = c0 + (uint32_t)(tid * ITEMS + r);
                if (e >= n) continue;
                const uint32_t sub = k[r] >> shift, w = sub >> 5, bit = 1u << (sub & 31u);
                if (w >= bit_words) {
                    HUGE_FAIL(kSiteGroupBits);
                    continue;
                }
                const uint32_t old = atomicOr(&s_seen[w], bit);
                if (old & bit) {
                    atomicOr(&s_dup[w], bit);
                    ++nR;
                } else if ((int64_t)k[r] >= N) {
                    ++nS;
                } else {
                    ++nT;
                }
            }
        }
        if (nS) atomicAdd(&s_stat[0], nS);
        if (nT) atomicAdd(&s_stat[1], nT);
        if (nR) atomicAdd(&s_nrep, nR);
        __syncthreads();
    }
    // with the bitmap: nothing repeated, nothing to group
    const bool any = !BM || uniform<THREADS>(s_nrep) != 0u;

    // With the bitmap and the whole bucket in LDS, only the items of
    // repeated keys are grouped: they are compacted to the front of the LDS
    // copy, in occurrence order (chunk by chunk; an item moves only to a
    // lower position, so no item is overwritten before it is read), and
    // the hash table is sized to them.
    uint32_t nw = n;  // items the count and the placement go through
    int tbits = most_tbits;
    if (BM && any && cached) {
        uint32_t out = 0;
        for (uint32_t c0 = 0; c0 < n; c0 += kGroupChunk) {
            uint32_t kk[ITEMS], vv[ITEMS];
            uint32_t mask = 0u, cnt = 0u;
            const uint32_t e0 = c0 + (uint32_t)(tid * ITEMS);
#pragma unroll
            for (int r = 0; r < ITEMS; ++r) {
                kk[r] = e0 + r < n ? s_ckey[e0 + r] : 0u;
                vv[r] = e0 + r < n ? s_cval[e0 + r] : 0u;
            }
#pragma unroll 1
            for (int r = 0; r < ITEMS; ++r) {
                if (e0 + r < n && repeated(kk[r])) {
                    mask |= 1u << r;
                    ++cnt;
                }
            }
            uint32_t total;
            uint32_t p = out + block_excl<THREADS>(cnt, s_tmp[0], &total);  // synchronises
#pragma unroll 1
            for (int r = 0; r < ITEMS; ++r) {
                if (mask & (1u << r)) {
                    s_ckey[p] = kk[r];
                    s_cval[p] = vv[r];
                    ++p;
                }
            }
            out += total;
            __syncthreads();  // s_tmp is reused
        }
        nw = out;
        tbits = 6;
        while (tbits < most_tbits && (1u << tbits) < 2u * nw) ++tbits;
    }
    const uint32_t tsize = 1u << tbits;
    const uint32_t tmask = tsize - 1u;
    const uint32_t tmax = tsize / 4u * 3u;   // distinct keys a range may hold
    const uint32_t tload = tsize / 8u * 7u;  // table load a count stays below

    // the bucket's record bounds and regions, and how many records it has written
    const uint32_t c_short = (uint32_t)(n / kShortDiv), c_piece = (uint32_t)(n / kPieceDiv);
    const uint32_t r_comb = (uint32_t)(s0 / kCombDiv), c_comb = (uint32_t)(n / kCombDiv);
    const uint32_t r_part = (uint32_t)(s0 / kPartDiv), c_part = (uint32_t)(n / kPartDiv);
    uint32_t nb_short = 0, nb_piece = 0, nb_comb = 0, nb_part = 0;

    uint32_t rep_base = 0;  // slots handed out to earlier ranges
    int level = 0, depth = 0;  // depth: where the next sibling range starts
    uint32_t ridx = 0;
    auto lookup = [&](uint32_t key) -> uint32_t {
        uint32_t h = slot_hash(key, tbits);
        for (int probe = 0; probe < kMaxProbe; ++probe) {
            const uint32_t kk = s_key[h];
            if (kk == key) return h;
            if (kk == kEmptyKey) return kEmptyKey;
            h = (h + 1u) & tmask;
        }
        return kEmptyKey;
    };
    while (any) {
        // ---- count ----
#pragma unroll 1
        for (uint32_t q = tid; q < tsize; q += THREADS) {
            s_key[q] = kEmptyKey;
            s_cnt[q] = 0u;
        }
        if (tid == 0) {
            s_distinct = 0u;
            s_fail = 0u;
        }
        __syncthreads();
        uint32_t seen = 0;  // items the count went through
        bool over = false;
        for (uint32_t c0 = 0; c0 < nw; c0 += kGroupChunk) {
            const uint32_t len = nw - c0 < (uint32_t)kGroupChunk ? nw - c0 : (uint32_t)kGroupChunk;
            if (uniform<THREADS>(s_distinct) + len > tload) {  // uniform: the table could fill up
                over = true;
                break;
            }
            uint32_t k[ITEMS];
            load_keys(c0, nw, k);
            uint32_t fresh = 0u;
#pragma unroll 1
            for (int r = 0; r < ITEMS; ++r) {
                const uint32_t e = c0 + (uint32_t)(tid * ITEMS + r);
                if (e >= nw || !in_range(k[r], level, ridx) || !repeated(k[r])) continue;
                uint32_t h = slot_hash(k[r], tbits);
                bool found = false;
                for (int probe = 0; probe < kMaxProbe; ++probe) {
                    const uint32_t old = atomicCAS(&s_key[h], kEmptyKey, k[r]);
                    if (old == kEmptyKey || old == k[r]) {
                        fresh += old == kEmptyKey ? 1u : 0u;
                        atomicAdd(&s_cnt[h], 1u);
                        found = true;
                        break;
                    }
                    h = (h + 1u) & tmask;
                }
                if (!found) s_fail = 1u;
            }
            if (fresh) atomicAdd(&s_distinct, fresh);
            __syncthreads();
            seen = c0 + len;
            if (uniform<THREADS>(s_fail) || uniform<THREADS>(s_distinct) > tmax) {  // uniform
                over = true;
                break;
            }
        }
        if (over) {
            // split the range; its first part next (uniform)
            int add = 1;
            if (!uniform<THREADS>(s_fail) && seen > 0u) {
                const uint64_t est = (uint64_t)uniform<THREADS>(s_distinct) * nw / seen;
                while (add < 8 && est > ((uint64_t)tmax << add) / 4u * 3u) ++add;
            }
            __syncthreads();
            if (level >= 32) {  // cannot happen: a depth-32 range holds one key value
                HUGE_FAIL(kSiteGroupDepth);
                goto finished;
            }
            if (add > 32 - level) add = 32 - level;
            level += add;
            ridx <<= add;
            if (depth < level) depth = level;
            continue;
        }

        {
        // ---- emit ----
        // this thread's table slots (tid, tid + THREADS, ...; conflict-free
        // LDS reads): statistics, slot counts, record counts; slots and
        // records are handed out thread by thread
        uint32_t nS = 0, nT = 0, nrep = 0, nshort = 0, npiece = 0, ncomb = 0, npart = 0;
#pragma unroll 1
        for (uint32_t q = tid; q < tsize; q += THREADS) {
            const uint32_t k = s_key[q];
            if (k == kEmptyKey) continue;
            if (!BM) {  // with BM the first pass counted the rows
                if ((int64_t)k >= N) ++nS; else ++nT;
            }
            const uint32_t c = s_cnt[q];
            if (c > 1u) {
                nrep += c;
                if (c <= kShortRun) {
                    ++nshort;
                } else if (c <= kPiece) {
                    ++npiece;
                } else {
                    const uint32_t np = (c + kPiece - 1) / kPiece;
                    npiece += np;
                    npart += np;
                    ++ncomb;
                }
            }
        }
        uint32_t t_rep, t_short, t_piece, t_comb, t_part;
        const uint32_t x_rep = block_excl<THREADS>(nrep, s_tmp[0], &t_rep);
        const uint32_t x_short = block_excl<THREADS>(nshort, s_tmp[1], &t_short);
        const uint32_t x_piece = block_excl<THREADS>(npiece, s_tmp[2], &t_piece);
        const uint32_t x_comb = block_excl<THREADS>(ncomb, s_tmp[3], &t_comb);
        const uint32_t x_part = block_excl<THREADS>(npart, s_tmp[4], &t_part);
        if (nS) atomicAdd(&s_stat[0], nS);
        if (nT) atomicAdd(&s_stat[1], nT);
        // the range's short runs and pieces are appended to the batch's lists
        // at positions reserved by one device-scope atomic each (the finish
        // kernel takes each record alone, so their order is free)
        if (tid == 0) {
            s_rbase[0] = t_short ? atomicAdd(&ctl->nshort, t_short) : 0u;
            s_rbase[1] = t_piece ? atomicAdd(&ctl->npiece, t_piece) : 0u;
        }
        __syncthreads();
        const uint32_t b_short = uniform<THREADS>(s_rbase[0]), b_piece = uniform<THREADS>(s_rbase[1]);
        // uniform: every thread has the same totals and bases
        const bool fits = (uint64_t)nb_short + t_short <= c_short &&
                          (uint64_t)nb_piece + t_piece <= c_piece &&
                          (uint64_t)nb_comb + t_comb <= c_comb &&
                          (uint64_t)nb_part + t_part <= c_part &&
                          (uint64_t)rep_base + t_rep <= n &&
                          (uint64_t)b_short + t_short <= caps.shorts &&
                          (uint64_t)b_piece + t_piece <= caps.pieces &&
                          (uint64_t)r_comb + c_comb <= caps.combs &&
                          (uint64_t)r_part + c_part <= caps.parts;
        if (!fits) {  // cannot happen: the regions bound every bucket
            HUGE_FAIL(kSiteGroupLists);
            goto finished;
        }
        {
            uint32_t pos = (uint32_t)s0 + rep_base + x_rep;
            uint32_t is = b_short + x_short, ip = b_piece + x_piece;
            uint32_t ic = r_comb + nb_comb + x_comb, ia = r_part + nb_part + x_part;
#pragma unroll 1
            for (uint32_t q = tid; q < tsize; q += THREADS) {
                const uint32_t k = s_key[q];
                const uint32_t c = s_cnt[q];
                if (k == kEmptyKey || c <= 1u) continue;
                if (c <= kShortRun) {
                    shorts[is++] = make_uint4(pos, c, k, 0u);
                } else if (c <= kPiece) {
                    pieces[ip++] = make_uint4(pos, c, k, 0u);
                } else {
                    const uint32_t np = (c + kPiece - 1) / kPiece;
                    for (uint32_t z = 0; z < np; ++z) {
                        const uint32_t len = (c - z * kPiece) < kPiece ? (c - z * kPiece) : kPiece;
                        pieces[ip++] = make_uint4(pos + z * kPiece, len, k, ic + 1u);
                    }
                    combs[ic] = make_uint4(k, ia, np, pos);
                    ccount[ic] = 0u;
                    ++ic;
                    ia += np;
                }
                s_cnt[q] = kRepFlag | pos;
                pos += c;
            }
        }
        nb_short += t_short;
        nb_piece += t_piece;
        nb_comb += t_comb;
        nb_part += t_part;
        if (tid == 0) s_stat[2] += t_rep;
        __syncthreads();

        // ---- place ----
        if (t_rep > 0u) {
            for (uint32_t c0 = 0; c0 < nw; c0 += kGroupChunk) {
                uint32_t k[ITEMS];
                load_keys(c0, nw, k);
                uint32_t mask = 0u, cnt = 0u;
#pragma unroll 1
                for (int r = 0; r < ITEMS; ++r) {
                    const uint32_t e = c0 + (uint32_t)(tid * ITEMS + r);
                    if (e >= nw || !in_range(k[r], level, ridx) || !repeated(k[r])) continue;
                    const uint32_t h = lookup(k[r]);
                    if (h == kEmptyKey) {
                        HUGE_FAIL(kSiteGroupLookup);
                        continue;
                    }
                    if (s_cnt[h] & kRepFlag) {
                        mask |= 1u << r;
                        ++cnt;
                    }
                }
                uint32_t chunk_rep;
                const uint32_t k0 = block_excl<THREADS>(cnt, s_tmp[5], &chunk_rep);  // synchronises
                {
                    uint32_t kk = k0;
#pragma unroll 1
                    for (int r = 0; r < ITEMS; ++r)
                        if (mask & (1u << r)) s_rep[kk++] = lookup(k[r]);
                }
                __syncthreads();
                if (wave == 0) {
                    for (uint32_t j0 = 0; j0 < chunk_rep; j0 += 64) {
                        const uint32_t j = j0 + (uint32_t)lane;
                        const bool act = j < chunk_rep;
                        const uint32_t sl = act ? s_rep[j] : 0u;
                        const uint64_t peers = match_peers(sl, tbits, __ballot(act));
                        const uint32_t before = (uint32_t)__popcll(peers & lanes_below());
                        const int ld = __ffsll((long long)peers) - 1;
                        const int leader = ld < 0 ? 0 : ld;
                        uint32_t st = 0u;
                        if (act && before == 0u) {
                            st = s_cnt[sl];
                            s_cnt[sl] = st + (uint32_t)__popcll(peers);
                        }
                        st = __shfl(st, leader, 64);
                        if (act) s_rep[j] = (st & ~kRepFlag) + before;
                    }
                }
                __syncthreads();
                uint32_t kk = k0;
#pragma unroll 1
                for (int r = 0; r < ITEMS; ++r) {
                    if (mask & (1u << r)) {
                        const uint32_t pos = s_rep[kk++];
                        const uint32_t e = c0 + (uint32_t)(tid * ITEMS + r);
                        const uint32_t o = cached ? s_cval[e] : vals[s0 + e];
                        if ((int64_t)pos >= s0 && (int64_t)pos < s0 + (int64_t)n &&
                            (int64_t)o < m) {
                            info[o] = (int32_t)pos;
                            occ[pos] = o;
                        } else {
                            HUGE_FAIL(kSiteGroupPlace);
                        }
                    }
                }
                __syncthreads();  // s_rep is reused by the next chunk
            }
        }
        rep_base += t_rep;
        }

        // ---- next range, depth first ----
        while (level > 0 && (ridx & 1u)) {
            --level;
            ridx >>= 1;
        }
        if (level == 0) break;
        ridx += 1u;
        if (level < depth) {  // the sibling is split as far as this one was
            ridx <<= (depth - level);
            level = depth;
        }
        __syncthreads();  // the table is cleared for the next range
    }
    __syncthreads();
    if (tid < 3) wstats[b * 3 + tid] = s_stat[tid];
    }
finished:
    if (bad) raise_internal(ctl, bad);
#undef HUGE_FAIL
}

hipError_t launch_group(Control* ctl, const uint32_t* keys, const uint32_t* vals, int64_t m,
                        int64_t N, const uint32_t* hist, const uint32_t* bstart, int32_t* info,
                        uint32_t* occ, uint4* shorts, uint4* pieces, uint4* combs, uint32_t* ccount,
                        ListCaps caps, uint32_t* wstats, int bins, int key_bits,
                        bool beside, hipEvent_t stop, bool* launched, hipStream_t s) {
    *launched = false;
    if (m == 0) return hipSuccess;
    if (bins < 2 || bins > kMaxBins || (bins & (bins - 1)) != 0) return hipErrorInvalidValue;
    const int shift = __builtin_ctz((unsigned)bins);
    const int sub_bits = key_bits > shift ? key_bits - shift : 0;
    const bool bm = sub_bits <= kBitmapBits;
    const GroupShape g = group_shape(m, bins, sub_bits, beside);
#define HUGE_GROUP_LAUNCH(BM, THREADS)                                                        \
    do {                                                                                      \
        const hipError_t set = allow_lds<&k_group<BM, THREADS>>(kLdsBytes - 1024);            \
        if (set != hipSuccess) return set;                                                    \
        hipExtLaunchKernelGGL((k_group<BM, THREADS>), dim3((unsigned)bins),                   \
                              dim3(THREADS), g.words * sizeof(uint32_t), s, nullptr, stop, 0, \
                              ctl, keys, vals, m, N, hist, bstart, info, occ, shorts, pieces, \
                              combs, ccount, caps, wstats, bins, shift, sub_bits,     \
                              g.cap, g.tbits);                                                \
    } while (0)
    if (bm && beside) {
        HUGE_GROUP_LAUNCH(true, kBlock);
    } else if (bm) {
        HUGE_GROUP_LAUNCH(true, kGroupAlone);
    } else if (beside) {
        HUGE_GROUP_LAUNCH(false, kBlock);
    } else {
        HUGE_GROUP_LAUNCH(false, kGroupAlone);
    }
#undef HUGE_GROUP_LAUNCH
    const hipError_t e = hipGetLastError();
    *launched = e == hipSuccess;
    return e;
}

}  // namespace huge
