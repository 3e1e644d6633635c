// Integer scan of packed 4-bit codes as a product on the matrix cores (Alg. 3; 16 or 32 tables of 16 entries).
//
// The sum of a code's table entries is the product of the tables, one row of 16 * tables numbers per query, and the code
// written as a column of as many numbers, one 1 per table and 0 elsewhere.  The scan needs the sums only to dismiss codes, so
// the product is formed from lower bounds of the entries in the narrowest types that the matrix cores have: the ones are 4-bit
// floats, a code's nibble n being the 64-bit word 2 << 4n, the entries 6-bit floats.  Of their steps, 1/8 up to 2, then 1/4 and
// 1/2, the entries use 76, centred so that the finest ones lie where the entries of codes that matter do:
//   e = min(75, floor((entry - least entry of its table) * s) + c),   s = min(1, R / (bound - sum of the least entries)),
// rounded down to a step and less 15, with R = 15 per table and the c of the tables making up what s times the difference is short of R.
// A code whose e add up to R has a sum beyond the bound: the sum of the 6-bit floats is not negative.  (The additions are exact
// in any order, multiples of 1/8 below 2^9.)  What is not dismissed is queued per wave in
// LDS, and its exact sum is formed from the 8-bit tables.
//
// Keys (sum, row) within the bound cost an atomic addition in device memory each, and a bound that falls while the scan goes on
// lets topk (1 + ln(n / codes of the first bound)) of them through per query: 25 M encoded codes, 1000 queries, top-1000 took 7.4 M
// additions to lists and as many to histograms, 1.8 of 3.6 ms.  The bounds are therefore found first, from a sample of the codes,
// by the same loop, whose keys are only counted: a quarter of the sample with a bound from a few thousand of its
// codes, the rest with the bound that the quarter gives.  Of the whole sample the r-th key is taken, r = mu + 4.5 sqrt(mu) + 4,
// which is so far above the number mu = topk / 2^shift of the results that such a sample holds that fewer than topk codes of all at
// or below it are one query in a million.  The sample has one row of every 2^shift, each in a place of its own, so that the results in it
// are as many as of independent rows, or closer to mu, whatever the order that the rows are stored in.  (Every 2^shift-th load of 1024
// bytes, as it was, is no such sample where neighbours lie together: 25 M codes in groups of 64 neighbours x 1000 queries, top-1000,
// left hundreds of queries short lists.)  It is gathered first: a line of memory
// per code, 12 us for 25 M codes (22 with twice as many).  Some 1.5 topk codes per query pass in the scan itself; their keys go to the query's list.  Queries whose
// list has fewer than topk keys, or more than it has room for, are left to the other loops.  25 M codes x 1000 queries, top-1000, before and after:
// in no order 2.64 and 2.50 ms, in groups of 64 neighbours 9.8 and 2.1, in the order of 8192 lists 11.3 and 2.7 (16-query loop 5.2, 3.9 and 8.0).
//
// What bounds it: v_mfma_f32_32x32x64_f8f6f4 on these types forms 1024 sums of 16 tables in 4 instructions of 32 cycles, 19.6 T
// sums/s at the nominal clock; under this load the device holds 13.3 T/s without any tests, 12.9 T/s with them in the shadow of the
// next product (loop alone, 25 M codes x 1000 queries 1.94 ms; the 16-query loop on 8-bit lower bounds from LDS, which
// issues its limit of vector instructions, 4.05).  A wave keeps the image of 128 queries (16 tables; 64 with 32) in
// 96 registers and forms a code's columns once for all of them; tests go over the sums of the product before.
#include <math.h>
#include <stddef.h>

#include "pq_internal.h"
#include "scan_common.h"
#include "scan_onehot.h"
#include "topk_device.h"

namespace pq {

typedef int v8i __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));

constexpr int OH_WAVES = 4, OH_THREADS = OH_WAVES * 64;
constexpr int OH_QUEUE = 512;                  // (row, query) pairs of a wave that wait for their exact sums
constexpr int OH_CENTRE = 15;                  // e is stored as e - 15, and a table's share of R is 15
constexpr int OH_MOST = 75;
constexpr int OH_PICK_THREADS = 512;            // of the last look at the counts (see onehot_pick_kernel)
enum { OH_FIRST, OH_REST, OH_LIST };           // a quarter of the sample, the rest of it, all codes

struct OnehotArgs {
    const uint8_t *codes;          // (of the sample: gathered)
    int64_t n;
    // Chunks: nhead ones of head_codes rows, then ones of chunk_codes (both multiples of a block's load of codes, below 2^25).  Where
    // sums tie by the ten thousand, the rows that are listed are the first ones: those come in small items.
    int64_t chunk_codes, head_codes;
    int nhead;
    int ntiles, nitems;    // item = chunk * ntiles + tile of queries
    const uint8_t *qluts;
    int nq, topk, hist_bins;       // (sample: the rank looked for in place of topk)
    int shift;                     // (sample: its i-th code is that of row onehot_sample_row(i, shift))
    unsigned long long *tau_key;   // [nq] whole key at or below which the query has topk codes
    uint32_t *cnt;                 // [nq][COUNT_PITCH] keys handed to the query's list
    uint32_t *hist;                // [nq][HIST_BINS]
    uint64_t *lists;               // [nq][cap]
    uint32_t cap;
    uint32_t *tie_val;             // [nq][ONEHOT_TIES] sums whose rows are counted, plus 1 (0: none yet)
    uint32_t *tie_rows;            // [nq][ONEHOT_TIES][ONEHOT_TIE_BINS] listed keys of that sum by row (see tie_bin)
    uint32_t *work_counter;
    unsigned long long *stats;
};

template <int NB, int G>
struct __align__(16) OnehotSmem {
    static constexpr int QT = 32 * G, ROW = NB * 32 + 16;   // (16 bytes more: the lanes of a wave read one column of 32 rows)
    uint8_t tab[QT][ROW];                     // entries less the least of their table
    uint32_t img[G * (NB / 2)][64][6];        // 6-bit floats as a lane of the product holds them
    uint32_t queue[OH_WAVES][OH_QUEUE];       // row in the item << 7 | query in the tile
    unsigned long long key[QT];               // bounds
    uint32_t off[QT];                         // sum of the tables' least entries
    uint32_t tie_val[QT][ONEHOT_TIES];
    OnehotArgs a;
    const uint8_t *chunk_ptr;
    int64_t begin;
    int ncodes, q0, item;
    uint32_t parked;
};

template <class T> using lds_ptr = __attribute__((address_space(3))) T *;

// 64-bit words of 4-bit floats, 1.0 (code 2) at the place that a nibble names: 32 numbers per code byte
__device__ __forceinline__ void onehot_columns(uint32_t w, v8i (&b)[4]) {
    const uint32_t even = (w << 2) & 0x3c3c3c3cu, odd = (w >> 2) & 0x3c3c3c3cu;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const uint64_t lo = 2ull << ((even >> (8 * s)) & 63u), hi = 2ull << ((odd >> (8 * s)) & 63u);
        b[s] = (v8i){(int)(uint32_t)lo, (int)(uint32_t)(lo >> 32), (int)(uint32_t)hi, (int)(uint32_t)(hi >> 32), 0, 0, 0, 0};
    }
}

// the 6-bit float (sign, 2 bits of exponent, 3 of mantissa) at or next below (e - 15) / 8
__device__ __forceinline__ uint32_t onehot_entry(uint32_t e) {
    const int m = (int)e - OH_CENTRE;
    const uint32_t small = m < 0 ? (uint32_t)(0x20 - m) : (uint32_t)m;
    const uint32_t shift = m < 32 ? 1u : 2u, large = (8u << (shift - 1u)) + ((uint32_t)m >> shift);
    return m < 16 ? small : large;
}

// Bins of rows, eight to an octave: ties that matter are the more and the earlier rows, the more there are of them (and with bins of equal
// widths the block that scans the first rows kept the others waiting: 25 M codes, 128 queries, top-100 640 us against 451).
__device__ __forceinline__ uint32_t tie_bin(uint32_t row) {
    const uint32_t e = 31u - (uint32_t)__builtin_clz(row | 1u);
    return row < 8u ? row : 8u * (e - 2u) + ((row >> (e - 3u)) & 7u);
}
__device__ __forceinline__ uint32_t tie_bin_last_row(uint32_t bin) {
    return bin < 8u ? bin : (uint32_t)(((uint64_t)((bin & 7u) + 9u) << ((bin >> 3) - 1u)) - 1u);
}

// the sign bit set if any of the 16 is negative
__device__ __forceinline__ uint32_t any_negative(const v16f &a) {
    uint32_t m = __float_as_uint(a[0]);
#pragma unroll
    for (int r = 1; r < 15; r += 2) m = m | __float_as_uint(a[r]) | __float_as_uint(a[r + 1]);
    return m | __float_as_uint(a[15]);
}

// Exact sums of the wave's first qn queued pairs, which leave the queue.  Out of line: it runs once per some thousand products.
template <int NB, int G, bool SAMPLE>
__device__ __noinline__ void onehot_flush(lds_ptr<OnehotSmem<NB, G>> sm, int wave, int qn) {
    constexpr int U = 2;
    const int lane = lane_id();
    const uint8_t *chunk_ptr = sm->chunk_ptr;
    const uint32_t ncodes = (uint32_t)sm->ncodes, row0 = (uint32_t)sm->begin;
    const int q0 = sm->q0, shift = sm->a.shift;
    for (int i0 = 0; i0 < qn; i0 += 64 * U) {
        uint32_t q[U], row[U], id[U], w[U][NB / 4];   // (id: the row in the database)
        bool in[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = i0 + 64 * u + lane;
            const uint32_t e = i < qn ? sm->queue[wave][i] : 0u;
            q[u] = e & 127u;
            row[u] = e >> 7;
            in[u] = i < qn && row[u] < ncodes;
            id[u] = SAMPLE ? onehot_sample_row(row0 + row[u], shift) : row0 + row[u];
            // (codes of the least sum that the tables allow: behind the bound's row nothing can qualify)
            if constexpr (!SAMPLE) {
                const unsigned long long bound = sm->key[q[u]];
                in[u] = in[u] && !((uint32_t)(bound >> 32) == sm->off[q[u]] && id[u] > (uint32_t)bound);
            }
        }
        if constexpr (!SAMPLE) {   // (they come by the thousand where they are stored side by side: 4 M codes in the order of 8192 lists, top-100, 929 -> 736 us)
            bool any = false;
#pragma unroll
            for (int u = 0; u < U; ++u) any = any || in[u];
            if (__ballot(any) == 0ull) continue;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int x = 0; x < NB / 4; ++x) w[u][x] = 0u;
            if (in[u]) {
                if constexpr (NB == 8) {
                    const uint2 v = *reinterpret_cast<const uint2 *>(chunk_ptr + (size_t)row[u] * 8);
                    w[u][0] = v.x; w[u][1] = v.y;
                } else {
                    const uint4 v = *reinterpret_cast<const uint4 *>(chunk_ptr + (size_t)row[u] * 16);
                    w[u][0] = v.x; w[u][1] = v.y; w[u][2] = v.z; w[u][3] = v.w;
                }
            }
        }
        uint32_t sum[U], base[U], rank[U];   // (places in the list: that of the lane named `leader`, and from there)
        int leader[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            sum[u] = sm->off[q[u]];
            lds_ptr<uint8_t> t = &sm->tab[q[u]][0];
#pragma unroll
            for (int j = 0; j < NB * 2; ++j) sum[u] += t[j * 16 + ((w[u][j >> 3] >> (4 * (j & 7))) & 15u)];
            const unsigned long long key = (unsigned long long)sum[u] << 32 | id[u];
            in[u] = in[u] && key <= sm->key[q[u]];
        }
        // Additions to one address are made one after the other, 8 ns each.  Ties by the ten thousand crowd in few queries, and so do
        // the candidates where neighbours are stored together: lanes that share what the first of them adds to add together, three times over
        // (all additions of the lanes in one instruction, whose answer takes a microsecond: 4 M codes in the order of 8192 lists, 1000 queries,
        // top-1000, 1750 -> 1265 us against an instruction a turn).
        auto add = [](uint32_t *at, uint32_t by) { return __hip_atomic_fetch_add(at, by, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
#pragma unroll
        for (int u = 0; u < U; ++u) {
            uint64_t todo = __ballot(in[u]);
            if constexpr (!SAMPLE) {
                uint32_t by = 1u;
                leader[u] = lane;
                rank[u] = base[u] = 0u;
                for (int turn = 0; turn < 3 && todo != 0ull; ++turn) {
                    const int first = __builtin_ctzll(todo);
                    const uint64_t same = __ballot(in[u] && q[u] == (uint32_t)__builtin_amdgcn_readlane(q[u], first)) & todo;
                    if (__popcll(same) < 6) break;
                    if ((same >> lane) & 1ull) {
                        leader[u] = first;
                        rank[u] = (uint32_t)mask_prefix(same);
                        by = (uint32_t)__popcll(same);
                    }
                    todo &= ~same;
                }
                if (in[u] && leader[u] == lane) base[u] = add(sm->a.cnt + (size_t)(q0 + q[u]) * COUNT_PITCH, by);
            } else {
                uint32_t *const bin = sm->a.hist + (size_t)(q0 + q[u]) * HIST_BINS + (sum[u] < HIST_BINS ? sum[u] : HIST_BINS - 1);
                uint32_t *tie = nullptr;
#pragma unroll
                for (int s = 0; s < ONEHOT_TIES; ++s)
                    if (in[u] && sum[u] + 1u == sm->tie_val[q[u]][s])
                        tie = sm->a.tie_rows + ((size_t)(q0 + q[u]) * ONEHOT_TIES + s) * ONEHOT_TIE_BINS + tie_bin(id[u]);
                for (int turn = 0; turn < 3 && todo != 0ull; ++turn) {
                    const int first = __builtin_ctzll(todo);
                    const uint64_t same = __ballot(in[u] && q[u] == (uint32_t)__builtin_amdgcn_readlane(q[u], first) && sum[u] == (uint32_t)__builtin_amdgcn_readlane(sum[u], first)) & todo;
                    if (__popcll(same) < 6) break;
                    const uint32_t bucket = tie_bin(id[u]);
                    const uint64_t near = __ballot(bucket == (uint32_t)__builtin_amdgcn_readlane(bucket, first)) & same;
                    if (lane == first) {
                        add(bin, (uint32_t)__popcll(same));
                        if (tie != nullptr) add(tie, (uint32_t)__popcll(near));
                    }
                    if ((near >> lane) & 1ull) tie = nullptr;   // (counted)
                    todo &= ~same;
                }
                if ((todo >> lane) & 1ull) add(bin, 1u);
                if (tie != nullptr) add(tie, 1u);
            }
        }
        if constexpr (!SAMPLE) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t at = (uint32_t)__shfl((int)base[u], leader[u]) + rank[u];
                if (in[u] && at < sm->a.cap) sm->a.lists[(size_t)(q0 + q[u]) * sm->a.cap + at] = (uint64_t)sum[u] << 32 | id[u];
            }
        }
    }
}

// The place of the counts by rows of the sum `bin`, -1 if there are none: they are kept from now on if there is a place left.
__device__ __forceinline__ int onehot_tie_slot(uint32_t *tie_val, uint32_t bin) {
    for (int s = 0; s < ONEHOT_TIES; ++s) {
        const uint32_t v = __builtin_amdgcn_readfirstlane(__hip_atomic_load(tie_val + s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        if (v == bin + 1u) return s;
        if (v == 0u) {
            if (lane_id() == 0) __hip_atomic_store(tie_val + s, bin + 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return -1;
        }
    }
    return -1;
}

// A bound, and where a better one is to be looked for: the need-th sampled row (0: nowhere) of its sum among those in tie bin `bin` (-1: all).
struct OnehotCut {
    uint64_t key;
    uint32_t need;
    int bin;
};

// For one wave: the key at or below which `topk` of the counted keys are (KEY_EMPTY: fewer, or beyond the bins that say something).
// Sums tie, in clustered data by the hundred thousand, and rows tell them apart: the first bound on a sum that far more than topk
// keys reach has the rows of that sum counted from then on (the least sum that the tables allow is counted from the start), later ones
// end at the last row of the bin in which the last tie that is needed falls.  Counts may lag behind, never run ahead.  Equal codes that are
// stored side by side all fall in one bin: where more than `most` beyond those needed do, the rows themselves are worth a look.
template <bool LAST>
__device__ __forceinline__ OnehotCut onehot_bound(const uint32_t *hist, uint32_t *tie_val, const uint32_t *tie_rows, int topk, int hist_bins, uint32_t most) {
    const int lane = lane_id();
    const int bin = hist_threshold(hist, topk);
    if (bin >= hist_bins) return {KEY_EMPTY, 0u, -1};
    uint32_t below = 0;
    for (int i = lane; i < bin; i += 64) below += hist[i];
    for (int o = 32; o > 0; o >>= 1) below += __shfl_xor(below, o);
    below = __builtin_amdgcn_readfirstlane(below);
    uint64_t key = (uint64_t)(uint32_t)bin << 32 | 0xffffffffull;
    // (the counts grow while they are read: more than topk below the bin bounds the sums by bin - 1)
    if (below >= (uint32_t)topk) return {bin > 0 ? key - (1ull << 32) : key, 0u, -1};
    const uint32_t ties = __builtin_amdgcn_readfirstlane(hist[bin]), need = (uint32_t)topk - below;
    if (below + ties < 2u * (uint32_t)topk + 64u) return {key, 0u, -1};
    const OnehotCut by_sum = {key, LAST && ties > need && ties - need > most ? need : 0u, -1};
    const int slot = onehot_tie_slot(tie_val, (uint32_t)bin);
    if (slot < 0) return by_sum;
    uint32_t c[ONEHOT_TIE_BINS / 64], incl = 0;
#pragma unroll
    for (int i = 0; i < ONEHOT_TIE_BINS / 64; ++i) {
        c[i] = __hip_atomic_load(tie_rows + (size_t)slot * ONEHOT_TIE_BINS + lane * (ONEHOT_TIE_BINS / 64) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        incl += c[i];
    }
    const uint32_t mine = incl;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
    }
    const uint64_t reach = __ballot(incl >= need);
    if (reach == 0ull) return by_sum;
    const int l = __builtin_ctzll(reach);
    uint32_t cum = incl - mine, last = 0, wanted = 0, there = 0;   // (of lane l; of the bin's ties: needed, counted)
#pragma unroll
    for (int i = 0; i < ONEHOT_TIE_BINS / 64; ++i) {
        if (cum < need) { last = (uint32_t)i; wanted = need - cum; there = c[i]; }
        cum += c[i];
    }
    const uint32_t last_bin = (uint32_t)l * (ONEHOT_TIE_BINS / 64) + (uint32_t)__builtin_amdgcn_readlane(last, l);
    wanted = (uint32_t)__builtin_amdgcn_readlane(wanted, l);
    there = (uint32_t)__builtin_amdgcn_readlane(there, l);
    return {(uint64_t)(uint32_t)bin << 32 | tie_bin_last_row(last_bin), LAST && there - wanted > most ? wanted : 0u, (int)last_bin};
}

// Whole block: the row of the cut's need-th tie in the sample (0xffffffff: there are fewer).
template <int NB>
__device__ __forceinline__ uint32_t onehot_tied_row(const OnehotArgs &a, int q, const OnehotCut cut) {
    constexpr int U = 4, WAVES = OH_PICK_THREADS / 64;
    __shared__ uint16_t pair[NB][256];
    __shared__ uint32_t got[2][U][WAVES], found;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint8_t *const tab = a.qluts + (size_t)q * (NB * 32);
    for (int i = tid; i < NB * 256; i += OH_PICK_THREADS) {
        const int r = i >> 8, byte = i & 255;
        pair[r][byte] = (uint16_t)(tab[r * 32 + (byte & 15)] + tab[r * 32 + 16 + (byte >> 4)]);
    }
    if (tid == 0) found = 0xffffffffu;
    __syncthreads();
    const uint32_t sum = (uint32_t)(cut.key >> 32), ns = (uint32_t)a.n;
    const uint32_t first = cut.bin <= 0 ? 0u : (tie_bin_last_row((uint32_t)cut.bin - 1u) + 1u) >> a.shift;
    const uint64_t last = cut.bin < 0 ? ns - 1u : tie_bin_last_row((uint32_t)cut.bin) >> a.shift;   // (in the sample)
    const uint32_t end = last < ns ? (uint32_t)last + 1u : ns;
    uint32_t seen = 0;
    for (uint32_t at = first, turn = 0; at < end; at += U * OH_PICK_THREADS, turn ^= 1u) {
        uint64_t tied[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = at + u * OH_PICK_THREADS + tid;
            uint32_t w[NB / 4] = {};
            if (i < end) {
                if constexpr (NB == 8) {
                    const uint2 v = reinterpret_cast<const uint2 *>(a.codes)[i];
                    w[0] = v.x; w[1] = v.y;
                } else {
                    const uint4 v = reinterpret_cast<const uint4 *>(a.codes)[i];
                    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
                }
            }
            uint32_t s = 0;
#pragma unroll
            for (int r = 0; r < NB; ++r) s += pair[r][(w[r >> 2] >> (8 * (r & 3))) & 255u];
            tied[u] = __ballot(i < end && s == sum && (cut.bin < 0 || tie_bin(onehot_sample_row(i, a.shift)) == (uint32_t)cut.bin));
            if (lane == 0) got[turn][u][wave] = (uint32_t)__popcll(tied[u]);
        }
        __syncthreads();   // (one per turn: the next one's counts go to the other half)
        uint32_t before = seen;
#pragma unroll
        for (int u = 0; u < U; ++u)
            for (int w = 0; w < WAVES; ++w) {
                const uint32_t c = got[turn][u][w];
                if (w == wave && before < cut.need && before + c >= cut.need) {
                    if (((tied[u] >> lane) & 1ull) && (uint32_t)mask_prefix(tied[u]) == cut.need - 1u - before) found = onehot_sample_row(at + u * OH_PICK_THREADS + tid, a.shift);
                }
                before += c;
            }
        seen = before;
        if (seen >= cut.need) break;
    }
    __syncthreads();
    return found;
}

// Whole block: the queries' bounds and the tables' image for the rows from row_lo on.
template <int NB, int G, bool SAMPLE>
__device__ __noinline__ void onehot_image(lds_ptr<OnehotSmem<NB, G>> sm, uint32_t row_lo) {
    constexpr int QT = 32 * G, PARTS = OH_THREADS / QT;
    constexpr uint32_t NT = 2 * NB, RANGE = OH_CENTRE * NT;
    const int tid = threadIdx.x;
    const int q0 = sm->q0, nq = sm->a.nq;
    if (tid < QT) {
        unsigned long long key = 0ull;
        if (q0 + tid < nq) {
            key = sm->a.tau_key[q0 + tid];
            // (a list without room: the call will be made another way)
            if (!SAMPLE && __hip_atomic_load(sm->a.cnt + (size_t)(q0 + tid) * COUNT_PITCH, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) > sm->a.cap) key = 0ull;
        }
        sm->key[tid] = key;
    }
    if (SAMPLE)
        for (int i = tid; i < QT * ONEHOT_TIES; i += OH_THREADS)
            sm->tie_val[i / ONEHOT_TIES][i % ONEHOT_TIES] = q0 + i / ONEHOT_TIES < nq ? sm->a.tie_val[(size_t)q0 * ONEHOT_TIES + i] : 0u;
    __syncthreads();
    const int q = tid % QT, part = tid / QT;
    const unsigned long long key = sm->key[q];
    // sums below `below` can still be candidates; at the bound's own sum its row decides
    const int64_t below = (int64_t)(key >> 32) + ((uint32_t)key >= row_lo ? 1 : 0) - (int64_t)sm->off[q];
    // (a query that the first codes gave no bound is left to the other loops)
    const bool none = q0 + q >= nq || below <= 0 || (uint32_t)(key >> 32) >= 0x7fffu;
    const float scale = none ? 0.f : below <= RANGE ? 1.f : (float)RANGE / (float)below;
    const uint32_t short_of = !none && below <= RANGE ? RANGE - (uint32_t)below : 0u;   // what the tables' c add up to
#pragma unroll 1
    for (int byte = part; byte < NB; byte += PARTS) {   // (32 entries)
        const int h = byte / (NB / 2), ks = byte % (NB / 2);
        uint32_t out[6] = {0u, 0u, 0u, 0u, 0u, 0u};
        uint32_t in[8];
        lds_ptr<uint32_t> t = (lds_ptr<uint32_t>)&sm->tab[q][byte * 32];
#pragma unroll
        for (int x = 0; x < 8; ++x) in[x] = t[x];
#pragma unroll
        for (int i = 0; i < 32; ++i) {
            const float v = (float)((in[i >> 2] >> (8 * (i & 3))) & 255u);
            // (the product may round up by 2^-24 of itself: 32 of them stay below the range for a sum below the bound by 1 or more)
            const uint32_t c = short_of / NT + ((uint32_t)(byte * 2 + i / 16) < short_of % NT ? 1u : 0u);
            const uint32_t e = none ? (uint32_t)OH_MOST : (uint32_t)(v * scale) + c;
            const uint32_t code = onehot_entry(e < (uint32_t)OH_MOST ? e : (uint32_t)OH_MOST);
            const int bit = 6 * i;
            out[bit >> 5] |= code << (bit & 31);
            if ((bit & 31) > 26) out[(bit >> 5) + 1] |= code >> (32 - (bit & 31));
        }
        lds_ptr<uint32_t> d = &sm->img[(q >> 5) * (NB / 2) + ks][h * 32 + (q & 31)][0];
#pragma unroll
        for (int x = 0; x < 6; ++x) d[x] = out[x];
    }
    __syncthreads();
}

// blocks of 4 waves that share a CU: by the 512 registers of a lane, and by LDS
constexpr int onehot_blocks_per_cu(int nb, int g) { return g * nb >= 32 ? 2 : 3; }

template <int NB, int G, int PASS>   // code bytes; groups of 32 queries that a block serves
__global__ __launch_bounds__(OH_THREADS, onehot_blocks_per_cu(NB, G)) void scan_onehot_kernel(OnehotArgs a) {
    typedef OnehotSmem<NB, G> SM;
    constexpr bool SAMPLE = PASS != OH_LIST;
    constexpr int QT = SM::QT, NK = NB / 8, NS = NB / 2;   // words of a code per lane, products per 32 codes and 32 queries
    constexpr int GU = G > 1 ? 2 : 1, TILES = 32 / NB;     // groups whose products run side by side; pieces of 32 codes per load
    constexpr int LOAD = 32 * TILES;                       // codes per 16-byte load of a wave
    static_assert(sizeof(SM) <= 72 * 1024, "two blocks share the 160 KB of a CU");
    __shared__ SM sm;
    lds_ptr<SM> smp = (lds_ptr<SM>)&sm;
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t h = (uint32_t)lane >> 5, col = (uint32_t)lane & 31u;
    if (tid == 0) { sm.a = a; sm.parked = 0u; }
    // least place that a row of the wave's queue entries starts from: row << 7 | query, the lane's own part
    const uint32_t lane_part = (NB == 8 ? 2u * col : col) << 7 | h << 2;
    uint32_t parked = 0;
    for (;;) {
        __syncthreads();
        if (tid == 0) sm.item = (int)atomicAdd(a.work_counter, 1u);
        __syncthreads();
        const int item = sm.item;
        if (item >= a.nitems) break;
        const int tile = item % a.ntiles;
        const int chunk = item / a.ntiles;
        const int64_t begin = chunk < a.nhead ? chunk * a.head_codes : a.nhead * a.head_codes + (chunk - a.nhead) * a.chunk_codes;
        const int64_t whole = chunk < a.nhead ? a.head_codes : a.chunk_codes;
        const int ncodes = (int)(begin + whole < a.n ? whole : a.n - begin);
        const int q0 = tile * QT;
        const uint8_t *const chunk_ptr = a.codes + (size_t)begin * NB;
        if (tid == 0) { sm.q0 = q0; sm.begin = begin; sm.ncodes = ncodes; sm.chunk_ptr = chunk_ptr; }
        if (tid < QT) sm.off[tid] = 0u;
        __syncthreads();
        for (int i = tid; i < QT * NB * 2; i += OH_THREADS) {
            const int q = i / (NB * 2), j = i % (NB * 2);
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (q0 + q < a.nq) v = *reinterpret_cast<const uint4 *>(a.qluts + (size_t)(q0 + q) * (NB * 32) + j * 16);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            uint32_t least = 255u;
#pragma unroll
            for (int x = 0; x < 16; ++x) {
                const uint32_t e = (w[x >> 2] >> (8 * (x & 3))) & 255u;
                least = e < least ? e : least;
            }
            const uint32_t all = least * 0x01010101u;   // (no byte is below it: no borrow)
            *reinterpret_cast<uint4 *>(&sm.tab[q][j * 16]) = make_uint4(v.x - all, v.y - all, v.z - all, v.w - all);
            if (least != 0u) atomicAdd(&sm.off[q], least);
        }
        // the loads that this pass looks at, and the one that is its x-th
        const int runs = (ncodes + LOAD - 1) / LOAD;
        const int nloads = PASS == OH_FIRST ? (runs + 3) / 4 : PASS == OH_REST ? runs - (runs + 3) / 4 : runs;
        auto row_of = [&](int x) -> int {   // (x beyond nloads by up to two rounds of the waves: below 2^25 all the same)
            return (PASS == OH_LIST ? x : PASS == OH_FIRST ? 4 * x : x + x / 3 + 1) * LOAD;
        };
        const int per_wave = (nloads + OH_WAVES - 1) / OH_WAVES;
        // 16 bytes per lane, rows beyond the item read as zeros
        auto load = [&](int x) -> uint4 {
            const int begin_row = row_of(x), row = begin_row + lane * (16 / NB);
            const uint8_t *const p = chunk_ptr + (size_t)row * NB;
            if (begin_row + LOAD <= ncodes) return *reinterpret_cast<const uint4 *>(p);
            if (row + 16 / NB <= ncodes) return *reinterpret_cast<const uint4 *>(p);
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (row < ncodes) {   // (8-byte codes only: the last one)
                const uint2 half = *reinterpret_cast<const uint2 *>(p);
                v.x = half.x; v.y = half.y;
            }
            return v;
        };
        uint4 code_a = load(wave), code_b = load(wave + OH_WAVES);   // (two loads on their way: one's products take 1 us, memory sometimes longer)
        __syncthreads();
        onehot_image<NB, G, SAMPLE>(smp, SAMPLE ? onehot_sample_row((uint32_t)begin, a.shift) : (uint32_t)begin);
        {
            v8i A[G][NS];
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int s = 0; s < NS; ++s) {
                    const uint2 *p = reinterpret_cast<const uint2 *>(&sm.img[g * NS + s][lane][0]);
                    const uint2 x = p[0], y = p[1], z = p[2];
                    A[g][s] = (v8i){(int)x.x, (int)x.y, (int)y.x, (int)y.y, (int)z.x, (int)z.y, 0, 0};
                }
            v16f acc[2][GU];
#pragma unroll
            for (int g = 0; g < GU; ++g)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[1][g][r] = 0.f;   // (the product before the first)
            int qn = 0;
            // queue what is negative among the sums of groups g0, g0 + 1 for the rows from `base` on
            auto test = [&](const v16f (&s)[GU], uint32_t base, int g0) {
                uint32_t neg[GU];
                neg[0] = any_negative(s[0]);
                if constexpr (GU == 2) neg[GU - 1] = any_negative(s[GU - 1]);
                if (__builtin_expect(__ballot((int)(neg[0] | neg[GU - 1]) < 0) == 0ull, 1)) return;
#pragma unroll
                for (int g = 0; g < GU; ++g) {
                    if (__ballot((int)neg[g] < 0) == 0ull) continue;
                    uint32_t bits = 0;   // bit 15 - r: number r is negative
#pragma unroll
                    for (int r = 0; r < 16; ++r) bits = __builtin_amdgcn_alignbit(bits, __float_as_uint(s[g][r]), 31);
                    const uint32_t entry = (base << 7) + lane_part + (uint32_t)(g0 + g) * 32u;
                    for (uint64_t mask; (mask = __ballot(bits != 0u)) != 0ull;) {
                        const uint32_t r = 15u - (uint32_t)__builtin_ctz(bits | 0x10000u);
                        if (bits != 0u) sm.queue[wave][qn + mask_prefix(mask)] = entry + 8u * (r >> 2) + (r & 3u);
                        qn += (int)__popcll(mask);
                        bits &= bits - 1u;
                        if (qn > OH_QUEUE - 64) {
                            onehot_flush<NB, G, SAMPLE>(smp, wave, qn);
                            parked += (uint32_t)qn;
                            qn = 0;
                        }
                    }
                }
            };
            uint32_t before = 0;   // first row of the product before
            auto products = [&](uint4 &code, int x) {
                const uint4 cur = code;
                // lanes 0-31 hold the first halves of 32 codes, lanes 32-63 the second ones
                uint32_t w[NK][TILES];
                if constexpr (NB == 8) {
                    const auto s0 = __builtin_amdgcn_permlane32_swap(cur.x, cur.y, false, false);   // even codes of the load
                    const auto s1 = __builtin_amdgcn_permlane32_swap(cur.z, cur.w, false, false);   // odd ones
                    w[0][0] = s0[0]; w[0][1] = s0[1]; w[0][2] = s1[0]; w[0][3] = s1[1];
                } else {
                    const auto s0 = __builtin_amdgcn_permlane32_swap(cur.x, cur.z, false, false);
                    const auto s1 = __builtin_amdgcn_permlane32_swap(cur.y, cur.w, false, false);
                    w[0][0] = s0[0]; w[0][1] = s0[1]; w[NK - 1][0] = s1[0]; w[NK - 1][1] = s1[1];
                }
                code = load(x + 2 * OH_WAVES);
                const uint32_t first = (uint32_t)row_of(x);
#pragma unroll
                for (int u = 0; u < TILES; ++u) {
                    const uint32_t base = first + (NB == 8 ? (uint32_t)((u & 1) * 64 + (u >> 1)) : (uint32_t)u * 32u);
                    v8i b[NS];
#pragma unroll
                    for (int k = 0; k < NK; ++k) {
                        v8i four[4];
                        onehot_columns(w[k][u], four);
#pragma unroll
                        for (int s = 0; s < 4; ++s) b[4 * k + s] = four[s];
                    }
#pragma unroll
                    for (int gp = 0; gp < G / GU; ++gp) {
                        constexpr bool BY_GROUP = G > GU;
                        const int now = BY_GROUP ? gp & 1 : u & 1;
#pragma unroll
                        for (int s = 0; s < NS; ++s)
#pragma unroll
                            for (int g = 0; g < GU; ++g)
                                acc[now][g] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(A[gp * GU + g][s], b[s], s == 0 ? (v16f){} : acc[now][g], 2, 4, 0, 0, 0, 0);
                        test(acc[now ^ 1], before, BY_GROUP && gp == 0 ? G - GU : BY_GROUP ? (gp - 1) * GU : 0);
                        before = base;
                    }
                }
            };
#pragma unroll 1
            for (int pos = 0; pos < per_wave; pos += 2) {
                products(code_a, pos * OH_WAVES + wave);
                products(code_b, (pos + 1) * OH_WAVES + wave);   // (of an odd number the last one: zeros)
            }
            test(acc[1], before, G - GU);
            if (qn > 0) {
                onehot_flush<NB, G, SAMPLE>(smp, wave, qn);
                parked += (uint32_t)qn;
            }
        }
    }
    if (a.stats != nullptr) {
        if (lane == 0 && parked != 0u) atomicAdd(&sm.parked, parked);
        __syncthreads();
        if (tid == 0 && sm.parked != 0u) atomicAdd(a.stats, (unsigned long long)sm.parked);
    }
}

// The bounds that the counts give: one wave per query, and behind the whole sample (LAST) a block that looks through it for the row at which
// ties end (only where a list might have no room for them).
template <int NB, bool LAST>
__global__ __launch_bounds__(LAST ? OH_PICK_THREADS : 64) void onehot_pick_kernel(OnehotArgs a) {
    const int q = blockIdx.x;
    __shared__ OnehotCut s_cut;
    const uint32_t most = (a.cap - a.cap / 4 >> a.shift) - (uint32_t)a.topk;   // (of a list's room three quarters; cap is far above the topk of both)
    if (threadIdx.x < 64) {
        const uint32_t *const hist = a.hist + (size_t)q * HIST_BINS;
        uint32_t *const tie_val = a.tie_val + (size_t)q * ONEHOT_TIES;
        const OnehotCut cut = onehot_bound<LAST>(hist, tie_val, a.tie_rows + (size_t)q * (ONEHOT_TIES * ONEHOT_TIE_BINS), a.topk, a.hist_bins, most);
        const unsigned long long before = a.tau_key[q];
        if (cut.key < before && threadIdx.x == 0) a.tau_key[q] = cut.key;
        if (LAST && threadIdx.x == 0) s_cut = cut;
        if (q == 0 && threadIdx.x == 0) *a.work_counter = 0u;
    }
    if constexpr (LAST) {
        __syncthreads();
        const OnehotCut cut = s_cut;
        if (cut.need == 0u) return;
        const uint32_t row = onehot_tied_row<NB>(a, q, cut);
        const unsigned long long key = cut.key >> 32 << 32 | row;
        if (threadIdx.x == 0 && key < a.tau_key[q]) a.tau_key[q] = key;
    }
}

// The sample gathered, and the least sum that a query's tables allow: the first whose rows are counted.  Bound by the lines of memory that the
// sample touches.
template <class CODE>
__global__ __launch_bounds__(256) void onehot_sample_kernel(const CODE *__restrict__ codes, uint32_t ns, int shift, CODE *__restrict__ sample,
                                                            const uint8_t *__restrict__ qluts, int nq, int tables, uint32_t *__restrict__ tie_val) {
    const int least_blocks = (nq + 3) / 4;   // (a wave per query)
    if ((int)blockIdx.x >= least_blocks) {
        const uint32_t i = (blockIdx.x - (uint32_t)least_blocks) * 256u + threadIdx.x;
        if (i < ns) sample[i] = codes[onehot_sample_row(i, shift)];
        return;
    }
    const int q = (int)blockIdx.x * 4 + (int)(threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (q >= nq) return;
    uint32_t least = 0;
    if (lane < tables) {
        const uint4 v = *reinterpret_cast<const uint4 *>(qluts + ((size_t)q * tables + lane) * 16);
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
        least = 255u;
#pragma unroll
        for (int x = 0; x < 16; ++x) least = min(least, (w[x >> 2] >> (8 * (x & 3))) & 255u);
    }
    for (int o = 32; o > 0; o >>= 1) least += __shfl_xor(least, o);
    if (lane == 0) tie_val[(size_t)q * ONEHOT_TIES] = least + 1u;
}

template <int NB, int G, int PASS>
static int launch_tiles(pq_ctx *ctx, OnehotArgs &a) {
    constexpr int QT = 32 * G, LOAD = 1024 / NB;
    constexpr int64_t step = (int64_t)LOAD * OH_WAVES;   // (and a round of the sample's four quarters)
    static_assert(OH_WAVES == 4, "a quarter of a chunk's loads of the sample is every fourth");
    const int most = onehot_blocks_per_cu(NB, G) * ctx->num_cu;
    a.ntiles = (a.nq + QT - 1) / QT;
    // As many items per block as have 64 loads of a wave and more (their set-up takes the time of 10), up to six: of the two blocks of a
    // compute unit the one that began first is served first, and items even that out.
    int64_t nchunks = most / a.ntiles, per_block = 1;
    if (PASS == OH_LIST) {
        per_block = a.n * a.ntiles / (most * 64 * step);
        per_block = per_block < 1 ? 1 : per_block > 6 ? 6 : per_block;
        nchunks = per_block * most / a.ntiles;
    }
    if (nchunks < 1) nchunks = 1;
    if (nchunks < (a.n >> 24) + 1) nchunks = (a.n >> 24) + 1;   // (25 bits of a queue entry for the row)
    auto whole_steps = [&](int64_t rows) { return (rows + step - 1) / step * step; };
    a.chunk_codes = whole_steps((a.n + nchunks - 1) / nchunks);
    a.head_codes = whole_steps((a.chunk_codes + 7) / 8);
    a.nhead = 0;
    // (the first 32nd of the rows, or the first chunk: 1 M codes, 2049 queries, top-10, 30 chunks 532 us without, 246 with)
    if (PASS == OH_LIST && nchunks >= 12 && a.head_codes < a.chunk_codes) a.nhead = (int)((nchunks < 64 ? 1 : nchunks / 32) * a.chunk_codes / a.head_codes);
    nchunks = a.nhead + (a.n - a.nhead * a.head_codes + a.chunk_codes - 1) / a.chunk_codes;
    a.nitems = (int)(nchunks * a.ntiles);
    const int nblocks = a.nitems < most ? a.nitems : most;
    scan_onehot_kernel<NB, G, PASS><<<nblocks, OH_THREADS, 0, ctx->stream>>>(a);
    PQ_HIP(ctx, hipGetLastError());
    return PQ_OK;
}

template <int NB, int G>
static int launch_passes(pq_ctx *ctx, OnehotArgs &a, const uint8_t *codes, int64_t n, int topk) {
    int rc = launch_tiles<NB, G, OH_FIRST>(ctx, a);
    if (rc) return rc;
    onehot_pick_kernel<NB, false><<<a.nq, 64, 0, ctx->stream>>>(a);
    PQ_HIP(ctx, hipGetLastError());
    rc = launch_tiles<NB, G, OH_REST>(ctx, a);
    if (rc) return rc;
    onehot_pick_kernel<NB, true><<<a.nq, OH_PICK_THREADS, 0, ctx->stream>>>(a);
    PQ_HIP(ctx, hipGetLastError());
    a.topk = topk;
    a.codes = codes;
    a.n = n;
    return launch_tiles<NB, G, OH_LIST>(ctx, a);
}

int onehot_queries_per_pass(int code_bytes, int nq) { return nq <= 32 ? 32 : nq <= 64 || code_bytes == 16 ? 64 : 128; }

// A greater shift makes the sample's gathering and passes cheaper and lets more keys through: 25 M codes, 1000 queries, top-100 and -1000, ms with shift 4 2.35
// and 2.74, 5 2.16 and 2.58, 6 2.08 and 2.48, 7 2.09 and 2.53; 8.4 M 0.96 and 1.32 with 5, 0.97 and 1.34 with 6; 256 queries, top-1000, 16 M 0.74 with 5, 0.80
// with 6; 4 M 0.66 and 0.93 with 4, 0.67 and 0.92 with 5; 1 M 0.38 and 0.61 with 3, 0.37 and 0.57 with 4.  (More where it has no room.)
int onehot_shift(int64_t n, int code_bytes, int nq, int topk, size_t room) {
    int shift = n >= 3 << 22 && (topk <= 512 || nq >= 512) ? 6 : n >= 1 << 23 ? 5 : n >= 1 << 21 ? 4 : 3;
    while (shift <= 8 && (size_t)(n >> shift) * code_bytes > room) ++shift;
    return shift <= 8 ? shift : 0;
}

int onehot_rank(int shift, int topk) {
    const double mu = (double)topk / (1 << shift);
    return (int)(mu + 4.5 * sqrt(mu) + 4.0);
}

int launch_onehot_sample(pq_ctx *ctx, const uint8_t *codes, int64_t n, int code_bytes, int shift, uint8_t *sample, const uint8_t *qluts, int nq, uint32_t *ties) {
    const uint32_t ns = (uint32_t)(n >> shift);
    const unsigned blocks = (unsigned)((nq + 3) / 4) + (ns + 255) / 256;
    if (code_bytes == 8) onehot_sample_kernel<uint2><<<blocks, 256, 0, ctx->stream>>>((const uint2 *)codes, ns, shift, (uint2 *)sample, qluts, nq, 16, ties);
    else onehot_sample_kernel<uint4><<<blocks, 256, 0, ctx->stream>>>((const uint4 *)codes, ns, shift, (uint4 *)sample, qluts, nq, 32, ties);
    PQ_HIP(ctx, hipGetLastError());
    return PQ_OK;
}

int launch_scan_onehot(pq_ctx *ctx, const uint8_t *codes, int64_t n, int code_bytes, const uint8_t *sample, int shift, const uint8_t *qluts, int nq, int topk, int hist_bins,
                       unsigned long long *tau_key, uint32_t *cnt, uint32_t *hist, uint64_t *lists, uint32_t cap,
                       uint32_t *ties, uint32_t *work_counter, unsigned long long *stats) {
    OnehotArgs a{sample, n >> shift, 0, 0, 0, 0, 0, qluts, nq, onehot_rank(shift, topk), hist_bins, shift, tau_key, cnt, hist, lists, cap,
                 ties, ties + (size_t)nq * ONEHOT_TIES, work_counter, stats};
    const int width = onehot_queries_per_pass(code_bytes, nq);
    if (code_bytes == 8) return width == 32 ? launch_passes<8, 1>(ctx, a, codes, n, topk) : width == 64 ? launch_passes<8, 2>(ctx, a, codes, n, topk) : launch_passes<8, 4>(ctx, a, codes, n, topk);
    return width == 32 ? launch_passes<16, 1>(ctx, a, codes, n, topk) : launch_passes<16, 2>(ctx, a, codes, n, topk);
}

}  // namespace pq
