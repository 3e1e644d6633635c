// IVFADC search with Quick ADC in the Scan step (chapter 5: packed 4-bit codes, m = 16 sub-quantizers of 16
// centroids, tables quantised to 8 bits, Section 5.2; Section 5.3 evaluates it inside the inverted index of
// Section 2.3.2).  Per query:
//   qmax     float ADC of the first `init` codes met when the probed lists are walked in probe order (each code with
//            the float tables of its own (query, list) pair); qmax = the topk-th smallest of these distances, the
//            distance to a temporary topk-th neighbour (Section 5.2.1, as Section 4.2.4);
//   8 bits   every pair's tables quantised between the pair's own smallest entry and the query's qmax
//            (launch_quantize_luts);
//   Scan     integer sums of the 8-bit entries (Alg. 3, plain sums) over the codes of the list; the kprime smallest
//            (sum, row) of a pair are its candidates;
//   Rerank   float ADC of the candidates with the pair's float tables; the topk smallest (distance, row) of the query.
// Sums of different pairs are not comparable (own qmin and scale each), so the candidates are chosen per pair.
//
// Where the thesis keeps the 16 tables of 16 bytes in SIMD registers and looks 16 codes up at once, the scan kernel
// here keeps the tables of EIGHT (query, list) pairs that probe the same list side by side in LDS: the entry for
// (sub-quantizer j, index i) is one 16-byte slot of eight 16-bit values, so one LDS read serves eight pairs and the
// eight sums are formed by four packed 16-bit additions per sub-quantizer.  The 16 slots of a sub-quantizer cover
// all 64 LDS banks once: lanes with different indexes never collide and lanes with equal indexes read one address.
//
// The kprime smallest sums of a work item (a chunk of a list x up to 8 pairs) are found by counting instead of
// sorting, because sums are small integers (at most 16 * 255): a first pass over the codes counts the sums of each
// pair in 512 bins, which gives the kprime-th smallest sum T of the pair exactly; a second pass collects the codes
// below T (fewer than kprime) and, in row order, those equal to T.  Every float sum of this file is formed in
// double in table order and rounded once, so that the bound, the 8-bit tables, the candidates and the distances are
// those of the plain definition bit for bit.
#include <stddef.h>
#include <type_traits>
#include "pq_internal.h"
#include "scan_common.h"
#include "topk_device.h"

namespace pq {

constexpr int QK_QS = 8;          // (query, list) pairs per work item
constexpr int QK_LONG_MIN = 1 << IVF_QUICK_LONG_CLASS;   // lists of this many rows and more take the blocks of 8 waves
constexpr int QK_BINS = 512;      // sums counted per pass: base .. base + 510, and one bin for everything above
constexpr int QK_KP = 128;        // kprime at most (the length of a result list)
constexpr int QK_BATCH = 4;       // codes of a thread on their way at a time
constexpr float QK_LB_RANGE = 104.f;   // units of the lower bounds between the sum of the minima and the cap (at most 118)
constexpr int QK_DBINS = IVF_QUICK_DBINS;   // bins of a query's float distances, over 0 .. qmax

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pk_add_u16(uint32_t a, uint32_t b) {
    const u16x2 r = __builtin_bit_cast(u16x2, a) + __builtin_bit_cast(u16x2, b);
    return __builtin_bit_cast(uint32_t, r);
}
// per 16-bit half: a - b, 0 where b > a
__device__ __forceinline__ uint32_t pk_sub_sat_u16(uint32_t a, uint32_t b) {
    const u16x2 r = __builtin_elementwise_sub_sat(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b));
    return __builtin_bit_cast(uint32_t, r);
}

// index j (0 .. 15) of a packed code: component 2i in the low half of byte i
__device__ __forceinline__ uint32_t code_index4(const uint2 c, int j) { return ((j < 8 ? c.x : c.y) >> (4 * (j & 7))) & 15u; }

// float ADC in double, table order, rounded once (tab: [16][16] floats)
__device__ __forceinline__ float adc16x4_exact(const float *tab, const uint2 c) {
    double s = 0.0;
#pragma unroll
    for (int j = 0; j < 16; ++j) s += (double)tab[j * 16 + code_index4(c, j)];
    return (float)s;
}

// ------------------------------------------------------------------------------------------
// qmax of every query, written once per (query, list) pair, and the query's bound for the final merge set to "none".
// One block per query.
constexpr int QK_INIT_MAX = 4096;
__global__ __launch_bounds__(256) void ivf_quick_qmax_kernel(const uint8_t *__restrict__ codes,
                                                             const int64_t *__restrict__ list_offsets,
                                                             const int32_t *__restrict__ probes, const float *__restrict__ luts,
                                                             int nprobe, int init, int topk, float *qmax_pair,
                                                             unsigned long long *tau_key, uint32_t *dist_bins, float *dist_inv) {
    __shared__ float tab[256];
    __shared__ uint32_t vals[QK_INIT_MAX];
    __shared__ uint32_t bins[256], state[2];
    const int q = blockIdx.x, tid = threadIdx.x;
    int count = 0;
    for (int r = 0; r < nprobe && count < init; ++r) {
        const int l = probes[(size_t)q * nprobe + r];
        const int64_t beg = list_offsets[l], size = list_offsets[l + 1] - beg;
        const int take = (int)(size < init - count ? size : init - count);
        if (take <= 0) continue;
        __syncthreads();
        tab[tid] = luts[((size_t)q * nprobe + r) * 256 + tid];
        __syncthreads();
        for (int i = tid; i < take; i += 256) {
            const uint2 c = *reinterpret_cast<const uint2 *>(codes + (size_t)(beg + i) * 8);
            vals[count + i] = f32_to_ord(adc16x4_exact(tab, c));
        }
        count += take;
    }
    __syncthreads();
    float qmax = __builtin_inff();
    if (count > 0) qmax = ord_to_f32(block_kth_smallest_u32(vals, count, (uint32_t)(topk < count ? topk : count), bins, state));
    for (int r = tid; r < nprobe; r += 256) qmax_pair[(size_t)q * nprobe + r] = qmax;
    static_assert(QK_DBINS == 256, "a thread per bin");
    if (dist_bins) dist_bins[(size_t)q * QK_DBINS + tid] = 0u;
    if (tid == 0) tau_key[q] = KEY_EMPTY;
    if (tid == 0 && dist_bins) {
        const float inv = (float)QK_DBINS / qmax;
        dist_inv[q] = qmax > 0.f && inv < __builtin_inff() ? inv : 0.f;   // (0, NaN, infinity or subnormal qmax: no bins)
    }
}

// What a query's bound says about the integer sums of one of its pairs.  A code of float distance D = sum of its entries t_j has
// 8-bit entries of at most (t_j - qmin) * scale each (rounded down, or 255 where that is more), so D <= tau implies
// sum <= (tau - 16 qmin) * scale: codes of greater sums are in no result, whether or not they are among the kprime smallest of
// their pair.  The factors 1 + 1e-6 and the unit on top cover the roundings of D, t_j - qmin and the product (2^-22 together).
// Returns the greatest sum that can matter, -1 if none can, QK_NO_CAP without a bound (no tau yet, or NaN anywhere).
constexpr int QK_NO_CAP = 0xfffe;
__device__ __forceinline__ int quick_sum_cap(unsigned long long tau_key, float qmin, float scale) {
    if (tau_key == KEY_EMPTY) return QK_NO_CAP;
    const double tau = (double)ord_to_f32((uint32_t)(tau_key >> 32));
    const double c = (tau + fabs(tau) * 1e-6 - 16.0 * (double)qmin) * (double)scale * (1.0 + 1e-6);
    if (!(c < (double)(QK_NO_CAP - 1))) return QK_NO_CAP;
    return c < 0.0 ? -1 : (int)c + 1;
}

// ------------------------------------------------------------------------------------------
// (256: slots are addressed by a bitwise or with their table's address, in sub-quantizers of 128 and of 256 bytes)
constexpr int QK_SMEM_ALIGN = 256;
template <int QK_WAVES, typename TieRow>
struct __align__(QK_SMEM_ALIGN) QuickSmem {
    uint2 lbtab[256];                            // slot j * 16 + i: 4-bit lower bounds of the entries (j, i) of the 8 pairs as bytes
    uint4 tab[256];                              // slot j * 16 + i: the 8-bit entries (j, i) of the 8 pairs as 16-bit values
    uint32_t hist[QK_QS][QK_BINS];
    unsigned long long sure[QK_QS][QK_KP];       // keys below the pair's T (fewer than kprime)
    TieRow tie[QK_WAVES][QK_QS][QK_KP];          // rows (within the item) with sum T, per wave in ascending order
    int sure_cnt[QK_QS];
    int tie_cnt[QK_WAVES][QK_QS];
    uint32_t tstar[QK_QS];                       // T: the kprime-th smallest sum (0xffff: every code is a candidate)
    uint32_t below[QK_QS];                       // sums below `base` (counted in earlier attempts)
    uint32_t base[QK_QS];                        // first sum of bin 0 in the current counting pass
    int found[QK_QS];
    uint32_t cap[QK_QS];                         // sums above it are not counted (the kprime-th smallest sum so far)
    uint32_t cum_t[QK_QS];                       // sums from `base` on below the cap (all counted sums while none is reached)
    int reached[QK_QS];
    int tcap[QK_QS];                             // the greatest sum that the query's bound leaves a chance (quick_sum_cap)
    float qmin[QK_QS], scale[QK_QS], dinv[QK_QS];
    unsigned long long tau[QK_QS];               // the query's bound when the item began
    int counted[QK_QS];                          // candidates put into the query's bins
    int alive[QK_QS];                            // some code of the pair can be in the result
    int pair[QK_QS];
    uint32_t out_idx[QK_QS];
    uint4 minw[16];                              // smallest entry of sub-quantizer j of the 8 pairs as 16-bit values
    uint2 lbbias;                                // per pair 0x80 minus its T in units of the bounds, as bytes
    uint32_t seg_saved[2];                       // rows saved in the last segment and in this one
    int pending;                                 // pairs whose T is not known yet
    int item;
    int single;                                  // the list is this one item: its candidates are final
};
// (lists of the blocks of 4 waves have fewer than QK_LONG_MIN = 2^16 rows, an item at most one row of alignment more: 16
// bits hold a row within the item)
typedef QuickSmem<4, uint16_t> QuickSmemShort;
typedef QuickSmem<8, uint32_t> QuickSmemLong;
static_assert(QK_LONG_MIN <= 65536, "rows of short items fit 16 bits");
static_assert(offsetof(QuickSmemShort, lbtab) % 128 == 0 && offsetof(QuickSmemLong, lbtab) % 128 == 0, "sub-quantizers of 128 bytes");
static_assert(offsetof(QuickSmemShort, tab) % 256 == 0 && offsetof(QuickSmemLong, tab) % 256 == 0, "sub-quantizers of 256 bytes");
static_assert(sizeof(QuickSmemShort) <= 40 * 1024, "four blocks of 4 waves share the 160 KB of a compute unit");
static_assert(sizeof(QuickSmemLong) <= 80 * 1024, "two blocks of 8 waves per compute unit");

// per pair: smallest entry (NaN: the tables hold one) and scale of the 8-bit tables; per query: bins of the candidates' float
// distances and their factor
struct QuickBound {
    const float *qmin, *scale;
    uint32_t *dist_bins;
    const float *dist_inv;
};

// Blocks of QK_WAVES waves.  LONG: the kernel takes the work items of lists of QK_LONG_MIN rows and more (8 waves, two blocks
// per compute unit: the longest item of a skewed index is what the call waits for), else the others (4 waves,
// four blocks per compute unit).  The table of items has those of the long lists first; blocks draw them from a counter.
// Both kernels are in flight together where the call has a second stream: blocks of the short items move in as
// those of the long ones leave, instead of waiting for the last long item.
// A list that is one item (all but the longest) has its candidates reranked here, while its codes are in the caches:
// the float keys go to the result list directly (the separate rerank fetched 82 M candidates' codes from memory again,
// one block of 128 threads per pair: 1.86 ms of the billion-code call).
// 10^9 codes in 65 536 lists, 10 000 queries x 64 probes: both scans and the rerank 14.2 -> 12.6 ms.
// BOUNDS: sums of different pairs have no common scale, but a query's bound on the float distance is a bound on each pair's
// sums (quick_sum_cap), so the lists scanned first cut down what the later ones count, save, collect and rerank: most lists
// then hold fewer than kprime codes that matter, and the whole prefix of sums up to the bound is kept, which is what makes
// the candidates of a pair those of the definition as far as the result can see them.  Both scans 12.4 -> 9.9 ms.
// Once a segment of an item saves less than a quarter of its rows, the next ones run on byte-wide lower bounds of the sums
// (build_lb), 16 8-byte LDS reads and 16 three-operand additions per code and eight pairs instead of twice that, and only rows that pass get their
// sums; with the next codes requested ahead and four waves per SIMD (128 registers, the cold parts spill) the long items take 5.1 -> 3.4 ms, call 13.5 ->
// 12.4.  Vector units busy 78 % of the cycles in the kernel of the long items, LDS 39 %; 59 and
// 34 % in that of the short ones (107 000 items, 5.2 ms by themselves: neither is full, what its waves wait for is not measured).
template <int QK_WAVES, bool LONG, bool BOUNDS>
__global__ __launch_bounds__(QK_WAVES * 64, LONG && !BOUNDS ? 2 : 4) void ivf_quick_scan_kernel(const uint8_t *__restrict__ codes,
                                                                       const uint8_t *__restrict__ qluts,
                                                                       const IvfItem *__restrict__ items,
                                                                       uint32_t *nitems_dev,
                                                                       const int32_t *__restrict__ pairs_by_list,
                                                                       const uint32_t *__restrict__ pair_out, int kprime,
                                                                       uint64_t *partial, uint32_t *saved_rows, int saved_cap,
                                                                       const float *__restrict__ luts, int nprobe, int topk,
                                                                       unsigned long long *tau_key, QuickBound qb) {
    constexpr int QK_THREADS = QK_WAVES * 64;
    extern __shared__ __align__(QK_SMEM_ALIGN) unsigned char quick_smem[];
    typedef typename std::conditional<LONG, uint32_t, uint16_t>::type TieRow;
    QuickSmem<QK_WAVES, TieRow> &sm = *reinterpret_cast<QuickSmem<QK_WAVES, TieRow> *>(quick_smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int first_item = LONG ? 0 : (int)nitems_dev[2], nitems = LONG ? (int)nitems_dev[2] : (int)nitems_dev[0];
    const bool share = BOUNDS && nitems - first_item > (int)gridDim.x;   // (items of one round all begin without bounds)
    uint32_t *const work_counter = nitems_dev + (LONG ? 4 : 5);
    // rows of the item that the counting pass found at or below some pair's cap of the moment, per wave in the order
    // the wave met them (ascending): the only rows the collecting pass has to look at again
    uint32_t *my_saved = saved_rows + ((size_t)blockIdx.x * QK_WAVES + wave) * (size_t)saved_cap;
    for (;;) {
        __syncthreads();   // the item before is done with the shared state
        if (tid == 0) sm.item = first_item + (int)atomicAdd(work_counter, 1u);
        __syncthreads();
        const int item = sm.item;
        if (item >= nitems) break;
        const IvfItem it = items[item];
        const int skip = (int)(it.skip_slots_chunk & 127u);
        const int nslots = (int)((it.skip_slots_chunk >> 8) & 255u);
        const uint32_t chunk = it.skip_slots_chunk >> 16;
        const int ncodes = (int)it.ncodes;            // rows from code_begin; the first `skip` belong to the list before
        const int nvalid = ncodes - skip;
        const uint32_t row0 = it.code_begin;
        const uint8_t *base_ptr = codes + (size_t)row0 * 8;
        if (tid == 0) sm.single = (it.skip_slots_chunk & 128u) != 0u ? 0 : 1;
        if (tid < QK_QS) {
            const int pair = tid < nslots ? pairs_by_list[it.pair_pos + tid] : -1;
            sm.pair[tid] = pair;
            sm.out_idx[tid] = pair >= 0 ? pair_out[pair] + chunk : 0u;
            sm.sure_cnt[tid] = 0;
            sm.below[tid] = 0u;
            sm.base[tid] = 0u;
            sm.counted[tid] = 0;
            if constexpr (!BOUNDS) {
                sm.alive[tid] = tid < nslots;
                sm.tcap[tid] = QK_NO_CAP;
                sm.tstar[tid] = 0xffffu;
                sm.found[tid] = (tid >= nslots || nvalid <= kprime) ? 1 : 0;
            }
        }
        __syncthreads();
        // (what the query's bound says of the pair: requested by the last wave, beside the tables)
        float cap_min = 0.f, cap_scale = 0.f, cap_inv = 0.f;
        unsigned long long cap_tau = 0ull;
        const int cap_slot = tid - (QK_THREADS - 64);
        const int cap_pair = cap_slot >= 0 && cap_slot < nslots ? sm.pair[cap_slot] : -1;
        if (BOUNDS && cap_pair >= 0) {
            cap_tau = __hip_atomic_load(tau_key + cap_pair / nprobe, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            cap_min = qb.qmin[cap_pair]; cap_scale = qb.scale[cap_pair]; cap_inv = qb.dist_inv[cap_pair / nprobe];
        }
        // ---- the 8-bit tables of the item's pairs, widened to 16 bits, pair s in half s of the slot
        if (tid < 256) {
            uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int s = 0; s < QK_QS; ++s) {
                const int pair = sm.pair[s];
                const uint32_t e = pair >= 0 ? (uint32_t)qluts[(size_t)pair * 256 + tid] : 0u;
                w[s >> 1] |= e << (16 * (s & 1));
            }
            sm.tab[tid] = make_uint4(w[0], w[1], w[2], w[3]);
        }
        if (BOUNDS && cap_slot >= 0 && cap_slot < QK_QS) {
            const int tcap = cap_pair >= 0 ? quick_sum_cap(cap_tau, cap_min, cap_scale) : -1;
            sm.tau[cap_slot] = cap_tau; sm.qmin[cap_slot] = cap_min; sm.scale[cap_slot] = cap_scale; sm.dinv[cap_slot] = cap_inv;
            sm.tcap[cap_slot] = tcap;
            sm.alive[cap_slot] = tcap >= 0;
            sm.tstar[cap_slot] = tcap == QK_NO_CAP ? 0xffffu : tcap < 0 ? 0u : (uint32_t)tcap;
            sm.found[cap_slot] = (tcap < 0 || nvalid <= kprime) ? 1 : 0;
        }
        if constexpr (!BOUNDS) {
            __syncthreads();
        } else if (__syncthreads_or(cap_slot >= 0 && cap_slot < QK_QS && sm.tcap[cap_slot] >= 0) == 0) {   // no code of the list can be in a result
            for (int e = tid; e < nslots * QK_KP; e += QK_THREADS) partial[(size_t)sm.out_idx[e / QK_KP] * QK_KP + e % QK_KP] = KEY_EMPTY;
            continue;
        }

        // sums of one code for the eight pairs: four registers of two 16-bit sums
        uint32_t tab_lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)sm.tab;   // LDS address of the tables
        asm volatile("" : "+v"(tab_lds));
        // Returns, per lane, whether some pair's sum is below its limit (`limit` holds the limits per 16-bit half; 0:
        // nothing passes).
        auto sums_below = [&](const uint2 c, bool valid, const uint32_t (&limit)[4], uint32_t (&acc)[4]) {
            acc[0] = acc[1] = acc[2] = acc[3] = 0u;
            // byte b of lo4 / hi4: index 2 b / 2 b + 1 of the code times 16, the offset of its slot within a sub-quantizer's 256 bytes
            uint32_t lo4[2] = {(c.x << 4) & 0xf0f0f0f0u, (c.y << 4) & 0xf0f0f0f0u};
            uint32_t hi4[2] = {c.x & 0xf0f0f0f0u, c.y & 0xf0f0f0f0u};
            // (kept as they are: the compiler would otherwise go back to a shift, a mask and an addition per entry)
            asm volatile("" : "+v"(lo4[0]), "+v"(lo4[1]), "+v"(hi4[0]), "+v"(hi4[1]));
            auto entry = [&](int j) {
                const uint32_t word = (j & 1) ? hi4[j >> 3] : lo4[j >> 3];
                const uint32_t addr = tab_lds | ((word >> (8 * ((j >> 1) & 3))) & 0xffu);   // (the tables start on a 256-byte boundary)
                return *(const __attribute__((address_space(3))) u32x4 *)(uintptr_t)(addr + (uint32_t)j * 256u);
            };
            // two 16-bit sums per register, added as 32-bit words (no half ever carries: a sum is at most 16 * 255), two
            // entries per three-operand addition
#pragma unroll
            for (int j = 0; j < 16; j += 2) {
                const u32x4 e0 = entry(j), e1 = entry(j + 1);
                acc[0] = acc[0] + e0.x + e1.x; acc[1] = acc[1] + e0.y + e1.y;
                acc[2] = acc[2] + e0.z + e1.z; acc[3] = acc[3] + e0.w + e1.w;
            }
            const uint32_t any = pk_sub_sat_u16(limit[0], acc[0]) | pk_sub_sat_u16(limit[1], acc[1]) |
                                 pk_sub_sat_u16(limit[2], acc[2]) | pk_sub_sat_u16(limit[3], acc[3]);
            return valid && any != 0u;
        };
        // f(row index within the item, code) for every code of the item; a thread meets its rows in ascending order,
        // and so does a wave (lane by lane within a step, step by step).  Long items with bounds request the next batch before the
        // current one is looked at; the short ones have no registers to spare for it (billion codes, call 12.5 ms; with it 13.0).
        constexpr bool AHEAD = LONG && BOUNDS;
        auto for_batches = [&](int begin, int end, auto &&f) {   // f(row of the first code, codes)
            uint2 c[QK_BATCH], next[QK_BATCH];
            auto load = [&](int i0, uint2 (&to)[QK_BATCH]) {
#pragma unroll
                for (int u = 0; u < QK_BATCH; ++u) {
                    const int i = i0 + u * QK_THREADS;
                    to[u] = i < end ? *reinterpret_cast<const uint2 *>(base_ptr + (size_t)i * 8) : make_uint2(0u, 0u);
                }
            };
            if constexpr (AHEAD) load(begin + tid, c);
            for (int i0 = begin + tid; i0 < end; i0 += QK_BATCH * QK_THREADS) {
                if constexpr (!AHEAD) load(i0, c);
                else load(i0 + QK_BATCH * QK_THREADS, next);
                f(i0, c);
                if constexpr (AHEAD) {
#pragma unroll
                    for (int u = 0; u < QK_BATCH; ++u) c[u] = next[u];
                }
            }
        };
        auto for_codes = [&](int begin, int end, auto &&f) {
            for_batches(begin, end, [&](int i0, const uint2 (&c)[QK_BATCH]) {
#pragma unroll
                for (int u = 0; u < QK_BATCH; ++u) f(i0 + u * QK_THREADS, c[u], i0 + u * QK_THREADS < end);
            });
        };

        // Lower bounds of the sums in bytes: entry (j, i) of a pair becomes min(15, floor((entry - min_j) * f)) with f = QK_LB_RANGE /
        // (cap - sum of the minima + 1), at most 1, so that a sum at or below the cap has a bound below T = floor((cap - sum of the
        // minima) * f) + 1 <= QK_LB_RANGE + 1.  Eight pairs fill an 8-byte slot: half the LDS traffic and half the additions of the
        // exact sums.  The first eight entries (at most 120) start from 0x80 - T, so bit 7 of a byte says that they reach T alone;
        // without it the other eight are added to its low seven bits and bit 7 says that all of them do.  No byte ever carries.
        // (all threads; after a barrier that follows the last change of the caps, ends with one)
        auto build_lb = [&](const bool first_time) {
            if (tid < 256) {
                const uint4 e = sm.tab[tid];
                const uint32_t ew[4] = {e.x, e.y, e.z, e.w};
                uint32_t mw[4];
                if (first_time) {
#pragma unroll
                    for (int p = 0; p < 4; ++p) mw[p] = ew[p];
#pragma unroll
                    for (int o = 1; o < 16; o <<= 1)   // (the 16 lanes of a sub-quantizer)
#pragma unroll
                        for (int p = 0; p < 4; ++p)
                            mw[p] = __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, mw[p]), __builtin_bit_cast(u16x2, (uint32_t)__shfl_xor(mw[p], o))));
                    if ((tid & 15) == 0) sm.minw[tid >> 4] = make_uint4(mw[0], mw[1], mw[2], mw[3]);
                }
            }
            if (first_time) __syncthreads();
            if (tid < 256) {
                uint32_t off[4] = {0u, 0u, 0u, 0u};   // sums of the minima
#pragma unroll 4
                for (int j = 0; j < 16; ++j) {
                    const uint4 m = sm.minw[j];
                    off[0] += m.x; off[1] += m.y; off[2] += m.z; off[3] += m.w;
                }
                const uint4 e = sm.tab[tid], mine = sm.minw[tid >> 4];
                const uint32_t ew[4] = {e.x, e.y, e.z, e.w}, mw[4] = {mine.x, mine.y, mine.z, mine.w};
                uint32_t l[2] = {0u, 0u}, bias[2] = {0u, 0u};
#pragma unroll
                for (int s = 0; s < QK_QS; ++s) {
                    const int sh = 16 * (s & 1);
                    const int room = (int)sm.cap[s] - (int)((off[s >> 1] >> sh) & 0xffffu);
                    float f = QK_LB_RANGE / (float)(room + 1);
                    f = room >= 0 && f < 1.f ? f : 1.f;
                    const float x = (float)(((ew[s >> 1] >> sh) & 0xffffu) - ((mw[s >> 1] >> sh) & 0xffffu)) * f;
                    l[s >> 2] |= (uint32_t)fminf(x, 15.f) << (8 * (s & 3));
                    const uint32_t t = sm.found[s] == 0 && room >= 0 ? (uint32_t)((float)room * f * (1.f + 1e-5f)) + 1u : 0u;   // (0: nothing passes)
                    bias[s >> 2] |= (0x80u - t) << (8 * (s & 3));
                }
                sm.lbtab[tid] = make_uint2(l[0], l[1]);
                if (tid == 0) sm.lbbias = make_uint2(bias[0], bias[1]);
            }
            __syncthreads();
        };
        uint32_t lb_lds = (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) char *)sm.lbtab;
        asm volatile("" : "+v"(lb_lds));
        // whether some pair's bound is below its T
        auto bound_passes = [&](const uint2 c, const uint2 bias) {
            uint32_t lo8[2] = {(c.x << 3) & 0x78787878u, (c.y << 3) & 0x78787878u};
            uint32_t hi8[2] = {(c.x >> 1) & 0x78787878u, (c.y >> 1) & 0x78787878u};
            asm volatile("" : "+v"(lo8[0]), "+v"(lo8[1]), "+v"(hi8[0]), "+v"(hi8[1]));
            auto entry = [&](int j) {
                const uint32_t word = (j & 1) ? hi8[j >> 3] : lo8[j >> 3];
                const uint32_t addr = lb_lds | ((word >> (8 * ((j >> 1) & 3))) & 0xffu);   // (the tables start on a 256-byte boundary)
                return *(const __attribute__((address_space(3))) u32x2 *)(uintptr_t)(addr + (uint32_t)j * 128u);
            };
            uint32_t a0 = bias.x, a1 = bias.y, b0 = 0u, b1 = 0u;
#pragma unroll
            for (int j = 0; j < 8; j += 2) {
                const u32x2 e0 = entry(j), e1 = entry(j + 1), f0 = entry(j + 8), f1 = entry(j + 9);
                a0 = a0 + e0.x + e1.x; a1 = a1 + e0.y + e1.y;
                b0 = b0 + f0.x + f1.x; b1 = b1 + f0.y + f1.y;
            }
            const uint32_t t0 = ((a0 & 0x7f7f7f7fu) + b0) | a0, t1 = ((a1 & 0x7f7f7f7fu) + b1) | a1;
            return (t0 & t1 & 0x80808080u) != 0x80808080u;
        };

        // ---- counting passes: T of every pair.  Sums of base .. base + 510 are counted (one pass unless fewer than
        // kprime sums lie in that range: then the next 511 values are counted in another pass).  The codes are taken
        // in segments of 1024, 2048, 4096, ... rows (twice that in blocks of 8 waves); after each segment the kprime-th smallest sum so far becomes the
        // pair's cap, and greater sums are no longer counted: the final T cannot exceed it.
        int scnt = 0;            // rows saved by this wave (uniform among the lanes still in the loop; lane 0 stays longest)
        bool use_saved = nvalid > kprime;
        if (nvalid > kprime) {
            for (int attempt = 0;; ++attempt) {
                if (attempt > 0) use_saved = false;   // (rows of a second counting pass would be saved twice: all rows are looked at again)
                for (int i = tid; i < QK_QS * QK_BINS; i += QK_THREADS) (&sm.hist[0][0])[i] = 0u;
                if (tid < QK_QS) {
                    const uint32_t last = sm.base[tid] + (uint32_t)(QK_BINS - 2);
                    sm.cap[tid] = BOUNDS && sm.tcap[tid] < (int)last ? (uint32_t)sm.tcap[tid] : last;   // (a pair without a chance is not counted)
                    sm.reached[tid] = 0;
                    sm.cum_t[tid] = 0u;
                }
                if (tid == 0) { sm.pending = 0; sm.seg_saved[0] = sm.seg_saved[1] = 0u; }
                __syncthreads();
                uint32_t seg_rows = 0u;   // rows of the segment before
                int seg_nr = 0;
                bool lb_ready = false;
                uint32_t lo[QK_QS];
                bool open[QK_QS];
#pragma unroll
                for (int s = 0; s < QK_QS; ++s) { lo[s] = sm.base[s]; open[s] = sm.found[s] == 0; }
                for (int seg_begin = skip, seg_len = QK_BATCH * QK_THREADS; seg_begin < ncodes; seg_len *= 2) {
                    const int seg_end = ncodes - seg_begin < seg_len ? ncodes : seg_begin + seg_len;
                    uint32_t capv[QK_QS], capplus[4] = {0u, 0u, 0u, 0u};   // cap + 1 per pair (0: pair not counted)
#pragma unroll
                    for (int s = 0; s < QK_QS; ++s) {
                        capv[s] = sm.cap[s];
                        if (open[s]) capplus[s >> 1] |= (capv[s] + 1u) << (16 * (s & 1));
                    }
                    if constexpr (BOUNDS) scnt = __builtin_amdgcn_readfirstlane(scnt);
                    const int scnt0 = scnt;
                    auto save = [&](int i, bool pass) {
                        const uint64_t mask = __ballot(pass);
                        if (mask == 0ull) return;
                        const int pos = scnt + mask_prefix(mask);
                        if (pass && pos < saved_cap) my_saved[pos] = (uint32_t)i;
                        scnt += __popcll(mask);
                    };
                    auto count = [&](const uint32_t (&acc)[4]) {
#pragma unroll
                        for (int s = 0; s < QK_QS; ++s) {
                            const uint32_t sum = (acc[s >> 1] >> (16 * (s & 1))) & 0xffffu;
                            if (open[s] && sum >= lo[s] && sum <= capv[s]) atomicAdd(&sm.hist[s][sum - lo[s]], 1u);
                        }
                    };
                    // Where the segment before saved few of its rows, this one is scanned by the lower bounds, and only the rows they
                    // let through get their sums, 64 at a time.
                    const bool by_bounds = BOUNDS && attempt == 0 && seg_nr > 0 && seg_end - seg_begin >= QK_THREADS * 2 &&
                                           sm.seg_saved[(seg_nr - 1) & 1] * 4u < seg_rows;   // (uniform: read behind the barriers of the segment before)
                    if (BOUNDS && by_bounds) {
                        build_lb(!lb_ready);
                        lb_ready = true;
                        const uint2 bias = sm.lbbias;
                        // (the bounds of a batch before any of them is looked at: their LDS reads overlap)
                        for_batches(seg_begin, seg_end, [&](int i0, const uint2 (&c)[QK_BATCH]) {
                            bool pass[QK_BATCH], some = false;
#pragma unroll
                            for (int u = 0; u < QK_BATCH; ++u) {
                                pass[u] = bound_passes(c[u], bias) & (i0 + u * QK_THREADS < seg_end);
                                some |= pass[u];
                            }
                            if (__ballot(some) == 0ull) return;
#pragma unroll
                            for (int u = 0; u < QK_BATCH; ++u) save(i0 + u * QK_THREADS, pass[u]);
                        });
                        scnt = __builtin_amdgcn_readfirstlane(scnt);
                        list_fence();   // (the rows were stored by other lanes)
                        const int have = scnt < saved_cap ? scnt : saved_cap;
                        for (int e0 = scnt0 + lane; e0 < have; e0 += QK_BATCH * 64) {
                            uint32_t r[QK_BATCH];
                            uint2 c[QK_BATCH];
#pragma unroll
                            for (int u = 0; u < QK_BATCH; ++u) r[u] = e0 + u * 64 < have ? my_saved[e0 + u * 64] : (uint32_t)skip;
#pragma unroll
                            for (int u = 0; u < QK_BATCH; ++u) c[u] = *reinterpret_cast<const uint2 *>(base_ptr + (size_t)r[u] * 8);
#pragma unroll
                            for (int u = 0; u < QK_BATCH; ++u) {
                                uint32_t acc[4];
                                if (sums_below(c[u], e0 + u * 64 < have, capplus, acc)) count(acc);
                            }
                        }
                    } else {
                        for_codes(seg_begin, seg_end, [&](int i, const uint2 c, bool valid) {
                            uint32_t acc[4];
                            const bool pass = sums_below(c, valid, capplus, acc);
                            if (__ballot(pass) == 0ull) return;
                            save(i, pass);
                            if (pass) count(acc);
                        });
                    }
                    if (BOUNDS && lane == 0) atomicAdd(&sm.seg_saved[seg_nr & 1], (uint32_t)(scnt - scnt0));
                    seg_rows = (uint32_t)(seg_end - seg_begin);
                    __syncthreads();
                    if (BOUNDS && tid == 0) sm.seg_saved[(seg_nr + 1) & 1] = 0u;   // (read above, and next added to behind the barriers below)
                    ++seg_nr;
                    const bool refresh = share && seg_len >= 8 * QK_BATCH * QK_THREADS;
                    // a wave reads the bins of a pair: lane l owns bins 8 l .. 8 l + 7 (the last bin stays empty)
                    for (int s = wave; s < QK_QS; s += QK_WAVES) {
                        if (sm.found[s]) continue;   // (uniform)
                        // (the bound falls while other lists of the query are scanned)
                        unsigned long long tau_now = KEY_EMPTY;
                        if (refresh) tau_now = __hip_atomic_load(tau_key + sm.pair[s] / nprobe, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        uint32_t b8[8], tot = 0u;
#pragma unroll
                        for (int t = 0; t < 8; ++t) { b8[t] = sm.hist[s][lane * 8 + t]; tot += b8[t]; }
                        uint32_t incl = tot;
#pragma unroll
                        for (int o = 1; o < 64; o <<= 1) {
                            const uint32_t up = __shfl_up(incl, o);
                            if (lane >= o) incl += up;
                        }
                        const uint32_t want = (uint32_t)kprime - sm.below[s];
                        const uint64_t reach = __ballot(incl >= want);
                        if (reach != 0ull) {
                            if (lane == __builtin_ctzll(reach)) {
                                uint32_t cum = incl - tot;
                                int t = 0;
                                while (cum + b8[t] < want) { cum += b8[t]; ++t; }   // (ends within the lane's bins)
                                sm.cap[s] = sm.base[s] + (uint32_t)(lane * 8 + t);   // the kprime-th smallest sum so far
                                sm.cum_t[s] = cum;                                    // sums below it, from base on
                                sm.reached[s] = 1;
                            }
                        } else if (lane == 63) {
                            sm.cum_t[s] = incl;   // all sums counted so far
                        }
                        if (refresh && lane == 0) sm.tcap[s] = quick_sum_cap(tau_now, sm.qmin[s], sm.scale[s]);
                    }
                    __syncthreads();
                    if constexpr (BOUNDS) {
                        if (tid < QK_QS && sm.found[tid] == 0 && sm.tcap[tid] < (int)sm.cap[tid]) sm.cap[tid] = sm.tcap[tid] < 0 ? 0u : (uint32_t)sm.tcap[tid];
                        __syncthreads();
                    }
                    seg_begin = seg_end;
                }
                if (tid < QK_QS && sm.found[tid] == 0) {
                    if (BOUNDS && (sm.tcap[tid] < 0 || (uint32_t)sm.tcap[tid] <= sm.cap[tid])) {   // every sum the bound leaves is counted: fewer than kprime, or as many with ties
                        sm.tstar[tid] = sm.cap[tid];
                        sm.found[tid] = 1;
                    } else if (sm.reached[tid]) {
                        sm.below[tid] += sm.cum_t[tid];
                        sm.tstar[tid] = sm.cap[tid];
                        sm.found[tid] = 1;
                    } else {
                        sm.below[tid] += sm.cum_t[tid];   // fewer than kprime sums up to base + 510: count the next 511 values
                        sm.base[tid] += (uint32_t)(QK_BINS - 1);
                        atomicAdd(&sm.pending, 1);
                    }
                }
                __syncthreads();
                if (sm.pending == 0) break;
                __syncthreads();   // (pending is cleared by thread 0 at the top of the next pass)
            }
        }

        // ---- collecting pass: keys below T, and the rows at T in ascending order per wave
        {
            uint32_t tplus[4] = {0u, 0u, 0u, 0u};   // T + 1 per pair (0 for empty slots: nothing passes)
            uint32_t tval[QK_QS];
            int need[QK_QS], tcnt[QK_QS];
            bool alive[QK_QS];
#pragma unroll
            for (int s = 0; s < QK_QS; ++s) {
                tval[s] = sm.tstar[s];
                alive[s] = BOUNDS ? sm.alive[s] != 0 : s < nslots;
                const uint32_t tp = alive[s] ? (tval[s] < 0xffffu ? tval[s] + 1u : 0xffffu) : 0u;
                tplus[s >> 1] |= tp << (16 * (s & 1));
                // rows at T that can still be candidates: kprime less the sums below T (none when every code is taken)
                need[s] = (alive[s] && tval[s] < 0xffffu) ? kprime - (int)sm.below[s] : 0;
                tcnt[s] = 0;
            }
            scnt = __builtin_amdgcn_readfirstlane(scnt);
            if (scnt > saved_cap) use_saved = false;   // (cannot happen: a wave saves at most the rows it meets)
            use_saved = __syncthreads_or(use_saved ? 0 : 1) == 0;   // (the same decision in every wave)
            // f(row, code, valid) for the rows to look at: the wave's saved rows in their order, or every row of the item
            auto for_rows = [&](auto &&f) {
                if (!use_saved) { for_codes(skip, ncodes, f); return; }
                for (int e0 = lane; e0 < scnt; e0 += QK_BATCH * 64) {
                    uint32_t r[QK_BATCH];
                    uint2 c[QK_BATCH];
#pragma unroll
                    for (int u = 0; u < QK_BATCH; ++u) r[u] = e0 + u * 64 < scnt ? my_saved[e0 + u * 64] : 0u;
#pragma unroll
                    for (int u = 0; u < QK_BATCH; ++u)
                        c[u] = e0 + u * 64 < scnt ? *reinterpret_cast<const uint2 *>(base_ptr + (size_t)r[u] * 8) : make_uint2(0u, 0u);
#pragma unroll
                    for (int u = 0; u < QK_BATCH; ++u) f((int)r[u], c[u], e0 + u * 64 < scnt);
                }
            };
            for_rows([&](int i, const uint2 c, bool valid) {
                uint32_t acc[4];
                const bool some = sums_below(c, valid, tplus, acc);
                if (__ballot(some) == 0ull) return;
#pragma unroll
                for (int s = 0; s < QK_QS; ++s) {
                    const uint32_t sum = (acc[s >> 1] >> (16 * (s & 1))) & 0xffffu;
                    const bool in = valid && alive[s];
                    if (in && sum < tval[s]) {
                        const int at = atomicAdd(&sm.sure_cnt[s], 1);   // (fewer than kprime such codes exist)
                        sm.sure[s][at] = ((unsigned long long)sum << 32) | (row0 + (uint32_t)i);
                    }
                    const bool at_t = in && sum == tval[s] && tval[s] < 0xffffu;
                    const uint64_t mask = __ballot(at_t);
                    if (mask != 0ull) {
                        const int pos = tcnt[s] + mask_prefix(mask);
                        if (at_t && pos < need[s]) sm.tie[wave][s][pos] = (TieRow)i;
                        tcnt[s] += __popcll(mask);
                        if (tcnt[s] > need[s]) tcnt[s] = need[s];   // (later rows of this wave are greater: not needed)
                    }
                }
            });
            if (lane == 0) {
#pragma unroll
                for (int s = 0; s < QK_QS; ++s) sm.tie_cnt[wave][s] = tcnt[s];
            }
        }
        __syncthreads();

        // ---- result lists: the keys below T, then the smallest rows at T up to kprime keys, then empty slots; put
        // together in LDS (the list of keys below T has room for kprime keys), then written out
        for (int e = tid; e < QK_QS * QK_KP; e += QK_THREADS) {
            const int s = e / QK_KP, idx = e % QK_KP;
            if (idx >= sm.sure_cnt[s]) sm.sure[s][idx] = KEY_EMPTY;
        }
        __syncthreads();
        for (int s = 0; s < nslots; ++s) {
            const int c = sm.sure_cnt[s];
            const uint32_t t = sm.tstar[s];
            const int need = t < 0xffffu ? kprime - c : 0;
            if (need <= 0) continue;
            // entry e of wave w's list: its rank among the rows at T of all waves (rows are distinct)
            for (int e = tid; e < QK_WAVES * QK_KP; e += QK_THREADS) {
                const int w = e / QK_KP, idx = e % QK_KP;
                if (idx >= sm.tie_cnt[w][s]) continue;
                const uint32_t row = (uint32_t)sm.tie[w][s][idx];
                int rank = idx;
#pragma unroll
                for (int w2 = 0; w2 < QK_WAVES; ++w2) {
                    if (w2 == w) continue;
                    int lo = 0, hi = sm.tie_cnt[w2][s];   // rows of w2 below `row`
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if ((uint32_t)sm.tie[w2][s][mid] < row) lo = mid + 1; else hi = mid;
                    }
                    rank += lo;
                }
                if (rank < need) sm.sure[s][c + rank] = ((unsigned long long)t << 32) | (row0 + row);
            }
        }
        __syncthreads();
        if (sm.single) {
            // float distances in place of the integer keys; the pairs' float tables take the memory of the bins
            float *const tabf = reinterpret_cast<float *>(&sm.hist[0][0]);
            static_assert(sizeof(sm.hist) >= QK_QS * 256 * sizeof(float), "the bins' memory holds the float tables");
            for (int e = tid; e < nslots * 256; e += QK_THREADS) {
                if (!BOUNDS || sm.sure[e >> 8][0] != KEY_EMPTY) tabf[e] = luts[(size_t)sm.pair[e >> 8] * 256 + (e & 255)];   // (no candidates: no tables)
            }
            __syncthreads();
            for (int e = tid; e < nslots * QK_KP; e += QK_THREADS) {
                const int s = e / QK_KP, idx = e % QK_KP;
                const unsigned long long key = sm.sure[s][idx];
                if (key == KEY_EMPTY) continue;
                const uint32_t row = (uint32_t)key;
                const uint2 c = *reinterpret_cast<const uint2 *>(codes + (size_t)row * 8);
                const float dist = adc16x4_exact(tabf + s * 256, c);
                const unsigned long long fkey = ((unsigned long long)f32_to_ord(dist) << 32) | row;
                sm.sure[s][idx] = fkey;
                if (share && fkey <= sm.tau[s] && sm.dinv[s] > 0.f) {   // (a key above the bound says nothing new)
                    const float at = dist * sm.dinv[s];
                    if (at >= 0.f && at < (float)QK_DBINS) {
                        atomicAdd(&qb.dist_bins[(size_t)(sm.pair[s] / nprobe) * QK_DBINS + (int)at], 1u);
                        sm.counted[s] = 1;
                    }
                }
            }
            __syncthreads();
            // two bounds of the query's result: the pair's topk-th key, and the bin edge at or below which topk candidates of all
            // the query's lists so far lie
            for (int s = wave; s < nslots; s += QK_WAVES) {
                if (sm.sure[s][BOUNDS ? 0 : topk - 1] == KEY_EMPTY) continue;   // (keys first, empty slots behind)
                const int q = sm.pair[s] / nprobe;
                const unsigned long long before = BOUNDS ? sm.tau[s] : KEY_EMPTY;
                unsigned long long bound = before;
                if (sm.sure[s][topk - 1] != KEY_EMPTY) {
                    const uint64_t two[2] = {sm.sure[s][lane], sm.sure[s][64 + lane]};
                    const uint64_t kth = wave_select_kth<2>(two, topk);
                    if (kth < bound) bound = kth;
                }
                if (BOUNDS && sm.counted[s]) {
                    uint32_t b4[4], tot = 0u;
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        b4[t] = __hip_atomic_load(qb.dist_bins + (size_t)q * QK_DBINS + lane * 4 + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        tot += b4[t];
                    }
                    uint32_t incl = tot;
#pragma unroll
                    for (int o = 1; o < 64; o <<= 1) {
                        const uint32_t up = __shfl_up(incl, o);
                        if (lane >= o) incl += up;
                    }
                    const uint64_t reach = __ballot(incl >= (uint32_t)topk);
                    if (reach != 0ull) {
                        const int first = __builtin_ctzll(reach);
                        int bin = lane * 4;
                        uint32_t cum = incl - tot;
#pragma unroll
                        for (int t = 0; t < 3; ++t) if (cum + b4[t] < (uint32_t)topk) { cum += b4[t]; ++bin; } else break;
                        bin = __builtin_amdgcn_readlane(bin, first);
                        // (dist * dinv < bin + 1 in fp32, so dist is below this edge)
                        const float edge = (float)(bin + 1) / sm.dinv[s] * (1.f + 1e-6f);
                        const unsigned long long key = ((unsigned long long)f32_to_ord(edge) << 32) | 0xffffffffull;
                        if (key < bound) bound = key;
                    }
                }
                if (lane == 0 && bound < before) atomicMin(&tau_key[q], bound);
            }
        }
        for (int e = tid; e < nslots * QK_KP; e += QK_THREADS) {
            const int s = e / QK_KP, idx = e % QK_KP;
            partial[(size_t)sm.out_idx[s] * QK_KP + idx] = sm.sure[s][idx];
        }
    }
}

// ------------------------------------------------------------------------------------------
// Rerank of the pairs whose list is cut into several chunks (the scan has seen to the others).  The kprime smallest integer
// keys over the pair's result lists (one per chunk, any number of them) are its candidates; their float distances replace
// them in the pair's first list, the other lists are emptied, and the pair's topk-th key (if it has one) bounds the query's
// result.  A block looks 256 pairs over for such ones, and takes in seven of a pair's lists at a time (128 threads and one
// list at a time: 82 sorts one after the other for the longest list of a billion codes, 0.45 ms).
constexpr int QK_RR_THREADS = 1024, QK_RR_PAIRS = 256, QK_RR_LISTS = QK_RR_THREADS / QK_KP - 1;
__global__ __launch_bounds__(QK_RR_THREADS) void ivf_quick_rerank_kernel(const uint8_t *__restrict__ codes, const float *__restrict__ luts,
                                                               const int32_t *__restrict__ probes, const uint32_t *__restrict__ nc_arr,
                                                               const uint32_t *__restrict__ pair_out, int npairs, int nprobe, int kprime,
                                                               int topk, uint64_t *partial, unsigned long long *tau_key, QuickBound qb) {
    __shared__ float tab[256];
    __shared__ uint64_t keys[QK_RR_THREADS];
    __shared__ int todo[QK_RR_PAIRS], ntodo;
    const int tid = threadIdx.x;
    if (tid == 0) ntodo = 0;
    __syncthreads();
    {
        const int pair = (int)blockIdx.x * QK_RR_PAIRS + tid;
        if (tid < QK_RR_PAIRS && pair < npairs && nc_arr[probes[pair]] > 1u) todo[atomicAdd(&ntodo, 1)] = pair;
    }
    __syncthreads();
    for (int i = 0; i < ntodo; ++i) {
        const int pair = todo[i], nc = (int)nc_arr[probes[pair]];
        uint64_t *lists = partial + (size_t)pair_out[pair] * QK_KP;
        __syncthreads();   // the pair before is done with the tables and keys
        if (tid < 256) tab[tid] = luts[(size_t)pair * 256 + tid];
        // the smallest keys so far in keys[0 .. 127], the next chunks' lists sorted in beside them
        if (tid < QK_KP) keys[tid] = lists[tid];
        for (int c = 1; c < nc; c += QK_RR_LISTS) {
            const size_t at = (size_t)c * QK_KP + (size_t)(tid - QK_KP);
            if (tid >= QK_KP) keys[tid] = at < (size_t)nc * QK_KP ? lists[at] : KEY_EMPTY;
            block_bitonic_sort(keys, QK_RR_THREADS);
        }
        // Chunks scanned under different bounds left out different sums; below the bound of now none did, and there the smallest
        // keys are those of the whole list.
        const int tcap = qb.qmin ? quick_sum_cap(__hip_atomic_load(tau_key + pair / nprobe, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT), qb.qmin[pair], qb.scale[pair])
                                 : QK_NO_CAP;
        uint64_t key = tid < kprime ? keys[tid] : KEY_EMPTY;
        if (tcap != QK_NO_CAP && (int64_t)(key >> 32) > (int64_t)tcap) key = KEY_EMPTY;
        __syncthreads();
        uint64_t fkey = KEY_EMPTY;
        if (key != KEY_EMPTY) {
            const uint32_t row = (uint32_t)key;
            const uint2 c = *reinterpret_cast<const uint2 *>(codes + (size_t)row * 8);
            fkey = ((uint64_t)f32_to_ord(adc16x4_exact(tab, c)) << 32) | row;
        }
        if (tid < QK_KP) keys[tid] = fkey;
        block_bitonic_sort(keys, QK_KP);
        if (tid < QK_KP) lists[tid] = keys[tid];
        for (size_t e = QK_KP + tid; e < (size_t)nc * QK_KP; e += QK_RR_THREADS) lists[e] = KEY_EMPTY;
        if (tid == 0 && keys[topk - 1] != KEY_EMPTY) atomicMin(&tau_key[pair / nprobe], (unsigned long long)keys[topk - 1]);
    }
}

// ------------------------------------------------------------------------------------------
// Rows a wave can meet in a work item of at most `rows` rows (+ the rows of alignment in front) scanned by `waves` waves.
static int ivf_quick_saved_cap(int64_t rows, int waves) { return (int)(((rows + 16) / (waves * 64) + 2) * 64); }

size_t ivf_quick_saved_bytes(const pq_ctx *ctx, int64_t max_item_rows) {
    return ((size_t)ctx->num_cu * 2 * 8 * ivf_quick_saved_cap(max_item_rows, 8) + (size_t)ctx->num_cu * 4 * 4 * ivf_quick_saved_cap(QK_LONG_MIN, 4)) * 4;
}

int launch_ivf_quick(pq_ctx *ctx, const uint8_t *codes, const int64_t *list_offsets, const int32_t *probes,
                     const float *luts, int nq, int nprobe, int init, int kprime, int topk, float *qmax_pair,
                     uint8_t *qluts, const IvfItem *items, uint32_t *nitems_dev, const int32_t *pairs_by_list,
                     const uint32_t *pair_out, const uint32_t *nc_arr, uint64_t *partial, unsigned long long *tau_key,
                     uint32_t *dist_bins, float *dist_inv, float *qmin, float *scale, uint32_t *saved_rows, int64_t max_item_rows, size_t most_items, bool two_streams, bool bounds) {
    if (kprime < 1 || kprime > QK_KP || topk < 1 || topk > QK_KP || init < 1 || init > QK_INIT_MAX)
        return fail(ctx, PQ_EUNSUPPORTED, "ivf quick adc: kprime and topk must be 1..%d, init 1..%d", QK_KP, QK_INIT_MAX);
    hipStream_t s = ctx->stream;
    const int npairs = nq * nprobe;
    ivf_quick_qmax_kernel<<<nq, 256, 0, s>>>(codes, list_offsets, probes, luts, nprobe, init, topk, qmax_pair, tau_key, bounds ? dist_bins : nullptr, dist_inv);
    PQ_HIP(ctx, hipGetLastError());
    const QuickBound qb = {bounds ? qmin : nullptr, bounds ? scale : nullptr, dist_bins, dist_inv};
    int rc = launch_quantize_luts(ctx, luts, npairs, 16, 16, qmax_pair, qluts, bounds ? qmin : nullptr, bounds ? scale : nullptr, bounds);
    if (rc) return rc;
    if (ctx->profiling) {
        PQ_HIP(ctx, hipEventRecord(ctx->ev_begin, s));
        snprintf(ctx->last_scan_name, sizeof(ctx->last_scan_name),
                 "ivf_quick_scan_kernel (16x4 codes, 8-bit tables of 8 (query, list) pairs per work item; blocks of 8 waves for lists of %d rows and more, of 4 waves for the others)", QK_LONG_MIN);
        ctx->last_scan_qpp = QK_QS;
        ctx->last_scan_passes = 2;
        ctx->stat_parked = nullptr;
        ctx->stat_ncand = nullptr;
        ctx->stat_ncand_len = 0;
        ctx->stat_onehot = nullptr;
    }
    {
        auto long_kernel = bounds ? ivf_quick_scan_kernel<8, true, true> : ivf_quick_scan_kernel<8, true, false>;
        auto short_kernel = bounds ? ivf_quick_scan_kernel<4, false, true> : ivf_quick_scan_kernel<4, false, false>;
        PQ_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(long_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)sizeof(QuickSmemLong)));
        PQ_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(short_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)sizeof(QuickSmemShort)));
        // the long items first, the many short ones beside them on the context's second stream (calls of few pairs: behind them)
        const int cap_long = ivf_quick_saved_cap(max_item_rows, 8), cap_short = ivf_quick_saved_cap(QK_LONG_MIN, 4);
        hipStream_t s2 = two_streams ? ctx->aux_stream : s;
        if (two_streams) PQ_HIP(ctx, hipEventRecord(ctx->aux_fork, s));
        // (no more blocks than there can be items: each draws from the counter, one after the other)
        auto blocks = [&](int full) { return (unsigned)(most_items < (size_t)full ? most_items : (size_t)full); };
        long_kernel<<<blocks(ctx->num_cu * 2), 8 * 64, sizeof(QuickSmemLong), s>>>(codes, qluts, items, nitems_dev, pairs_by_list, pair_out,
                                                                       kprime, partial, saved_rows, cap_long, luts, nprobe, topk, tau_key, qb);
        PQ_HIP(ctx, hipGetLastError());
        if (two_streams) PQ_HIP(ctx, hipStreamWaitEvent(s2, ctx->aux_fork, 0));
        short_kernel<<<blocks(ctx->num_cu * 4), 4 * 64, sizeof(QuickSmemShort), s2>>>(codes, qluts, items, nitems_dev, pairs_by_list, pair_out,
                                                                          kprime, partial,
                                                                          saved_rows + (size_t)ctx->num_cu * 2 * 8 * cap_long, cap_short, luts, nprobe, topk, tau_key, qb);
        PQ_HIP(ctx, hipGetLastError());
        if (two_streams) {
            PQ_HIP(ctx, hipEventRecord(ctx->aux_join, s2));
            PQ_HIP(ctx, hipStreamWaitEvent(s, ctx->aux_join, 0));
        }
    }
    if (ctx->profiling) {
        PQ_HIP(ctx, hipEventRecord(ctx->ev_end, s));
        ctx->ev_valid = 1;
    }
    ivf_quick_rerank_kernel<<<(npairs + QK_RR_PAIRS - 1) / QK_RR_PAIRS, QK_RR_THREADS, 0, s>>>(codes, luts, probes, nc_arr, pair_out, npairs, nprobe, kprime, topk, partial, tau_key, qb);
    PQ_HIP(ctx, hipGetLastError());
    return PQ_OK;
}

}  // namespace pq
