// Search with derived quantizers (chapter 6; Section 6.2.3, Alg. 5) for 64-bit codes of four
// 16-bit indexes whose low 8 bits name the centroid of the derived 8-bit quantizer (property P1
// of Section 6.2.2).
//
//   Step 1.1  compact tables from the derived codebooks      -> the Tables kernel (lut_kernels.hip)
//   Step 1.2  qmax = greatest compact distance of the first r2 codes (derived_qmax_kernel),
//             8-bit tables                                   -> the quantiser (lut_kernels.hip)
//   Step 1.3  adc_low_bits over the whole database into buckets indexed by the integer distance
//   Step 2    precise distances from the full codebooks for the vectors of the buckets taken in
//             increasing order until r2 vectors are in (the bucket of the r2-th is finished)
//
// Capped buckets on a GPU.  The thesis appends every vector to the list of its bucket and keeps
// an upper bound on the bucket index so that the lists stay short.  Here the lists are replaced
// by counts: a first pass over the codes counts, per query, the vectors of every bucket up to a
// bound that is lowered in the same way (the smallest bucket below which r2 counted vectors lie
// bounds the bucket of the r2-th from above, so every vector at or below the final bucket is
// always counted); the bucket b* of the r2-th vector and the exact number of vectors in the
// buckets 0..b* follow from the counts.  A second pass over the codes, with b* fixed, writes the
// ids of exactly those vectors into a list whose size is known beforehand.  Where the database is large, the first pass looks
// at a sample only (see launch_derived_search), the second lists what its bounds let through, and the counts are taken from
// the lists.  Both passes run the
// same loop: 8 queries per pass over a chunk of codes, tables in LDS as 16-bit entries (8 queries
// per 16-byte slot, the four tables stored four times in the rotated slot order of lds_walk.h,
// so every read is conflict-free), four lookups and three packed adds per code, one packed
// compare for 8 queries x 2 codes.

#include "pq_internal.h"
#include "scan_common.h"
#include "topk_device.h"
#include "lds_walk.h"

namespace pq {
namespace {

constexpr int DQ_WAVES = 16;
constexpr int DQ_THREADS = DQ_WAVES * 64;
constexpr int DQ_QB = 8;            // queries per pass
constexpr int DQ_M = 4;             // sub-quantizers (16-bit indexes per code)
constexpr int DQ_BINS = 1024;       // buckets: integer distances are at most 4 * 255
constexpr int DQ_SUB = 128;         // codes per wave sub-tile (16 bytes = two codes per lane)
constexpr uint32_t DQ_THR_MAX = 0x7fffu;   // "every sum passes" (sums stay below 1024)
constexpr int DQ_DEPTH = 4;         // sub-tiles per group of a wave
constexpr int64_t DQ_SAMPLE_PAIRS = (int64_t)5 << 24;   // (code, query) pairs from which on a sample may replace the counting pass
constexpr int DQ_RING = 64 * (DQ_DEPTH + 1);   // parked rows per wave: a group's worth behind an unflushed rest

struct DqArgs {
    const uint8_t *codes;        // [n][8]
    int64_t n, chunk_codes;
    int nchunks, ngroups, nitems, nq, r2;
    const uint8_t *qluts;        // [nq][4][256]
    uint32_t *work_counter;
    uint32_t *g_hist;            // [nq][DQ_BINS] vectors counted per bucket
    uint32_t *g_bound;           // [nq] bucket bound shared by the blocks (counting pass)
    const uint32_t *bucket;      // [nq] b* (collecting pass)
    const uint64_t *cand_off;    // [nq + 1]
    uint32_t *cand_cnt;          // [nq]
    uint64_t *cand;              // keys (integer distance << 32 | row)
    uint2 *cand_code;            // the codes at those rows (nullptr: not wanted)
};

struct __align__(16) DqSmem {
    uint4 lut[4096];                   // row b: 16 slots; slot s = table s >> 2 (four copies)
    uint32_t hist[DQ_QB][DQ_BINS];     // this block's counts of the current item
    uint32_t thr[DQ_QB];               // a vector is kept for query q if its sum is below thr[q]
    uint32_t ring[DQ_WAVES][DQ_RING];  // rows whose sums passed a threshold, waiting to be counted or listed
    int item;
};

// first bin at which the running count reaches k, and that count; DQ_BINS if it never does.
// `load(i)` returns the count of bin i.  One wave.
template <class Load>
__device__ __forceinline__ int first_bin_reaching(Load load, uint32_t k, uint32_t *count_out) {
    const int lane = lane_id();
    uint32_t carry = 0;
    for (int j = 0; j < DQ_BINS / 64; ++j) {
        uint32_t v = load(j * 64 + lane);
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t up = __shfl_up(v, o);
            if (lane >= o) v += up;
        }
        v += carry;
        const uint64_t reached = __ballot(v >= k);
        if (reached != 0ull) {
            const int first = __builtin_ctzll(reached);
            if (count_out) *count_out = __shfl(v, first);
            return j * 64 + first;
        }
        carry = __shfl(v, 63);
    }
    if (count_out) *count_out = carry;
    return DQ_BINS;
}

// Collecting passes: where the keys of a batch go.  Lane q holds the number of the batch's keys of query q of the group
// (0 for empty slots); one atomic instruction reserves their places for all queries together (one after the other, each
// with its own round trip to the counter, a batch took longer than the scan that found it: 25 M encoded codes,
// 1000 queries, 48 M keys: 6.7 -> 3.9 ms).
struct DqPlaces {
    uint64_t begin, end;   // the query's list
    uint32_t slot;         // first place reserved in it
    // (readlane returns an int: a low word from 2^31 on must not be sign-extended into the high one)
    static __device__ __forceinline__ uint64_t of_lane(uint64_t v, int lane) {
        return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((uint32_t)(v >> 32), lane) << 32 | (uint32_t)__builtin_amdgcn_readlane((uint32_t)v, lane);
    }
    __device__ __forceinline__ void list_of(const DqArgs &a, int gq) {
        begin = gq < a.nq ? a.cand_off[gq] : 0;
        end = gq < a.nq ? a.cand_off[gq + 1] : 0;
    }
    __device__ __forceinline__ void reserve(const DqArgs &a, int gq, uint32_t count) { slot = count != 0u ? atomicAdd(&a.cand_cnt[gq], count) : 0u; }
    // place `index` of query q's.  After a counting pass the list has room for exactly the vectors it counted.  Room estimated
    // from a sample may be too small: the comparison is what keeps the keys beyond it out of the next query's list, cand_cnt still
    // counts them, and derived_settle_kernel sees from that that the call has to make the two passes.
    __device__ __forceinline__ void store(const DqArgs &a, int q, bool pass, uint32_t index, uint32_t sum, uint32_t row, uint32_t w0, uint32_t w1) const {
        const uint64_t first = of_lane(begin, q) + (uint32_t)__builtin_amdgcn_readlane(slot, q);
        const uint64_t stop = of_lane(end, q);
        const uint64_t at = first + index;
        if (pass && at < stop) {
            a.cand[at] = ((uint64_t)sum << 32) | row;
            if (a.cand_code != nullptr) a.cand_code[at] = make_uint2(w0, w1);
        }
    }
};

// MODE 0: counting pass (buckets), MODE 1: collecting pass (ids of the buckets 0..b*)
template <int MODE>
__global__ __launch_bounds__(DQ_THREADS) void derived_scan_kernel(DqArgs a) {
    __shared__ DqSmem sm;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id();
    const uint32_t lane15 = (uint32_t)lane & 15u;
    // Lane l reads slot ((l & 15) + 4 s) & 15 at step s, which holds table ((l >> 2) + s) & 3;
    // rotating the code right by 2 * ((l >> 2) & 3) bytes brings that table's index byte to
    // byte 2 s.  bases[g]: slot offsets of steps 2g (byte 0) and 2g + 1 (byte 2).
    const uint32_t rot = 2u * ((lane15 >> 2) & 3u);
    uint32_t bases[2];
#pragma unroll
    for (int g = 0; g < 2; ++g)
        bases[g] = (((lane15 + 4u * (2 * g)) & 15u) << 4) | ((((lane15 + 4u * (2 * g + 1)) & 15u) << 4) << 16);
    const char *lut_bytes = reinterpret_cast<const char *>(sm.lut);

    for (;;) {
        if (threadIdx.x == 0) sm.item = (int)atomicAdd(a.work_counter, 1u);
        __syncthreads();
        const int item = sm.item;
        if (item >= a.nitems) break;
        const int group = item % a.ngroups, chunk = item / a.ngroups;
        const int64_t cbeg = (int64_t)chunk * a.chunk_codes;
        const int64_t cend = cbeg + a.chunk_codes < a.n ? cbeg + a.chunk_codes : a.n;
        const int ncodes = cend > cbeg ? (int)(cend - cbeg) : 0;

        if (threadIdx.x < DQ_QB) {
            const int gq = group * DQ_QB + threadIdx.x;
            uint32_t thr = 0;   // empty slot: nothing passes
            if (gq < a.nq) {
                const uint32_t b = MODE == 0 ? __hip_atomic_load(&a.g_bound[gq], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                             : a.bucket[gq];
                thr = b + 1u < DQ_THR_MAX ? b + 1u : DQ_THR_MAX;
            }
            sm.thr[threadIdx.x] = thr;
        }
        if (MODE == 0)
            for (int i = threadIdx.x; i < DQ_QB * DQ_BINS; i += DQ_THREADS) (&sm.hist[0][0])[i] = 0u;
        {   // tables of the group's queries: entry (byte b, table t) of all 8 queries in one slot
            const int b = threadIdx.x >> 2, t = threadIdx.x & 3;
            uint32_t v[DQ_QB];
#pragma unroll
            for (int q = 0; q < DQ_QB; ++q) {
                const int gq = group * DQ_QB + q;
                v[q] = gq < a.nq ? (uint32_t)a.qluts[((size_t)gq * DQ_M + t) * 256 + b] : 0u;
            }
            const uint4 pk = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
#pragma unroll
            for (int c = 0; c < 4; ++c) sm.lut[b * 16 + t * 4 + c] = pk;
        }
        __syncthreads();

        const uint8_t *chunk_ptr = a.codes + cbeg * 8;
        const int nfull = ncodes / DQ_SUB;                       // sub-tiles with every code present
        const int nsub = (ncodes + DQ_SUB - 1) / DQ_SUB;         // the last one may be ragged
        uint32_t tau[4];   // thresholds of the 8 queries, two per register
        auto reload_tau = [&]() {
            const uint32_t t = sm.thr[lane & (DQ_QB - 1)];
#pragma unroll
            for (int p = 0; p < 4; ++p)
                tau[p] = __builtin_amdgcn_readlane(t, 2 * p) | (__builtin_amdgcn_readlane(t, 2 * p + 1) << 16);
        };
        typedef uint32_t v4u __attribute__((ext_vector_type(4)));
        typedef const __attribute__((address_space(1))) v4u *global_v4u;
        auto load_full = [&](int t) -> uint4 {
            const v4u v = *(global_v4u)(chunk_ptr + (size_t)t * (DQ_SUB * 8) + lane * 16);
            return make_uint4(v.x, v.y, v.z, v.w);
        };
        // the two codes at rows pos, pos + 1 of the chunk (zeros for rows past its end)
        auto load_pair = [&](int pos) -> uint4 {
            uint4 c = make_uint4(0, 0, 0, 0);
            const uint8_t *p = chunk_ptr + (size_t)pos * 8;
            if (pos + 2 <= ncodes) {
                c = *reinterpret_cast<const uint4 *>(p);
            } else if (pos < ncodes) {
                const uint2 half = *reinterpret_cast<const uint2 *>(p);
                c.x = half.x; c.y = half.y;
            }
            return c;
        };

        // the eight table reads of the lane's two codes (four tables each, in the lane's rotated order)
        auto issue = [&](const uint4 c, uint4 (&v)[8]) {
            uint32_t w[4] = {c.x, c.y, c.z, c.w};
            rot8(w[0], w[1], (rot & 4u) != 0, rot & 3u);
            rot8(w[2], w[3], (rot & 4u) != 0, rot & 3u);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const uint32_t word = w[2 * h + (s >> 1)];
                    const uint32_t off = (s & 1) ? lut_offset<2>(word, bases[s >> 1]) : lut_offset<0>(word, bases[s >> 1]);
                    v[4 * h + s] = *reinterpret_cast<const uint4 *>(lut_bytes + off);
                }
            }
        };
        // integer distances of the two codes for the 8 queries, as four packed pairs per code
        auto add_up = [&](const uint4 (&v)[8], uint32_t (&d)[2][4]) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                d[h][0] = v[4 * h].x + v[4 * h + 1].x + v[4 * h + 2].x + v[4 * h + 3].x;
                d[h][1] = v[4 * h].y + v[4 * h + 1].y + v[4 * h + 2].y + v[4 * h + 3].y;
                d[h][2] = v[4 * h].z + v[4 * h + 1].z + v[4 * h + 2].z + v[4 * h + 3].z;
                d[h][3] = v[4 * h].w + v[4 * h + 1].w + v[4 * h + 2].w + v[4 * h + 3].w;
            }
        };

        // One sub-tile whose reads are on their way: sums, one packed test for 8 queries x 2 codes,
        // and the rows of the lanes with a sum below a threshold parked in the wave's ring.
        int ring_cnt = 0;
        auto finish = [&](const uint4 (&v)[8], const int sidx) {
            uint32_t d[2][4];
            add_up(v, d);
            // 16-bit fields below 0x8000: the smaller of the two sums minus the threshold wraps
            // (sets bit 15) iff one of them is below the threshold
            typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
            uint32_t below = 0;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const u16x2 mn = __builtin_elementwise_min(__builtin_bit_cast(u16x2, d[0][p]), __builtin_bit_cast(u16x2, d[1][p]));
                below |= __builtin_bit_cast(uint32_t, (u16x2)(mn - __builtin_bit_cast(u16x2, tau[p])));
            }
            const uint64_t hit = __ballot((below & 0x80008000u) != 0u);
            if (__builtin_expect(hit != 0ull, 0)) {
                if ((hit >> lane) & 1ull) sm.ring[wave][ring_cnt + mask_prefix(hit)] = (uint32_t)(sidx * DQ_SUB + lane * 2);
                ring_cnt += __popcll(hit);
            }
        };
        auto scan_sub = [&](const uint4 c, const int sidx) {
            uint4 v[8];
            issue(c, v);
            asm volatile("" : : : "memory");   // all eight reads are issued before the first add
            finish(v, sidx);
        };

        // Parked rows, 64 at a time: the sums again, the test against the thresholds of now, and
        // for every (code, query) that passes the bucket count or the list append.
        auto flush = [&](const int count) {
            reload_tau();
            DqPlaces places;
            const int my_q = lane & (DQ_QB - 1), my_gq = group * DQ_QB + my_q;
            if (MODE == 1) places.list_of(a, my_gq);
            for (int base = 0; base < count; base += 64) {
                const bool have = base + lane < count;
                const int pos = have ? (int)sm.ring[wave][base + lane] : ncodes;
                const uint4 c = load_pair(pos);
                uint32_t d[2][4];
                {
                    uint4 v[8];
                    issue(c, v);
                    add_up(v, d);
                }
                auto passes = [&](int h, int q, uint32_t &sum) {
                    sum = (d[h][q >> 1] >> (16 * (q & 1))) & 0xffffu;
                    return pos + h < ncodes && sum < ((tau[q >> 1] >> (16 * (q & 1))) & 0xffffu);
                };
                uint32_t sum;
                if (MODE == 0) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int q = 0; q < DQ_QB; ++q)
                            if (passes(h, q, sum)) atomicAdd(&sm.hist[q][sum], 1u);
                } else {
                    uint32_t mine = 0;
#pragma unroll
                    for (int q = 0; q < DQ_QB; ++q) {
                        const uint32_t keys = (uint32_t)__popcll(__ballot(passes(0, q, sum))) + (uint32_t)__popcll(__ballot(passes(1, q, sum)));
                        mine = lane == q ? keys : mine;
                    }
                    if (__ballot(mine != 0u) == 0ull) continue;
                    places.reserve(a, my_gq, mine);
#pragma unroll
                    for (int q = 0; q < DQ_QB; ++q) {
                        const bool p0 = passes(0, q, sum);
                        const uint32_t s0 = sum;
                        const bool p1 = passes(1, q, sum);
                        const uint64_t m0 = __ballot(p0), m1 = __ballot(p1);
                        if ((m0 | m1) == 0ull) continue;
                        places.store(a, q, p0, (uint32_t)mask_prefix(m0), s0, (uint32_t)(cbeg + pos), c.x, c.y);
                        places.store(a, q, p1, (uint32_t)(__popcll(m0) + mask_prefix(m1)), sum, (uint32_t)(cbeg + pos + 1), c.z, c.w);
                    }
                }
            }
        };

        // Counting pass: the bound of a query is lowered from the block's own counts while the item
        // runs (waves 0..7, one query each), early and then every 16 groups.
        auto refresh = [&]() {
            const int q = wave;
            if (group * DQ_QB + q >= a.nq) return;
            const int b = first_bin_reaching([&](int i) { return sm.hist[q][i]; }, (uint32_t)a.r2, nullptr);
            if (b < DQ_BINS && lane == 0) atomicMin(&sm.thr[q], (uint32_t)b + 1u);
        };

        // A wave works through groups of DQ_DEPTH full sub-tiles (group g = sub-tiles g * DEPTH ...);
        // the codes of its next group are requested into the registers of the sub-tile just scanned;
        // full batches of parked rows are flushed between groups.
        const int ngroups_t = nfull / DQ_DEPTH;
        int it = 0;
        uint4 cur[DQ_DEPTH];
#pragma unroll
        for (int u = 0; u < DQ_DEPTH; ++u) cur[u] = make_uint4(0, 0, 0, 0);
        // this lane's 16 bytes of sub-tile 0 of the wave's current group, then of its next group
        const uint8_t *gp = chunk_ptr + (size_t)wave * (DQ_DEPTH * DQ_SUB * 8) + lane * 16;
        auto load_group_sub = [&](const uint8_t *p, int u) -> uint4 {
            const v4u v = *(global_v4u)(p + u * (DQ_SUB * 8));
            return make_uint4(v.x, v.y, v.z, v.w);
        };
        if (wave < ngroups_t) {
#pragma unroll
            for (int u = 0; u < DQ_DEPTH; ++u) cur[u] = load_group_sub(gp, u);
        }
        reload_tau();
        for (int g = wave; g < ngroups_t; g += DQ_WAVES) {
            const bool more = g + DQ_WAVES < ngroups_t;
            gp += (size_t)DQ_WAVES * (DQ_DEPTH * DQ_SUB * 8);
            // the table reads of sub-tile u + 1 are issued before the sums of sub-tile u are formed
            uint4 va[8], vb[8];
            issue(cur[0], va);
            if (more) cur[0] = load_group_sub(gp, 0);
#pragma unroll
            for (int u = 0; u < DQ_DEPTH; ++u) {
                if (u + 1 < DQ_DEPTH) {
                    issue(cur[u + 1], (u & 1) ? va : vb);
                    if (more) cur[u + 1] = load_group_sub(gp, u + 1);
                }
                asm volatile("" : : : "memory");
                finish((u & 1) ? vb : va, g * DQ_DEPTH + u);
            }
            if (__builtin_expect(ring_cnt >= 64, 0)) {
                const int whole = ring_cnt & ~63;
                flush(whole);
                for (int i = lane; i < ring_cnt - whole; i += 64) {   // the rest moves to the front
                    const uint32_t v = sm.ring[wave][whole + i];
                    sm.ring[wave][i] = v;
                }
                ring_cnt -= whole;
            }
            if (MODE == 0) {
                if (wave < DQ_QB && ((it & (it + 1)) == 0 || (it & 15) == 15)) refresh();
                reload_tau();
            }
            ++it;
        }
        // sub-tiles past the last whole group, the ragged one included
        for (int sidx = ngroups_t * DQ_DEPTH + wave; sidx < nsub; sidx += DQ_WAVES)
            scan_sub(load_pair(sidx * DQ_SUB + lane * 2), sidx);
        if (ring_cnt > 0) flush(ring_cnt);

        if (MODE == 0) {
            // the block's counts join the query's device-wide buckets, whose bound then serves
            // every block that starts an item of this query later
            __syncthreads();
            for (int i = threadIdx.x; i < DQ_QB * DQ_BINS; i += DQ_THREADS) {
                const int q = i / DQ_BINS, bin = i % DQ_BINS;
                const uint32_t v = sm.hist[q][bin];
                const int gq = group * DQ_QB + q;
                if (v != 0u && gq < a.nq) atomicAdd(&a.g_hist[(size_t)gq * DQ_BINS + bin], v);
            }
            __syncthreads();
            if (wave < DQ_QB && group * DQ_QB + wave < a.nq) {
                const int gq = group * DQ_QB + wave;
                const uint32_t *gh = a.g_hist + (size_t)gq * DQ_BINS;
                const int b = first_bin_reaching(
                    [&](int i) { return __hip_atomic_load(&gh[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                    (uint32_t)a.r2, nullptr);
                if (b < DQ_BINS && lane == 0) atomicMin(&a.g_bound[gq], (uint32_t)b);
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// The same loop for many queries (640 and more; used by the collecting pass): 16 queries per pass over the codes.  The entries of the
// 8-bit tables are bytes, so the entries of 16 queries for one (table, byte) fill a 16-byte LDS slot exactly;
// their sums of four do not fit a byte, so the scan loop adds 5-bit lower bounds instead,
//   L[t][b] = min(31, floor((Q[t][b] - min_b Q[t][b]) * scale)),   scale = DQ16_RANGE / (thr - off),
// (off = the sum of the four minima, thr = the query's threshold: sums below it are wanted), four of which stay
// below 128: the 16 sums of a code add up byte-wise in four 32-bit adds per table, and one add per word tests them
// against 0x80 - threshold (bit 7 of a byte stays clear iff that sum is below its threshold).  A code with
// sum <= thr - 1 has a bound of at most floor((thr - 1 - off) * scale) + 1 (fp32 rounding of the products), so
// testing "bound < that + 2" loses none.  Lanes that pass park their rows; the parked rows get their exact sums
// from the exact tables, which wait in LDS as well (16 KB), and are counted or listed as in the 8-query kernel.
// In the counting pass the thresholds fall quickly at the start of an item; the bounds are rebuilt from the
// exact tables at the thresholds of the moment after 4, 16 and 64 groups of a wave.
constexpr int DQ16_QB = 16;
constexpr int DQ16_DEPTH = 2;
constexpr int DQ16_RING = 64 * (DQ16_DEPTH + 1);
constexpr float DQ16_RANGE = 48.f;
constexpr float DQ16_ENTRY_MAX = 31.f;

template <int MODE>
struct __align__(16) DqSmem16 {
    uint4 lut[4096];                   // lower bounds: row b, 16 slots; slot s = table s >> 2 (four copies); 16 queries per slot
    uint4 lutx[DQ_M][256];             // exact entries: table t, byte b, 16 queries
    uint32_t hist[MODE == 0 ? DQ16_QB : 1][DQ_BINS];   // this block's counts of the current item (counting pass)
    uint32_t thr[DQ16_QB];             // a vector is kept for query q if its sum is below thr[q] (0: empty slot)
    uint32_t tmin[DQ16_QB][DQ_M];      // minima of the exact tables
    float off[DQ16_QB], scale[DQ16_QB];
    uint32_t ring[DQ_WAVES][DQ16_RING];
    int item;
};

template <int MODE>
__global__ __launch_bounds__(DQ_THREADS) void derived_scan16_kernel(DqArgs a) {
    typedef DqSmem16<MODE> SM;
    __shared__ SM sm;
    static_assert(sizeof(SM) <= 160 * 1024, "LDS of a CU");
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = lane_id();
    const uint32_t lane15 = (uint32_t)lane & 15u;
    // the walk over the slots of a row is that of the 8-query kernel (same layout of the rows)
    const uint32_t rot = 2u * ((lane15 >> 2) & 3u);
    uint32_t bases[2];
#pragma unroll
    for (int g = 0; g < 2; ++g)
        bases[g] = (((lane15 + 4u * (2 * g)) & 15u) << 4) | ((((lane15 + 4u * (2 * g + 1)) & 15u) << 4) << 16);
    const char *lut_bytes = reinterpret_cast<const char *>(sm.lut);

    for (;;) {
        if (threadIdx.x == 0) sm.item = (int)atomicAdd(a.work_counter, 1u);
        __syncthreads();
        const int item = sm.item;
        if (item >= a.nitems) break;
        const int group = item % a.ngroups, chunk = item / a.ngroups;
        const int64_t cbeg = (int64_t)chunk * a.chunk_codes;
        const int64_t cend = cbeg + a.chunk_codes < a.n ? cbeg + a.chunk_codes : a.n;
        const int ncodes = cend > cbeg ? (int)(cend - cbeg) : 0;

        if (threadIdx.x < DQ16_QB) {
            const int gq = group * DQ16_QB + threadIdx.x;
            uint32_t thr = 0;   // empty slot: nothing passes
            if (gq < a.nq) {
                const uint32_t b = MODE == 0 ? __hip_atomic_load(&a.g_bound[gq], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                             : a.bucket[gq];
                thr = b + 1u;   // at most DQ_BINS
            }
            sm.thr[threadIdx.x] = thr;
        }
        if (MODE == 0)
            for (int i = threadIdx.x; i < DQ16_QB * DQ_BINS; i += DQ_THREADS) (&sm.hist[0][0])[i] = 0u;
        {   // exact tables of the group's queries: entry (table t, byte b) of all 16 queries in one slot
            const int b = threadIdx.x >> 2, t = threadIdx.x & 3;
            uint32_t v[DQ16_QB];
#pragma unroll
            for (int q = 0; q < DQ16_QB; ++q) {
                const int gq = group * DQ16_QB + q;
                v[q] = gq < a.nq ? (uint32_t)a.qluts[((size_t)gq * DQ_M + t) * 256 + b] : 255u;
            }
            sm.lutx[t][b] = make_uint4(v[0] | (v[1] << 8) | (v[2] << 16) | (v[3] << 24), v[4] | (v[5] << 8) | (v[6] << 16) | (v[7] << 24),
                                       v[8] | (v[9] << 8) | (v[10] << 16) | (v[11] << 24), v[12] | (v[13] << 8) | (v[14] << 16) | (v[15] << 24));
        }
        __syncthreads();
        {   // minima: wave w takes rows (q, t) = 4w .. 4w + 3 of the 64, four entries per lane
            const uint8_t *xb = reinterpret_cast<const uint8_t *>(sm.lutx);
            for (int row = wave * 4; row < wave * 4 + 4; ++row) {
                const int q = row >> 2, t = row & 3;
                uint32_t mn = 255u;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t v = xb[((size_t)t * 256 + lane + 64 * i) * 16 + q];
                    mn = v < mn ? v : mn;
                }
                for (int o = 32; o > 0; o >>= 1) { const uint32_t other = __shfl_xor(mn, o); mn = other < mn ? other : mn; }
                if (lane == 0) sm.tmin[q][t] = mn;
            }
        }
        __syncthreads();
        // lower-bound tables from the exact ones at the thresholds of the moment (all threads; ends with a barrier)
        auto build_bounds = [&]() {
            if (threadIdx.x < DQ16_QB) {
                const int q = threadIdx.x;
                const uint32_t off = sm.tmin[q][0] + sm.tmin[q][1] + sm.tmin[q][2] + sm.tmin[q][3];
                const uint32_t thr = sm.thr[q];
                float scale = 0.f;   // every bound 0: every code goes to the exact test
                if (thr > off) scale = DQ16_RANGE / (float)(thr - off);
                sm.off[q] = (float)off;
                sm.scale[q] = scale;
            }
            __syncthreads();
            {
                const int b = threadIdx.x >> 2, t = threadIdx.x & 3;
                const uint4 x = sm.lutx[t][b];
                const uint32_t xw[4] = {x.x, x.y, x.z, x.w};
                uint32_t l[DQ16_QB];
#pragma unroll
                for (int q = 0; q < DQ16_QB; ++q) {
                    const uint32_t e = (xw[q >> 2] >> (8 * (q & 3))) & 255u;
                    const float v = (float)(e - sm.tmin[q][t]) * sm.scale[q];
                    l[q] = sm.thr[q] != 0u ? (uint32_t)fminf(floorf(v), DQ16_ENTRY_MAX) : (uint32_t)DQ16_ENTRY_MAX;
                }
                const uint4 pk = make_uint4(l[0] | (l[1] << 8) | (l[2] << 16) | (l[3] << 24), l[4] | (l[5] << 8) | (l[6] << 16) | (l[7] << 24),
                                            l[8] | (l[9] << 8) | (l[10] << 16) | (l[11] << 24), l[12] | (l[13] << 8) | (l[14] << 16) | (l[15] << 24));
#pragma unroll
                for (int c = 0; c < 4; ++c) sm.lut[b * 16 + t * 4 + c] = pk;
            }
            __syncthreads();
        };
        build_bounds();

        const uint8_t *chunk_ptr = a.codes + cbeg * 8;
        const int nfull = ncodes / DQ_SUB;                       // sub-tiles with every code present
        const int nsub = (ncodes + DQ_SUB - 1) / DQ_SUB;         // the last one may be ragged
        uint32_t tau[4];   // 0x80 minus the threshold (in units of the bounds) of the 16 queries, four per register
        auto reload_tau = [&]() {
            const int ql = lane & (DQ16_QB - 1);
            const uint32_t thr = sm.thr[ql];
            const float t = floorf(((float)thr - 1.f - sm.off[ql]) * sm.scale[ql]) + 2.f;
            const uint32_t t8 = thr != 0u ? (uint32_t)fmaxf(fminf(t, 127.f), 0.f) : 0u;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                tau[p] = 0x80808080u - (__builtin_amdgcn_readlane(t8, 4 * p) | (__builtin_amdgcn_readlane(t8, 4 * p + 1) << 8) |
                                        (__builtin_amdgcn_readlane(t8, 4 * p + 2) << 16) | (__builtin_amdgcn_readlane(t8, 4 * p + 3) << 24));
        };
        typedef uint32_t v4u __attribute__((ext_vector_type(4)));
        typedef const __attribute__((address_space(1))) v4u *global_v4u;
        // the two codes at rows pos, pos + 1 of the chunk (zeros for rows past its end)
        auto load_pair = [&](int pos) -> uint4 {
            uint4 c = make_uint4(0, 0, 0, 0);
            const uint8_t *p = chunk_ptr + (size_t)pos * 8;
            if (pos + 2 <= ncodes) {
                c = *reinterpret_cast<const uint4 *>(p);
            } else if (pos < ncodes) {
                const uint2 half = *reinterpret_cast<const uint2 *>(p);
                c.x = half.x; c.y = half.y;
            }
            return c;
        };
        // the eight table reads of the lane's two codes (four tables each, in the lane's rotated order)
        auto issue = [&](const uint4 c, uint4 (&v)[8]) {
            uint32_t w[4] = {c.x, c.y, c.z, c.w};
            rot8(w[0], w[1], (rot & 4u) != 0, rot & 3u);
            rot8(w[2], w[3], (rot & 4u) != 0, rot & 3u);
#pragma unroll
            for (int h = 0; h < 2; ++h) {
#pragma unroll
                for (int s = 0; s < 4; ++s) {
                    const uint32_t word = w[2 * h + (s >> 1)];
                    const uint32_t off = (s & 1) ? lut_offset<2>(word, bases[s >> 1]) : lut_offset<0>(word, bases[s >> 1]);
                    v[4 * h + s] = *reinterpret_cast<const uint4 *>(lut_bytes + off);
                }
            }
        };
        // One sub-tile whose reads are on their way: the bounds of the two codes for the 16 queries (four bytes per
        // word), one add per word against the thresholds, the rows of the lanes with a bound below one parked.
        int ring_cnt = 0;
        auto finish = [&](const uint4 (&v)[8], const int sidx) {
            uint32_t keep = 0x80808080u;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                keep &= v[4 * h].x + v[4 * h + 1].x + v[4 * h + 2].x + v[4 * h + 3].x + tau[0];
                keep &= v[4 * h].y + v[4 * h + 1].y + v[4 * h + 2].y + v[4 * h + 3].y + tau[1];
                keep &= v[4 * h].z + v[4 * h + 1].z + v[4 * h + 2].z + v[4 * h + 3].z + tau[2];
                keep &= v[4 * h].w + v[4 * h + 1].w + v[4 * h + 2].w + v[4 * h + 3].w + tau[3];
            }
            const uint64_t hit = __ballot(keep != 0x80808080u);
            if (__builtin_expect(hit != 0ull, 0)) {
                if ((hit >> lane) & 1ull) sm.ring[wave][ring_cnt + mask_prefix(hit)] = (uint32_t)(sidx * DQ_SUB + lane * 2);
                ring_cnt += __popcll(hit);
            }
        };
        auto scan_sub = [&](const uint4 c, const int sidx) {
            uint4 v[8];
            issue(c, v);
            asm volatile("" : : : "memory");   // all eight reads are issued before the first add
            finish(v, sidx);
        };

        // Parked rows, 64 at a time: the exact sums of the two codes of a row for the 16 queries (the 16 bytes of a
        // slot split into even and odd queries, two 16-bit sums per word: word p of `ev` holds queries 4p and 4p + 2,
        // word p of `od` queries 4p + 1 and 4p + 3), the test against the thresholds of now, and for every
        // (code, query) that passes the bucket count or the list append.
        auto flush = [&](const int count) {
            const uint32_t thr_lane = sm.thr[lane & (DQ16_QB - 1)];
            uint32_t comp_ev[4], comp_od[4];   // 0x8000 - threshold (thresholds are at most 1024)
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                comp_ev[p] = 0x80008000u - (__builtin_amdgcn_readlane(thr_lane, 4 * p) | (__builtin_amdgcn_readlane(thr_lane, 4 * p + 2) << 16));
                comp_od[p] = 0x80008000u - (__builtin_amdgcn_readlane(thr_lane, 4 * p + 1) | (__builtin_amdgcn_readlane(thr_lane, 4 * p + 3) << 16));
            }
            DqPlaces places;
            const int my_q = lane & (DQ16_QB - 1), my_gq = group * DQ16_QB + my_q;
            if (MODE == 1) places.list_of(a, my_gq);
            for (int base = 0; base < count; base += 64) {
                const bool have = base + lane < count;
                const int pos = have ? (int)sm.ring[wave][base + lane] : ncodes;
                const uint4 c = load_pair(pos);
                uint32_t ev[2][4], od[2][4];
                uint32_t m = 0;   // bit h * 16 + q: code h of the row is wanted by query q
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t w0 = h == 0 ? c.x : c.z, w1 = h == 0 ? c.y : c.w;
                    const uint32_t idx[4] = {w0 & 255u, (w0 >> 16) & 255u, w1 & 255u, (w1 >> 16) & 255u};
#pragma unroll
                    for (int p = 0; p < 4; ++p) { ev[h][p] = 0; od[h][p] = 0; }
#pragma unroll
                    for (int t = 0; t < DQ_M; ++t) {
                        const uint4 x = sm.lutx[t][idx[t]];
                        const uint32_t xw[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            ev[h][p] += xw[p] & 0x00ff00ffu;
                            od[h][p] += (xw[p] >> 8) & 0x00ff00ffu;
                        }
                    }
                    if (pos + h < ncodes) {
#pragma unroll
                        for (int p = 0; p < 4; ++p) {
                            // bit 15 / 31 of sum + (0x8000 - threshold) is clear iff the sum is below the threshold
                            const uint32_t fe = ~(ev[h][p] + comp_ev[p]), fo = ~(od[h][p] + comp_od[p]);
                            const uint32_t nib = ((fe >> 15) & 1u) | (((fo >> 15) & 1u) << 1) | (((fe >> 31) & 1u) << 2) | (((fo >> 31) & 1u) << 3);
                            m |= nib << (h * 16 + 4 * p);
                        }
                    }
                }
                if (MODE == 0) {
                    uint32_t bits = m;
                    while (bits != 0u) {
                        const int bit = __builtin_ctz(bits);
                        bits &= bits - 1u;
                        const int q = bit & 15, h = bit >> 4, p = q >> 2;
                        uint32_t word = (q & 1) ? (h == 0 ? od[0][0] : od[1][0]) : (h == 0 ? ev[0][0] : ev[1][0]);
#pragma unroll
                        for (int i = 1; i < 4; ++i)
                            word = p == i ? ((q & 1) ? (h == 0 ? od[0][i] : od[1][i]) : (h == 0 ? ev[0][i] : ev[1][i])) : word;
                        const uint32_t sum = (q & 2) ? word >> 16 : word & 0xffffu;
                        atomicAdd(&sm.hist[q][sum], 1u);
                    }
                } else {
                    if (__ballot(m != 0u) == 0ull) continue;
                    uint32_t mine = 0;
#pragma unroll
                    for (int q = 0; q < DQ16_QB; ++q) {
                        const uint32_t keys = (uint32_t)__popcll(__ballot((m >> q) & 1u)) + (uint32_t)__popcll(__ballot((m >> (16 + q)) & 1u));
                        mine = lane == q ? keys : mine;
                    }
                    places.reserve(a, my_gq, mine);
#pragma unroll
                    for (int q = 0; q < DQ16_QB; ++q) {
                        const bool p0 = ((m >> q) & 1u) != 0u, p1 = ((m >> (16 + q)) & 1u) != 0u;
                        const uint64_t m0 = __ballot(p0), m1 = __ballot(p1);
                        if ((m0 | m1) == 0ull) continue;
                        auto sum_of = [&](int h) {
                            const uint32_t word = (q & 1) ? od[h][q >> 2] : ev[h][q >> 2];
                            return (q & 2) ? word >> 16 : word & 0xffffu;
                        };
                        places.store(a, q, p0, (uint32_t)mask_prefix(m0), sum_of(0), (uint32_t)(cbeg + pos), c.x, c.y);
                        places.store(a, q, p1, (uint32_t)(__popcll(m0) + mask_prefix(m1)), sum_of(1), (uint32_t)(cbeg + pos + 1), c.z, c.w);
                    }
                }
            }
        };

        // Counting pass: the bound of a query is lowered from the block's own counts while the item
        // runs (one wave per query), early and then every 16 groups.
        auto refresh = [&]() {
            const int q = wave;
            if (group * DQ16_QB + q >= a.nq) return;
            const int b = first_bin_reaching([&](int i) { return sm.hist[q][i]; }, (uint32_t)a.r2, nullptr);
            if (b < DQ_BINS && lane == 0) atomicMin(&sm.thr[q], (uint32_t)b + 1u);
        };

        const int ngroups_t = nfull / DQ16_DEPTH;
        int it = 0;
        uint4 cur[DQ16_DEPTH];
#pragma unroll
        for (int u = 0; u < DQ16_DEPTH; ++u) cur[u] = make_uint4(0, 0, 0, 0);
        const uint8_t *gp = chunk_ptr + (size_t)wave * (DQ16_DEPTH * DQ_SUB * 8) + lane * 16;
        auto load_group_sub = [&](const uint8_t *p, int u) -> uint4 {
            const v4u v = *(global_v4u)(p + u * (DQ_SUB * 8));
            return make_uint4(v.x, v.y, v.z, v.w);
        };
        if (wave < ngroups_t) {
#pragma unroll
            for (int u = 0; u < DQ16_DEPTH; ++u) cur[u] = load_group_sub(gp, u);
        }
        reload_tau();
        for (int g = wave; g < ngroups_t; g += DQ_WAVES) {
            const bool more = g + DQ_WAVES < ngroups_t;
            gp += (size_t)DQ_WAVES * (DQ16_DEPTH * DQ_SUB * 8);
            // the table reads of sub-tile u + 1 are issued before the sums of sub-tile u are formed
            uint4 va[8], vb[8];
            issue(cur[0], va);
            if (more) cur[0] = load_group_sub(gp, 0);
#pragma unroll
            for (int u = 0; u < DQ16_DEPTH; ++u) {
                if (u + 1 < DQ16_DEPTH) {
                    issue(cur[u + 1], (u & 1) ? va : vb);
                    if (more) cur[u + 1] = load_group_sub(gp, u + 1);
                }
                asm volatile("" : : : "memory");
                finish((u & 1) ? vb : va, g * DQ16_DEPTH + u);
            }
            if (__builtin_expect(ring_cnt >= 64, 0)) {
                const int whole = ring_cnt & ~63;
                flush(whole);
                for (int i = lane; i < ring_cnt - whole; i += 64) {   // the rest moves to the front
                    const uint32_t v = sm.ring[wave][whole + i];
                    sm.ring[wave][i] = v;
                }
                ring_cnt -= whole;
            }
            if (MODE == 0) {
                if ((it & (it + 1)) == 0 || (it & 15) == 15) refresh();
                // every wave of the block runs iteration `it` iff its last wave does: then all of them meet here
                if ((it == 3 || it == 15 || it == 63) && DQ_WAVES * it + DQ_WAVES - 1 < ngroups_t) {
                    __syncthreads();
                    build_bounds();
                }
                reload_tau();
            }
            ++it;
        }
        // sub-tiles past the last whole group, the ragged one included
        for (int sidx = ngroups_t * DQ16_DEPTH + wave; sidx < nsub; sidx += DQ_WAVES)
            scan_sub(load_pair(sidx * DQ_SUB + lane * 2), sidx);
        if (ring_cnt > 0) flush(ring_cnt);

        if (MODE == 0) {
            // the block's counts join the query's device-wide buckets, whose bound then serves
            // every block that starts an item of this query later
            __syncthreads();
            for (int i = threadIdx.x; i < DQ16_QB * DQ_BINS; i += DQ_THREADS) {
                const int q = i / DQ_BINS, bin = i % DQ_BINS;
                const uint32_t v = sm.hist[q][bin];
                const int gq = group * DQ16_QB + q;
                if (v != 0u && gq < a.nq) atomicAdd(&a.g_hist[(size_t)gq * DQ_BINS + bin], v);
            }
            __syncthreads();
            if (group * DQ16_QB + wave < a.nq) {
                const int gq = group * DQ16_QB + wave;
                const uint32_t *gh = a.g_hist + (size_t)gq * DQ_BINS;
                const int b = first_bin_reaching(
                    [&](int i) { return __hip_atomic_load(&gh[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); },
                    (uint32_t)a.r2, nullptr);
                if (b < DQ_BINS && lane == 0) atomicMin(&a.g_bound[gq], (uint32_t)b);
            }
        }
    }
}

__global__ void derived_init_kernel(uint32_t *work_counter, uint32_t *g_hist, size_t nhist, uint32_t *g_bound, int nq) {
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    if (i0 == 0) *work_counter = 0;
    for (size_t i = i0; i < nhist; i += stride) g_hist[i] = 0u;
    for (size_t i = i0; i < (size_t)nq; i += stride) g_bound[i] = DQ_BINS - 1;   // no bound yet: every bucket is counted
}

// One wave per query: the bucket in which the r2-th vector falls (all vectors if there are fewer)
// and the number of vectors in the buckets up to it.
__global__ __launch_bounds__(64) void derived_bucket_kernel(const uint32_t *g_hist, int64_t n, int r2, uint32_t *bucket,
                                                            uint32_t *count) {
    const int q = blockIdx.x;
    const uint32_t *gh = g_hist + (size_t)q * DQ_BINS;
    const uint32_t want = (int64_t)r2 < n ? (uint32_t)r2 : (uint32_t)n;
    uint32_t cnt = 0;
    int b = 0;
    if (want > 0) b = first_bin_reaching([&](int i) { return gh[i]; }, want, &cnt);
    if (threadIdx.x == 0) {
        bucket[q] = (uint32_t)(b < DQ_BINS ? b : DQ_BINS - 1);
        count[q] = cnt;
    }
}

// A sample of the codes: one of every `step`, at a place in its step that its number's hash picks (the database may be periodic),
// so that a run of similar codes, as in a database ordered by cluster, is represented to within a code or two.
__global__ __launch_bounds__(256) void derived_sample_kernel(const uint2 *__restrict__ codes, int64_t nsample, uint32_t step, uint2 *__restrict__ sample) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < nsample) sample[i] = codes[i * step + (((uint32_t)i * 2654435761u) >> 16) % step];
}

// As derived_bucket_kernel from the counts of a sample (a share 1 / ratio of the codes): the bucket in which the sample's want-th vector falls, and
// room for the vectors up to it: six standard deviations of the sample's count more than it says.
__global__ __launch_bounds__(64) void derived_sample_bucket_kernel(const uint32_t *g_hist, int64_t n, uint32_t want, double ratio, uint32_t *bucket,
                                                                   uint32_t *room) {
    const int q = blockIdx.x;
    const uint32_t *gh = g_hist + (size_t)q * DQ_BINS;
    uint32_t cnt = 0;
    const int b = first_bin_reaching([&](int i) { return gh[i]; }, want, &cnt);
    if (threadIdx.x == 0) {
        bucket[q] = (uint32_t)(b < DQ_BINS ? b : DQ_BINS - 1);
        const double most = ((double)cnt + 6.0 * sqrt((double)cnt) + 16.0) * ratio;
        room[q] = most < (double)n ? (uint32_t)most : (uint32_t)n;
    }
}

// After a collecting pass on the bounds of a sample: per query the bucket of its r2-th vector and the number of vectors up to it, from the
// keys of its list (all vectors up to the sample's bucket, in no order); count 2^32 - 1 where the list did not fit or holds
// fewer than r2 vectors.  One block per query.
__global__ __launch_bounds__(1024) void derived_settle_kernel(const uint64_t *__restrict__ cand, const uint64_t *__restrict__ cand_off,
                                                              uint32_t *cand_cnt, int r2, uint32_t *bucket, uint32_t *count) {
    __shared__ uint32_t hist[DQ_BINS];
    const int q = blockIdx.x, tid = threadIdx.x;
    for (int i = tid; i < DQ_BINS; i += 1024) hist[i] = 0u;
    const uint64_t begin = cand_off[q], room = cand_off[q + 1] - begin;
    const uint32_t len = cand_cnt[q];
    __syncthreads();
    if (len <= room)
        for (uint32_t i0 = 0; i0 < len; i0 += 4096u) {   // (four keys of a thread on their way)
            uint32_t sum[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint32_t i = i0 + (uint32_t)(u * 1024 + tid);
                sum[u] = i < len && i >= i0 ? (uint32_t)(cand[begin + i] >> 32) : (uint32_t)DQ_BINS;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) wave_count_bin(hist, sum[u] < (uint32_t)DQ_BINS, sum[u]);
            if (i0 + 4096u < i0) break;   // (a list may end near 2^32)
        }
    __syncthreads();
    if (tid >= 64) return;
    uint32_t cnt = 0;
    const int b = first_bin_reaching([&](int i) { return hist[i]; }, (uint32_t)r2, &cnt);
    if (tid == 0) {
        const bool open = b >= DQ_BINS;   // fewer than r2 vectors, or a list that did not fit
        bucket[q] = open ? 0u : (uint32_t)b;
        count[q] = open ? 0xffffffffu : cnt;
    }
}

// What the host needs of the settled lists: summary[0] = keys in all lists, summary[1] = the first query whose count exceeds `cap`
// (nq if none; cap < 0: no limit), summary[2] = that query's count, summary[3] = queries left open.  One block.
__global__ __launch_bounds__(1024) void derived_summary_kernel(const uint32_t *__restrict__ count, const uint32_t *__restrict__ cand_cnt, int nq, long long cap,
                                                               unsigned long long *__restrict__ summary) {
    __shared__ unsigned long long total;
    __shared__ int bad, open;
    if (threadIdx.x == 0) { total = 0; bad = nq; open = 0; }
    __syncthreads();
    for (int q = threadIdx.x; q < nq; q += 1024) {
        if (count[q] == 0xffffffffu) atomicAdd(&open, 1);
        else if (cap >= 0 && (long long)count[q] > cap) atomicMin(&bad, q);
        atomicAdd(&total, (unsigned long long)cand_cnt[q]);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        summary[0] = total;
        summary[1] = (unsigned long long)bad;
        summary[2] = bad < nq ? count[bad] : 0;
        summary[3] = (unsigned long long)open;
    }
}

__global__ void derived_reset_kernel(uint32_t *work_counter, uint32_t *cand_cnt, int nq) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i == 0) *work_counter = 0;
    if (i < nq) cand_cnt[i] = 0u;
}

// Offsets of the candidate lists (exclusive prefix sum of the nq counts, one block) and what the host
// needs of them: summary[0] = total, summary[1] = the first query whose count exceeds `cap` (nq if
// none), summary[2] = that query's count.
__global__ __launch_bounds__(1024) void derived_offsets_kernel(const uint32_t *__restrict__ count, int nq, long long cap,
                                                                unsigned long long *__restrict__ cand_off,
                                                                unsigned long long *__restrict__ summary) {
    __shared__ unsigned long long wsum[16];
    __shared__ unsigned long long carry;
    __shared__ int bad;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) { carry = 0; bad = nq; }
    __syncthreads();
    for (int base = 0; base < nq; base += 1024) {
        const int q = base + tid;
        const unsigned long long c = q < nq ? count[q] : 0;
        if (q < nq && cap >= 0 && (long long)c > cap) atomicMin(&bad, q);
        unsigned long long incl = c;   // inclusive scan over the wave
        for (int o = 1; o < 64; o <<= 1) {
            const unsigned long long other = __shfl_up(incl, o);
            if (lane >= o) incl += other;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        unsigned long long before = carry;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        if (q < nq) cand_off[q] = before + incl - c;
        __syncthreads();
        if (tid == 1023) carry = before + incl;
        __syncthreads();
    }
    if (tid == 0) {
        cand_off[nq] = carry;
        summary[0] = carry;
        summary[1] = (unsigned long long)bad;
        summary[2] = bad < nq ? count[bad] : 0;
    }
}

// Step 1.2: greatest compact distance (float tables of the derived quantizers, low bits of the
// indexes; entries added in double in table order, rounded once) among the first `init` codes.
__global__ __launch_bounds__(256) void derived_qmax_kernel(const uint8_t *codes, int init, const float *dluts, float *qmax) {
    __shared__ float red[256];
    const int q = blockIdx.x;
    const float *lut = dluts + (size_t)q * DQ_M * 256;
    float best = 0.f;   // distances are not negative; no code at all gives 0
    for (int i = threadIdx.x; i < init; i += 256) {
        const uint2 c = *reinterpret_cast<const uint2 *>(codes + (size_t)i * 8);
        const double s = (double)lut[c.x & 255u] + (double)lut[256 + ((c.x >> 16) & 255u)] +
                         (double)lut[512 + (c.y & 255u)] + (double)lut[768 + ((c.y >> 16) & 255u)];
        best = fmaxf(best, (float)s);
    }
    red[threadIdx.x] = best;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + o]);
        __syncthreads();
    }
    if (threadIdx.x == 0) qmax[q] = red[0];
}

// What follows from the counts, in one launch before the collecting pass: the work items of Step 2 (a query's candidates in
// pieces of `piece`; item_off [nq + 1], item_query [item]; list_len: entries of the lists, more than the counts where they hold
// vectors of later buckets too), the counters of that pass (if given) and the bounds of Step 2 reset, the caller's buckets and
// counts (optional).  One block.
__global__ __launch_bounds__(1024) void derived_items_kernel(const uint32_t *__restrict__ count, const uint32_t *list_len, int nq, uint32_t piece,
                                                             uint32_t *__restrict__ item_off, uint32_t *__restrict__ item_query,
                                                             unsigned long long *__restrict__ tau_key, uint32_t *work_counter, uint32_t *__restrict__ cand_cnt,
                                                             const uint32_t *__restrict__ bucket, uint32_t *__restrict__ bucket_out, int64_t *__restrict__ ncand_out) {
    __shared__ uint32_t wsum[16];
    __shared__ uint32_t carry;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) {
        carry = 0;
        if (work_counter) *work_counter = 0;
    }
    __syncthreads();
    for (int base = 0; base < nq; base += 1024) {
        const int q = base + tid;
        if (q < nq) {
            if (cand_cnt) cand_cnt[q] = 0u;
            if (bucket_out) bucket_out[q] = bucket[q];
            if (ncand_out) ncand_out[q] = (int64_t)count[q];
        }
        const uint32_t c = q < nq ? list_len[q] / piece + (list_len[q] % piece != 0u ? 1u : 0u) : 0u;   // (a length may be close to 2^32)
        uint32_t incl = c;   // inclusive scan over the wave
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t other = __shfl_up(incl, o);
            if (lane >= o) incl += other;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        uint32_t before = carry;
        for (int w = 0; w < wave; ++w) before += wsum[w];
        if (q < nq) {
            const uint32_t first = before + incl - c;
            item_off[q] = first;
            tau_key[q] = KEY_EMPTY;
            for (uint32_t i = 0; i < c; ++i) item_query[first + i] = (uint32_t)q;
        }
        __syncthreads();
        if (tid == 1023) carry = before + incl;
        __syncthreads();
    }
    if (tid == 0) item_off[nq] = carry;
}

// Step 2: precise distance of every candidate from the full codebooks (each of the four terms ||y^j - C^j[c[j]]||^2
// summed in double and rounded to float as the table entry of Eq. (tables) would be, the four entries added in double
// and rounded once, Eq. (adc1)).  A block takes a piece of one query's candidates and leaves the topk smallest
// (distance, row) keys of it for the merge; the topk-th key of a piece is a bound for the other pieces of the query.
// What bounds it is the traffic of the centroid rows (four per candidate, dsub floats each, from codebooks of
// 4 k rows that no L2 holds), so a row is read by 8 lanes together, 16 bytes each, two candidates per wave and read,
// RR_ILP reads on their way.  (A thread per candidate read 4 bytes of 64 different rows per instruction, and one
// block per query waited for the longest list: 48 M candidates of 1000 queries, the longest 455 000: 11.3 -> 3.2 ms.)
constexpr int RR_THREADS = 512, RR_WAVES = RR_THREADS / 64;
constexpr int RR_KEEP = 128;            // best keys carried from tile to tile (topk <= 128)
constexpr int RR_TILE = 2 * RR_THREADS; // candidates per tile: two batches of 64 per wave
constexpr int RR_ILP = 8;               // pairs of candidates whose rows are on their way together
constexpr uint32_t RR_PIECE_MIN = RR_THREADS, RR_PIECE_MAX = 16 * RR_TILE;
constexpr size_t RR_TABLE_BYTES = (size_t)256 << 20;   // complete tables of a batch of queries (the last-level cache's size)
constexpr int RR_TABLE_QUERIES = 8192;   // of a batch, and of their sub-vectors as doubles

// v + (v of the lane that the DPP control names)
template <int CTRL>
__device__ __forceinline__ double dpp_add(double v) {
    const uint64_t b = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, true);
    const uint32_t hi = __builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, true);
    return v + __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}
// odd rows of 16 lanes of a <-> even rows of b
__device__ __forceinline__ void swap_rows16(double &a, double &b) {
    typedef uint32_t pair2 __attribute__((ext_vector_type(2)));
    const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
    const pair2 lo = __builtin_bit_cast(pair2, __builtin_amdgcn_permlane16_swap((uint32_t)x, (uint32_t)y, false, false));
    const pair2 hi = __builtin_bit_cast(pair2, __builtin_amdgcn_permlane16_swap((uint32_t)(x >> 32), (uint32_t)(y >> 32), false, false));
    a = __builtin_bit_cast(double, (uint64_t)hi[0] << 32 | lo[0]);
    b = __builtin_bit_cast(double, (uint64_t)hi[1] << 32 | lo[1]);
}

// VEC: floats per load (4 where rows start on 16 bytes and hold a multiple of 4 dimensions, else 1); 0: the queries'
// complete tables [4][k] stand in `tables` (from query q_first on), and a candidate is four entries added up, a thread
// each.  Consecutive items go to blocks of one die (blocks are dealt to the 8 dies in turn), so that what its L2
// holds is the tables of the few queries at hand.
template <int VEC>
__global__ __launch_bounds__(RR_THREADS, 4) void derived_rerank_kernel(const uint8_t *codes, const float *codebooks, int k, int dsub, const float *queries,
                                                                      const uint64_t *cand, const uint2 *cand_code, const uint64_t *cand_off,
                                                                      const uint32_t *cand_len, const uint32_t *bucket, const uint32_t *item_off, const uint32_t *item_query, int q_first, int q_end,
                                                                      uint32_t piece, int topk, unsigned long long *tau_key, uint64_t *partial,
                                                                      const float *tables) {
    extern __shared__ float4 rr_dyn[];
    __shared__ uint64_t keys[2048];   // KEEP + TILE, a power of two
    __shared__ uint2 wcode[RR_WAVES][64];
    __shared__ float wdist[RR_WAVES][64];
    __shared__ int nnew;
    static_assert(RR_KEEP + RR_TILE <= 2048 && RR_ILP % 2 == 0, "layout");
    float *const y = reinterpret_cast<float *>(rr_dyn);   // [4 * dsub]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, j = (lane >> 3) & 3, l8 = lane & 7;
    const float *const cb = codebooks + (size_t)j * k * dsub;
    uint32_t item = item_off[q_first], item_end = item_off[q_end], step = gridDim.x;
    if (VEC == 0) {   // (the grid is a multiple of 8)
        const uint32_t share = (item_end - item + 7) / 8, die = blockIdx.x & 7;
        const uint32_t stop = item + (die + 1) * share;
        item += die * share + (blockIdx.x >> 3);
        item_end = stop < item_end ? stop : item_end;
        step /= 8;
    } else {
        item += blockIdx.x;
    }
    for (; item < item_end; item += step) {
        const int q = (int)item_query[item];
        const uint64_t begin = cand_off[q] + (uint64_t)(item - item_off[q]) * piece;
        const uint64_t list_end = cand_off[q] + cand_len[q], end = begin + piece < list_end ? begin + piece : list_end;
        const uint32_t last_sum = bucket[q];   // (entries of later buckets are no candidates)
        __syncthreads();   // the previous item's keys and query have been read
        if (VEC > 0) for (int i = tid; i < DQ_M * dsub; i += RR_THREADS) y[i] = queries[(size_t)q * (DQ_M * dsub) + i];
        for (int i = tid; i < RR_KEEP; i += RR_THREADS) keys[i] = KEY_EMPTY;
        if (tid == 0) nnew = 0;
        __syncthreads();
        const float *const yj = y + j * dsub;
        for (uint64_t base = begin; base < end; base += RR_TILE) {
            uint64_t bound = keys[topk - 1];
            const uint64_t shared = __hip_atomic_load(&tau_key[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bound = shared < bound ? shared : bound;
            for (int u = 0; u < 2; ++u) {
                const uint64_t c0 = base + (uint64_t)(u * RR_THREADS + wave * 64);
                if (c0 >= end) break;
                const uint64_t ci = c0 + lane;
                bool have = ci < end;
                const uint64_t entry = cand[have ? ci : c0];
                const uint32_t row = (uint32_t)entry;
                if constexpr (VEC == 0) {
                    const uint2 c = cand_code != nullptr ? cand_code[have ? ci : c0] : *reinterpret_cast<const uint2 *>(codes + (size_t)row * 8);
                    have = have && (uint32_t)(entry >> 32) <= last_sum;
                    const float *const tab = tables + (size_t)(q - q_first) * DQ_M * k;
                    const uint32_t idx[DQ_M] = {c.x & 0xffffu, c.x >> 16, c.y & 0xffffu, c.y >> 16};
                    double e[DQ_M];
#pragma unroll
                    for (int t = 0; t < DQ_M; ++t)   // indexes are below k by contract
                        e[t] = (double)tab[(size_t)t * k + (idx[t] < (uint32_t)k ? idx[t] : (uint32_t)k - 1u)];
                    const double total = (e[0] + e[1]) + (e[2] + e[3]);   // (the order of the other forms)
                    const uint64_t key = ((uint64_t)f32_to_ord((float)total) << 32) | row;
                    if (have && key < bound) keys[RR_KEEP + atomicAdd(&nnew, 1)] = key;
                    continue;
                }
                constexpr int W = VEC > 0 ? VEC : 1;
                wcode[wave][lane] = cand_code != nullptr ? cand_code[have ? ci : c0] : *reinterpret_cast<const uint2 *>(codes + (size_t)row * 8);
                asm volatile("" : : : "memory");   // (the wave's LDS accesses stay in order)
                const uint16_t *const idx16 = reinterpret_cast<const uint16_t *>(wcode[wave]);
                const int left = end - c0 < 64 ? (int)(end - c0) : 64;
                for (int s = 0; s < left; s += 2 * RR_ILP) {
                    // lanes 32 h .. 32 h + 31: candidate s + 2 v + h, row j, dimensions VEC * l8 .. of every 8 * VEC
                    const float *p[RR_ILP];
                    double sum[RR_ILP];
#pragma unroll
                    for (int v = 0; v < RR_ILP; ++v) {
                        uint32_t idx = idx16[(s + 2 * v + half) * 4 + j];
                        idx = idx < (uint32_t)k ? idx : (uint32_t)k - 1u;   // indexes are below k by contract
                        p[v] = cb + (size_t)idx * dsub;
                        sum[v] = 0.0;
                    }
                    for (int t = W * l8; t < dsub; t += 8 * W) {
                        float yv[W], cv[RR_ILP][W];
#pragma unroll
                        for (int v = 0; v < RR_ILP; ++v) {
                            if (W == 4) {
                                const float4 f = *reinterpret_cast<const float4 *>(p[v] + t);
                                cv[v][0] = f.x; cv[v][W > 1 ? 1 : 0] = f.y; cv[v][W > 2 ? 2 : 0] = f.z; cv[v][W > 3 ? 3 : 0] = f.w;
                            } else {
                                cv[v][0] = p[v][t];
                            }
                        }
#pragma unroll
                        for (int i = 0; i < W; ++i) yv[i] = yj[t + i];
#pragma unroll
                        for (int v = 0; v < RR_ILP; ++v)
#pragma unroll
                            for (int i = 0; i < W; ++i) {
                                const double diff = (double)yv[i] - (double)cv[v][i];
                                sum[v] = fma(diff, diff, sum[v]);
                            }
                    }
#pragma unroll
                    for (int v = 0; v < RR_ILP; v += 2) {
                        double pairsum[2];
#pragma unroll
                        for (int w = 0; w < 2; ++w) {
                            double x = dpp_add<0xB1>(sum[v + w]);   // lane ^ 1 (quad_perm 1,0,3,2)
                            x = dpp_add<0x4E>(x);                   // lane ^ 2 (quad_perm 2,3,0,1)
                            x = dpp_add<0x141>(x);                  // the other four of eight (row_half_mirror)
                            x = (double)(float)x;                   // the table entry
                            pairsum[w] = dpp_add<0x128>(x);         // tables j and j ^ 1 (row_ror 8)
                        }
                        swap_rows16(pairsum[0], pairsum[1]);
                        const float total = (float)(pairsum[0] + pairsum[1]);   // row of 16 lanes r: candidate s + 2 (v + (r & 1)) + (r >> 1)
                        if ((lane & 15) == 0) wdist[wave][s + 2 * (v + ((lane >> 4) & 1)) + half] = total;
                    }
                }
                asm volatile("" : : : "memory");   // (the wave's LDS accesses stay in order)
                const uint64_t key = ((uint64_t)f32_to_ord(wdist[wave][lane]) << 32) | row;
                have = have && (uint32_t)(entry >> 32) <= last_sum;
                if (have && key < bound) keys[RR_KEEP + atomicAdd(&nnew, 1)] = key;   // (room: see the end of the tile)
                asm volatile("" : : : "memory");   // (the wave's LDS accesses stay in order)
            }
            __syncthreads();
            // sorted while there is no bound yet, when the next tile might not fit, and at the end
            const int added = nnew, total = RR_KEEP + added;
            const bool later = keys[topk - 1] != KEY_EMPTY && total + RR_TILE <= 2048 && base + RR_TILE < end;
            __syncthreads();   // (every thread has read the counter before the next tile adds to it)
            if (later) continue;
            if (added > 0) {
                int n2 = 256;
                while (n2 < total) n2 <<= 1;
                for (int i = total + tid; i < n2; i += RR_THREADS) keys[i] = KEY_EMPTY;
                block_bitonic_sort(keys, n2);
            }
            __syncthreads();
            if (tid == 0) {
                nnew = 0;
                if (added > 0 && keys[topk - 1] != KEY_EMPTY) atomicMin(&tau_key[q], (unsigned long long)keys[topk - 1]);
            }
            __syncthreads();
        }
        for (int i = tid; i < RR_KEEP; i += RR_THREADS) partial[(size_t)item * RR_KEEP + i] = i < topk ? keys[i] : KEY_EMPTY;
    }
}

// The queries' sub-vectors as doubles, padded with zeros to DIMS dimensions: [nq][4][DIMS].
template <int DIMS>
__global__ __launch_bounds__(256) void derived_widen_kernel(const float *__restrict__ queries, int nq, int dsub, double *__restrict__ wide) {
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= (size_t)nq * DQ_M * DIMS) return;
    const int t = (int)(i % DIMS);
    wide[i] = t < dsub ? (double)queries[i / DIMS * dsub + t] : 0.0;   // (a sub-vector follows the other in the query as well)
}

// Complete tables of a batch of queries for Step 2: entry ||y^j - C^j[i]||^2 from the differences, summed in double and rounded
// to float, in the very order of derived_rerank_kernel<4> (eight partial sums over dimensions 4 l .. 4 l + 3 of every 32, added
// pairwise), so that a candidate has the same distance, bit for bit, whichever form measures it.  (The expanded form of the
// Tables step loses bits where a query nearly hits a centroid, and makes a NaN of an infinite component.)  A thread has one
// centroid in registers, as doubles, and goes through the queries, whose dimensions are the same for the whole wave and come
// through scalar loads: two fp64 instructions per dimension, nothing else.  Padding adds zeros and changes no sum.
constexpr int DT_QUERIES = 64;   // queries per block: what a centroid row's conversion is spread over
template <int DIMS>
__global__ __launch_bounds__(256) void derived_tables_kernel(const double *__restrict__ wide, const float *__restrict__ codebooks, int nq, int k, int dsub,
                                                             float *__restrict__ tables) {
    const int i = blockIdx.x * 256 + threadIdx.x, j = blockIdx.y, q0 = blockIdx.z * DT_QUERIES;
    const float4 *const row = reinterpret_cast<const float4 *>(codebooks + ((size_t)j * k + (i < k ? i : k - 1)) * dsub);
    double c[DIMS];
#pragma unroll
    for (int t = 0; t < DIMS; t += 4) {
        const bool inside = t < dsub;   // (dsub is a multiple of 4)
        const float4 f = row[inside ? t / 4 : 0];
        c[t] = inside ? (double)f.x : 0.0; c[t + 1] = inside ? (double)f.y : 0.0;
        c[t + 2] = inside ? (double)f.z : 0.0; c[t + 3] = inside ? (double)f.w : 0.0;
    }
    const int q1 = q0 + DT_QUERIES < nq ? q0 + DT_QUERIES : nq;
    for (int q = q0; q < q1; ++q) {
        const double *const y = wide + ((size_t)q * DQ_M + j) * DIMS;
        auto part = [&](int l) {
            double sum = 0.0;
#pragma unroll
            for (int t = 4 * l; t < DIMS; t += 32)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const double diff = y[t + u] - c[t + u];
                    sum = fma(diff, diff, sum);
                }
            return sum;
        };
        auto four = [&](int l) {
            const double a = part(l) + part(l + 1);
            return a + (part(l + 2) + part(l + 3));
        };
        const double a = four(0);
        const double entry = a + four(4);
        if (i < k) tables[((size_t)q * DQ_M + j) * k + i] = (float)entry;
    }
}

template <int DIMS>
static int launch_derived_tables(pq_ctx *ctx, const float *queries, const float *codebooks, int nq, int k, int dsub, double *wide, float *tables) {
    const size_t values = (size_t)nq * DQ_M * DIMS;
    derived_widen_kernel<DIMS><<<(unsigned)((values + 255) / 256), 256, 0, ctx->stream>>>(queries, nq, dsub, wide);
    PQ_HIP(ctx, hipGetLastError());
    const dim3 grid((k + 255) / 256, DQ_M, (nq + DT_QUERIES - 1) / DT_QUERIES);
    derived_tables_kernel<DIMS><<<grid, 256, 0, ctx->stream>>>(wide, codebooks, nq, k, dsub, tables);
    PQ_HIP(ctx, hipGetLastError());
    return PQ_OK;
}

// candidate rows of every query as [nq][cap] ids (ascending positions in the list are not sorted), padded with -1.  Lists that hold
// nothing else (place == nullptr), or, from place[q] on (0 at the start), the entries of the buckets up to bucket[q].
__global__ void derived_export_kernel(const uint64_t *cand, const uint64_t *cand_off, const uint32_t *cand_len, const uint32_t *bucket,
                                      const uint32_t *count, uint32_t *place, int64_t cap, int64_t *out) {
    const int q = blockIdx.y;
    const uint64_t begin = cand_off[q], cnt = count[q];
    const int64_t first = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = first; i < cap; i += stride) {
        if ((uint64_t)i >= cnt) out[(size_t)q * cap + i] = -1;
        else if (place == nullptr) out[(size_t)q * cap + i] = (int64_t)(uint32_t)cand[begin + i];
    }
    if (place == nullptr) return;
    const int64_t len = cand_len[q];
    for (int64_t i = first; i < len; i += stride) {
        const uint64_t entry = cand[begin + i];
        if ((uint32_t)(entry >> 32) > bucket[q]) continue;
        const uint32_t at = atomicAdd(&place[q], 1u);
        if ((int64_t)at < cap) out[(size_t)q * cap + at] = (int64_t)(uint32_t)entry;
    }
}

}  // namespace

int launch_derived_search(pq_ctx *ctx, const uint16_t *codes16, int64_t n, const float *derived_codebooks,
                          const float *codebooks, int k, const float *queries, int nq, int d, int r2, int topk,
                          float *out_dist, int64_t *out_ids, uint32_t *bucket_out, int64_t *ncand_out,
                          int64_t *cand_ids_out, int64_t cand_cap) {
    const uint8_t *codes = reinterpret_cast<const uint8_t *>(codes16);
    const int dsub = d / DQ_M;
    hipStream_t s = ctx->stream;
    // 640 queries and more (measured on 25 M codes: 512 queries 4.45 -> 4.90 ms per call, 700 queries 6.23 -> 6.06 ms,
    // 1000 queries 8.30 -> 7.87 ms): the collecting pass takes 16 queries per pass over the codes (PQ_SCAN_Q8=0: 8, as
    // for fewer queries).  The counting pass stays with 8: its bound is the loose one of the block's own counts for most of
    // an item, so a large share of the codes needs exact sums, which the 8-query loop has at hand and the 16-query
    // loop fetches again (measured: 3.7 ms against 5.0 ms, 4.7 ms with a first bound from a sample).
    const bool wide = nq >= 640 && opt_int(ctx, PQ_OPT_SCAN_Q8, 1) != 0;

    // work items: chunk of codes x group of 8 or 16 queries, chunk-major (blocks running together share chunks)
    struct Geometry { int ngroups, nblocks; int64_t nchunks, chunk_codes, nitems; };
    auto geometry = [&](int qb, int64_t n, int min_tiles) {
        Geometry g;
        g.ngroups = (nq + qb - 1) / qb;
        const int64_t block_tile = (int64_t)DQ_SUB * DQ_WAVES;
        int nblocks_max = opt_int(ctx, PQ_OPT_SCAN_BLOCKS, ctx->num_cu);
        if (nblocks_max < 1) nblocks_max = 1;
        int64_t nchunks = ((int64_t)opt_int(ctx, PQ_OPT_SCAN_ITEMS_PER_BLOCK, 4) * nblocks_max + g.ngroups - 1) / g.ngroups;
        const int64_t max_by_n = (n + min_tiles * block_tile - 1) / (min_tiles * block_tile);
        if (nchunks > max_by_n) nchunks = max_by_n;
        const int64_t min_chunks = (n + ((int64_t)1 << 30) - 1) >> 30;   // a chunk's rows are counted in 32 bits
        if (nchunks < min_chunks) nchunks = min_chunks;
        if (nchunks < 1) nchunks = 1;
        int64_t chunk_codes = (n + nchunks - 1) / nchunks;
        chunk_codes = (chunk_codes + block_tile - 1) / block_tile * block_tile;
        if (chunk_codes < block_tile) chunk_codes = block_tile;
        g.chunk_codes = chunk_codes;
        g.nchunks = n > 0 ? (n + chunk_codes - 1) / chunk_codes : 0;
        g.nitems = g.nchunks * g.ngroups;
        g.nblocks = (int)(g.nitems < nblocks_max ? g.nitems : nblocks_max);
        return g;
    };
    const Geometry g_count = geometry(DQ_QB, n, 8), g_collect = geometry(wide ? DQ16_QB : DQ_QB, n, 8);
    if (g_count.nitems > 0x3fffffff) return fail(ctx, PQ_EUNSUPPORTED, "derived_search: too many work items (%lld)", (long long)g_count.nitems);
    auto bind_geometry = [&](DqArgs &a, const Geometry &g) {
        a.chunk_codes = g.chunk_codes; a.nchunks = (int)g.nchunks; a.ngroups = g.ngroups; a.nitems = (int)g.nitems;
    };

    // One pass over the codes instead of two where the counting pass is long and a share of the codes says where the r2-th vector
    // falls: a sample, one code of every sample_step, gives each query a bucket that holds the r2-th vector with 4.5 standard
    // deviations of the sample's count to spare and the room for its list, the collecting pass lists everything up to it, and
    // the buckets and counts are taken from the lists (derived_settle_kernel).  Entries of later buckets stay in the lists and are
    // passed over by Step 2.  A query whose list turns out too short or does not fit sends the call to the two passes.
    // The sample holds 150 of the r2 vectors at least; below 84 M pairs the additional launches and the second wait cost what the
    // shorter count saves.  Call: 25 M codes, 1000 queries, r2 = 10 000 9.95 -> 6.75 ms, r2 = 1000 8.30 -> 5.88; 8 M, 100,
    // 10 000 0.73 -> 0.59; 25 M, 8, 10 000 0.556 -> 0.527; 1 M, 100, 1000 0.233 -> 0.218; but 2 M, 30, 10 000 0.272 -> 0.307
    // and 8 M, 8, 10 000 0.307 -> 0.318.  A call that its sample misleads pays for both ways: with a far code at half of the sample's
    // rows, 25 M codes, 1000 queries, r2 = 10 000 9.97 -> 14.65 ms, 8 M, 100, 10 000 0.72 -> 1.07.  Rows that do not follow the hash
    // mislead a query once in 300 000 (4.5 deviations), a call of 1000 queries once in 300.
    int sample_step = r2 / 150 < 16 ? r2 / 150 : 16;
    if (sample_step < 3 || n < (int64_t)r2 * 32 || n * nq < DQ_SAMPLE_PAIRS || opt_int(ctx, PQ_OPT_DERIVED_SAMPLE, 1) == 0) sample_step = 0;
    const int64_t nsample = sample_step > 0 ? n / sample_step : 0;

    // workspace, first part: tables and counts
    size_t off = 0;
    auto take = [&](size_t bytes) { const size_t o = off; off += align_up(bytes, 256); return o; };
    const size_t o_counter = take(256);
    const size_t o_dluts = take((size_t)nq * DQ_M * 256 * 4);
    const size_t o_qmax = take((size_t)nq * 4);
    const size_t o_qmin = take((size_t)nq * 4);
    const size_t o_scale = take((size_t)nq * 4);
    const size_t o_qluts = take((size_t)nq * DQ_M * 256);
    const size_t o_hist = take((size_t)nq * DQ_BINS * 4);
    const size_t o_bound = take((size_t)nq * 4);
    const size_t o_bucket = take((size_t)nq * 4);
    const size_t o_count = take((size_t)nq * 4);
    const size_t o_candcnt = take((size_t)nq * 4);
    const size_t o_candoff = take((size_t)(nq + 1) * 8);

    auto prepare = [&](uint8_t *ws) -> int {   // Steps 1.1 and 1.2
        float *dluts = (float *)(ws + o_dluts), *qmax = (float *)(ws + o_qmax);
        int rc = launch_build_luts(ctx, queries, derived_codebooks, nq, d, DQ_M, 256, dluts);
        if (rc) return rc;
        const int init = (int)((int64_t)r2 < n ? (int64_t)r2 : n);
        derived_qmax_kernel<<<nq, 256, 0, s>>>(codes, init, dluts, qmax);
        PQ_HIP(ctx, hipGetLastError());
        return launch_quantize_luts(ctx, dluts, nq, DQ_M, 256, qmax, ws + o_qluts, (float *)(ws + o_qmin),
                                    (float *)(ws + o_scale));
    };

    const size_t o_summary = take(256);
    const size_t o_sbucket = take((size_t)nq * 4);
    const size_t o_room = take((size_t)nq * 4);
    const size_t o_sample = take((size_t)nsample * 8);
    int rc = ws_reserve(ctx, off);
    if (rc == PQ_ENOMEM && sample_step > 0) {   // (the two passes do without)
        sample_step = 0;
        rc = ws_reserve(ctx, o_sample);
    }
    if (rc) return rc;
    if (!ctx->host_pin) {   // a few words of pinned host memory, kept by the context
        void *p = nullptr;
        PQ_HIP(ctx, hipHostMalloc(&p, 256, hipHostMallocDefault));
        ctx->host_pin = p;
    }
    DqArgs a;
    a.nq = nq;
    auto summary_to_host = [&](uint8_t *ws) -> int {   // (a handful of words through pinned memory)
        PQ_HIP(ctx, hipMemcpyAsync(ctx->host_pin, ws + o_summary, 32, hipMemcpyDeviceToHost, s));
        PQ_HIP(ctx, hipStreamSynchronize(s));
        return PQ_OK;
    };
    auto cap_error = [&]() {
        const unsigned long long *pin = (const unsigned long long *)ctx->host_pin;
        return fail(ctx, PQ_ESHAPE, "derived_search: query %d has %u candidates, cand_cap is %lld", (int)pin[1], (unsigned)pin[2], (long long)cand_cap);
    };
    const long long cap_arg = cand_ids_out ? (long long)cand_cap : -1;
    // The counts of `len` codes up to the bucket of a query's `want`-th vector among them, in the workspace.
    auto count_codes = [&](uint8_t *ws, const Geometry &g, const uint8_t *some, int64_t len, int want) -> int {
        bind_geometry(a, g);
        a.codes = some; a.n = len;
        a.qluts = ws + o_qluts;
        a.work_counter = (uint32_t *)(ws + o_counter);
        a.g_hist = (uint32_t *)(ws + o_hist);
        a.g_bound = (uint32_t *)(ws + o_bound);
        a.bucket = nullptr; a.cand_off = nullptr; a.cand_cnt = nullptr; a.cand = nullptr; a.cand_code = nullptr;
        a.r2 = want;
        derived_init_kernel<<<256, 256, 0, s>>>(a.work_counter, a.g_hist, (size_t)nq * DQ_BINS, a.g_bound, nq);
        PQ_HIP(ctx, hipGetLastError());
        if (g.nblocks > 0) {
            derived_scan_kernel<0><<<g.nblocks, DQ_THREADS, 0, s>>>(a);
            PQ_HIP(ctx, hipGetLastError());
        }
        return PQ_OK;
    };
    // Steps 1.1 to 1.3 (counting pass) in the workspace `ws`; leaves the buckets, the counts and the
    // offsets of the candidate lists there and brings their total (and the first list beyond
    // cand_cap, if any) to the host: three words through pinned memory.
    auto count_pass = [&](uint8_t *ws, unsigned long long *total) -> int {
        if (ctx->profiling) {
            note_plain_scan(ctx, "derived_scan_kernel<count> (8 queries per pass)", 8, g_count.ngroups);
            PQ_HIP(ctx, hipEventRecord(ctx->ev_begin, s));
        }
        int rc = count_codes(ws, g_count, codes, n, r2);
        if (rc) return rc;
        if (ctx->profiling) {
            PQ_HIP(ctx, hipEventRecord(ctx->ev_end, s));
            ctx->ev_valid = 1;
        }
        derived_bucket_kernel<<<nq, 64, 0, s>>>(a.g_hist, n, r2, (uint32_t *)(ws + o_bucket), (uint32_t *)(ws + o_count));
        PQ_HIP(ctx, hipGetLastError());
        derived_offsets_kernel<<<1, 1024, 0, s>>>((const uint32_t *)(ws + o_count), nq, cap_arg, (unsigned long long *)(ws + o_candoff),
                                                  (unsigned long long *)(ws + o_summary));
        PQ_HIP(ctx, hipGetLastError());
        rc = summary_to_host(ws);
        if (rc) return rc;
        const unsigned long long *pin = (const unsigned long long *)ctx->host_pin;
        if (pin[1] < (unsigned long long)nq) return cap_error();
        *total = pin[0];
        return PQ_OK;
    };
    uint8_t *ws = (uint8_t *)ctx->ws;
    rc = prepare(ws);
    if (rc) return rc;
    const bool rr_vec = (dsub & 3) == 0 && ((uintptr_t)codebooks & 15) == 0;
    const size_t table_bytes = (size_t)DQ_M * k * 4;
    int table_batch = (int)(RR_TABLE_BYTES / table_bytes / 128 * 128);   // (k <= 65536: 256 at least)
    if (table_batch > RR_TABLE_QUERIES) table_batch = RR_TABLE_QUERIES;
    const int table_dims = dsub <= 32 ? 32 : 64;   // of a padded sub-vector
    unsigned long long total = 0;
    uint32_t piece = RR_PIECE_MIN;
    bool with_tables = false;
    size_t max_items = 0, o_partial = 0, o_cand = 0, o_code = 0, o_table = 0, o_wide = 0;
    uint8_t *lists = nullptr;
    uint32_t *item_off = nullptr, *item_query = nullptr;
    unsigned long long *tau_key = nullptr;
    for (;; sample_step = 0) {   // (once more, with the two passes, if the lists of a sample's bounds do not do)
        const bool sampled = sample_step > 0;
        if (sampled) {
            derived_sample_kernel<<<(unsigned)((nsample + 255) / 256), 256, 0, s>>>((const uint2 *)codes, nsample, (uint32_t)sample_step, (uint2 *)(ws + o_sample));
            PQ_HIP(ctx, hipGetLastError());
            const double ratio = (double)n / (double)nsample, w = (double)r2 / ratio;
            const uint32_t want = (uint32_t)ceil(w + 4.5 * sqrt(w) + 4.0);
            rc = count_codes(ws, geometry(DQ_QB, nsample, 32), ws + o_sample, nsample, (int)want);
            if (rc) return rc;
            derived_sample_bucket_kernel<<<nq, 64, 0, s>>>(a.g_hist, n, want, ratio, (uint32_t *)(ws + o_sbucket), (uint32_t *)(ws + o_room));
            PQ_HIP(ctx, hipGetLastError());
            derived_offsets_kernel<<<1, 1024, 0, s>>>((const uint32_t *)(ws + o_room), nq, -1, (unsigned long long *)(ws + o_candoff),
                                                      (unsigned long long *)(ws + o_summary));
            PQ_HIP(ctx, hipGetLastError());
            rc = summary_to_host(ws);
            if (rc) return rc;
            total = *(const unsigned long long *)ctx->host_pin;   // (room for that many)
        } else {
            rc = count_pass(ws, &total);
            if (rc) return rc;
        }
        // The sizes of the candidate lists are known now; they live in a buffer of their own, so that what the counting pass left
        // in the workspace stays.  Pieces of Step 2: as many as there are blocks four times over.
        const uint64_t per_block = total / (8ull * (unsigned)ctx->num_cu);
        piece = per_block > RR_PIECE_MAX ? RR_PIECE_MAX : (uint32_t)per_block / RR_PIECE_MIN * RR_PIECE_MIN;
        if (piece < RR_PIECE_MIN) piece = RR_PIECE_MIN;
        // Long lists: the complete tables of the queries cost less than the rows of the candidates.  65 536 centroids of 32 dimensions
        // per sub-space: 0.78 us of the GPU per query and 29 ps per candidate for its four entries, against 50 to 67 ps for its four
        // rows: from half as many candidates as centroids on.  (25 M codes, 1000 queries with 41 000 candidates each on average:
        // call 9.33 -> 8.83 ms, with 52 000: 10.98 -> 10.42; 100 000 codes, 100 queries, 32 768 each 508 -> 468 us, 16 384 each
        // 345 against 395.)  Rows below 24 dimensions cost less and the tables the same: from as many candidates as centroids on.
        // Fewer than 128 queries count as 128.  Queries go in batches whose tables stay below RR_TABLE_BYTES.
        // (the room of a sample's lists is about a fifth more than their entries)
        const uint64_t entries = sampled ? total / 6 * 5 : total;
        with_tables = entries * (dsub < 24 ? 1 : 2) >= (uint64_t)((nq + 127) / 128 * 128) * (uint64_t)k;
        with_tables = rr_vec && dsub >= 8 && dsub < 64 && opt_int(ctx, PQ_OPT_DERIVED_TABLES, with_tables ? 1 : 0) != 0;
        if (with_tables) piece = 8 * RR_TILE;   // (shorter than at most: what the blocks of a die work on belongs to few queries; 2, 4, 16 tiles: 10.8, 10.6, 10.5 against 10.4 ms per call)
        max_items = (size_t)(total / piece) + (size_t)nq;
        o_partial = 0;
        const size_t o_items = o_partial + align_up(max_items * RR_KEEP * 8, 256);
        const size_t o_itemoff = o_items + align_up(max_items * 4, 256);
        const size_t o_tau = o_itemoff + align_up((size_t)(nq + 1) * 4, 256);
        o_cand = o_tau + align_up((size_t)nq * 8, 256);
        o_code = o_cand + align_up((size_t)total * 8, 256);
        o_table = o_code + align_up((size_t)total * 8, 256);
        const size_t batch_queries = (size_t)(nq < table_batch ? nq : table_batch);
        o_wide = o_table + align_up(batch_queries * table_bytes, 256);
        const size_t table_end = o_wide + batch_queries * DQ_M * table_dims * 8;
        // (a copy of the candidates' codes beside the list saves Step 2 a random read of the database per candidate; it is
        // left out if there is no memory for it)
        bool with_codes = opt_int(ctx, PQ_OPT_DERIVED_CODE_COPY, 1) != 0;
        auto reserve_lists = [&](size_t bytes) { return buf_reserve(ctx, &ctx->derived_lists, bytes, "the candidate lists"); };
        rc = reserve_lists(with_tables ? table_end : o_table);
        if (rc == PQ_ENOMEM && sampled) continue;   // (lists of the exact sizes are shorter)
        if (rc == PQ_ENOMEM && with_tables) {
            with_tables = false;
            rc = reserve_lists(o_table);
        }
        if (rc == PQ_ENOMEM) {
            with_codes = false;
            rc = reserve_lists(o_code);
        }
        if (rc) return rc;
        lists = (uint8_t *)ctx->derived_lists.p;
        item_off = (uint32_t *)(lists + o_itemoff);
        item_query = (uint32_t *)(lists + o_items);
        tau_key = (unsigned long long *)(lists + o_tau);

        // Step 1.3, collecting pass
        a.qluts = ws + o_qluts;
        a.work_counter = (uint32_t *)(ws + o_counter);
        a.g_hist = nullptr; a.g_bound = nullptr;
        a.codes = codes; a.n = n;
        a.bucket = (const uint32_t *)(ws + (sampled ? o_sbucket : o_bucket));
        a.cand_off = (const uint64_t *)(ws + o_candoff);
        a.cand_cnt = (uint32_t *)(ws + o_candcnt);
        a.cand = (uint64_t *)(lists + o_cand);
        a.cand_code = with_codes ? (uint2 *)(lists + o_code) : nullptr;
        auto make_items = [&](const uint32_t *list_len, uint32_t *reset_counter, uint32_t *reset_cnt) -> int {
            derived_items_kernel<<<1, 1024, 0, s>>>((const uint32_t *)(ws + o_count), list_len, nq, piece, item_off, item_query, tau_key, reset_counter, reset_cnt,
                                                    (const uint32_t *)(ws + o_bucket), bucket_out, ncand_out);
            PQ_HIP(ctx, hipGetLastError());
            return PQ_OK;
        };
        if (sampled) {
            derived_reset_kernel<<<(nq + 255) / 256, 256, 0, s>>>(a.work_counter, a.cand_cnt, nq);
            PQ_HIP(ctx, hipGetLastError());
        } else {
            rc = make_items((const uint32_t *)(ws + o_count), a.work_counter, a.cand_cnt);
            if (rc) return rc;
        }
        bind_geometry(a, g_collect);
        if (sampled && ctx->profiling) {
            note_plain_scan(ctx, wide ? "derived_scan16_kernel<collect> (16 queries per pass, up to the buckets of a sample)"
                                      : "derived_scan_kernel<collect> (8 queries per pass, up to the buckets of a sample)", wide ? DQ16_QB : DQ_QB, g_collect.ngroups);
            PQ_HIP(ctx, hipEventRecord(ctx->ev_begin, s));
        }
        if (g_collect.nblocks > 0) {
            if (wide) derived_scan16_kernel<1><<<g_collect.nblocks, DQ_THREADS, 0, s>>>(a);
            else derived_scan_kernel<1><<<g_collect.nblocks, DQ_THREADS, 0, s>>>(a);
            PQ_HIP(ctx, hipGetLastError());
        }
        if (!sampled) break;
        if (ctx->profiling) {
            PQ_HIP(ctx, hipEventRecord(ctx->ev_end, s));
            ctx->ev_valid = 1;
        }
        derived_settle_kernel<<<nq, 1024, 0, s>>>(a.cand, a.cand_off, a.cand_cnt, r2, (uint32_t *)(ws + o_bucket), (uint32_t *)(ws + o_count));
        PQ_HIP(ctx, hipGetLastError());
        derived_summary_kernel<<<1, 1024, 0, s>>>((const uint32_t *)(ws + o_count), a.cand_cnt, nq, cap_arg, (unsigned long long *)(ws + o_summary));
        PQ_HIP(ctx, hipGetLastError());
        rc = summary_to_host(ws);
        if (rc) return rc;
        const unsigned long long *pin = (const unsigned long long *)ctx->host_pin;
        if (pin[3] != 0) continue;
        if (pin[1] < (unsigned long long)nq) return cap_error();
        total = pin[0];
        max_items = (size_t)(total / piece) + (size_t)nq;   // (no more than there is room for)
        rc = make_items(a.cand_cnt, nullptr, nullptr);
        if (rc) return rc;
        break;
    }
    // Step 2
    const unsigned rr_grid = (unsigned)(max_items < 4 * (size_t)ctx->num_cu ? max_items : 4 * (size_t)ctx->num_cu);
    const size_t rr_lds = with_tables ? 0 : align_up((size_t)d * 4, 16);
    uint64_t *partial = (uint64_t *)(lists + o_partial);
    if (with_tables) {
        float *tables = (float *)(lists + o_table);
        double *wide_queries = (double *)(lists + o_wide);
        for (int q0 = 0; q0 < nq; q0 += table_batch) {
            const int q1 = nq - q0 < table_batch ? nq : q0 + table_batch;
            const float *batch = queries + (size_t)q0 * d;
            rc = table_dims == 32 ? launch_derived_tables<32>(ctx, batch, codebooks, q1 - q0, k, dsub, wide_queries, tables)
                                  : launch_derived_tables<64>(ctx, batch, codebooks, q1 - q0, k, dsub, wide_queries, tables);
            if (rc) return rc;
            derived_rerank_kernel<0><<<(rr_grid + 7) / 8 * 8, RR_THREADS, rr_lds, s>>>(codes, codebooks, k, dsub, queries, a.cand, a.cand_code, a.cand_off, a.cand_cnt,
                                                                                    (const uint32_t *)(ws + o_bucket), item_off, item_query, q0, q1, piece, topk, tau_key, partial, tables);
            PQ_HIP(ctx, hipGetLastError());
        }
    } else {
        auto rerank = rr_vec ? derived_rerank_kernel<4> : derived_rerank_kernel<1>;
        rerank<<<rr_grid, RR_THREADS, rr_lds, s>>>(codes, codebooks, k, dsub, queries, a.cand, a.cand_code, a.cand_off, a.cand_cnt, (const uint32_t *)(ws + o_bucket), item_off, item_query, 0, nq, piece,
                                                   topk, tau_key, partial, nullptr);
        PQ_HIP(ctx, hipGetLastError());
    }
    rc = launch_merge_filtered(ctx, (const uint64_t *)(lists + o_partial), item_off, 0, 1, 1, tau_key, RR_KEEP, nq, topk, nullptr, false, out_dist, out_ids);
    if (rc) return rc;
    if (cand_ids_out && cand_cap > 0) {
        const bool mixed = sample_step > 0;   // (lists with entries of later buckets)
        if (mixed) {
            derived_reset_kernel<<<(nq + 255) / 256, 256, 0, s>>>(a.work_counter, (uint32_t *)(ws + o_room), nq);
            PQ_HIP(ctx, hipGetLastError());
        }
        derived_export_kernel<<<dim3(64, nq), 256, 0, s>>>(a.cand, a.cand_off, a.cand_cnt, (const uint32_t *)(ws + o_bucket), (const uint32_t *)(ws + o_count),
                                                           mixed ? (uint32_t *)(ws + o_room) : nullptr, cand_cap, cand_ids_out);
        PQ_HIP(ctx, hipGetLastError());
    }
    return PQ_OK;
}

}  // namespace pq
