// Scan step (Alg. 1 `scan`/`adc`, Eq. (adc1)): the general kernel for shapes outside the tuned
// ones, the kernel that merges the per-block candidate lists into the final top-k, and the
// dispatcher behind pq_adc_scan_topk.
//
// Top-k in the general kernel.  Each wave keeps a candidate buffer in device scratch and a
// threshold.  A code is a candidate if its value is below the threshold; when the buffer is
// nearly full the wave selects its k smallest keys, keeps them and lowers its threshold to the
// k-th.  Thresholds are shared (block LDS and a per-query device word, atomic min).  A bound
// learnt from another wave is the k-th smallest of a different subset: codes equal to it may
// still belong to the result, so foreign bounds prune with "<=" and the wave's own with "<"
// (the wave meets ids in increasing order, so a later code equal to its own k-th key can never
// replace it).  At the end of the block the 8 wave lists are merged to one list of k keys; the
// merge kernel sorts the lists of all chunks of a query and writes the result.
#include <math.h>
#include <type_traits>

#include "pq_internal.h"
#include "scan_common.h"
#include "topk_device.h"
#include "lds_walk.h"

namespace pq {

constexpr int SCAN_WAVES = 8;
constexpr int SCAN_THREADS = SCAN_WAVES * 64;

struct ScanArgs {
    const uint8_t *codes;
    int64_t n;
    int64_t chunk_codes;   // multiple of the block tile
    int nchunks;
    int ngroups;
    const void *luts;      // [nq][m][k] f32 or u8
    int nq;
    int topk;
    uint32_t *tau_global;  // [ngroups*QB], ordered-value domain
    uint64_t *scratch;     // [nblocks][SCAN_WAVES][QB][CAP]
    uint64_t *partial;     // [nchunks*ngroups][QB][KPAD]
};

// ------------------------------------------------------------------------------------------
// End of block: every wave has left at most k keys per query in its scratch list and its
// count in wave_cnt.  Wave q (q < QB) folds the 8 lists of query q into the list of wave 0
// and writes KPAD keys (padded with KEY_EMPTY) to `out`.
template <int QB, int E, int KPAD>
__device__ __forceinline__ void block_merge_lists(uint64_t *block_scratch, int (*wave_cnt)[QB], int k,
                                                   uint64_t *out_item, uint32_t queries = ~0u) {
    constexpr int CAP = 64 * E;
    const int wave = threadIdx.x >> 6, lane = lane_id();
    if (wave < QB && ((queries >> wave) & 1u) != 0u) {
        const int q = wave;
        uint64_t *acc = block_scratch + (size_t)(0 * QB + q) * CAP;
        int cnt = wave_cnt[0][q];
        for (int w = 1; w < SCAN_WAVES; ++w) {
            const uint64_t *src = block_scratch + (size_t)(w * QB + q) * CAP;
            const int cw = wave_cnt[w][q];
            for (int i = lane; i < cw; i += 64) key_store(acc + cnt + i, key_load(src + i));
            cnt += cw;
            if (cnt > k) wave_compact<E>(acc, cnt, k);
        }
        list_fence();
        uint64_t *out = out_item + (size_t)q * KPAD;
        for (int i = lane; i < KPAD; i += 64) out[i] = i < cnt ? key_load(acc + i) : KEY_EMPTY;
    }
}

// ------------------------------------------------------------------------------------------
// General kernel: any m, k with m*k <= 8192 entries, float or 8-bit tables, either code
// format, one query per block.  Used for shapes outside the two tuned kernels.
template <bool LUT_U8, int E, int KPAD>
__global__ __launch_bounds__(SCAN_THREADS) void scan_generic_kernel(ScanArgs a, int m, int k, int cf) {
    constexpr int QB = 1;
    constexpr int CAP = 64 * E;
    typedef typename std::conditional<LUT_U8, U32Val, F32Val>::type V;
    __shared__ float lutf[8192];
    __shared__ uint32_t tau_blk[QB];
    __shared__ int wave_cnt[SCAN_WAVES][QB];

    const int group = blockIdx.x % a.ngroups;   // = query
    const int chunk = blockIdx.x / a.ngroups;
    const int wave = threadIdx.x >> 6, lane = lane_id();
    const int cb = cf == PQ_CODES_U4_PACKED ? m / 2 : m;
    uint32_t *lutu = (uint32_t *)lutf;

    for (int e = threadIdx.x; e < m * k; e += SCAN_THREADS) {
        if (LUT_U8) lutu[e] = ((const uint8_t *)a.luts)[(size_t)group * m * k + e];
        else lutf[e] = ((const float *)a.luts)[(size_t)group * m * k + e];
    }
    if (threadIdx.x < QB) tau_blk[threadIdx.x] = a.tau_global[group];
    __syncthreads();

    WaveTopK<V, QB, E> st;
    uint64_t *block_scratch = a.scratch + (size_t)blockIdx.x * SCAN_WAVES * QB * CAP;
    st.k = a.topk;
    st.buf[0] = block_scratch + (size_t)wave * CAP;
    st.cnt[0] = 0;
    st.own_ord[0] = V::ord_inf();
    if (LUT_U8) st.own_ord[0] = 0xfffffffeu;   // sums of up to 8192 bytes exceed the 16-bit bound of the packed kernel
    st.set_tau(0, tau_blk[0]);

    const int64_t cbeg = (int64_t)chunk * a.chunk_codes;
    const int64_t cend = cbeg + a.chunk_codes < a.n ? cbeg + a.chunk_codes : a.n;
    int iter = 0;
    for (int64_t base = cbeg + (int64_t)wave * 64; base < cend; base += SCAN_WAVES * 64, ++iter) {
        const int64_t i = base + lane;
        const bool valid = i < cend;
        typename V::type val = 0;
        if (valid) {
            const uint8_t *c = a.codes + i * cb;
            for (int j = 0; j < m; ++j) {
                int idx;
                if (cf == PQ_CODES_U4_PACKED) {
                    const uint32_t byte = c[j >> 1];
                    idx = (j & 1) ? (byte >> 4) : (byte & 15u);
                } else {
                    idx = c[j];
                }
                if (idx < k) {
                    if (LUT_U8) val += lutu[j * k + idx]; else val += lutf[j * k + idx];
                }
            }
        }
        const bool pass = valid && val < st.tau[0];
        if (__ballot(pass) != 0ull) {
            if (st.insert(0, pass, val, (uint32_t)i)) {
                atomicMin(&tau_blk[0], st.own_ord[0]);
                atomicMin(&a.tau_global[group], st.own_ord[0]);
                st.set_tau(0, tau_blk[0]);
            }
        }
        if ((iter & 15) == 15) {
            uint32_t s = tau_blk[0];
            if ((iter & 63) == 63) {
                const uint32_t g = __hip_atomic_load(&a.tau_global[group], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (g < s) { atomicMin(&tau_blk[0], g); s = g; }
            }
            st.set_tau(0, s);
        }
    }
    if (st.cnt[0] > st.k) wave_compact<E>(st.buf[0], st.cnt[0], st.k);
    if (lane == 0) wave_cnt[wave][0] = st.cnt[0];
    list_fence();
    __syncthreads();
    block_merge_lists<QB, E, KPAD>(block_scratch, wave_cnt, a.topk, a.partial + (size_t)blockIdx.x * QB * KPAD);
}

// ------------------------------------------------------------------------------------------
// 32-bit codes: 4 float tables of 256 entries, 4 queries per block, two blocks of 8 waves per CU.
//
// Row b of the tables in LDS (256 bytes) holds the entries of code byte b for the four queries as 16-byte slots, every table
// in four copies; a lane reads slot (lane + 4 s) & 15 at step s, so the 16 lanes that the LDS serves together always read 16
// different bank groups and a code costs four reads without conflicts for four queries.  What bounds the kernel is
// vector instructions, 79 M for 4 M codes and 100 queries: their units are busy 76 % of its 197 us, the LDS 30 %; 10^6 codes and 6
// queries (28 us) are bound by the latency of few short items, 24 and 10 %.  The rotated order of the
// additions makes the sum a filter only, with a margin of its rounding; codes at or below the bound are added up again in table
// order, so values and ids are those of the general kernel.
// Bounds: a sample of the codes is counted first in the bins of a histogram per query (codes4_sample_kernel), the scan adds
// the candidates beyond the sample's rows, and waves that find many read the bin of the k-th from it; keys cut from a wave's
// or a block's lists bound the rows of tied codes as well.
// Call, general kernel -> this one: 10^6 codes, 6 queries, top-100 337 -> 67 us; 4 M codes, top-100, 25 queries 1060 -> 147,
// 100 queries 1830 -> 260, top-1024 7380 -> 381; 30 000 codes, 3 queries 64 -> 38; 4096 codes, one query 59 -> 37, 16 queries,
// top-1024 471 -> 114.  An atomic for each of the
// equal values counted made the 25 queries' call 441 us, folding the longer lists instead of sorting them the 100 queries' 596.
constexpr int C4_QB = 4, C4_TAB = 4 * 256;
constexpr int64_t C4_MIN_N = 4096;     // smaller databases: the general kernel (its merge sorts few lists there, and there is little to sample)

struct Codes4Args {
    const uint32_t *codes;
    int64_t n, chunk_codes, nsample;   // the first nsample rows are counted by the sampling pass
    int nitems, ngroups, nq, topk;     // item = chunk * ngroups + group
    const float *luts;
    unsigned long long *tau_key;       // [nq] at least topk keys are at or below it
    uint32_t *hist;                    // [nq][HIST_BINS], bins of 2^HIST_SHIFT ordered-value units that end at ref
    uint32_t *ref;                     // [nq]
    float *margin;                     // [nq] between a sum in rotated order and the value (NaN: sums may overflow, no filter)
    uint64_t *scratch;                 // [nblocks][SCAN_WAVES][C4_QB][64 * E]
    uint64_t *partial;                 // [nitems][C4_QB][KPAD]
};

// One wave: the sum of a query's greatest finite entries per table (the reference of its histogram: whatever lies above it is
// not counted) and of their greatest magnitudes.
__device__ __forceinline__ void codes4_table_sums(const float *__restrict__ lut, float &top, float &mag) {
    const int lane = lane_id();
    top = mag = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float t = -__builtin_inff(), a = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float e = lut[j * 256 + i * 64 + lane];
            if (e < __builtin_inff()) t = fmaxf(t, e);
            if (fabsf(e) < __builtin_inff()) a = fmaxf(a, fabsf(e));
        }
        for (int o = 32; o > 0; o >>= 1) { t = fmaxf(t, __shfl_xor(t, o)); a = fmaxf(a, __shfl_xor(a, o)); }
        top += t;
        mag += a;
    }
}

__global__ void codes4_clear_kernel(uint4 *hist, size_t n4) {
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = i0; i < n4; i += stride) hist[i] = make_uint4(0, 0, 0, 0);
}

// Block (q, s) counts the values of slice s of the sample.  Of its bins only those up to its own k-th can hold the sample's
// k-th: they go to the query's bins in device memory.
__global__ __launch_bounds__(SCAN_THREADS) void codes4_sample_kernel(Codes4Args a, int slice, int nslices) {
    __shared__ float tab[C4_TAB];
    __shared__ __align__(16) uint32_t hist[HIST_BINS];
    __shared__ uint32_t ref_s;
    __shared__ int bin_s;
    const int q = blockIdx.x / nslices, tid = threadIdx.x;
    const float *lut = a.luts + (size_t)q * C4_TAB;
    for (int i = tid; i < C4_TAB; i += SCAN_THREADS) tab[i] = lut[i];
    for (int i = tid; i < HIST_BINS; i += SCAN_THREADS) hist[i] = 0;
    if (tid < 64) {
        float top, mag;
        codes4_table_sums(lut, top, mag);
        if (tid == 0) ref_s = f32_to_ord(top);
    }
    __syncthreads();
    const uint32_t ref = ref_s;
    const int64_t begin = (int64_t)(blockIdx.x % nslices) * slice, end = begin + slice < a.nsample ? begin + slice : a.nsample;
    for (int64_t i0 = begin + tid; i0 < end; i0 += 4 * SCAN_THREADS) {
        uint32_t c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) c[u] = i0 + u * SCAN_THREADS < end ? a.codes[i0 + u * SCAN_THREADS] : 0u;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            float d = 0.f;
#pragma unroll
            for (int j = 0; j < 4; ++j) d += tab[j * 256 + ((c[u] >> (8 * j)) & 255u)];
            const uint32_t ord = f32_to_ord(d);
            if (i0 + u * SCAN_THREADS < end && d < __builtin_inff() && ord <= ref) {
                const uint32_t below = (ref - ord) >> HIST_SHIFT;
                atomicAdd(&hist[HIST_BINS - 1 - (below < HIST_BINS ? below : HIST_BINS - 1)], 1u);
            }
        }
    }
    __syncthreads();
    if (tid < 64) {
        const int b = hist_threshold(hist, a.topk);
        if (tid == 0) bin_s = b;
    }
    __syncthreads();
    for (int i = tid; i < HIST_BINS && i <= bin_s; i += SCAN_THREADS)
        if (hist[i] != 0u) atomicAdd(&a.hist[(size_t)q * HIST_BINS + i], hist[i]);
}

// What the items of a query start from, one wave per query.  (Read off the histogram by every item instead, which has to
// drop its L2's copies for that: 10^6 codes, 6 queries, scan 64 us.)
__global__ __launch_bounds__(64) void codes4_pick_kernel(Codes4Args a) {
    const int q = blockIdx.x;
    float top, mag;
    codes4_table_sums(a.luts + (size_t)q * C4_TAB, top, mag);
    const uint32_t ref = f32_to_ord(top);
    const int b = hist_threshold(a.hist + (size_t)q * HIST_BINS, a.topk);
    if (threadIdx.x == 0) {
        a.ref[q] = ref;
        // two orders of four additions differ by at most six roundings of the magnitudes' sum (3.6e-7 of it)
        a.margin[q] = mag < 1e38f ? mag * 1e-6f : __builtin_nanf("");
        a.tau_key[q] = (unsigned long long)(b < HIST_BINS ? ref - ((uint32_t)(HIST_BINS - 1 - b) << HIST_SHIFT) : 0xff800000u) << 32 | 0xffffffffull;
    }
}

template <int E, int KPAD>
__global__ __launch_bounds__(SCAN_THREADS, 4) void scan_codes4_kernel(Codes4Args a) {
    constexpr int QB = C4_QB, CAP = 64 * E, UNROLL = 4, STEP = 64 * UNROLL;
    __shared__ uint4 lut[4096];
    __shared__ unsigned long long key_blk[QB];   // at least topk keys of the query are at or below it
    __shared__ float margin[QB];
    __shared__ int found;
    __shared__ uint32_t ref_s[QB];
    __shared__ int wave_cnt[SCAN_WAVES][QB];
    __shared__ uint32_t ring[SCAN_WAVES][STEP + 64];   // rows of the item whose sums passed, waiting for the exact test
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = lane_id();
    const char *const lut_bytes = (const char *)lut;
    uint64_t *const block_scratch = a.scratch + (size_t)blockIdx.x * SCAN_WAVES * QB * CAP;
    uint64_t *const wave_buf = block_scratch + (size_t)wave * QB * CAP;
    uint32_t bases = 0;   // slot offsets of the four steps
#pragma unroll
    for (int s = 0; s < 4; ++s) bases |= ((((uint32_t)lane + 4u * s) & 15u) << 4) << (8 * s);
    const uint32_t rot = ((uint32_t)lane >> 2) & 3u;   // the table of step 0
    // keys of a wave's list at which it is cut to the k smallest: there must be room for 64 more, and short results find their
    // k-th key, which rules out ties, long before that
    const int list_most = 2 * a.topk + 32 < CAP - 64 ? 2 * a.topk + 32 : CAP - 64;

    for (int item = blockIdx.x; item < a.nitems; item += gridDim.x) {
        const int q0 = item % a.ngroups * QB;
        const int64_t begin = (int64_t)(item / a.ngroups) * a.chunk_codes;
        const int64_t end = begin + a.chunk_codes < a.n ? begin + a.chunk_codes : a.n;
        auto publish = [&](int q, unsigned long long key) {   // (one lane)
            __hip_atomic_fetch_min(&key_blk[q], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            atomicMin(&a.tau_key[q0 + q], key);
        };
        auto bound_of = [&](int q) { return __hip_atomic_load(&key_blk[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };
        auto edge_key = [&](int q) -> unsigned long long {   // (one wave) the edge of the bin that holds the k-th counted value
            const int b = hist_threshold(a.hist + (size_t)(q0 + q) * HIST_BINS, a.topk);
            return b < HIST_BINS ? (unsigned long long)(ref_s[q] - ((uint32_t)(HIST_BINS - 1 - b) << HIST_SHIFT)) << 32 | 0xffffffffull : KEY_EMPTY;
        };
        __syncthreads();   // the last item is done with the tables and the counts
        for (int e = tid; e < C4_TAB; e += SCAN_THREADS) {
            uint32_t v[QB];
#pragma unroll
            for (int q = 0; q < QB; ++q) v[q] = q0 + q < a.nq ? __float_as_uint(a.luts[(size_t)(q0 + q) * C4_TAB + e]) : 0u;
            const int j = e >> 8, b = e & 255;
#pragma unroll
            for (int c = 0; c < 4; ++c) lut[b * 16 + 4 * j + ((c + b) & 3)] = make_uint4(v[0], v[1], v[2], v[3]);
        }
        if (lane < QB) wave_cnt[wave][lane] = 0;
        if (tid < QB) {
            const bool used = q0 + tid < a.nq;   // (a slot without a query: no code passes, see reload)
            key_blk[tid] = used ? __hip_atomic_load(&a.tau_key[q0 + tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
            margin[tid] = used ? a.margin[q0 + tid] : 0.f;
            ref_s[tid] = used ? a.ref[q0 + tid] : 0u;
        }
        __syncthreads();

        float thr[QB];   // a rotated sum above it is no candidate
        auto reload = [&]() {
#pragma unroll
            for (int q = 0; q < QB; ++q) {
                const float t = q0 + q < a.nq ? ord_to_f32((uint32_t)(bound_of(q) >> 32)) + margin[q] : -__builtin_inff();
                thr[q] = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(t)));
            }
        };
        reload();
        int added = 0;   // keys this wave has added since it last looked at a histogram
        // Parked rows, 64 at a time: the values in table order, and the lists.
        auto flush = [&](int count) {
#pragma unroll 1
            for (int base = 0; base < count; base += 64) {
                const bool have = base + lane < count;
                const int64_t row = begin + (have ? ring[wave][base + lane] : 0u);
                const uint32_t code = a.codes[row];
                float val[QB] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const uint4 e = lut[((code >> (8 * j)) & 255u) * 16 + 4 * j + (lane & 3)];
                    val[0] += __uint_as_float(e.x); val[1] += __uint_as_float(e.y);
                    val[2] += __uint_as_float(e.z); val[3] += __uint_as_float(e.w);
                }
#pragma unroll 1
                for (int q = 0; q < QB && q0 + q < a.nq; ++q) {
                    const float v = q == 0 ? val[0] : q == 1 ? val[1] : q == 2 ? val[2] : val[3];
                    const uint32_t ord = f32_to_ord(v);
                    const uint64_t key = (uint64_t)ord << 32 | (uint32_t)row;
                    const bool pass = have && v < __builtin_inff() && key <= bound_of(q);
                    const uint64_t mask = __ballot(pass);
                    if (mask == 0ull) continue;
                    uint64_t *const buf = wave_buf + (size_t)q * CAP;
                    int cnt = wave_append(buf, wave_cnt[wave][q], pass, key);
                    const uint32_t below = (ref_s[q] - ord) >> HIST_SHIFT;   // (equal values add together: one atomic for them)
                    wave_count_bin(a.hist + (size_t)(q0 + q) * HIST_BINS, pass && row >= a.nsample && ord <= ref_s[q],
                                   HIST_BINS - 1 - (below < HIST_BINS ? below : HIST_BINS - 1));
                    added += __popcll(mask);
                    if (cnt > list_most) {
                        const uint64_t kth = wave_compact<E>(buf, cnt, a.topk);
                        if (kth != KEY_EMPTY && lane == 0) publish(q, kth);
                    }
                    wave_cnt[wave][q] = cnt;   // (the same from every lane)
                }
            }
        };
        // steps of 256 codes, the next step's codes on their way while one is scanned
        const int ncodes = (int)(end - begin), nsteps = (ncodes + STEP - 1) / STEP;
        const uint32_t *const codes = a.codes + begin;
        auto load_step = [&](int s, uint32_t (&c)[UNROLL]) {
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const int i = s * STEP + u * 64 + lane;
                c[u] = codes[i < ncodes ? i : ncodes - 1];
            }
        };
        uint32_t next[UNROLL];
        load_step(wave, next);
        int iter = 0, parked = 0;
        for (int s = wave; s < nsteps; s += SCAN_WAVES, ++iter) {
            uint32_t cur[UNROLL];
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) cur[u] = next[u];
            load_step(s + SCAN_WAVES, next);
#pragma unroll
            for (int u = 0; u < UNROLL; ++u) {
                const uint32_t w = __builtin_amdgcn_alignbyte(cur[u], cur[u], rot);
                float d[QB];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint32_t off = t == 0 ? lut_offset<0>(w, bases) : t == 1 ? lut_offset<1>(w, bases) : t == 2 ? lut_offset<2>(w, bases) : lut_offset<3>(w, bases);
                    const float4 e = *reinterpret_cast<const float4 *>(lut_bytes + off);
                    if (t == 0) { d[0] = e.x; d[1] = e.y; d[2] = e.z; d[3] = e.w; }
                    else { d[0] += e.x; d[1] += e.y; d[2] += e.z; d[3] += e.w; }
                }
                // (written as "not above": NaN sums and thresholds pass to the exact test)
                const int i = s * STEP + u * 64 + lane;
                const uint64_t hit = __ballot(i < ncodes && (!(d[0] > thr[0]) || !(d[1] > thr[1]) || !(d[2] > thr[2]) || !(d[3] > thr[3])));
                if (__builtin_expect(hit != 0ull, 0)) {
                    if ((hit >> lane) & 1ull) ring[wave][parked + mask_prefix(hit)] = (uint32_t)i;
                    parked += __popcll(hit);
                }
            }
            const bool last = s + SCAN_WAVES >= nsteps;
            if (parked >= 64 || (last && parked > 0)) {   // whole batches; what is left moves to the front
                const int take = last ? parked : parked & ~63;
                flush(take);
                parked -= take;
                if (lane < parked) ring[wave][lane] = ring[wave][take + lane];
                if (added >= KPAD / 2) {
                    added = 0;
                    const int q = wave & (QB - 1);
                    if (q0 + q < a.nq) {
                        const unsigned long long key = edge_key(q);
                        if (lane == 0) publish(q, key);
                    }
                }
                reload();
            }
            if ((iter & 3) == 3) reload();
        }
        list_fence();
        __syncthreads();
        // End of item.  Lists that fit side by side are copied; longer ones (encoded data ties: 4 M codes hold thousands of
        // copies of a near code) are sorted in the memory of the tables, and their k-th key bounds the items that follow; the
        // longest are folded one into the other.
        int total[QB];
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            total[q] = 0;
            for (int w = 0; w < SCAN_WAVES; ++w) total[q] += wave_cnt[w][q];
        }
        uint64_t *const out = a.partial + (size_t)item * QB * KPAD;
        uint64_t *const keys = (uint64_t *)lut;
        constexpr int SORT_KEYS = sizeof(lut) / 8;
        uint32_t fold = 0;
#pragma unroll
        for (int q = 0; q < QB; ++q) {
            const uint64_t *const src = wave_buf + (size_t)q * CAP;
            uint64_t *const to = out + (size_t)q * KPAD;
            if (total[q] <= KPAD) {
                int at = 0;
                for (int w = 0; w < wave; ++w) at += wave_cnt[w][q];
                for (int i = lane; i < wave_cnt[wave][q]; i += 64) to[at + i] = key_load(src + i);
                for (int i = total[q] + tid; i < KPAD; i += SCAN_THREADS) to[i] = KEY_EMPTY;
            } else if (total[q] <= SORT_KEYS) {
                __syncthreads();   // (the last query's keys have been read)
                if (tid == 0) found = 0;
                __syncthreads();
                const uint64_t bound = bound_of(q);
                const int cnt = wave_cnt[wave][q];
                for (int i0 = 0; i0 < cnt; i0 += 64) {
                    const uint64_t key = i0 + lane < cnt ? key_load(src + i0 + lane) : KEY_EMPTY;
                    const bool in = key <= bound;
                    const int at = wave_place(&found, in);
                    if (in) keys[at] = key;
                }
                __syncthreads();
                const int nkeys = found;
                int n2 = 64;
                while (n2 < nkeys) n2 <<= 1;
                for (int i = nkeys + tid; i < n2; i += SCAN_THREADS) keys[i] = KEY_EMPTY;
                block_bitonic_sort(keys, n2);
                for (int i = tid; i < KPAD; i += SCAN_THREADS) to[i] = i < n2 ? keys[i] : KEY_EMPTY;
                if (tid == 0 && nkeys >= a.topk) atomicMin(&a.tau_key[q0 + q], (unsigned long long)keys[a.topk - 1]);
            } else {
                fold |= 1u << q;
            }
        }
        if (fold != 0u) {
            __syncthreads();   // every wave has read the counts before any of them changes
            for (int q = 0; q < QB; ++q) {   // (the fold makes room list by list: at most k keys in each)
                if (((fold >> q) & 1u) == 0u) continue;
                int cnt = wave_cnt[wave][q];
                if (cnt > a.topk) wave_compact<E>(wave_buf + (size_t)q * CAP, cnt, a.topk);
                wave_cnt[wave][q] = cnt;
            }
            list_fence();
            __syncthreads();
            block_merge_lists<QB, E, KPAD>(block_scratch, wave_cnt, a.topk, out, fold);
        }
    }
}

// ------------------------------------------------------------------------------------------
__global__ void init_tau_kernel(uint32_t *tau, int count, uint32_t value) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < count) tau[i] = value;
}

// One block per query: gather the KPAD-key lists of all chunks, sort, write the first topk.
template <bool VAL_U32>
__global__ __launch_bounds__(1024) void merge_topk_kernel(const uint64_t *partial, int nchunks, int ngroups, int qb,
                                                           int kpad, int n2, int topk, void *out_val,
                                                           int64_t *out_ids) {
    extern __shared__ uint64_t skeys[];
    const int gq = blockIdx.x, group = gq / qb, q = gq % qb;
    const int total = nchunks * kpad;
    for (int i = threadIdx.x; i < n2; i += blockDim.x) {
        uint64_t key = KEY_EMPTY;
        if (i < total) {
            const int c = i / kpad, e = i % kpad;
            key = partial[((size_t)(c * ngroups + group) * qb + q) * kpad + e];
        }
        skeys[i] = key;
    }
    block_bitonic_sort(skeys, n2);
    for (int i = threadIdx.x; i < topk; i += blockDim.x) {
        const uint64_t key = skeys[i];
        const bool empty = key == KEY_EMPTY;
        if (VAL_U32) ((uint32_t *)out_val)[(size_t)gq * topk + i] = empty ? 0xffffffffu : (uint32_t)(key >> 32);
        else ((float *)out_val)[(size_t)gq * topk + i] = empty ? __builtin_inff() : ord_to_f32((uint32_t)(key >> 32));
        out_ids[(size_t)gq * topk + i] = empty ? -1 : (int64_t)(uint32_t)key;
    }
}

// One block per query: the k smallest keys over all result lists of the query, for scans that
// leave a final bound per query (at least k keys are at or below it): keys above the bound cannot
// be in the result and are dropped before the sort, so the number of lists is not limited by the
// sort.  The lists of query gq are either lists qlist_off[gq] .. qlist_off[gq + 1] of `partial`
// (inverted-list search) or, with qlist_off == nullptr, list (c * ngroups + gq / qb) * qb + gq % qb
// for every chunk c (flat scan).  ids (optional) maps rows to the ids to return.
// MERGE_CAP keys are kept in LDS (more than that at or below the bound: the rounds below).  Calls of few queries
// give every query a block of 1024 threads and room for 8192 keys; calls of many queries take blocks of 256 threads
// and 2048 keys (512 threads and 4096 keys for topk above 512), of which a compute unit holds several.
constexpr int MERGE_COUNT = 256;   // as many kept keys find their ranks by counting, without a selection before
constexpr int merge_lds_bytes(int cap) { return cap * 8 + cap * 4 + 1024 * 8; }   // kept keys, 32-bit values for the selection, the result's keys
enum { MERGE_LISTS, MERGE_COUNTED, MERGE_AGAIN };   // (the latter two: see AgainArgs; kernels of their own: 1 us of a call that wants neither)
template <bool VAL_U32, int MERGE_CAP, int MODE = MERGE_LISTS>
__global__ __launch_bounds__(1024) void merge_filtered_kernel(const uint64_t *__restrict__ partial,
                                                              const uint32_t *__restrict__ qlist_off, int nchunks,
                                                              int ngroups, int qb,
                                                              const unsigned long long *__restrict__ tau_key, int kpad, int topk,
                                                              const int64_t *__restrict__ ids, void *out_val,
                                                              int64_t *out_ids, const uint32_t *__restrict__ hist,
                                                              const uint32_t *__restrict__ hist_ref, int hist_bins,
                                                              const uint32_t *__restrict__ counts, uint32_t cap, AgainArgs again) {
    extern __shared__ uint64_t skeys[];
    __shared__ int s_count;
    constexpr bool COUNTED = MODE == MERGE_COUNTED;
    const int tid = threadIdx.x, slot = blockIdx.x;
    int gq = slot, per = qb;   // (per: queries per group)
    if constexpr (MODE == MERGE_AGAIN) {
        const int count = (int)*again.count;
        if (slot >= count) return;
        gq = (int)again.query[slot];
        per = again_per_group(count, qb, again.ngroups, again.spread);
        ngroups = (count + per - 1) / per;
    }
    // (with counts a query has one list of up to cap keys, read as if it were lists of 64)
    uint32_t listed = 0;
    if constexpr (COUNTED) {
        listed = counts[(size_t)gq * COUNT_PITCH];
        if (gq == 0 && tid == 0) *again.work_counter = 0u;
        if (listed < (uint32_t)topk || listed > cap) {
            // (the bound of a short list is none, but the sample's topk-th key is one, if it has counted as many)
            uint32_t *const bins = again.hist + (size_t)gq * HIST_BINS;
            if (tid < 64 && listed < (uint32_t)topk) {
                const int bin = hist_threshold(bins, topk);
                if (tid == 0) again.tau_key[gq] = (uint64_t)(bin < hist_bins ? (uint32_t)bin : 0x7fffu) << 32 | 0xffffffffull;
            }
            __syncthreads();
            for (int i = tid; i < HIST_BINS; i += blockDim.x) bins[i] = 0u;
            if (tid == 0) again.query[atomicAdd(again.count, 1u)] = (uint32_t)gq;
            return;
        }
    }
    const size_t nlists = COUNTED ? (size_t)((listed + 63u) / 64u) : qlist_off ? (size_t)(qlist_off[gq + 1] - qlist_off[gq]) : (size_t)nchunks;
    // Every list is packed (its keys first, KEY_EMPTY behind them; kpad is a multiple of 64): a wave
    // takes whole lists, 64 keys at a time, and leaves a list at the first empty slot it sees.
    const int wave = tid >> 6, lane = tid & 63, nwaves = (int)(blockDim.x >> 6);
    // (The first 64 keys of four lists are requested together, and the rest of a list whose first 64 places are taken five
    // pieces at a time: otherwise a walk over a thousand short lists, or the 16 pieces of a full list of 1024 keys, is a chain of
    // memory round trips.  8 queries, 24 lists of up to 1024 keys each: 271 -> 79 us with the selections below.)
    auto list_ptr = [&](size_t l) {
        if constexpr (COUNTED) return partial + (size_t)gq * cap + l * 64;
        const size_t list = qlist_off ? (size_t)qlist_off[gq] + l : (l * ngroups + slot / per) * qb + slot % per;
        return partial + list * kpad;
    };
    constexpr int MLP = 4, REST = 5;
    auto load_heads = [&](size_t l0, uint64_t (&first)[MLP]) {
#pragma unroll
        for (int u = 0; u < MLP; ++u) {
            const size_t l = l0 + (size_t)u * nwaves;
            first[u] = l < nlists && (!COUNTED || (uint32_t)l * 64u + (uint32_t)lane < listed) ? list_ptr(l)[lane] : KEY_EMPTY;
        }
    };
    auto for_each_key = [&](auto &&f, uint64_t (&first)[MLP], bool loaded) {
        for (size_t l0 = wave; l0 < nlists; l0 += (size_t)MLP * nwaves) {
            if (!loaded) load_heads(l0, first);
            loaded = false;
            uint32_t full = 0;   // lists whose first 64 places are taken
#pragma unroll
            for (int u = 0; u < MLP; ++u) {
                f(first[u]);
                full |= __ballot(first[u] == KEY_EMPTY) == 0ull ? 1u << u : 0u;
            }
#pragma unroll 1
            for (; full != 0u; full &= full - 1u) {
                const uint64_t *const lp = list_ptr(l0 + (size_t)__builtin_ctz(full) * nwaves);
                bool more = true;
#pragma unroll 1
                for (int e0 = 64; more && e0 < kpad; e0 += 64 * REST) {
                    uint64_t key[REST];
#pragma unroll
                    for (int r = 0; r < REST; ++r) key[r] = e0 + 64 * r < kpad ? lp[e0 + 64 * r + lane] : KEY_EMPTY;
#pragma unroll
                    for (int r = 0; r < REST; ++r) {
                        if (!more) break;
                        f(key[r]);
                        more = __ballot(key[r] == KEY_EMPTY) == 0ull;
                    }
                }
            }
        }
    };
    uint64_t heads[MLP];
    load_heads(wave, heads);
    // keys up to `most` go to LDS, as many as there is room for
    auto keep = [&](uint64_t key, uint64_t most) {
        const bool in = key != KEY_EMPTY && key <= most;
        const int at = wave_place(&s_count, in);
        if (in && at < MERGE_CAP) skeys[at] = key;
    };
    // The topk-th smallest of the first `cnt` kept keys (cnt > topk): radix selection of its value, then of the row among the
    // keys that tie with it.
    uint32_t *vals = reinterpret_cast<uint32_t *>(skeys + MERGE_CAP);          // [MERGE_CAP]
    uint64_t *shortlist = skeys + MERGE_CAP + MERGE_CAP / 2;                   // [1024]
    __shared__ uint32_t sel_bins[256], sel_state[2];
    __shared__ int s_below, s_ties;
    auto kth_kept = [&](int cnt) -> uint64_t {
        for (int i = tid; i < cnt; i += blockDim.x) vals[i] = (uint32_t)(skeys[i] >> 32);
        if (tid == 0) { s_below = 0; s_ties = 0; }
        __syncthreads();
        const uint32_t vk = block_kth_smallest_u32(vals, cnt, (uint32_t)topk, sel_bins, sel_state);
        // rows of the keys that tie with the topk-th value (into vals, which has served its purpose), keys below it counted
        __syncthreads();
        int below = 0;
        for (int i = tid; i < cnt; i += blockDim.x) {
            const uint32_t v = (uint32_t)(skeys[i] >> 32);
            below += v < vk ? 1 : 0;
        }
        for (int o = 32; o > 0; o >>= 1) below += __shfl_xor(below, o);
        if (lane == 0) atomicAdd(&s_below, below);
        for (int i = tid; i < cnt; i += blockDim.x) {
            const uint64_t key = skeys[i];
            const bool tie = (uint32_t)(key >> 32) == vk;
            const int at = wave_place(&s_ties, tie);
            if (tie) vals[at] = (uint32_t)key;
        }
        __syncthreads();
        const uint32_t rk = block_kth_smallest_u32(vals, s_ties, (uint32_t)(topk - s_below), sel_bins, sel_state);
        __syncthreads();
        return ((uint64_t)vk << 32) | rk;
    };
    // The topk-th smallest key at or below `most`, of which the lists hold more than topk: radix selection, one byte of the key
    // and one walk over the lists per pass, most significant byte first.
    auto kth_of_lists = [&](uint64_t most) -> uint64_t {
        uint64_t prefix = 0;
        uint32_t want = (uint32_t)topk;
        __shared__ uint32_t sel_byte;
        for (int shift = 56; shift >= 0; shift -= 8) {
            for (int i = tid; i < 256; i += blockDim.x) sel_bins[i] = 0u;
            __syncthreads();
            const uint64_t fixed = shift == 56 ? 0ull : ~0ull << (shift + 8);   // bytes decided in earlier passes
            for_each_key([&](uint64_t key) {
                wave_count_bin(sel_bins, key != KEY_EMPTY && key <= most && (key & fixed) == prefix, (uint32_t)(key >> shift) & 255u);
            }, heads, false);
            __syncthreads();
            if (tid < 64) {   // one wave: the byte value whose bin holds the `want`-th key
                const uint32_t h[4] = {sel_bins[4 * tid], sel_bins[4 * tid + 1], sel_bins[4 * tid + 2], sel_bins[4 * tid + 3]};
                const uint32_t tot = h[0] + h[1] + h[2] + h[3];
                uint32_t incl = tot;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const uint32_t up = __shfl_up(incl, o);
                    if (tid >= o) incl += up;
                }
                const uint64_t reach = __ballot(incl >= want);   // (not empty: there are more than topk such keys)
                if (reach != 0ull && tid == __builtin_ctzll(reach)) {
                    uint32_t cum = incl - tot;
                    int b = 4 * tid;
                    for (int t = 0; t < 3 && cum + h[t] < want; ++t) { cum += h[t]; ++b; }
                    sel_byte = (uint32_t)b;
                    sel_state[0] = want - cum;
                }
            }
            __syncthreads();
            prefix |= (uint64_t)sel_byte << shift;
            want = sel_state[0];
            __syncthreads();
        }
        return prefix;
    };
    // More keys at or below the bound than there is room for (loose bounds, massive ties): the topk-th smallest of those
    // kept is a bound as well, usually a far better one, and the lists are walked once more.  Two walks are the rule.  But a
    // round is only sure to rule out the MERGE_CAP - topk greatest of the kept keys, and keys that are met from the
    // greatest to the smallest would make it a round for every few lists (520 queries with 1024 lists of 128 keys: call 20 ms, now 6.1), so
    // after three walks the topk-th key is selected exactly, in eight.
    uint64_t bound = tau_key[gq];   // a whole key at or below which k keys exist (rows separate ties of the value)
    // The scan's histogram of the keys that any block inserted is complete by now, where each block's last look at it was not:
    // the edge of the bin that holds the k-th.  (25 M codes of 16 4-bit indexes, 8 queries, top-1000: 29 000 keys at or below the
    // shared bound, 3000 below the edge.)
    if (hist != nullptr) {
        __shared__ uint64_t s_edge;
        if (wave == 0) {
            const int bin = hist_threshold(hist + (size_t)gq * HIST_BINS, topk);
            const uint32_t ref = VAL_U32 ? 0u : hist_ref[gq];
            uint64_t edge = KEY_EMPTY;
            if (bin < hist_bins && ref != TAU_REF_UNSET)
                edge = (uint64_t)(VAL_U32 ? (uint32_t)bin : ref - ((uint32_t)(HIST_BINS - 1 - bin) << HIST_SHIFT)) << 32 | 0xffffffffull;
            if (lane == 0) s_edge = edge;
        }
        __syncthreads();
        if (s_edge < bound) bound = s_edge;
    }
    int kept;
    for (int walk = 1;; ++walk) {
        if (tid == 0) s_count = 0;
        __syncthreads();
        for_each_key([&](uint64_t key) { keep(key, bound); }, heads, walk == 1);
        __syncthreads();
        kept = s_count;
        __syncthreads();
        if (kept <= MERGE_CAP) break;
        bound = walk < 3 ? kth_kept(MERGE_CAP) : kth_of_lists(bound);
    }
    auto emit = [&](int i, uint64_t key) {
        const bool empty = key == KEY_EMPTY;
        const uint32_t row = (uint32_t)key;
        if (VAL_U32) ((uint32_t *)out_val)[(size_t)gq * topk + i] = empty ? 0xffffffffu : (uint32_t)(key >> 32);
        else ((float *)out_val)[(size_t)gq * topk + i] = empty ? __builtin_inff() : ord_to_f32((uint32_t)(key >> 32));
        out_ids[(size_t)gq * topk + i] = empty ? -1 : (ids ? ids[row] : (int64_t)row);
    };
    // The topk smallest of the kept keys without sorting them all (a bitonic sort of a few thousand keys is dozens of
    // barrier stages): the keys up to the topk-th are moved to a short list, where every thread finds the rank of its keys by
    // counting the smaller ones and writes them straight to their places.
    // (a few hundred keys at once)
    int nshort = kept;
    uint64_t *src = skeys;
    if (kept > topk && kept > MERGE_COUNT) {
        const uint64_t kth = kth_kept(kept);
        if (tid == 0) s_count = 0;
        __syncthreads();
        for (int i = tid; i < kept; i += blockDim.x) {
            const uint64_t key = skeys[i];
            const int at = wave_place(&s_count, key <= kth);
            if (key <= kth) shortlist[at] = key;   // exactly topk keys (keys are distinct)
        }
        __syncthreads();
        nshort = s_count;
        src = shortlist;
    }
    if (nshort > MERGE_COUNT) {
        // long results: counting the smaller keys is nshort^2 broadcast reads (a thousand keys: 40 us of LDS time on a
        // compute unit that holds four such blocks); the short list is sorted instead (at most 1024 keys: 55 stages)
        uint64_t *buf = src;   // (nshort <= topk <= 1024 either way)
        int n2 = 512;
        while (n2 < nshort) n2 <<= 1;
        for (int i = nshort + tid; i < n2; i += blockDim.x) buf[i] = KEY_EMPTY;
        block_bitonic_sort(buf, n2);
        for (int i = tid; i < topk; i += blockDim.x) emit(i, i < nshort ? buf[i] : KEY_EMPTY);
        return;
    }
    for (int i = tid; i < nshort; i += blockDim.x) {
        const uint64_t mine = src[i];
        int rank = 0;
        for (int j = 0; j < nshort; ++j) rank += src[j] < mine ? 1 : 0;
        if (rank < topk) emit(rank, mine);
    }
    for (int i = nshort + tid; i < topk; i += blockDim.x) emit(i, KEY_EMPTY);
}

int launch_merge_filtered(pq_ctx *ctx, const uint64_t *partial, const uint32_t *qlist_off, int nchunks, int ngroups, int qb,
                          const unsigned long long *tau_key, int kpad, int nq, int topk, const int64_t *ids, bool val_u32,
                          void *out_val, int64_t *out_ids, const uint32_t *hist, const uint32_t *hist_ref, int hist_bins) {
    if (nq == 0) return PQ_OK;
    // (the histograms' bound: 16 KB read per query; with many queries the keys are fewer and the selection is the shorter way:
    // 1000 queries, top-100 34 us without, 44 with)
    auto launch = [&](auto kernel, int cap, int threads, const uint32_t *hist = nullptr) -> int {
        PQ_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, merge_lds_bytes(cap)));
        kernel<<<nq, threads, merge_lds_bytes(cap), ctx->stream>>>(partial, qlist_off, nchunks, ngroups, qb, tau_key, kpad, topk, ids, out_val, out_ids, hist, hist_ref, hist_bins, nullptr, 0u, AgainArgs{});
        PQ_HIP(ctx, hipGetLastError());
        return PQ_OK;
    };
    // calls of many queries: several smaller blocks per compute unit (room for at least four times topk keys)
    const bool many = nq >= 2 * ctx->num_cu;
    if (many && topk <= 512) {
        if (val_u32) return launch(merge_filtered_kernel<true, 2048>, 2048, 256);
        return launch(merge_filtered_kernel<false, 2048>, 2048, 256);
    }
    if (many) {
        if (val_u32) return launch(merge_filtered_kernel<true, 4096>, 4096, 512);
        return launch(merge_filtered_kernel<false, 4096>, 4096, 512);
    }
    // (nor where few lists cannot hold more keys than there is room for: 22 034 codes, 135 queries, top-19, call 56 us without, 61 with)
    if ((int64_t)nchunks * kpad <= 8192) hist = nullptr;
    if (val_u32) return launch(merge_filtered_kernel<true, 8192>, 8192, 1024, hist);
    return launch(merge_filtered_kernel<false, 8192>, 8192, 1024, hist);
}

int launch_merge_counted(pq_ctx *ctx, const uint64_t *lists, const uint32_t *counts, uint32_t cap, const AgainArgs &again, int nq, int topk,
                         void *out_val, int64_t *out_ids, int hist_bins) {
    auto launch = [&](auto kernel, int room, int threads) -> int {   // (sized as above)
        PQ_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, merge_lds_bytes(room)));
        kernel<<<nq, threads, merge_lds_bytes(room), ctx->stream>>>(lists, nullptr, 0, 1, 1, again.tau_key, 64, topk, nullptr, out_val, out_ids, nullptr, nullptr, hist_bins, counts, cap, again);
        PQ_HIP(ctx, hipGetLastError());
        return PQ_OK;
    };
    const bool many = nq >= 2 * ctx->num_cu;
    if (many && topk <= 512) return launch(merge_filtered_kernel<true, 2048, MERGE_COUNTED>, 2048, 256);
    if (many) return launch(merge_filtered_kernel<true, 4096, MERGE_COUNTED>, 4096, 512);
    return launch(merge_filtered_kernel<true, 8192, MERGE_COUNTED>, 8192, 1024);
}

int launch_merge_again(pq_ctx *ctx, const uint64_t *partial, const AgainArgs &again, int kpad, int nq, int topk, void *out_val, int64_t *out_ids,
                       int hist_bins) {
    auto kernel = merge_filtered_kernel<true, 8192, MERGE_AGAIN>;
    PQ_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, merge_lds_bytes(8192)));
    kernel<<<nq, 1024, merge_lds_bytes(8192), ctx->stream>>>(partial, nullptr, again.nchunks, 1, again.qb, again.tau_key, kpad, topk, nullptr, out_val, out_ids, again.hist, nullptr, hist_bins, nullptr, 0u, again);
    PQ_HIP(ctx, hipGetLastError());
    return PQ_OK;
}

// ------------------------------------------------------------------------------------------
static int next_pow2(int x) { int p = 1; while (p < x) p <<= 1; return p; }

int launch_merge_topk(pq_ctx *ctx, const uint64_t *partial, int nchunks, int ngroups, int qb, int kpad, int nq,
                      int topk, bool val_u32, void *out_val, int64_t *out_ids) {
    const int n2 = next_pow2(nchunks * kpad);
    if (n2 > 16384) return fail(ctx, PQ_EUNSUPPORTED, "merge: %d keys per query exceed the LDS sort", n2);
    const int mthreads = n2 / 2 < 1024 ? (n2 / 2 < 64 ? 64 : n2 / 2) : 1024;
    if (val_u32) {
        PQ_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(merge_topk_kernel<true>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 131072));
        merge_topk_kernel<true><<<nq, mthreads, (size_t)n2 * 8, ctx->stream>>>(partial, nchunks, ngroups, qb, kpad, n2,
                                                                               topk, out_val, out_ids);
    } else {
        PQ_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void *>(merge_topk_kernel<false>),
                                        hipFuncAttributeMaxDynamicSharedMemorySize, 131072));
        merge_topk_kernel<false><<<nq, mthreads, (size_t)n2 * 8, ctx->stream>>>(partial, nchunks, ngroups, qb, kpad, n2,
                                                                                topk, out_val, out_ids);
    }
    PQ_HIP(ctx, hipGetLastError());
    return PQ_OK;
}

// General kernel: one block per (chunk, query).
static int run_generic(pq_ctx *ctx, const uint8_t *codes, int64_t n, int cf, const void *luts, bool lut_u8, int nq,
                       int m, int k, int topk, void *out_val, int64_t *out_ids) {
    const bool small = topk <= 128;
    const int kpad = small ? 128 : 1024, cap = 2 * kpad, qb = 1;
    const int ngroups = nq;
    const int64_t block_tile = 64 * SCAN_WAVES;
    // enough blocks to keep every CU busy for several rounds, but chunks of at least 8 block tiles
    int64_t nchunks = (16 * ctx->num_cu + ngroups - 1) / ngroups;
    const int64_t max_by_n = (n + 8 * block_tile - 1) / (8 * block_tile);
    const int64_t max_by_merge = 16384 / kpad;
    if (nchunks > max_by_n) nchunks = max_by_n;
    if (nchunks > max_by_merge) nchunks = max_by_merge;
    if (nchunks < 1) nchunks = 1;
    int64_t chunk_codes = (n + nchunks - 1) / nchunks;
    chunk_codes = (chunk_codes + block_tile - 1) / block_tile * block_tile;
    if (chunk_codes < block_tile) chunk_codes = block_tile;
    nchunks = n > 0 ? (n + chunk_codes - 1) / chunk_codes : 1;
    const int64_t nblocks = nchunks * ngroups;
    if (nblocks > 0x7fffffff) return fail(ctx, PQ_EUNSUPPORTED, "scan grid too large (%lld blocks)", (long long)nblocks);

    const size_t tau_bytes = align_up((size_t)ngroups * qb * sizeof(uint32_t), 256);
    const size_t scratch_bytes = (size_t)nblocks * SCAN_WAVES * qb * cap * sizeof(uint64_t);
    const size_t partial_bytes = (size_t)nblocks * qb * kpad * sizeof(uint64_t);
    int rc = ws_reserve(ctx, tau_bytes + scratch_bytes + partial_bytes);
    if (rc) return rc;
    uint8_t *ws = (uint8_t *)ctx->ws;

    ScanArgs a;
    a.codes = codes; a.n = n; a.chunk_codes = chunk_codes; a.nchunks = (int)nchunks; a.ngroups = ngroups;
    a.luts = luts; a.nq = nq; a.topk = topk;
    a.tau_global = (uint32_t *)ws;
    a.scratch = (uint64_t *)(ws + tau_bytes);
    a.partial = (uint64_t *)(ws + tau_bytes + scratch_bytes);

    const int ntau = ngroups * qb;
    init_tau_kernel<<<(ntau + 255) / 256, 256, 0, ctx->stream>>>(a.tau_global, ntau,
                                                                 lut_u8 ? 0xfffffffeu : 0xff800000u /* ordered +inf */);
    PQ_HIP(ctx, hipGetLastError());
    if (ctx->profiling) {
        note_plain_scan(ctx, "scan_generic_kernel (one query per block)", 1, nq);
        PQ_HIP(ctx, hipEventRecord(ctx->ev_begin, ctx->stream));
    }
    hipStream_t s = ctx->stream;
    if (lut_u8) {
        if (small) scan_generic_kernel<true, 4, 128><<<nblocks, SCAN_THREADS, 0, s>>>(a, m, k, cf);
        else scan_generic_kernel<true, 32, 1024><<<nblocks, SCAN_THREADS, 0, s>>>(a, m, k, cf);
    } else {
        if (small) scan_generic_kernel<false, 4, 128><<<nblocks, SCAN_THREADS, 0, s>>>(a, m, k, cf);
        else scan_generic_kernel<false, 32, 1024><<<nblocks, SCAN_THREADS, 0, s>>>(a, m, k, cf);
    }
    PQ_HIP(ctx, hipGetLastError());
    if (ctx->profiling) {
        PQ_HIP(ctx, hipEventRecord(ctx->ev_end, ctx->stream));
        ctx->ev_valid = 1;
    }
    return launch_merge_topk(ctx, a.partial, (int)nchunks, ngroups, qb, kpad, nq, topk, lut_u8, out_val, out_ids);
}

// 32-bit codes (see scan_codes4_kernel).  The sample: its counting costs about as much as the candidates its bound lets
// through, topk n / sample per query, near 4 sqrt(topk n) codes.
static int run_codes4(pq_ctx *ctx, const uint8_t *codes, int64_t n, const float *luts, int nq, int topk, void *out_val, int64_t *out_ids) {
    const bool small = topk <= 128;
    const int kpad = small ? 128 : 1024, cap = small ? 256 : 2048;
    Codes4Args a;
    a.codes = (const uint32_t *)codes; a.n = n; a.nq = nq; a.topk = topk; a.luts = luts;
    a.ngroups = (nq + C4_QB - 1) / C4_QB;
    // chunks for one round of two blocks per CU, of at least 4096 codes; large ones in four rounds, of which the later find
    // the bounds of the earlier
    int64_t nchunks = 2 * ctx->num_cu / a.ngroups;
    if (nchunks > n / 4096) nchunks = n / 4096;
    if (nchunks >= 1 && n / nchunks >= (1 << 17)) nchunks = 8 * ctx->num_cu / a.ngroups;
    if (nchunks < (n >> 28) + 1) nchunks = (n >> 28) + 1;   // (rows of an item are counted in 32 bits)
    a.chunk_codes = ((n + nchunks - 1) / nchunks + 255) / 256 * 256;
    nchunks = (n + a.chunk_codes - 1) / a.chunk_codes;
    a.nitems = (int)(nchunks * a.ngroups);
    const int nblocks = a.nitems < 2 * ctx->num_cu ? a.nitems : 2 * ctx->num_cu;
    int64_t sample = (int64_t)(4.0 * sqrt((double)topk * (double)n));
    if (sample < 16 * (int64_t)topk) sample = 16 * (int64_t)topk;
    a.nsample = sample < n ? sample : n;

    const size_t tau_bytes = align_up((size_t)nq * 8, 256), ref_bytes = align_up((size_t)nq * 4, 256), hist_bytes = (size_t)nq * HIST_BINS * 4;
    const size_t scratch_bytes = (size_t)nblocks * SCAN_WAVES * C4_QB * cap * 8;
    int rc = ws_reserve(ctx, tau_bytes + 2 * ref_bytes + hist_bytes + scratch_bytes + (size_t)a.nitems * C4_QB * kpad * 8);
    if (rc) return rc;
    uint8_t *ws = (uint8_t *)ctx->ws;
    a.tau_key = (unsigned long long *)ws; ws += tau_bytes;
    a.ref = (uint32_t *)ws; ws += ref_bytes;
    a.margin = (float *)ws; ws += ref_bytes;
    a.hist = (uint32_t *)ws; ws += hist_bytes;
    a.scratch = (uint64_t *)ws; ws += scratch_bytes;
    a.partial = (uint64_t *)ws;

    hipStream_t s = ctx->stream;
    codes4_clear_kernel<<<nq < 1024 ? nq : 1024, 256, 0, s>>>((uint4 *)a.hist, hist_bytes / 16);
    PQ_HIP(ctx, hipGetLastError());
    // slices for four blocks per CU, of at least 2048 codes
    const int64_t per_query = 4 * ctx->num_cu / nq > 1 ? 4 * ctx->num_cu / nq : 1;
    int64_t slice = ((a.nsample + per_query - 1) / per_query + 2047) / 2048 * 2048;
    const int nslices = (int)((a.nsample + slice - 1) / slice);
    codes4_sample_kernel<<<(unsigned)nslices * (unsigned)nq, SCAN_THREADS, 0, s>>>(a, (int)slice, nslices);
    PQ_HIP(ctx, hipGetLastError());
    codes4_pick_kernel<<<nq, 64, 0, s>>>(a);
    PQ_HIP(ctx, hipGetLastError());
    if (ctx->profiling) {
        note_plain_scan(ctx, "scan_codes4_kernel (4 queries per block)", C4_QB, a.ngroups);
        PQ_HIP(ctx, hipEventRecord(ctx->ev_begin, s));
    }
    if (small) scan_codes4_kernel<4, 128><<<nblocks, SCAN_THREADS, 0, s>>>(a);
    else scan_codes4_kernel<32, 1024><<<nblocks, SCAN_THREADS, 0, s>>>(a);
    PQ_HIP(ctx, hipGetLastError());
    if (ctx->profiling) {
        PQ_HIP(ctx, hipEventRecord(ctx->ev_end, s));
        ctx->ev_valid = 1;
    }
    return launch_merge_filtered(ctx, a.partial, nullptr, (int)nchunks, a.ngroups, C4_QB, a.tau_key, kpad, nq, topk, nullptr, false,
                                 out_val, out_ids, a.hist, a.ref, HIST_BINS);
}

int launch_scan(pq_ctx *ctx, const uint8_t *codes, int64_t n, int cf, const void *luts, int lf, int nq, int m, int k,
                int topk, void *out_val, int64_t *out_ids) {
    const bool general = opt_int(ctx, PQ_OPT_SCAN_FORCE_GENERAL, 0) != 0;
    if (!general && cf == PQ_CODES_U8 && lf == PQ_LUT_F32 && k == 256 && (m == 8 || m == 16))
        return w16::launch_scan_tuned(ctx, m == 8 ? 0 : 1, codes, n, luts, nq, topk, out_val, out_ids);
    if (!general && cf == PQ_CODES_U4_PACKED && lf == PQ_LUT_U8 && k == 16 && m == 16)
        return w16::launch_scan_tuned(ctx, 2, codes, n, luts, nq, topk, out_val, out_ids);
    // 32 tables: scan of 1 M codes, 100 queries, top-1000 10.5 -> 0.24 ms, two-pass call 10.8 -> 0.38.  Under 1024 codes and
    // with short results the general kernel's single launch is the shorter way (300 codes, 29 queries, call 60 us against 79;
    // 2500 codes 100 against 78), and so it is where every code is in the result (600 codes, 29 queries, top-1000: 34 us against
    // 97; top-500 208 against 103).  With the fixed scratch of the call that allocates nothing, requests that do not fit there go
    // on to the general kernel, which may need less.
    if (!general && cf == PQ_CODES_U4_PACKED && lf == PQ_LUT_U8 && k == 16 && m == 32 && (n >= 1024 || (topk > 128 && n > topk))) {
        const int rc = w16::launch_scan_tuned(ctx, 7, codes, n, luts, nq, topk, out_val, out_ids);
        if (!(rc == PQ_ENOMEM && ctx->ws_fixed)) return rc;
    }
    if (!general && cf == PQ_CODES_U8 && lf == PQ_LUT_F32 && k == 256 && m == 4 && n >= C4_MIN_N) {
        const int rc = run_codes4(ctx, codes, n, (const float *)luts, nq, topk, out_val, out_ids);
        if (!(rc == PQ_ENOMEM && ctx->ws_fixed)) return rc;
    }
    if ((int64_t)m * k <= 8192)
        return run_generic(ctx, codes, n, cf, luts, lf == PQ_LUT_U8, nq, m, k, topk, out_val, out_ids);
    return fail(ctx, PQ_EUNSUPPORTED, "scan: no kernel for m=%d k=%d code_fmt=%d lut_fmt=%d", m, k, cf, lf);
}

}  // namespace pq
