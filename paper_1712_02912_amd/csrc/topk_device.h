// Device-side building blocks of the top-k selection used by the scan kernels.
//
// A candidate is one 64-bit key: (ordered value << 32) | id.  Unsigned comparison of keys
// is the total order (value, id) of Alg. 1's heap, so "the k smallest keys" is exactly the
// content of that heap after the scan.  For float values the upper word is the usual
// order-preserving map of IEEE-754 bits to unsigned integers.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pq {

constexpr uint64_t KEY_EMPTY = ~0ull;

__device__ __forceinline__ uint32_t f32_to_ord(float f) {
    uint32_t b = __float_as_uint(f);
    return b ^ ((b >> 31) ? 0xffffffffu : 0x80000000u);
}
// The same with every NaN behind all numbers (above, one with its sign set comes first): a distance that is none is no result.
__device__ __forceinline__ uint32_t f32_to_ord_nan_last(float f) { return f == f ? f32_to_ord(f) : 0xffffffffu; }
__device__ __forceinline__ float ord_to_f32(uint32_t o) {
    uint32_t b = o ^ ((o >> 31) ? 0x80000000u : 0xffffffffu);
    return __uint_as_float(b);
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }

// number of set bits of `mask` below this lane
__device__ __forceinline__ int mask_prefix(uint64_t mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// Candidate lists in device scratch are written and read back by different lanes of a wave and,
// when a block merges its lists, by different waves of the same block: never by another block.
// Work-group scope is therefore enough, which keeps the lists in the caches of the block's own CU
// and XCD (device scope would send every access, and every fence, past the L2 to memory).
__device__ __forceinline__ void key_store(uint64_t *p, uint64_t v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint64_t key_load(const uint64_t *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// orders the list accesses of the block's waves (stores before, loads after)
__device__ __forceinline__ void list_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup"); }

// k-th smallest (1-based) of the wave's 64*E keys, by bitwise bisection on the key value:
// the smallest v with count(key <= v) >= k.  Every lane must call it; the result is uniform.
// If fewer than k non-empty keys exist the result is KEY_EMPTY.
template <int E>
__device__ __forceinline__ uint64_t wave_select_kth(const uint64_t (&key)[E], int k) {
    uint64_t v = 0;
    for (int bit = 63; bit >= 0; --bit) {
        const uint64_t trial = v | ((1ull << bit) - 1ull);
        int c = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) c += __popcll(__ballot(key[e] <= trial));
        if (c < k) v |= (1ull << bit);
    }
    return v;
}

// Keep the k smallest of buf[0..cnt) (cnt <= 64*E) in buf[0..min(cnt,k)), in no particular
// order.  Returns a key t with exactly min(cnt,k) keys <= t, at least the k-th smallest key
// (KEY_EMPTY if cnt < k), and updates cnt.  Lists of up to 512 keys are held in registers;
// longer ones are re-read from memory in every bisection step (rare path, few registers).
template <int E>
__device__ __forceinline__ uint64_t wave_compact(uint64_t *buf, int &cnt, int k) {
    const int lane = lane_id();
    list_fence();  // the appends of every lane are visible to the other lanes
    if constexpr (E <= 8) {
        uint64_t key[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int idx = e * 64 + lane;
            key[e] = idx < cnt ? key_load(buf + idx) : KEY_EMPTY;
        }
        const uint64_t kth = wave_select_kth<E>(key, k);
        int base = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const bool keep = key[e] <= kth && key[e] != KEY_EMPTY;
            const uint64_t mask = __ballot(keep);
            if (keep) key_store(buf + base + mask_prefix(mask), key[e]);
            base += __popcll(mask);
        }
        cnt = base;
        return kth;
    } else {
        uint64_t v = 0;
        for (int bit = 63; bit >= 0; --bit) {
            const uint64_t trial = v | ((1ull << bit) - 1ull);
            int c = 0;
#pragma unroll 8
            for (int e = 0; e < E; ++e) {
                const int idx = e * 64 + lane;
                const uint64_t key = idx < cnt ? key_load(buf + idx) : KEY_EMPTY;
                c += __popcll(__ballot(key <= trial));
            }
            if (c == k) { v = trial; break; }   // exactly k keys at or below the trial: good enough
            if (c < k) v |= (1ull << bit);
        }
        // in-place compaction, 64 keys per round: the write position never passes the read position
        int base = 0;
#pragma unroll 4
        for (int e = 0; e < E; ++e) {
            const int idx = e * 64 + lane;
            const uint64_t key = idx < cnt ? key_load(buf + idx) : KEY_EMPTY;
            const bool keep = key <= v && key != KEY_EMPTY;
            const uint64_t mask = __ballot(keep);
            if (keep) key_store(buf + base + mask_prefix(mask), key);
            base += __popcll(mask);
        }
        cnt = base;
        return v;
    }
}

// Append the lanes with `pass` set to buf at position cnt (uniform).  Returns the new count.
__device__ __forceinline__ int wave_append(uint64_t *buf, int cnt, bool pass, uint64_t key) {
    const uint64_t mask = __ballot(pass);
    if (pass) key_store(buf + cnt + mask_prefix(mask), key);
    return cnt + __popcll(mask);
}

// One more in bins[bin] (LDS) for every lane with `in` set.  Values that share their leading bytes count in one bin, and 64
// atomics to one address are served one after the other: the lanes that share the first lane's bin add together.
__device__ __forceinline__ void wave_count_bin(uint32_t *bins, bool in, uint32_t bin) {
    const uint64_t mask = __ballot(in);
    if (mask == 0ull) return;
    const int first = __builtin_ctzll(mask);
    const uint32_t common = __builtin_amdgcn_readlane(bin, first);
    const uint64_t same = __ballot(in && bin == common);
    if (lane_id() == first) atomicAdd(&bins[common], (uint32_t)__popcll(same));
    if (in && bin != common) atomicAdd(&bins[bin], 1u);
}

// A place from the counter *count (LDS) for every lane with `in` set: one atomic per wave.
__device__ __forceinline__ int wave_place(int *count, bool in) {
    const uint64_t mask = __ballot(in);
    if (mask == 0ull) return 0;
    const int first = __builtin_ctzll(mask);
    int at = 0;
    if (lane_id() == first) at = atomicAdd(count, __popcll(mask));
    return __builtin_amdgcn_readlane(at, first) + (int)mask_prefix(mask);
}

// The k-th smallest (k = 1 .. n) of n 32-bit values in LDS, by the whole block (at least 256 threads), by radix
// selection, most significant byte first: four rounds of a 256-bin count over the values that share the bytes
// fixed so far.  `bins`: 256 LDS words, `state`: 2 LDS words.  Every thread gets the value; a few barriers in all.
__device__ inline uint32_t block_kth_smallest_u32(const uint32_t *vals, int n, uint32_t k, uint32_t *bins, uint32_t *state) {
    const int tid = threadIdx.x;
    if (tid == 0) { state[0] = 0u; state[1] = k; }
    for (int pass = 3; pass >= 0; --pass) {
        if (tid < 256) bins[tid] = 0u;
        __syncthreads();
        const int shift = 8 * pass;
        const uint32_t fixed = pass == 3 ? 0u : 0xffffffffu << (shift + 8);   // bytes decided in earlier rounds
        const uint32_t prefix = state[0], want = state[1];
        for (int i = tid; i < n; i += blockDim.x) {
            const uint32_t v = vals[i];
            wave_count_bin(bins, (v & fixed) == prefix, (v >> shift) & 255u);
        }
        __syncthreads();
        if (tid < 64) {   // one wave: the byte value whose bin holds the `want`-th value
            const uint32_t h[4] = {bins[4 * tid], bins[4 * tid + 1], bins[4 * tid + 2], bins[4 * tid + 3]};
            const uint32_t tot = h[0] + h[1] + h[2] + h[3];
            uint32_t incl = tot;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t up = __shfl_up(incl, o);
                if (tid >= o) incl += up;
            }
            const uint64_t reach = __ballot(incl >= want);   // never empty: want <= values that share the prefix
            if (reach != 0ull && tid == __builtin_ctzll(reach)) {
                uint32_t cum = incl - tot;
                int b = 4 * tid;
                for (int t = 0; t < 3 && cum + h[t] < want; ++t) { cum += h[t]; ++b; }
                state[0] = prefix | ((uint32_t)b << shift);
                state[1] = want - cum;
            }
        }
        __syncthreads();
    }
    return state[0];
}

// The 32 bits that lane ^ STRIDE holds, by lane moves of the vector unit: a shuffle takes each half of a key through LDS instead.
template <int STRIDE>
__device__ __forceinline__ uint32_t wave_xor_u32(uint32_t v) {
    static_assert(STRIDE == 1 || STRIDE == 2 || STRIDE == 4 || STRIDE == 8 || STRIDE == 16 || STRIDE == 32, "a power of two within the wave");
    if constexpr (STRIDE == 1) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0xb1, 0xf, 0xf, true);         // quad_perm [1,0,3,2]
    else if constexpr (STRIDE == 2) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x4e, 0xf, 0xf, true);    // quad_perm [2,3,0,1]
    else if constexpr (STRIDE == 4)                                                                             // half row mirrored (^ 7), quads mirrored (^ 3)
        return (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp((int)v, 0x141, 0xf, 0xf, true), 0x1b, 0xf, 0xf, true);
    else if constexpr (STRIDE == 8) return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x128, 0xf, 0xf, true);   // row of 16 rotated by 8
    else if constexpr (STRIDE == 16) {   // odd rows of the first with even rows of the second: the pair's lower row twice, its upper row twice
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (lane_id() & 16) ? r[0] : r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return (lane_id() & 32) ? r[0] : r[1];
    }
}

// One step of a bitonic network within the wave: the key of lane ^ STRIDE, the smaller one kept by the lower lane where `up`.
template <int STRIDE>
__device__ __forceinline__ uint64_t wave_bitonic_step(uint64_t key, int lane, bool up) {
    const uint64_t other = (uint64_t)wave_xor_u32<STRIDE>((uint32_t)(key >> 32)) << 32 | wave_xor_u32<STRIDE>((uint32_t)key);
    const bool keep_small = ((lane & STRIDE) == 0) == up;
    return (other < key) == keep_small ? other : key;
}
// The steps of strides STRIDE, STRIDE / 2 .. 1.
template <int STRIDE>
__device__ __forceinline__ uint64_t wave_bitonic_merge(uint64_t key, int lane, bool up) {
    key = wave_bitonic_step<STRIDE>(key, lane, up);
    if constexpr (STRIDE > 1) key = wave_bitonic_merge<STRIDE / 2>(key, lane, up);
    return key;
}

// In-LDS bitonic sort (ascending) of n2 keys, n2 a power of two, by the whole block: few registers and little code, a barrier
// per step.
__device__ inline void block_bitonic_sort_plain(uint64_t *s, int n2) {
    for (int size = 2; size <= n2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            __syncthreads();
            for (int i = threadIdx.x; i < (n2 >> 1); i += blockDim.x) {
                const int lo = 2 * i - (i & (stride - 1));
                const int hi = lo + stride;
                const bool asc = (lo & size) == 0;
                const uint64_t a = s[lo], b = s[hi];
                if ((a > b) == asc) { s[lo] = b; s[hi] = a; }
            }
        }
    }
    __syncthreads();
}

// The same for blocks of whole waves and n2 of at least 64: steps between keys less than 64 apart are done by a wave on 64 keys
// in registers, so that only the others cost a barrier (1024 keys: 15 barriers instead of 55; pq_rerank_f32 of 8 x 1000 candidates
// 22 -> 18 us, of 100 27 -> 23, probe selection of one query among 1024 lists 11 -> 9).
__device__ inline void block_bitonic_sort(uint64_t *s, int n2) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwaves = (int)(blockDim.x >> 6);
    if (n2 < 64) { block_bitonic_sort_plain(s, n2); return; }
#pragma unroll 1
    for (int size = 64; size <= n2; size <<= 1) {
#pragma unroll 1
        for (int stride = size >> 1; stride >= 64; stride >>= 1) {
            __syncthreads();
            for (int i = tid; i < (n2 >> 1); i += blockDim.x) {
                const int lo = 2 * i - (i & (stride - 1));
                const int hi = lo + stride;
                const bool asc = (lo & size) == 0;
                const uint64_t a = s[lo], b = s[hi];
                if ((a > b) == asc) { s[lo] = b; s[hi] = a; }
            }
        }
        __syncthreads();
        for (int t = wave; t < (n2 >> 6); t += nwaves) {
            const bool asc = ((t * 64) & size) == 0;
            uint64_t key = s[t * 64 + lane];
            if (size == 64) {   // (sorted from scratch: ascending and descending runs in turn)
                key = wave_bitonic_merge<1>(key, lane, (lane & 2) == 0);
                key = wave_bitonic_merge<2>(key, lane, (lane & 4) == 0);
                key = wave_bitonic_merge<4>(key, lane, (lane & 8) == 0);
                key = wave_bitonic_merge<8>(key, lane, (lane & 16) == 0);
                key = wave_bitonic_merge<16>(key, lane, (lane & 32) == 0);
            }
            key = wave_bitonic_merge<32>(key, lane, asc);
            s[t * 64 + lane] = key;
        }
    }
    __syncthreads();
}

}  // namespace pq
