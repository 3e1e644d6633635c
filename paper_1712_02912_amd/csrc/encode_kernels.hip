// Encoder of the product quantizer (Section 2.3.1): a vector x is cut into m sub-vectors and
// sub-vector x^j is replaced by the index of the closest centroid of codebook j,
//   code_j(x) = argmin_i || x^j - C^j[i] ||^2          (ties: smallest i),
// decided in double.  Two forms:
//   encode_split16_kernel  sub-vectors of up to 64 dimensions: the centroids are ranked by inner products on the fp16
//                          matrix cores (operands as two halves); where the ranking's error bound leaves the nearest
//                          one open, the plain definition in double decides.
//   pq_encode_kernel       longer sub-vectors: the expanded form ||x||^2 + ||c||^2 - 2<x, c> with the inner products
//                          on the fp64 matrix cores, entries that cancel almost completely recomputed from the
//                          differences.
#include "pq_internal.h"

namespace pq {

// ------------------------------------------------------------------------------------------
// Ranking on the fp16 matrix cores.  Both operands are taken relative to the mean centroid of the sub-space (which
// leaves distances alone and makes the operands, and with them the error, small), and multiplied by a power of two S_j
// that brings the largest centroid component into [2^10, 2^11).  Maximised is s_i = <x, c_i> - ||c_i||^2 / 2 (the squared
// distance is ||x||^2 - 2 s_i), with x and c_i split into two fp16 halves.  A 16 x 16 matrix tile has 16 centroids as rows
// and 16 vectors as columns; the 32 products of an instruction are 16 dimensions times (high half, low half) of the
// centroids, against the vectors' high halves and, in a second instruction with the same centroid operand, their low
// halves.  A lane so holds 4 centroids of one vector per tile, and its running best needs no other lane until all
// centroids are done.  The centroid's number within the lane (tile, register) takes the place of the lowest bits of
// s_i, so that the two largest values are kept with 2.25 instructions per value.
//
// |approximate - exact s_i| <= bound (||x||^2 + ||c||_max^2), with P = ||x|| ||c|| + ||c||^2 / 2 <= ||x||^2 / 2 + ||c||_max^2:
//   rounding of x - mean, c - mean   2^-22 P
//   representation in halves         2^-21 P, and where a half falls below fp16's normal range 2^-14 per component, which is
//                                    2^-24 of the largest centroid component: sqrt(dims) 2^-23 (||x||^2 + ||c||_max^2) in all
//   additions                        one unit of 2^-23 of P for each of the 4 dims products, the start value and its rounding
//   number in the low bits           2^-17 P (6 bits of 24)
// The nearest centroid is settled if the second largest value lies more than twice this bound below the largest.  Else
// (also for NaN, infinities and vectors more than 2^4 times larger than the codebook, whose halves may overflow) the
// centroids within twice the bound of the largest value are measured as the definition has it, in double; which these
// are is known if no lane has two of them, else the ranking of the 16 vectors concerned is repeated.
//
// Bound by issue: vector instructions (2.25 per (vector, centroid) pair of a lane) hold the SIMDs for 59 % of the cycles, matrix
// instructions, which do not overlap with them, for 26 %; with 16 centroids 59 % and 4 %, the rest waits for rows.  Measured, against the fp64 form
// below (which reads each centroid tile once per 64 vectors and is bound by fp64 conversions, LDS and the fp64 matrix rate):
//   4 M vectors, d = 128, 8 x 256    17.0 -> 1.7 ms (0.09 ms of it measuring what the ranking leaves open)
//   4 M vectors, d = 128, 16 x 16     7.5 -> 1.3 ms
//   500 k, d = 960, 16 x 256         10.9 -> 1.8 ms (0.36 ms)      500 k, d = 960, 32 x 16   3.3 -> 0.97 ms
//   1000 vectors, d = 128, 8 x 256    159 -> 28 us
// Tried: images of one sub-space at a time in LDS for all sizes (2.0 against 1.7 ms: barriers, and no wave can fetch
// ahead of the others); a whole wave measuring all 256 centroids of an open vector (3.9 ms in all: strided reads).
typedef _Float16 enc_half8 __attribute__((ext_vector_type(8)));
typedef float enc_float4 __attribute__((ext_vector_type(4)));

constexpr int ENC_MAX_DS = 64;      // 4 chunks of 16 dimensions: 64 KB of LDS for the centroids, 128 registers for the vectors
constexpr int ENC_VECS = 64;        // vectors per wave (4 tiles of 16): one LDS read of centroids feeds 8 matrix instructions
constexpr size_t ENC_RESIDENT_BYTES = 156 * 1024;   // of 160 KB of LDS
constexpr float ENC_NO_CENTROID = -1e38f;   // start value of rows past the last centroid and of copies of an earlier one

struct EncodeInfo { float scale, bound, cmax2, pad; };   // per sub-space: S_j; error bound; ||c||_max^2 in scaled units (inf: nothing is settled)

// One block per sub-space.  Image of a sub-space: the centroids as matrix operands [tile of 16][chunk][lane][8 halves],
// then the start values -||c||^2 / 2 [tiles * 16], the mean centroid times S_j [chunks * 16] and an EncodeInfo.
// A chain of passes over one codebook on one compute unit, bound by their latency: the codebook is read once into LDS (rows of
// an odd length: no bank is met twice by lanes of neighbouring rows).  8 x 256 of 16 dimensions 15 -> 11.5 us, 16 x 256 of 60 25 -> 18.
constexpr int enc_prep_row(int ds) { return ds | 1; }
__host__ __device__ constexpr int encode_image_len(int tiles, int nch) { return tiles * nch * 64 + tiles * 4 + nch * 4 + 1; }   // in uint4

__global__ __launch_bounds__(1024) void encode_prep_kernel(const float *__restrict__ codebooks, int k, int ds, int nch, int tiles,
                                                           uint4 *__restrict__ images) {
    __shared__ float red[16], mean[ENC_MAX_DS];
    __shared__ unsigned int cmax_bits, row_hash[256], part_hash[4][256];
    __shared__ double part_norm[4][256];
    __shared__ bool copy_of_earlier[256];
    const int j = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
    extern __shared__ float cb[];   // component t of centroid c at c * row + t
    const int row = enc_prep_row(ds);
    // 16, 32 or 64 lanes per centroid, so that no index is divided
    const int seg_bits = ds <= 16 ? 4 : ds <= 32 ? 5 : 6, my_t = tid & ((1 << seg_bits) - 1), my_c = tid >> seg_bits, c_step = 1024 >> seg_bits;
    if (my_t < ds) {
        const float *const src = codebooks + (size_t)j * k * ds;
#pragma unroll 4
        for (int c = my_c; c < k; c += c_step) cb[c * row + my_t] = src[(size_t)c * ds + my_t];
    }
    __syncthreads();
    uint4 *const image = images + (size_t)j * encode_image_len(tiles, nch);
    float *const start = reinterpret_cast<float *>(image + tiles * nch * 64), *const offset = start + tiles * 16;
    for (int t = tid >> 6; t < ENC_MAX_DS; t += 16) {   // (any value near the centroids does)
        float sum = 0.f;
        if (t < ds)
            for (int c = lane; c < k; c += 64) sum += cb[c * row + t] / (float)k;
        for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o);
        if (lane == 0) mean[t] = sum;
    }
    if (tid == 0) cmax_bits = 0;
    __syncthreads();
    float amax = 0.f;
    bool finite = true;
    if (my_t < ds)
        for (int c = my_c; c < k; c += c_step) {
            const float v = fabsf(cb[c * row + my_t] - mean[my_t]);
            finite = finite && v < __builtin_inff();
            amax = v > amax ? v : amax;
        }
    if (!finite) amax = __builtin_inff();
    for (int o = 32; o > 0; o >>= 1) {
        const float other = __shfl_xor(amax, o);
        amax = other > amax ? other : amax;
    }
    if (lane == 0) red[tid >> 6] = amax;
    __syncthreads();
    for (int w = 0; w < 16; ++w) amax = red[w] > amax ? red[w] : amax;
    // amax in [2^e, 2^(e+1)) becomes [2^10, 2^11), which the error bound relies on.  Where that takes a factor beyond the
    // powers of two of fp32 (centroids within 2^-116 of their mean), nothing is settled by the ranking.
    int e = amax > 0.f && amax < __builtin_inff() ? ilogbf(amax) : 10;
    e = 10 - e;   // (-117 at least)
    const bool ranked = amax < __builtin_inff() && e <= 126;
    e = e > 126 ? 126 : e;
    const float scale = ldexpf(1.f, e);
    {   // norms and hashes, a quarter of the dimensions per thread (256 centroids at most)
        const int c = tid & 255, quarter = tid >> 8, len = (ds + 3) / 4;
        double norm = 0.0;
        unsigned int hash = 2166136261u;
        if (c < k)
            for (int t = quarter * len; t < (quarter + 1) * len && t < ds; ++t) {
                const float x = cb[c * row + t];
                const double v = (double)((x - mean[t]) * scale);
                norm += v * v;
                hash = (hash ^ __float_as_uint(x)) * 16777619u;
            }
        part_norm[quarter][c] = norm;
        part_hash[quarter][c] = hash;
    }
    __syncthreads();
    if (tid < tiles * 16) {
        const int c = tid;
        const double norm = (part_norm[0][c] + part_norm[1][c]) + (part_norm[2][c] + part_norm[3][c]);
        row_hash[c] = ((part_hash[0][c] * 16777619u ^ part_hash[1][c]) * 16777619u ^ part_hash[2][c]) * 16777619u ^ part_hash[3][c];
        copy_of_earlier[c] = false;
        start[c] = c < k ? (float)(-0.5 * norm) : ENC_NO_CENTROID;
        if (c < k) {
            const float nf = (float)norm;
            atomicMax(&cmax_bits, __float_as_uint(nf == nf ? nf : __builtin_inff()));   // (non-negative floats order like their bits)
        }
    }
    __syncthreads();
    // Equal centroids (a sub-space that is constant in the data has nothing else) tie for every vector they are nearest to, and the
    // ranking would leave them all open.  The smallest index wins a tie, so the copies take no part, like rows past the last one.
    // (400 000 vectors, 8 x 256: all centroids equal 9.1 -> 0.20 ms, every one there twice 0.55 -> 0.21; looking for them 2 us.)
    {
        const int c = tid & 255, quarter = tid >> 8;   // four threads per centroid
        int equal = -1;   // (an earlier row of the same hash)
        if (c < k) {
            const unsigned int hash = row_hash[c];
#pragma unroll 8
            for (int e = quarter; e < c; e += 4) equal = row_hash[e] == hash ? e : equal;
        }
        if (equal >= 0) {
            bool same = true;
#pragma unroll 4
            for (int t = 0; t < ds; ++t) same = same && __float_as_uint(cb[equal * row + t]) == __float_as_uint(cb[c * row + t]);
            if (same) {
                copy_of_earlier[c] = true;
                start[c] = ENC_NO_CENTROID;
            }
        }
    }
    if (tid < nch * 16) offset[tid] = mean[tid] * scale;
    __syncthreads();
    if (tid == 0) {
        const float p17 = 7.6293945e-6f, p21 = 4.7683716e-7f, p22 = 2.3841858e-7f, p23 = 1.1920929e-7f;
        const float dims = (float)(nch * 16);
        EncodeInfo r;
        r.scale = scale;
        r.bound = 1.01f * (p22 + p21 + sqrtf(dims) * p23 + (4.f * dims + 8.f) * p23 + p17);
        r.cmax2 = ranked ? 1.001f * __uint_as_float(cmax_bits) : __builtin_inff();
        r.pad = 0.f;
        *reinterpret_cast<EncodeInfo *>(offset + nch * 16) = r;
    }
    for (int i = tid; i < tiles * nch * 64; i += 1024) {
        const int ch = (i >> 6) % nch, tile = (i >> 6) / nch;
        const int c = tile * 16 + (lane & 15), g = lane >> 4;
        enc_half8 h;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int t = ch * 16 + 8 * (g & 1) + q;
            const float v = c < k && t < ds && !copy_of_earlier[c] ? (cb[c * row + t] - mean[t]) * scale : 0.f;
            const _Float16 hi = (_Float16)v;
            h[q] = g >> 1 ? (_Float16)(v - (float)hi) : hi;
        }
        image[i] = __builtin_bit_cast(uint4, h);
    }
}

// the two largest values of a lane and, of two lanes' pairs, those of both
__device__ __forceinline__ float enc_with_number(float v, uint32_t keep, uint32_t number) { return __uint_as_float((__float_as_uint(v) & keep) | number); }
__device__ __forceinline__ void enc_two_more(float &m1, float &m2, float a, float b) {
    m2 = fmaxf(m2, __builtin_amdgcn_fmed3f(m1, a, b));
    m1 = fmaxf(fmaxf(m1, a), b);
}
struct EncBest { float m1, m2; int idx; };
__device__ __forceinline__ EncBest enc_merge(const EncBest &a, const EncBest &b) {
    EncBest r;
    r.m2 = fmaxf(fminf(a.m1, b.m1), fmaxf(a.m2, b.m2));
    r.idx = a.m1 >= b.m1 ? a.idx : b.idx;
    r.m1 = fmaxf(a.m1, b.m1);
    return r;
}
// lanes of b's first half <-> lanes of a's second half (halves of 32 or, within each 32 lanes, of 16)
template <int HALF>
__device__ __forceinline__ void enc_swap(uint32_t &a, uint32_t &b) {
    typedef uint32_t pair2 __attribute__((ext_vector_type(2)));
    pair2 r;
    if (HALF == 32) r = __builtin_bit_cast(pair2, __builtin_amdgcn_permlane32_swap(a, b, false, false));
    else r = __builtin_bit_cast(pair2, __builtin_amdgcn_permlane16_swap(a, b, false, false));
    a = r[0];
    b = r[1];
}
template <int HALF>
__device__ __forceinline__ EncBest enc_swap_merge(EncBest a, EncBest b) {
    uint32_t a1 = __float_as_uint(a.m1), b1 = __float_as_uint(b.m1), a2 = __float_as_uint(a.m2), b2 = __float_as_uint(b.m2), ai = a.idx, bi = b.idx;
    enc_swap<HALF>(a1, b1);
    enc_swap<HALF>(a2, b2);
    enc_swap<HALF>(ai, bi);
    return enc_merge(EncBest{__uint_as_float(a1), __uint_as_float(a2), (int)ai}, EncBest{__uint_as_float(b1), __uint_as_float(b2), (int)bi});
}

struct EncodeArgs {
    const float *x, *codebooks;
    uint8_t *codes;
    int64_t n;
    int d, ds, m, k, packed, code_bytes, tiles;
    int bytes_per_y;        // code bytes of one block (blockIdx.y numbers the parts)
    int words;              // codes may be written as 32-bit words
    const uint4 *images;
};

// VEC consecutive floats
template <int VEC>
__device__ __forceinline__ void enc_load(const float *p, float *v) {
    if (VEC == 4) {
        const float4 f = *reinterpret_cast<const float4 *>(p);
        v[0] = f.x; v[1] = f.y; v[VEC > 2 ? 2 : 0] = f.z; v[VEC > 2 ? 3 : 0] = f.w;
    } else if (VEC == 2) {
        const float2 f = *reinterpret_cast<const float2 *>(p);
        v[0] = f.x; v[VEC > 1 ? 1 : 0] = f.y;
    } else {
        v[0] = *p;
    }
}

// VEC: dimensions per load (what the alignment of a sub-vector allows).  FULL: 256 centroids.  RESIDENT: the images of all
// sub-spaces stay in LDS and every wave goes through its share of the vectors without meeting the others; else the
// block's waves take one sub-space after the other together.
template <int NCH, int VEC, bool FULL, bool RESIDENT>
__global__ __launch_bounds__(RESIDENT && NCH == 1 ? 1024 : 512, NCH == 1 ? 4 : 2) void encode_split16_kernel(EncodeArgs A) {
    extern __shared__ uint4 enc_lds[];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4;
    const int ds = A.ds, tiles = FULL ? 16 : A.tiles, image_len = encode_image_len(tiles, NCH);
    const int waves = blockDim.x >> 6;
    const int byte0 = blockIdx.y * A.bytes_per_y;
    const int byte1 = byte0 + A.bytes_per_y < A.code_bytes ? byte0 + A.bytes_per_y : A.code_bytes;
    const int j0 = A.packed ? 2 * byte0 : byte0, j1 = A.packed ? 2 * byte1 : byte1;
    int low_bits = 3;   // of the values: number of the centroid within the lane
    while (low_bits < tiles * 4 - 1) low_bits = 2 * low_bits + 1;
    uint32_t keep = ~(uint32_t)low_bits;
    asm("" : "+v"(keep));   // (in a vector register: mask and number then go into one instruction, which takes one scalar operand)
    if (RESIDENT) {
        for (int i = tid; i < A.m * image_len; i += blockDim.x) enc_lds[i] = A.images[i];
        __syncthreads();
    }
    const int64_t stride = (int64_t)gridDim.x * waves * ENC_VECS;
    for (int64_t v0 = ((int64_t)blockIdx.x * waves + __builtin_amdgcn_readfirstlane(tid >> 6)) * ENC_VECS;; v0 += stride) {
        if (RESIDENT && v0 >= A.n) break;
        const int64_t mine = v0 + lane;   // the vector whose codes this lane writes
        const float *xrow[4];
#pragma unroll
        for (int tv = 0; tv < 4; ++tv) {
            const int64_t row = v0 + tv * 16 + (lane & 15);
            xrow[tv] = A.x + (size_t)(row < A.n ? row : A.n - 1) * A.d;
        }
        uint32_t word = 0;
        for (int j = j0; j < j1; ++j) {
            if (!RESIDENT) {
                __syncthreads();   // the previous sub-space's centroids have been read
                for (int i = tid; i < image_len; i += blockDim.x) enc_lds[i] = A.images[(size_t)j * image_len + i];
                __syncthreads();
            }
            const uint4 *const image = enc_lds + (RESIDENT ? j * image_len : 0);
            const float *const start = reinterpret_cast<const float *>(image + tiles * NCH * 64), *const offset = start + tiles * 16;
            const EncodeInfo info = *reinterpret_cast<const EncodeInfo *>(offset + NCH * 16);
            enc_half8 xh[4][NCH], xl[4][NCH];
            float xx[4];
#pragma unroll
            for (int tv = 0; tv < 4; ++tv) {
                xx[tv] = 0.f;
                if (NCH > 1) __builtin_amdgcn_sched_barrier(0);   // (one tile's floats in registers at a time)
#pragma unroll
                for (int ch = 0; ch < NCH; ++ch) {
                    float v[8];
#pragma unroll
                    for (int q = 0; q < 8; q += VEC) {
                        const int t = ch * 16 + 8 * (g & 1) + q;
                        const bool inside = t < ds;   // (VEC divides ds: the whole group is, or none of it)
                        enc_load<VEC>(xrow[tv] + (size_t)j * ds + (inside ? t : 0), v + q);
#pragma unroll
                        for (int u = 0; u < VEC; ++u) v[q + u] = inside ? v[q + u] : 0.f;   // (offset is 0 there)
                    }
                    float mu[8];
                    enc_load<4>(offset + ch * 16 + 8 * (g & 1), mu);
                    enc_load<4>(offset + ch * 16 + 8 * (g & 1) + 4, mu + 4);
#pragma unroll
                    for (int q = 0; q < 8; ++q) {
                        const float s = fmaf(v[q], info.scale, -mu[q]);   // (x - mean) S_j, rounded once: S_j is a power of two
                        const _Float16 hi = (_Float16)s;
                        xh[tv][ch][q] = hi;
                        xl[tv][ch][q] = (_Float16)(s - (float)hi);
                        xx[tv] = fmaf(s, s, xx[tv]);
                    }
                }
                asm volatile("" : "+v"(xx[tv]));   // (summed here: moved below the ranking it would hold all floats in registers)
            }
            // lane: rows 4 g .. 4 g + 3 (centroids) of column lane % 16 (vector)
            auto products = [&](int t, const enc_half8 *a, int tv) {
                enc_float4 acc = *reinterpret_cast<const enc_float4 *>(start + t * 16 + 4 * g);
#pragma unroll
                for (int ch = 0; ch < NCH; ++ch) {
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[ch], xh[tv][ch], acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(a[ch], xl[tv][ch], acc, 0, 0, 0);
                }
                return acc;
            };
            float m1[4], m2[4];
            constexpr int TILES_AT_ONCE = FULL ? 2 : 1;
#pragma unroll
            for (int tv = 0; tv < 4; ++tv) { m1[tv] = -3e38f; m2[tv] = -3e38f; }
#pragma unroll TILES_AT_ONCE
            for (int t = 0; t < tiles; ++t) {
                uint32_t number[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    number[r] = 4 * t + r;
                    asm volatile("" : "+s"(number[r]));
                }
                enc_half8 a[NCH];
#pragma unroll
                for (int ch = 0; ch < NCH; ++ch) a[ch] = __builtin_bit_cast(enc_half8, image[(t * NCH + ch) * 64 + lane]);
#pragma unroll
                for (int tv = 0; tv < 4; ++tv) {
                    const enc_float4 acc = products(t, a, tv);
                    enc_two_more(m1[tv], m2[tv], enc_with_number(acc[0], keep, number[0]), enc_with_number(acc[1], keep, number[1]));
                    enc_two_more(m1[tv], m2[tv], enc_with_number(acc[2], keep, number[2]), enc_with_number(acc[3], keep, number[3]));
                }
            }
            // the four groups of 16 lanes hold a quarter of the centroids each: group g ends up with tile g's vectors
            EncBest best[4];
            float norm2 = 0.f;
#pragma unroll
            for (int tv = 0; tv < 4; ++tv) {
                const int number = (int)(__float_as_uint(m1[tv]) & ~keep);
                best[tv] = EncBest{m1[tv], m2[tv], (number >> 2) * 16 + g * 4 + (number & 3)};
                const float whole = xx[tv] + __shfl_xor(xx[tv], 16);
                norm2 = g == tv ? whole : norm2;
            }
            const EncBest half0 = enc_swap_merge<32>(best[0], best[2]), half1 = enc_swap_merge<32>(best[1], best[3]);
            const EncBest fin = enc_swap_merge<16>(half0, half1);
            int code = fin.idx;
            // settled (false for NaN): the gap exceeds twice the error bound; 2^31: no component above fp16's range
            const float twice = 2.f * info.bound * (norm2 + info.cmax2);
            const bool valid = norm2 < 2147483648.f && fin.m1 > -1e37f && twice < 1e37f;
            const unsigned long long open = __ballot(!(valid && fin.m1 - fin.m2 > twice) && mine < A.n);
            if (open) {
                // from here on lane = (group, column) again: every group takes its centroids of its column's vector
                const float least = valid ? fin.m1 - twice : -__builtin_inff();
#pragma unroll
                for (int tv = 0; tv < 4; ++tv) {
                    const uint32_t cols = (uint32_t)(open >> (16 * tv)) & 0xffffu;
                    if (cols == 0) continue;
                    const bool wanted = (cols >> (lane & 15)) & 1;
                    const float floor_ = __shfl(least, tv * 16 + (lane & 15));
                    unsigned long long near = 0;   // bit 4 t + r: centroid 16 t + 4 g + r
                    if (!__any(wanted && !(m2[tv] < floor_))) {
                        // at most one centroid of each lane is near, and its number is known
                        if (m1[tv] >= floor_) near = 1ull << (__float_as_uint(m1[tv]) & ~keep);
                    } else {
#pragma unroll 1
                        for (int t = 0; t < tiles; ++t) {
                            enc_half8 a[NCH];
#pragma unroll
                            for (int ch = 0; ch < NCH; ++ch) a[ch] = __builtin_bit_cast(enc_half8, image[(t * NCH + ch) * 64 + lane]);
                            const enc_float4 acc = products(t, a, tv);
#pragma unroll
                            for (int r = 0; r < 4; ++r)
                                if (!(acc[r] < floor_) && t * 16 + 4 * g + r < A.k) near |= 1ull << (4 * t + r);   // (NaN: near)
                        }
                    }
                    if (!wanted) near = 0;
                    const float *const xr = xrow[tv] + (size_t)j * ds;
                    double bd = __builtin_inf();
                    int bi = 0;
#pragma unroll 1
                    while (near) {
                        const int bit = __builtin_ctzll(near);
                        near &= near - 1;
                        const int i = (bit >> 2) * 16 + 4 * g + (bit & 3);
                        const float *const cr = A.codebooks + ((size_t)j * A.k + i) * ds;
                        double dist = 0.0;
#pragma unroll 4
                        for (int t = 0; t < ds; t += VEC) {
                            float v[VEC], c[VEC];
                            enc_load<VEC>(xr + t, v);
                            enc_load<VEC>(cr + t, c);
#pragma unroll
                            for (int u = 0; u < VEC; ++u) {
                                const double df = (double)v[u] - (double)c[u];
                                dist += df * df;
                            }
                        }
                        if (dist < bd) { bd = dist; bi = i; }   // (a lane's centroids ascend: ties keep the smaller one)
                    }
#pragma unroll
                    for (int o = 16; o < 64; o <<= 1) {
                        const double od = __shfl_xor(bd, o);
                        const int oi = __shfl_xor(bi, o);
                        if (od < bd || (od == bd && oi < bi)) { bd = od; bi = oi; }
                    }
                    if (g == tv && wanted) code = bd < __builtin_inf() ? bi : 0;   // (no finite distance at all: index 0)
                }
            }
            // codes: one byte per index, or two indexes per byte
            const int byte = A.packed ? j >> 1 : j;
            const int shift = A.words ? 8 * (byte & 3) : 0;
            word |= (uint32_t)code << (shift + (A.packed && (j & 1) ? 4 : 0));
            if (!A.packed || (j & 1)) {
                if (A.words) {
                    if ((byte & 3) == 3) {
                        if (mine < A.n) *reinterpret_cast<uint32_t *>(A.codes + (size_t)mine * A.code_bytes + (byte & ~3)) = word;
                        word = 0;
                    }
                } else {
                    if (mine < A.n) A.codes[(size_t)mine * A.code_bytes + byte] = (uint8_t)word;
                    word = 0;
                }
            }
        }
        if (!RESIDENT) break;
    }
}

template <int NCH, int VEC, bool FULL, bool RESIDENT>
static int launch_encode_split16(pq_ctx *ctx, const EncodeArgs &A, dim3 grid, int threads, size_t lds) {
    if (lds > 64 * 1024)
        PQ_HIP(ctx, hipFuncSetAttribute((const void *)encode_split16_kernel<NCH, VEC, FULL, RESIDENT>,
                                        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    encode_split16_kernel<NCH, VEC, FULL, RESIDENT><<<grid, threads, lds, ctx->stream>>>(A);
    PQ_HIP(ctx, hipGetLastError());
    return PQ_OK;
}
template <int NCH, int VEC>
static int launch_encode_split16(pq_ctx *ctx, const EncodeArgs &A, dim3 grid, int threads, size_t lds, bool resident) {
    if (A.tiles == 16)
        return resident ? launch_encode_split16<NCH, VEC, true, true>(ctx, A, grid, threads, lds)
                        : launch_encode_split16<NCH, VEC, true, false>(ctx, A, grid, threads, lds);
    return resident ? launch_encode_split16<NCH, VEC, false, true>(ctx, A, grid, threads, lds)
                    : launch_encode_split16<NCH, VEC, false, false>(ctx, A, grid, threads, lds);
}
template <int NCH>
static int launch_encode_split16(pq_ctx *ctx, const EncodeArgs &A, int vec, dim3 grid, int threads, size_t lds, bool resident) {
    if (vec == 4) return launch_encode_split16<NCH, 4>(ctx, A, grid, threads, lds, resident);
    if (vec == 2) return launch_encode_split16<NCH, 2>(ctx, A, grid, threads, lds, resident);
    return launch_encode_split16<NCH, 1>(ctx, A, grid, threads, lds, resident);
}

// ------------------------------------------------------------------------------------------
constexpr int ER = 64;   // vectors per block (4 waves x 16 rows)
constexpr int EC = 64;   // centroids per tile
constexpr int EK = 16;   // dimensions per LDS chunk

// One block of 256 threads encodes 64 vectors, one sub-space after the other.  Wave w owns rows
// 16 w .. 16 w + 15 and all 64 centroids of a tile (four 16 x 16 MFMA tiles), so the arg-min of a
// row is reduced inside one wave.
__global__ __launch_bounds__(256) void pq_encode_kernel(const float *__restrict__ x, const float *__restrict__ codebooks,
                                                        int64_t n, int d, int m, int k, int packed,
                                                        uint8_t *__restrict__ codes) {
    typedef double double4_t __attribute__((ext_vector_type(4)));
    __shared__ double xs[EK][ER + 2];
    __shared__ double cs[EK][EC + 2];
    __shared__ double nx[ER], nc[EC];
    const int ds = d / m;
    const int64_t r0 = (int64_t)blockIdx.x * ER;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lrow = tid >> 2, lk = (tid & 3) * 4;   // staging: 4 consecutive dimensions of one row
    const bool xrow_ok = r0 + lrow < n;
    const int code_bytes = packed ? m / 2 : m;
    int prev_idx[4] = {0, 0, 0, 0};   // packed codes: index of the even sub-space, kept for the odd one

    for (int j = 0; j < m; ++j) {
        const float *xrow = x + (size_t)(xrow_ok ? r0 + lrow : 0) * d + (size_t)j * ds;
        const float *cbase = codebooks + (size_t)j * k * ds;
        double best[4];
        int best_idx[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) { best[v] = __builtin_inf(); best_idx[v] = 0; }

        for (int c0 = 0; c0 < k; c0 += EC) {
            const bool crow_ok = c0 + lrow < k;
            const float *crow = cbase + (size_t)(crow_ok ? c0 + lrow : 0) * ds;
            double4_t acc[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = (double4_t){0.0, 0.0, 0.0, 0.0};
            double norm = 0.0;   // thread t < 64: ||x_t||^2, thread 64 + t: ||c_t||^2
            for (int k0 = 0; k0 < ds; k0 += EK) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int t = k0 + lk + i;
                    xs[lk + i][lrow] = xrow_ok && t < ds ? (double)xrow[t] : 0.0;
                    cs[lk + i][lrow] = crow_ok && t < ds ? (double)crow[t] : 0.0;
                }
                __syncthreads();
                if (tid < ER + EC) {
                    const double(*src)[ER + 2] = tid < ER ? xs : cs;
                    const int r = tid & (ER - 1);
#pragma unroll
                    for (int kk = 0; kk < EK; ++kk) norm += src[kk][r] * src[kk][r];
                }
#pragma unroll
                for (int ks = 0; ks < EK; ks += 4) {
                    const double a = xs[ks + (lane >> 4)][wave * 16 + (lane & 15)];
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const double b = cs[ks + (lane >> 4)][t * 16 + (lane & 15)];
                        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[t], 0, 0, 0);
                    }
                }
                __syncthreads();
            }
            if (tid < ER) nx[tid] = norm;
            else if (tid < ER + EC) nc[tid - ER] = norm;
            __syncthreads();
            // lane l holds rows l / 16 + 4 v of column l % 16 of each 16 x 16 tile
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int r = wave * 16 + (lane >> 4) + 4 * v;
                double dmin = __builtin_inf();
                int imin = 0x7fffffff;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int c = t * 16 + (lane & 15), ci = c0 + c;
                    if (ci >= k) continue;
                    const double sum = nx[r] + nc[c];
                    double dist = sum - 2.0 * acc[t][v];
                    if (dist < 1e-9 * sum && r0 + r < n) {   // nearly complete cancellation: the plain definition
                        dist = 0.0;
                        const float *xr = x + (size_t)(r0 + r) * d + (size_t)j * ds, *cr = cbase + (size_t)ci * ds;
                        for (int t2 = 0; t2 < ds; ++t2) {
                            const double df = (double)xr[t2] - (double)cr[t2];
                            dist += df * df;
                        }
                    }
                    if (dist < dmin) { dmin = dist; imin = ci; }   // columns ascend with t: the first minimum stays
                }
                // smallest (distance, index) over the 16 lanes that share the row
#pragma unroll
                for (int o = 1; o < 16; o <<= 1) {
                    const double od = __shfl_xor(dmin, o);
                    const int oi = __shfl_xor(imin, o);
                    if (od < dmin || (od == dmin && oi < imin)) { dmin = od; imin = oi; }
                }
                if (dmin < best[v]) { best[v] = dmin; best_idx[v] = imin; }   // tiles ascend: ties keep the smaller index
            }
            __syncthreads();
        }
        if ((lane & 15) == 0) {
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t row = r0 + wave * 16 + (lane >> 4) + 4 * v;
                if (row >= n) continue;
                if (!packed) {
                    codes[(size_t)row * code_bytes + j] = (uint8_t)best_idx[v];
                } else if (j & 1) {
                    codes[(size_t)row * code_bytes + (j >> 1)] = (uint8_t)(prev_idx[v] | (best_idx[v] << 4));
                } else {
                    prev_idx[v] = best_idx[v];
                }
            }
        }
    }
}

int launch_encode(pq_ctx *ctx, const float *vectors, const float *codebooks, int64_t n, int d, int m, int k, int cf,
                  uint8_t *codes) {
    if (n == 0) return PQ_OK;
    const int ds = d / m, packed = cf == PQ_CODES_U4_PACKED ? 1 : 0;
    const int64_t nblocks = (n + ER - 1) / ER;
    if (nblocks > 0x7fffffff) return fail(ctx, PQ_EUNSUPPORTED, "encode: more than 2^37 vectors");
    // The centroids as matrix operands need scratch memory.  A call that cannot have it takes the form that needs none, and so
    // does every call on a stream that is being captured: its graph holds no memory of the context, which a later call may
    // give back, and can be replayed for as long as the caller's own buffers live.
    const int chunks = (ds + 15) / 16, nch = chunks <= 2 ? chunks : 4, tiles = (k + 15) / 16;
    const size_t image_bytes = (size_t)encode_image_len(tiles, nch) * sizeof(uint4);
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(ctx->stream, &capture) != hipSuccess) {
        (void)hipGetLastError();
        capture = hipStreamCaptureStatusActive;
    }
    if (ds <= ENC_MAX_DS && capture == hipStreamCaptureStatusNone && opt_int(ctx, PQ_OPT_ENCODE_SPLIT16, 1) != 0 &&
        buf_reserve(ctx, &ctx->encode_images, (size_t)m * image_bytes, "the centroid images of the encoder") == PQ_OK) {
        EncodeArgs A{};
        A.x = vectors; A.codebooks = codebooks; A.codes = codes; A.n = n; A.d = d; A.ds = ds; A.m = m; A.k = k; A.packed = packed;
        A.code_bytes = packed ? m / 2 : m; A.tiles = tiles;
        A.images = (const uint4 *)ctx->encode_images.p;
        A.words = (A.code_bytes & 3) == 0 && ((uintptr_t)codes & 3) == 0;
        const uintptr_t bases = (uintptr_t)vectors | (uintptr_t)codebooks;
        const int vec = (ds & 3) == 0 && (bases & 15) == 0 ? 4 : ((ds & 1) == 0 && (bases & 7) == 0 ? 2 : 1);
        // All images in LDS where they fit and every wave of the chip has a tile of vectors (a block copies all of
        // them).  Else blocks of 8 waves share one image at a time; few vectors, and those of small images (nothing to share), go
        // in blocks of 2 waves.  The code bytes are dealt to several blocks until there are two for every compute unit (d = 960,
        // 16 x 256, blocks of 2 waves while there were few vectors, whole words dealt -> now: call of 2000 vectors 119 -> 52 us, 60 000 403 -> 250,
        // 250 000 1525 -> 908; d = 128, 8 x 256: 1000 vectors 53 -> 28, 100 000 96 -> 69; 100 000 of d = 960, 32 x 16 in blocks of 8 waves 335 -> 351).
        const int resident_waves = nch == 1 ? 16 : 8;
        const bool resident = m * image_bytes <= ENC_RESIDENT_BYTES && n >= (int64_t)ctx->num_cu * resident_waves * ENC_VECS;
        const int64_t big = (n + 8 * ENC_VECS - 1) / (8 * ENC_VECS);
        const int waves = resident ? resident_waves : (big >= 2 * ctx->num_cu || (big * A.code_bytes >= ctx->num_cu && image_bytes >= 8192) ? 8 : 2);
        const int64_t bx = resident ? ctx->num_cu : (n + waves * ENC_VECS - 1) / (waves * ENC_VECS);
        int parts = resident ? 1 : (int)((2 * (int64_t)ctx->num_cu + bx - 1) / bx);
        if (parts > A.code_bytes / 4) A.words = 0;   // (more parts than words: byte by byte)
        const int unit = A.words ? 4 : 1, units = A.code_bytes / unit;
        parts = parts < 1 ? 1 : (parts > units ? units : parts);
        A.bytes_per_y = (units + parts - 1) / parts * unit;
        parts = (A.code_bytes + A.bytes_per_y - 1) / A.bytes_per_y;
        const size_t prep_lds = (size_t)k * enc_prep_row(ds) * 4;
        if (prep_lds > 32 * 1024)
            PQ_HIP(ctx, hipFuncSetAttribute((const void *)encode_prep_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)prep_lds));
        encode_prep_kernel<<<m, 1024, prep_lds, ctx->stream>>>(codebooks, k, ds, nch, tiles, (uint4 *)ctx->encode_images.p);
        PQ_HIP(ctx, hipGetLastError());
        const dim3 grid((unsigned)bx, (unsigned)parts);
        const size_t lds = image_bytes * (resident ? m : 1);
        if (nch == 1) return launch_encode_split16<1>(ctx, A, vec, grid, waves * 64, lds, resident);
        if (nch == 2) return launch_encode_split16<2>(ctx, A, vec, grid, waves * 64, lds, resident);
        return launch_encode_split16<4>(ctx, A, vec, grid, waves * 64, lds, resident);
    }
    pq_encode_kernel<<<(unsigned)nblocks, 256, 0, ctx->stream>>>(vectors, codebooks, n, d, m, k, packed, codes);
    PQ_HIP(ctx, hipGetLastError());
    return PQ_OK;
}

}  // namespace pq
