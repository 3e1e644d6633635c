// Integer scan of packed 4-bit codes on the matrix cores (scan_onehot.hip).
#pragma once
#include "pq_internal.h"

namespace pq {

// Sums per query whose rows are counted, and the bins of their rows (see onehot_bound).
constexpr int ONEHOT_TIES = 3, ONEHOT_TIE_BINS = 256;
constexpr size_t onehot_tie_words(size_t nq) { return nq * (ONEHOT_TIES + ONEHOT_TIES * ONEHOT_TIE_BINS); }

int onehot_queries_per_pass(int code_bytes, int nq);

// The sample: of every 2^shift rows one, in a place that the row's number in the sample is mixed into (Knuth's multiplicative hash, twice).  Rows
// stored by what they are near (list by list, as they came) would be in a sample of adjacent rows together or not at all.
__device__ __forceinline__ uint32_t onehot_sample_row(uint32_t i, int shift) {
    uint32_t x = (i ^ (i >> 15)) * 0x9e3779b9u;
    x = (x ^ (x >> 15)) * 0x9e3779b9u;
    return (i << shift) | (x >> (32 - shift));
}
// shift of a sample that fits `room` bytes (0: none), and the rank in it that bounds the scan
int onehot_shift(int64_t n, int code_bytes, int nq, int topk, size_t room);
int onehot_rank(int shift, int topk);
// The sample's codes side by side, and the queries' least sums, whose rows are the first to be counted (`ties` as below).
int launch_onehot_sample(pq_ctx *ctx, const uint8_t *codes, int64_t n, int code_bytes, int shift, uint8_t *sample, const uint8_t *qluts, int nq, uint32_t *ties);

// Lists every key (sum << 32 | row) up to a bound that it leaves in tau_key[q] (a valid one only if at least topk are listed):
// cnt[q * COUNT_PITCH] of them, the first cap in lists[q][cap].  tau_key holds bounds to start from: keys at or below which the sample has at
// least onehot_rank codes.  The lists may lie where the sample is.  cnt[nq * COUNT_PITCH], hist[nq][HIST_BINS], ties[onehot_tie_words(nq)] and *work_counter are clear.
int launch_scan_onehot(pq_ctx *ctx, const uint8_t *codes, int64_t n, int code_bytes, const uint8_t *sample, int shift, const uint8_t *qluts, int nq, int topk, int hist_bins,
                       unsigned long long *tau_key, uint32_t *cnt, uint32_t *hist, uint64_t *lists, uint32_t cap,
                       uint32_t *ties, uint32_t *work_counter, unsigned long long *stats);

}  // namespace pq
