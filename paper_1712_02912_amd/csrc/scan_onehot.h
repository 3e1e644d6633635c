// Integer scan of packed 4-bit codes on the matrix cores (scan_onehot.hip).
#pragma once
#include "pq_internal.h"

namespace pq {

// Sums per query whose rows are counted, and the bins of their rows (see onehot_bound).
constexpr int ONEHOT_TIES = 3, ONEHOT_TIE_BINS = 256;
constexpr size_t onehot_tie_words(size_t nq) { return nq * (ONEHOT_TIES + ONEHOT_TIES * ONEHOT_TIE_BINS); }

int onehot_queries_per_pass(int code_bytes, int nq);

// The sample: every onehot_stride-th load of 1024 code bytes, and the rank in it that bounds the scan.
int onehot_stride(int64_t n);
int onehot_rank(int64_t n, int topk);

// Lists every key (sum << 32 | row) up to a bound that it leaves in tau_key[q] (a valid one only if at least topk are listed):
// cnt[q * COUNT_PITCH] of them, the first cap in lists[q][cap].  tau_key holds bounds to start from: keys at or below which the sample has at
// least onehot_rank codes.  cnt[nq * COUNT_PITCH], hist[nq][HIST_BINS], ties[onehot_tie_words(nq)] and *work_counter are clear.
int launch_scan_onehot(pq_ctx *ctx, const uint8_t *codes, int64_t n, int code_bytes, const uint8_t *qluts, int nq, int topk, int hist_bins,
                       unsigned long long *tau_key, uint32_t *cnt, uint32_t *hist, uint64_t *lists, uint32_t cap,
                       uint32_t *ties, uint32_t *work_counter, unsigned long long *stats);

}  // namespace pq
