// Sampling rows of many ids look for the K largest among candidates first (sample_rows_sparse_kernel): the keys above a bound that
// kSamples of the row's V keys suggest.  Which rows do, which ids are sampled, and the bound.  Plain C++ (constexpr: host and device), so
// that a test can play rows through without a GPU.
#pragma once
#include <stdint.h>

constexpr uint32_t kSamples = 1024, kCand = 6 * 1024;   // one sample and at most six candidates a thread
constexpr int kSelBins = 2048;
constexpr int kBin0Shift = 17;   // round 0 of the select: 2^17 order keys per bin = 64 bins per binade of the logit

// Sample t: one id of each of kSamples equal parts of the row, at a place in its part that varies (V >= kSamples)
constexpr uint32_t sample_id(uint32_t t, uint32_t V) {
    return (uint32_t)(((uint64_t)t * V) >> 10) + ((((t * 2654435761u) >> 16) * (V >> 10)) >> 16);
}
// Where r samples lie above the bound, some r x V / kSamples keys do, give or take sqrt(r) x V / kSamples.  1.5 x the share that K is
// and 12 more: 3.2 such spreads at least above what K needs.
constexpr uint32_t candidate_rank(uint32_t K, uint32_t V) { return (uint32_t)((uint64_t)K * (kSamples + kSamples / 2) / V) + 12u; }
// The bound: the lowest key of the round-0 bin that the sample of that rank is in
constexpr uint32_t candidate_bound(uint32_t kmax, uint32_t bin) {
    const uint32_t off = (bin + 1u) << kBin0Shift;   // (2048 x 2^17 = 2^28: no overflow)
    return bin < (uint32_t)(kSelBins - 1) && kmax > off ? kmax - off + 1u : 1u;
}
// A row that has looked in vain starts over with all its keys, and the launch lasts as long as its slowest row: only where the
// candidates find room with three spreads to spare, and only where a thread has more than 16 keys (12 000 ids, K = 500, without ->
// with candidates: 14.8 -> 14.7 us, 4097 ids 13.3 -> 14.3, 256 rows of 16 384 18.6 -> 21.5).
constexpr bool candidates_fit(uint32_t K, uint32_t V) {
    const uint64_t room = (uint64_t)kCand * kSamples / V, r = candidate_rank(K, V);
    return V > 16 * 1024 && K < V && r < room && 9 * r <= (room - r) * (room - r);
}
