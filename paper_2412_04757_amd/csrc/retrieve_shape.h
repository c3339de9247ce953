// How a launch of step 2 is shaped (retrieve.hip): what its Q^R is made of, whether one kernel does everything behind that, and
// how many sequences a launch takes. Plain C++, so that the host tests can look at every size.
#pragma once
#include <stddef.h>

namespace ltri {

constexpr int RT1_MAX_SPANS = 8192;
constexpr int rt1_pow2(int n) { int m = 64; while (m < n) m <<= 1; return m; }
// dynamic LDS of the selection: keys, ids, clipped lengths
constexpr size_t rt1_lds_bytes(int bound) { return (size_t)rt1_pow2(bound) * 12 + (size_t)bound * 4; }

constexpr int QREP_PIECE = 128;                    // tokens of a piece of a query span
// Chunks whose query rows every scoring workgroup sums itself: their tokens; and for calls of few sequences and KV heads, whose
// sums a launch spreads over the chip, bytes of a KV head's rows. A compute unit's reading bounds it: 128 rows of 8 heads of 128 bf16
// (256 KB) are as fast as with a launch before, of 16 heads 27.4 us against 24.9; but 24 sequences of 100 such rows 38.5 us with a
// launch before, 23.3 without.
constexpr int QREP_SHORT = 128;
constexpr int QREP_ROWS_BYTES = 256 * 1024;
constexpr int QREP_FEW_PROBLEMS = 8;
constexpr size_t RETRIEVE_LDS = 116 * 1024;        // dynamic LDS of retrieve_chunk_kernel, at most

// Partial sums of the query rows that a launch of qrep_partial_kernel leaves per problem, at most.
constexpr int qrep_units(int n_q) { return n_q / QREP_PIECE + n_q; }

// Whether retrieve_chunk_kernel takes the table: its arrays of keys, ids and lengths share the 160 KB of LDS with 26 KB of masks
// and list scratch.
inline bool retrieve_one_tail(int span_bound, int item_bound) {
  return span_bound >= 1 && span_bound <= RT1_MAX_SPANS && item_bound <= RT1_MAX_SPANS && rt1_lds_bytes(item_bound) <= RETRIEVE_LDS;
}

struct RetrieveShape {
  bool one_tail;        // one launch (retrieve_chunk_kernel) for everything behind the sums
  bool from_sums;       // Q^R from the running sums of the query rows
  bool from_rows;       // Q^R by every scoring workgroup for itself
  bool spans;           // Q^R by a workgroup per query span, launched first (chunks of up to QREP_PIECE tokens)
  bool pieces;          // Q^R from sums of pieces, launched first
  int per;              // sequences a trip of launches takes
};

// reads_sums: running sums serve the configuration and chunk length (retrieve_reads_running_sums); votes: collaborative retrieval;
// stored: Q^R of the chunk's spans is in place already; row_bytes: bytes of a token's query rows of a KV head; count: sequences of the
// call, of `heads` KV heads; buffer_seqs: sequences that the buffer of pieces and running sums has room for.
inline RetrieveShape retrieve_shape(bool reads_sums, bool votes, bool stored, int n_q, int row_bytes, int span_bound, int item_bound,
                                    int count, int heads, int buffer_seqs) {
  RetrieveShape s;
  s.one_tail = !votes && retrieve_one_tail(span_bound, item_bound);
  s.from_sums = s.one_tail && reads_sums;
  s.from_rows = s.one_tail && !s.from_sums && n_q <= QREP_SHORT &&
                (n_q * row_bytes <= QREP_ROWS_BYTES || count * heads > QREP_FEW_PROBLEMS);
  const bool summed = !s.from_sums && !s.from_rows && !(s.one_tail && stored);       // (very long tables: whatever is in place)
  s.spans = summed && n_q <= QREP_PIECE;
  s.pieces = summed && n_q > QREP_PIECE;
  s.per = s.from_sums || s.pieces ? buffer_seqs : count;
  return s;
}

// Whether step 2 of a chunk with index vectors reads a Q^R that is in place: not where its workgroups sum the rows themselves, nor
// with very long tables, so that the step before need not take it there.
inline bool retrieve_reads_stored(int n_q, int row_bytes, int span_bound, int item_bound, int count, int heads) {
  const RetrieveShape s = retrieve_shape(false, false, true, n_q, row_bytes, span_bound, item_bound, count, heads, 1);
  return !s.from_rows && !s.spans && !s.pieces;
}

}  // namespace ltri
