// How a launch of the matrix-core attention is shaped: key groups per workgroup and splits of the key range. Plain C++.
//
// A workgroup (one per compute unit: its registers fill it) covers 256 (row, head) pairs with every wavefront on all keys
// (KS = 1), or 128 with two groups on alternate tiles (KS = 2, merged in LDS): twice the workgroups, half the stages, twice
// the rows fetched per product. Splits divide the stages further but write and read back partial results. The launch takes
// (rounds of workgroups over the chip) x (stages per workgroup x time of a stage + start) + merge; the least of that model
// over both KS and 1 .. 16 splits is taken. Its constants (us): a stage 1.5 on a nearly empty chip .. 1.85 on a full one
// (the clock falls), 7 % more with KS = 2, 4 to start and drain a workgroup, 5 + 1.7e-4 per partial row for the merge (with
// the write-back of the rows at the end of the kernel).
// Measured at 173 launches (64, 32, 16 and 8 query heads on 8 or 2 KV heads, 1 to 16 sequences, 64 to 2048 rows behind up to
// 12300 context tokens; profiles/attend_shapes.txt) in every shape: the model is 8 % low with 11 % of scatter, what it takes is
// 0.9 % above the best shape in the geometric mean, and never slower than one group without splits, which all launches were
// before. That one against what is taken, context + rows, 32 heads: 12292 + 1024 326 -> 225 (two groups), 2052 + 700
// 74 -> 47, four sequences of 2052 + 256 69 -> 49, 12292 + 512 315 -> 119 (four splits), 2052 + 128 63 -> 22 (two groups, six
// splits), 0 + 700 22 -> 19. A full chip keeps one group (12292 + 2048: 427 against 452 with two, 2052 + 2048: 116 against 119).
#pragma once
#include <math.h>
#include <stddef.h>

namespace ltri {

constexpr int ATT_NW = 8;                // wavefronts per workgroup of the matrix-core kernel
constexpr int ATT_MAX_SPLITS = 16;       // key-range splits of an attention launch, at most
constexpr int ATT_SPLIT_MAX_ROWS = 4;    // longest query block whose split does not depend on the context (decoding)
// Partial rows of a longer block, at most (34 MB at head_dim 128). Twice what one round of workgroups writes: with more,
// 1100 to 1536 rows of 32 heads would be split into three rounds of workgroups, which the model favours over the two
// rounds of one group but which took 1 to 5 % longer (two groups and splits, 12292 + 1400: 342 against 336, 12292 + 1536: 363 against 348).
constexpr size_t ATT_PART_MAX_ROWS = 65536;

struct AttShape { int ks, ns; };

// Modelled time of a launch in ks groups and ns splits; chunk: share of the chunk's tiles that a workgroup walks.
inline float attend_cost(int Hq, int seq_count, int n_q, int n_ctx, int n_chunk, long long blocks, int ks, int ns, float chunk, int n_cus) {
  const float tiles = (float)((n_ctx + 63) / 64) + (float)((n_chunk + 63) / 64) * chunk;
  const long long rounds = (blocks * ns + n_cus - 1) / n_cus;
  const float fill = (float)(blocks * ns) / (float)(rounds * n_cus);
  const float stages = ceilf(tiles / (float)(ks * ns));
  return (float)rounds * (stages * (1.5f + 0.35f * fill) * (ks == 2 ? 1.07f : 1.f) + 4.f) +
         (ns > 1 ? 5.f + 1.7e-4f * (float)((size_t)seq_count * Hq * n_q * ns) : 0.f);
}

// n_ctx context and n_chunk chunk tokens; part_rows: partial rows there is room for.
inline AttShape attend_shape(int Hq, int Hkv, int seq_count, int n_q, int n_ctx, int n_chunk, size_t part_rows, int n_cus) {
  const int G = Hq / Hkv, HG = G < 4 ? G : 4;
  AttShape best{1, 1};
  float best_cost = 0.f;
  for (int ks = 1; ks <= 2; ++ks) {
    const int rs = ATT_NW / ks / HG, rpb = 32 * rs;
    const long long blocks = (long long)Hkv * (G / HG) * ((n_q + rpb - 1) / rpb) * seq_count;
    for (int ns = 1; ns <= ATT_MAX_SPLITS; ++ns) {
      // The causal part: workgroups end at rows all over the chunk or its upper half. In a single round the longest walks
      // set the pace, in several they average out.
      const float chunk = blocks * ns > n_cus ? 0.75f : 0.85f;
      const float tiles = (float)((n_ctx + 63) / 64) + (float)((n_chunk + 63) / 64) * chunk;
      const size_t rows = (size_t)seq_count * Hq * n_q * ns;
      if (ns > 1 && (rows > part_rows || ns * ks > tiles)) break;
      const float cost = attend_cost(Hq, seq_count, n_q, n_ctx, n_chunk, blocks, ks, ns, chunk, n_cus);
      if ((ks == 1 && ns == 1) || cost < best_cost) { best_cost = cost; best = AttShape{ks, ns}; }
    }
  }
  return best;
}

// The most partial rows that attend_shape takes for the blocks of more than ATT_SPLIT_MAX_ROWS rows of a context: up to
// n_seqs sequences, chunk_max rows and max_ctx context tokens. Row counts are walked by whole workgroups, contexts by
// eighths of their size; a launch between them that wants more takes the best shape there is room for.
inline size_t attend_most_part_rows(int Hq, int Hkv, int n_seqs, int chunk_max, long long max_ctx, int n_cus) {
  const int G = Hq / Hkv, step = 32 * (ATT_NW / 2 / (G < 4 ? G : 4));
  size_t most = 0;
  for (int seqs = 1; seqs <= n_seqs; ++seqs)
    for (int rows = step; rows < chunk_max + step; rows += step) {
      const int n_q = rows < chunk_max ? rows : chunk_max;
      if (n_q <= ATT_SPLIT_MAX_ROWS) continue;
      if ((size_t)2 * seqs * Hq * n_q > ATT_PART_MAX_ROWS) break;
      for (long long ctx = 0;; ctx = ctx + (ctx / 8 > 64 ? ctx / 8 : 64)) {
        const AttShape s = attend_shape(Hq, Hkv, seqs, n_q, (int)(ctx < max_ctx ? ctx : max_ctx), n_q, ATT_PART_MAX_ROWS, n_cus);
        const size_t need = s.ns > 1 ? (size_t)seqs * Hq * n_q * s.ns : 0;
        if (need > most) most = need;
        if (ctx >= max_ctx) break;
      }
      if (most > ATT_PART_MAX_ROWS - ATT_PART_MAX_ROWS / 16) return ATT_PART_MAX_ROWS;
    }
  return most;
}

// ---- fp32 (attend_f32.hip) ----
constexpr int F32_WAVES = 8;             // wavefronts per workgroup, which has 16 (row, head) pairs and takes tiles of 16 keys
constexpr int F32_MAX_SPLITS = 4;
constexpr int F32_SPLIT_WGS = 256;       // workgroups of a split launch, at most (tickets: ATT_EVEN_WGS)

// Splits of the key range: as many as fit one round of workgroups, one per compute unit, while every wavefront keeps two tiles.
inline int attend_f32_splits(int G, int Hkv, int seq_count, int n_q, long long n_ctx) {
  const long long wgs = (long long)((n_q * G + 15) / 16) * Hkv * seq_count, tiles = (n_ctx + n_q + 15) / 16;
  int ns = 1;
  while (ns < F32_MAX_SPLITS && wgs * (ns + 1) <= F32_SPLIT_WGS && tiles >= 2LL * F32_WAVES * (ns + 1)) ++ns;
  return ns;
}

// ---- even shares ----
constexpr int ATT_EVEN_LEAST = 96;       // fewest blocks of a launch: below, a compute unit would fold in many pieces
constexpr int ATT_EVEN_BLOCKS = 512;     // blocks of a die at most (one per thread of the workgroup that counts their stages)
constexpr int ATT_EVEN_WGS = 256;        // workgroups (compute units) there are flags for
// a piece that its workgroup does not finish: 32 / KS pairs of sums, and maximum and sum, per lane
constexpr size_t att_even_place_bytes(int ks) { return (size_t)ATT_NW * (32 / ks + 1) * 64 * 8; }

// Modelled time of a launch in even shares of ks groups, and its blocks.
inline float attend_even_cost(int Hq, int Hkv, int seq_count, int n_q, int n_ctx, int ks, int n_cus, long long* blocks) {
  const int G = Hq / Hkv, HG = G < 4 ? G : 4, rs = ATT_NW / ks / HG, rpb = 32 * rs, n_rb = (n_q + rpb - 1) / rpb;
  const long long slots = (long long)Hkv * (G / HG) * seq_count;
  long long stages = 0;
  for (int y = 0; y < n_rb; ++y) {                         // (as the kernel counts them, but for the lists' lengths)
    const int end = rs == 1 ? (n_rb - y) * 32 : (n_rb * rs - y * (rs / 2)) * 32;
    stages += ((n_ctx + 63) / 64 + ((end < n_q ? end : n_q) + 63) / 64 + ks - 1) / ks;
  }
  *blocks = slots * n_rb;
  const float cu = 1.f / (float)n_cus;
  const float block = ks == 2 ? 8.f : HG == 4 ? 4.5f : 0.5f;
  return (float)(slots * stages) * cu * (ks == 2 ? 2.13f : 1.9f) + (float)*blocks * cu * block + (ks == 2 ? 13.f : 19.f);
}

// Whether a launch is cut into even shares (attend.hip), and then its key groups (else 0). They help where an ordinary launch
// ends with most of the chip idle: just over one round of workgroups, or a second or third round that is nearly empty. They
// do not where it merely starts with some units idle: the chip is limited by power, and the others run faster meanwhile (700
// rows behind 2052 tokens on 176 units take 1.3 us a stage, on all of them 2.3). Nor for a chunk without much of a context: its
// blocks are short, and a share that goes through several of them pays for the start and end of each, which ordinary workgroups
// of several rounds spend beside each other's walks (1121 rows of two sequences, no context, 32 heads: 47 us, in even shares 82).
// Modelled as the share of a compute unit, in stages of 256 pairs x 64 keys at 1.9 us (two groups 2.13), its blocks at 4.5 (less
// than four heads per KV head 0.5, two groups 8), and 19 us (13) for the count of the stages, a second piece, and the partial
// result written, awaited and folded in. Taken where that is below 0.88 of the ordinary shape's cost, which is some 8 % high (and
// more where a workgroup has one sub-tile and several rounds average half the chunk: 0.6 of it counts here). Two groups behind a
// context of less than half the chunk were slower whatever the model said, and are left out.
// Measured in all forms at 1101 launches (64 to 4 query heads, 1 to 24 sequences, 64 to 2048 rows behind 0 to 12292 tokens;
// profiles/attend_even_shares.txt), most of them near the line: taken at 506, 14 % faster there in the mean, at one more than 2 %
// slower (4). With one constant for all blocks the rule took 797 of them, 1 % slower in the mean and 46 % at worst.
// 12292 + 1100 rows 331 -> 245, 2052 + 1050 81 -> 63, 12292 + 700 178 -> 162, three sequences of 8196 + 700 388 -> 299.
inline int attend_even(int Hq, int Hkv, int seq_count, int n_q, int n_ctx, size_t part_bytes, size_t part_rows, int n_cus) {
  const int G = Hq / Hkv, HG = G < 4 ? G : 4;
  if (n_cus % 8 != 0) return 0;
  float cost[3] = {};
  int even = 0;
  for (int ks = 1; ks <= 2; ++ks) {
    long long blocks;
    cost[ks] = attend_even_cost(Hq, Hkv, seq_count, n_q, n_ctx, ks, n_cus, &blocks);
    // (above the limit a die's blocks would outnumber the threads)
    if (blocks < ATT_EVEN_LEAST || blocks > (long long)8 * (ATT_EVEN_BLOCKS - 1) || (size_t)n_cus * att_even_place_bytes(ks) > part_bytes) continue;
    if (ks == 2 && 2 * n_ctx < n_q) continue;
    if (!even || cost[ks] < cost[even]) even = ks;
  }
  if (!even) return 0;
  const AttShape s = attend_shape(Hq, Hkv, seq_count, n_q, n_ctx, n_q, part_rows, n_cus);
  const int rs = ATT_NW / s.ks / HG, rpb = 32 * rs;
  const long long blocks = (long long)Hkv * (G / HG) * ((n_q + rpb - 1) / rpb) * seq_count;
  const float chunk = blocks * s.ns <= n_cus ? 0.85f : rs == 1 ? 0.6f : 0.75f;
  return cost[even] < 0.88f * attend_cost(Hq, seq_count, n_q, n_ctx, n_q, blocks, s.ks, s.ns, chunk, n_cus) ? even : 0;
}

// The most room for pieces that the launches of a context can take.
inline size_t attend_most_even_bytes(int Hq, int Hkv, int n_seqs, int chunk_max, int n_cus) {
  const int G = Hq / Hkv, HG = G < 4 ? G : 4;
  for (int ks = 1; ks <= 2; ++ks) {                        // (the larger place first)
    const int rpb = 32 * (ATT_NW / ks / HG);
    if ((long long)Hkv * (G / HG) * ((chunk_max + rpb - 1) / rpb) * n_seqs >= ATT_EVEN_LEAST) return (size_t)n_cus * att_even_place_bytes(ks);
  }
  return 0;
}

}  // namespace ltri
