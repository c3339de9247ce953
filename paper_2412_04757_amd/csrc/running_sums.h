// Running sums of a chunk's query rows (summed over the query heads of a KV head) and key rows, for step 2 of long
// chunks with mean representatives: Q^R of a query span (Eq. 8's query side) and the mean key of a new span
// (Sec. 3.3.1) are each a difference of two running sums divided by the span's length, and running sums need no
// span boundaries, so they are taken while, or before, the chunk is segmented.
// Layout: out[problem][token][128] (fp64, `rows` rows per problem) holds, for token t, the sum of the rows of the
// tokens of t's block of RUNSUM_BLOCK tokens up to and including t; the reader adds the last rows of the earlier
// blocks. The key rows' sums follow `keys_off` elements behind the query rows'. bf16 rows, head_dim 128 only. Sums of bf16
// values in fp64 are exact while the values of a column span less than 2^30 in magnitude over the chunk (8 bits
// each, 13 for the row count, 53 in all), so the result does not depend on the order of the additions and a
// difference of two running sums is the sum over the rows between them.
#pragma once
#include "device_common.h"

namespace ltri {

constexpr int RUNSUM_BLOCK = 128;

// Workgroups per problem that running_sums_block is to be called by: one per block of query rows, one per two blocks of
// key rows (a key block is a quarter of the rows of a query block of the paper's model).
__host__ __device__ inline int running_sums_blocks(const RunSums& r) {
  const int nblk = (r.n_q + RUNSUM_BLOCK - 1) / RUNSUM_BLOCK;
  return nblk + (r.k_arena ? (nblk + 1) / 2 : 0);
}

// One block of tokens (query or key rows) for problem p = (sequence batch_off + p / Hkv, KV head p % Hkv). Called by all
// 1024 threads of a workgroup; wt: LDS, 16 x 128 doubles. A wavefront takes 8 tokens and a lane two columns of them, so
// that the running sums of a lane's tokens need no exchange, a row is read in one piece and a token's sums are written
// in one piece; the 16 wavefronts meet once, over the totals of their tokens. A chunk of 1024 tokens (96 workgroups on
// an otherwise idle chip, 10 MB in and 16 MB out) is bound by the latency of a workgroup. With 8 columns and two tokens
// per lane, whose sums went through 48 lane exchanges and left in 16-byte pieces 64 bytes apart, it took 12 us and the
// launch it rides in 19.4; now that launch takes 13.5 (700 tokens: 18.1 and 10.4) and its selections bound it.
// The sums leave past the caches: other dies read them, and a launch ends when its writes are out (2048 tokens, 32 MB: that
// launch 18.4 -> 16.6 us and step 2, which reads them, 18.4 -> 18.75; 1024 tokens 18.1 -> 17.1 and 13.75 -> 14.1).
__device__ __forceinline__ void running_sums_one(const Dims& D, const BatchPos& bp, int layer, int batch_off,
                                                 const RunSums& r, int blk, bool keys, int p, double* wt) {
  constexpr int TOK = RUNSUM_BLOCK / 16;                // tokens per wavefront
  const int d = 128, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, col = 2 * lane;
  const int bi = batch_off + p / D.Hkv, h = p % D.Hkv;
  const int inner = keys ? 1 : D.G;                     // rows per token
  const size_t tok_stride = keys ? (size_t)d : (size_t)D.Hq * d;
  const uint16_t* base;
  if (keys && r.k_chunk) {
    base = reinterpret_cast<const uint16_t*>(r.k_chunk) + (size_t)(bi * D.Hkv + h) * r.n_q * d + col;
  } else if (keys) {
    const int c0 = bp.c0[bi];
    base = reinterpret_cast<const uint16_t*>(r.k_arena) + arena_off(D, slot_of(D, layer, bp.seq[bi], h)) +
           (size_t)chunk_tok_row(D, c0, c0) * d + col;
  } else {
    base = reinterpret_cast<const uint16_t*>(r.q) + (size_t)bi * r.n_q * D.Hq * d + (size_t)h * D.G * d + col;
  }
  const int t0 = blk * RUNSUM_BLOCK + TOK * wave;
  double x[TOK], y[TOK];                                // sums of a token's rows, then running sums over the tokens
#pragma unroll
  for (int t = 0; t < TOK; ++t) x[t] = y[t] = 0.0;
  for (int g0 = 0; g0 < inner; g0 += 4) {               // 4 rows of 8 tokens in flight
    uint32_t v[4][TOK];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (g0 + g >= inner) break;                       // uniform
#pragma unroll
      for (int t = 0; t < TOK; ++t)
        v[g][t] = *reinterpret_cast<const uint32_t*>(base + (size_t)min(t0 + t, r.n_q - 1) * tok_stride + (size_t)(g0 + g) * d);
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      if (g0 + g >= inner) break;
#pragma unroll
      for (int t = 0; t < TOK; ++t) {
        x[t] += (double)__uint_as_float(v[g][t] << 16);
        y[t] += (double)__uint_as_float(v[g][t] & 0xffff0000u);
      }
    }
  }
#pragma unroll
  for (int t = 1; t < TOK; ++t) { x[t] += x[t - 1]; y[t] += y[t - 1]; }   // (tokens past the chunk come last and are not written)
  *reinterpret_cast<double2*>(wt + wave * d + col) = make_double2(x[TOK - 1], y[TOK - 1]);
  __syncthreads();
  double cx = 0.0, cy = 0.0;
  for (int w = 0; w < wave; ++w) {
    const double2 u = *reinterpret_cast<const double2*>(wt + w * d + col);
    cx += u.x;
    cy += u.y;
  }
  typedef double f64x2_t __attribute__((ext_vector_type(2)));
  double* out = r.out + (keys ? r.keys_off : (size_t)0) + ((size_t)p * r.rows + t0) * d + col;
#pragma unroll
  for (int t = 0; t < TOK; ++t)
    if (t0 + t < r.n_q) __builtin_nontemporal_store(f64x2_t{cx + x[t], cy + y[t]}, reinterpret_cast<f64x2_t*>(out + (size_t)t * d));
}

// Workgroup `w` (0 .. running_sums_blocks - 1) of problem p.
__device__ __forceinline__ void running_sums_block(const Dims& D, const BatchPos& bp, int layer, int batch_off,
                                                   const RunSums& r, int w, int p, double* wt) {
  const int nblk = (r.n_q + RUNSUM_BLOCK - 1) / RUNSUM_BLOCK;
  const bool keys = w >= nblk;
  const int b0 = keys ? 2 * (w - nblk) : w, b1 = keys ? min(b0 + 2, nblk) : w + 1;
  for (int b = b0; b < b1; ++b) {                       // uniform over the workgroup
    if (b > b0) __syncthreads();                        // wt is written again
    running_sums_one(D, bp, layer, batch_off, r, b, keys, p, wt);
  }
}

}  // namespace ltri
