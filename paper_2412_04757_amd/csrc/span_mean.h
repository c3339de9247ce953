// Mean of a run of rows, used for the representative keys of new spans (Sec. 3.3.1, mean
// pooling) and for the query-span representatives of step 2. One workgroup of 16 wavefronts
// per span; every lane streams 16-byte pieces, so a long span has tens of KB in flight.
// Sums are fp64 in a fixed order (per lane, then across lanes, then across wavefronts): the
// result is deterministic, and exact before the final division for bf16 inputs.
#pragma once
#include "device_common.h"

namespace ltri {

// Accumulates rows r = 0 .. n_rows-1, row r = `inner` consecutive d-vectors of token r / inner:
// address base + (r / inner) * tok_stride + (r % inner) * d. Writes mean over tokens (sum over
// all rows divided by n_tokens) to out[0..d), or, when out_sum is given, the undivided fp64
// sums to out_sum[0..d). Called by all 1024 threads of a workgroup.
// With tokmask (global or LDS words, bit bit0 + t for token t) only the marked tokens are summed and
// the result is their sum, not a mean (the stored vector of a span's index tokens, Sec. 3.3.2).
template <int DT>
__device__ __forceinline__ void span_mean_block(const typename Elt<DT>::type* base, size_t tok_stride,
                                                int inner, int n_tokens, int d,
                                                typename Elt<DT>::type* out, double (*part)[128],
                                                double* out_sum = nullptr,
                                                const uint32_t* tokmask = nullptr, int bit0 = 0) {
  typedef typename Elt<DT>::type T;
  constexpr int EPP = 16 / (int)sizeof(T);           // elements per 16-byte piece
  const int R = d / EPP;                             // lanes per d-vector (16 or 32)
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int sub = lane / R, piece = lane - sub * R;
  const int rpw = 64 / R;                            // rows per wavefront per load
  const int step = 16 * rpw;
  const int n_rows = n_tokens * inner;
  double acc[EPP];
#pragma unroll
  for (int e = 0; e < EPP; ++e) acc[e] = 0.0;
  for (int r0 = wave * rpw + sub; r0 < n_rows; r0 += 4 * step) {
    uint4 v[4];
    bool ok[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = r0 + u * step;
      ok[u] = r < n_rows;
      const int rr = ok[u] ? r : r0;
      const int tok = rr / inner, g = rr - tok * inner;
      const T* row = base + (size_t)tok * tok_stride + (size_t)g * d + piece * EPP;
      if (tokmask) {                                 // few tokens are marked: only their rows are fetched
        ok[u] = ok[u] && ((tokmask[(bit0 + tok) >> 5] >> ((bit0 + tok) & 31)) & 1u);
        if (ok[u]) v[u] = *reinterpret_cast<const uint4*>(row);
      } else {
        v[u] = *reinterpret_cast<const uint4*>(row);
      }
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (ok[u]) {
        const T* pv = reinterpret_cast<const T*>(&v[u]);
#pragma unroll
        for (int e = 0; e < EPP; ++e) acc[e] += Elt<DT>::to_f64(pv[e]);
      }
    }
  }
  for (int o = R; o < 64; o <<= 1) {
#pragma unroll
    for (int e = 0; e < EPP; ++e) acc[e] += __shfl_xor(acc[e], o, 64);
  }
  if (lane < R) {
#pragma unroll
    for (int e = 0; e < EPP; ++e) part[wave][piece * EPP + e] = acc[e];
  }
  __syncthreads();
  if ((int)threadIdx.x < d) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) s += part[w][threadIdx.x];
    // raw sum of a piece of a span, stored through to device scope: another workgroup of the same launch may
    // add the pieces up (the one that takes the last ticket)
    if (out_sum) __hip_atomic_store(out_sum + threadIdx.x, s, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else         out[threadIdx.x] = Elt<DT>::from_f64(tokmask ? s : s / (double)n_tokens);
  }
  __syncthreads();
}

// ---- the same for all spans of a short chunk, by one workgroup ----
// put(q, c, sum, n): column c of the sum over the tokens of span q (with a mask: its marked ones; n of them), q < nq, of the
// `inner` rows of every token (tok_stride elements apart). start(q): chunk-local start of span q, start(nq) the last one's
// end. Chunks of up to SHORT_SUMS_TOKENS tokens; called by all 64 NW threads; lds: short_sums_lds() bytes. Wavefront w takes
// the w-th share of the tokens (with a mask, of a list of the marked ones, so that only their rows are read), eight loads in
// flight, and leaves one partial sum per span it meets (spans and shares both ascend, so the places differ), which are added
// up in ascending order. It takes the place of a launch with a workgroup per span. What bounds it: one compute unit reads
// about 25 GB/s of rows that are in no cache (128 bf16 tokens of four heads 5 us, 256 fp32 ones, 64 wide, 9.3: longer chunks
// keep a workgroup per span or piece, also for the 64 KB of keys, where this took 5 us behind the selection and the launch 4).
constexpr int SHORT_SUMS_TOKENS = 128;
constexpr int SHORT_SUMS_SPANS = 32;                       // spans at a time
__host__ __device__ constexpr size_t short_sums_lds(int d) {
  return (size_t)(SHORT_SUMS_SPANS + 15) * d * 8 + (SHORT_SUMS_SPANS + 1 + SHORT_SUMS_TOKENS) * 4;
}
template <int DT, int NW, class Start, class Put>
__device__ __forceinline__ void short_span_sums(const typename Elt<DT>::type* base, size_t tok_stride, int inner, int n_tok,
                                                int d, int nq, Start start_of, const uint32_t* mask, unsigned char* lds, Put put) {
  typedef typename Elt<DT>::type T;
  static_assert(NW <= 16, "places of the partial sums");
  constexpr int EPP = 16 / (int)sizeof(T), MW = SHORT_SUMS_TOKENS / 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int R = d / EPP, rpw = 64 / R;                     // lanes per row, rows per load
  const int sub = lane / R, piece = lane - sub * R;
  const int GL = (inner + rpw - 1) / rpw;                  // loads per token
  double* part = reinterpret_cast<double*>(lds);
  int* start = reinterpret_cast<int*>(lds + (size_t)(SHORT_SUMS_SPANS + 15) * d * 8);      // places in the list
  int* list = start + SHORT_SUMS_SPANS + 1;
  uint32_t mw[MW];
  auto place = [&](int t) {                                // marked tokens before token t
    if (!mask) return t;
    int c = 0;
#pragma unroll
    for (int w = 0; w < MW; ++w) {
      const int bits = min(max(t - 32 * w, 0), 32);
      c += __popc(bits == 32 ? mw[w] : mw[w] & ((1u << bits) - 1u));
    }
    return c;
  };
  if (mask) {
#pragma unroll
    for (int w = 0; w < MW; ++w) mw[w] = mask[w];
    if (tid < n_tok && ((mask[tid >> 5] >> (tid & 31)) & 1u)) list[place(tid)] = tid;
  }
  const int n_list = place(n_tok), S = max((n_list + NW - 1) / NW, 1);
  for (int s0 = 0; s0 < nq; s0 += SHORT_SUMS_SPANS) {
    const int ns = min(SHORT_SUMS_SPANS, nq - s0);
    if (s0) __syncthreads();                               // the partial sums of the spans before are read
    if (tid <= ns) start[tid] = place(start_of(s0 + tid));
    __syncthreads();
    const int t_lo = max(wave * S, start[0]), t_hi = min((wave + 1) * S, start[ns]);
    if (t_lo < t_hi) {
      const uint64_t begun = __ballot(lane < ns && start[min(lane, ns)] <= t_lo);
      int s = __popcll(begun) - 1, next = start[s + 1];
      double acc[EPP];
#pragma unroll
      for (int e = 0; e < EPP; ++e) acc[e] = 0.0;
      auto flush = [&]() {
#pragma unroll
        for (int e = 0; e < EPP; ++e) {
          if (R <= 16) acc[e] += lane_xor_f64<16>(acc[e]);
          acc[e] += lane_xor_f64<32>(acc[e]);
        }
        if (lane < R) {
#pragma unroll
          for (int e = 0; e < EPP; ++e) part[(s + wave) * d + piece * EPP + e] = acc[e];
        }
#pragma unroll
        for (int e = 0; e < EPP; ++e) acc[e] = 0.0;
      };
      int lt = t_lo, lg = 0, ct = t_lo, cg = 0;            // (token, load) to request next, and to add next
      while (ct < t_hi) {
        uint4 v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {                      // (past the end: the last token again)
          const int i = min(lt, t_hi - 1), tok = mask ? list[i] : i;
          v[e] = *reinterpret_cast<const uint4*>(base + (size_t)tok * tok_stride + (size_t)min(lg * rpw + sub, inner - 1) * d + piece * EPP);
          if (++lg == GL) { lg = 0; ++lt; }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (ct >= t_hi) break;                           // uniform
          while (cg == 0 && ct == next) { flush(); ++s; next = start[s + 1]; }      // (a span without a marked token: 0)
          if (cg * rpw + sub < inner) {
            const T* pv = reinterpret_cast<const T*>(&v[e]);
#pragma unroll
            for (int k = 0; k < EPP; ++k) acc[k] += Elt<DT>::to_f64(pv[k]);
          }
          if (++cg == GL) { cg = 0; ++ct; }
        }
      }
      flush();
    }
    __syncthreads();
    for (int i = tid; i < ns * d; i += 64 * NW) {
      const int q = i / d, c = i - q * d, b0 = start[q], b1 = start[q + 1];
      double sum = 0.0;
      if (b1 > b0)
        for (int w = b0 / S; w <= (b1 - 1) / S; ++w) sum += part[(q + w) * d + c];
      put(s0 + q, c, sum, b1 - b0);
    }
  }
}

}  // namespace ltri
