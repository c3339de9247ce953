// Step 3 for fp32 contexts: the same exact attention, on the fp32 matrix cores.
//
// v_mfma_f32_16x16x4f32 with 16 (query row, head) pairs of one KV head as columns, so that every group size fills the
// tile and the rows of a tile are few (the causal edge costs one tile). A wavefront walks every 8th tile of 16 keys of
// its workgroup's pairs with all operands in registers: nothing is shared between wavefronts but the caches, and a
// chunk of 256 rows x 4 heads still runs 512 wavefronts. S^T = K Q^T leaves the probabilities of one query in four
// lanes as the B operand of O^T = V^T P^T; key k of a tile is fed as product step k % 4, lane group k / 4, which is the
// order they come in. The partial results of the wavefronts (own maximum, sum and O) are merged in LDS at the end, in a
// fixed order.
// Launches that reach few compute units (256 rows x 4 heads: 64 workgroups) split the key range over workgroups as well: each
// leaves its partial result (16 queries, 4 or 8 KB), and the one of a tile of pairs that finishes last (a ticket counter,
// left at zero again) adds them up, in a fixed order.
// What bounds it: the chain list -> rows -> products before and the merges after, and the fp32 matrix rate (256 flop per cycle
// and compute unit) of the compute units it reaches. 256 rows of 4 / 1 heads x 64 behind some 900 tokens: 18.9 us without
// splits, 13.2 with four.
// Measured against one wavefront per row and head on the vector ALU, context + rows (us): 4 / 1 heads x 64
// wide, 1028 + 256: 223 -> 22, 1540 + 1: 249 -> 22; 8 / 2 x 64, 1504 + 1000: 680 -> 75; 4 / 2 x 128, 1504 + 512:
// 673 -> 61, two sequences of 1504 + 2048: 4692 -> 311. Error against fp64 there: 6e-7 .. 1e-6 -> 3e-7 .. 5e-7.
// 16 wavefronts per workgroup: 24.5 (a smaller share of the tiles each, a larger merge), 4: 25.9; 32 pairs per
// wavefront (half the row loads): 37.4 and no faster on large launches.
#include "device_common.h"
#include "attend_args.h"

namespace ltri {

typedef float f32x4u_t __attribute__((ext_vector_type(4), aligned(4)));      // the caller's query rows: element alignment

__device__ __forceinline__ bool not_finite(float x) { return (__float_as_uint(x) & 0x7f800000u) == 0x7f800000u; }
__device__ __forceinline__ float group_max(float v) {      // over the four lanes of a query
  v = fmaxf(v, __uint_as_float(lane_xor_c<16>(__float_as_uint(v))));
  return fmaxf(v, __uint_as_float(lane_xor_c<32>(__float_as_uint(v))));
}

constexpr int F32_PITCH = 68;                                // floats per query of a wavefront's 64 columns in LDS

template <int DIM>
__global__ __launch_bounds__(64 * F32_WAVES, DIM == 64 ? 4 : 2) void attend_f32_kernel(AttArgs a) {
  constexpr int NP = DIM / 16;                               // 4-element pieces of a row for each of its four lanes
  constexpr int NC = DIM / 64;                               // 64-column parts of a row
  __shared__ float part[F32_WAVES * 16 * F32_PITCH];
  __shared__ float s_m[F32_WAVES][16], s_l[F32_WAVES][16];
  const Dims& D = a.D;
  const int G = D.G, L = a.n_q;
  __shared__ int s_last;
  const int h = blockIdx.y, bi = blockIdx.z, ns = a.n_splits;
  const int n_blocks = (int)gridDim.x / ns, split = (int)blockIdx.x % ns, block = n_blocks - 1 - (int)blockIdx.x / ns;
  const int p0 = block * 16;                                 // the latest rows, which see the most keys, first
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, r = lane & 15, g = lane >> 4;
  const int seq = a.bp.seq[bi], c0 = a.bp.c0[bi];
  const int slot = slot_of(D, a.layer, seq, h);
  const float* Kb = reinterpret_cast<const float*>(a.k_arena) + arena_off(D, slot);
  const float* Vb = reinterpret_cast<const float*>(a.v_arena) + arena_off(D, slot);
  const int list_len = a.st.meta[(size_t)slot * META_WORDS + META_LIST_LEN];
  const int32_t* list = a.st.row_list + (size_t)slot * D.list_cap;
  const int chunk_row = chunk_tok_row(D, c0, c0);
  const int last_pair = min(p0 + 16, L * G) - 1;
  const int n_keys = list_len + last_pair / G + 1;           // keys the latest row of the workgroup sees
  const int n_open = list_len + p0 / G + 1;                  // keys every row of it sees
  const int n_tiles = (n_keys + 15) / 16;
  const float scale = 1.0f / sqrtf((float)DIM);

  const int pair = min(p0 + r, last_pair);
  const int vis = list_len + pair / G + 1;                   // keys the lane's query sees
  f32x4_t qf[NP];
  {
    const float* qrow = reinterpret_cast<const float*>(a.q) + (((size_t)bi * L + pair / G) * D.Hq + h * G + pair % G) * DIM;
#pragma unroll
    for (int u = 0; u < NP; ++u) qf[u] = *reinterpret_cast<const f32x4u_t*>(qrow + 4 * (g + 4 * u));
  }
  f32x4_t o[NC][4];                                          // O[query r][64 c + 16 g + 4 v + e] = o[c][e][v]
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) o[c][e] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = -1e30f, l_run = 0.f;                         // l_run: the lane's own keys only

  auto token = [&](int t) -> int {                           // row of key 16 t + r (past the end: the last key)
    const int k = min(16 * t + r, n_keys - 1);
    return k < list_len ? list[k] : chunk_row + (k - list_len);
  };
  f32x4_t kf[NP], vf[4][NC];
  auto load_k = [&](int tok) {
    const float* row = Kb + (size_t)tok * DIM + 4 * g;
#pragma unroll
    for (int u = 0; u < NP; ++u) kf[u] = *reinterpret_cast<const f32x4_t*>(row + 16 * u);
  };
  auto load_v = [&](int tok) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const float* row = Vb + (size_t)__shfl(tok, 4 * g + v, 64) * DIM + 4 * r;
#pragma unroll
      for (int c = 0; c < NC; ++c) vf[v][c] = *reinterpret_cast<const f32x4_t*>(row + 64 * c);
    }
  };
  const int step = F32_WAVES * ns, t0 = split * F32_WAVES + wave;
  int tok = token(t0), tok_next = token(t0 + step);
  load_k(tok);
  load_v(tok);
  for (int t = t0; t < n_tiles; t += step) {
    f32x4_t s = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int u = 0; u < NP; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[u][e], qf[u][e], s, 0, 0, 0);
    // the rows of the wavefront's next tile are requested as soon as this one's registers are free
    tok = tok_next;
    load_k(tok);
    tok_next = token(t + 2 * step);
    const bool edge = 16 * t + 16 > n_open;                  // uniform: some row does not see the whole tile
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      s[v] *= scale;
      if (edge && 16 * t + 4 * g + v >= vis) s[v] = -INFINITY;
    }
    const float m_new = fmaxf(m_run, group_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]))));
    if (__any(m_new > m_run)) {
      const float alpha = expf(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int c = 0; c < NC; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[c][e] *= alpha;
      m_run = m_new;
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) s[v] = expf(s[v] - m_run);
    l_run += (s[0] + s[1]) + (s[2] + s[3]);
    bool apart = false;                                      // an infinity or NaN in a row that some query must not see
    if (edge) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) apart |= not_finite(vf[v][c][e]);
      apart = __any(apart);
    }
    if (!apart) {
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
          for (int e = 0; e < 4; ++e) o[c][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[v][c][e], s[v], o[c][e], 0, 0, 0);
    } else {
      // key by key; a query that must not see a key keeps its sums (a product with a probability of 0 would not do)
      for (int gg = 0; gg < 4; ++gg)
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
          for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const f32x4_t x = __builtin_amdgcn_mfma_f32_16x16x4f32(g == gg ? vf[v][c][e] : 0.f, g == gg ? s[v] : 0.f,
                                                                    o[c][e], 0, 0, 0);
              if (16 * t + 4 * gg + v < vis) o[c][e] = x;
            }
    }
    load_v(tok);
  }

  // ---- merge of the wavefronts, in a fixed order ----
  l_run += __uint_as_float(lane_xor_c<16>(__float_as_uint(l_run)));
  l_run += __uint_as_float(lane_xor_c<32>(__float_as_uint(l_run)));
  if (g == 0) { s_m[wave][r] = m_run; s_l[wave][r] = l_run; }
  __syncthreads();
  float m_all = -1e30f;
#pragma unroll
  for (int w = 0; w < F32_WAVES; ++w) m_all = fmaxf(m_all, s_m[w][r]);
  const float f = expf(m_run - m_all);                       // 0 for a wavefront without a key
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    if (c) __syncthreads();                                  // the columns before are read
#pragma unroll
    for (int v = 0; v < 4; ++v)
      *reinterpret_cast<f32x4_t*>(part + (wave * 16 + r) * F32_PITCH + 16 * g + 4 * v) =
          f32x4_t{o[c][0][v] * f, o[c][1][v] * f, o[c][2][v] * f, o[c][3][v] * f};
    __syncthreads();
#pragma unroll
    for (int qq = 0; qq < 16 / F32_WAVES; ++qq) {            // one query per wavefront, a column per lane
      const int q = wave + F32_WAVES * qq, p = p0 + q;
      if (p <= last_pair) {
        float m = -1e30f, l = 0.f, sum = 0.f;
#pragma unroll
        for (int w = 0; w < F32_WAVES; ++w) m = fmaxf(m, s_m[w][q]);
#pragma unroll
        for (int w = 0; w < F32_WAVES; ++w) {
          l = fmaf(s_l[w][q], expf(s_m[w][q] - m), l);
          sum += part[(w * 16 + q) * F32_PITCH + lane];
        }
        if (ns > 1) {                                        // unnormalised, with its maximum and sum; device scope (see below)
          float* pr = a.part + (((size_t)(bi * D.Hkv + h) * n_blocks + block) * ns + split) * (16 * (DIM + 2)) + q * (DIM + 2);
          __hip_atomic_store(pr + 64 * c + lane, sum, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          if (c == 0 && lane < 2) __hip_atomic_store(pr + DIM + lane, lane ? l : m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          continue;
        }
        const size_t rh = ((size_t)bi * L + p / G) * D.Hq + h * G + p % G;
        reinterpret_cast<float*>(a.out)[rh * DIM + 64 * c + lane] = sum * (1.f / l);
        if (c == 0 && a.lse && lane == 0) a.lse[rh] = m + logf(l);
      }
    }
  }
  if (ns == 1) return;
  // the workgroup that takes the last ticket of its tile of pairs adds the splits up
  wait_for_own_stores();
  __syncthreads();
  int32_t* ticket = a.even_flags + (size_t)(bi * D.Hkv + h) * n_blocks + block;
  if (threadIdx.x == 0) s_last = atomicAdd(ticket, 1) == ns - 1;
  __syncthreads();
  if (!s_last) return;
  if (threadIdx.x == 0) *ticket = 0;
  const float* base = a.part + ((size_t)(bi * D.Hkv + h) * n_blocks + block) * ns * (16 * (DIM + 2));
  auto get = [&](int s, int i) { return __hip_atomic_load(base + (size_t)s * (16 * (DIM + 2)) + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); };
  for (int q = wave; q < 16 && p0 + q <= last_pair; q += F32_WAVES) {
    float mv[F32_MAX_SPLITS], lv[F32_MAX_SPLITS], ov[F32_MAX_SPLITS][NC];
#pragma unroll
    for (int s = 0; s < F32_MAX_SPLITS; ++s) {
      const int ss = min(s, ns - 1);
      mv[s] = get(ss, q * (DIM + 2) + DIM);
      lv[s] = get(ss, q * (DIM + 2) + DIM + 1);
#pragma unroll
      for (int c = 0; c < NC; ++c) ov[s][c] = get(ss, q * (DIM + 2) + 64 * c + lane);
    }
    float m = mv[0], l = 0.f, sum[NC] = {};
#pragma unroll
    for (int s = 1; s < F32_MAX_SPLITS; ++s) m = fmaxf(m, mv[s]);
#pragma unroll
    for (int s = 0; s < F32_MAX_SPLITS; ++s) {
      const float f = expf(mv[s] - m);                       // 0 for a split without a key, whose sums are 0
      l = s < ns ? fmaf(lv[s], f, l) : l;
#pragma unroll
      for (int c = 0; c < NC; ++c) sum[c] = s < ns ? fmaf(ov[s][c], f, sum[c]) : sum[c];
    }
    const int p = p0 + q;
    const size_t rh = ((size_t)bi * L + p / G) * D.Hq + h * G + p % G;
#pragma unroll
    for (int c = 0; c < NC; ++c) reinterpret_cast<float*>(a.out)[rh * DIM + 64 * c + lane] = sum[c] * (1.f / l);
    if (a.lse && lane == 0) a.lse[rh] = m + logf(l);
  }
}

// Rows of partial results (of head_dim + 2 floats) a split launch takes, at most.
size_t attend_f32_part_rows() { return (size_t)F32_SPLIT_WGS * 16; }

size_t attend_f32_short_bytes(const Dims& D) {
  if (D.dtype != LTRI_F32) return 0;
  const size_t wgs = (size_t)((ATT_SPLIT_MAX_ROWS * D.G + 15) / 16) * D.Hkv * (D.n_seqs < LTRI_MAX_BATCH ? D.n_seqs : LTRI_MAX_BATCH);
  const size_t split = wgs * F32_MAX_SPLITS;
  return (split < (size_t)F32_SPLIT_WGS ? split : (size_t)F32_SPLIT_WGS) * 16 * (D.d + 2) * sizeof(float);
}

// n_ctx: context tokens that the chunk is expected to attend.
hipError_t launch_attend_f32(const AttArgs& args, long long n_ctx, hipStream_t s) {
  AttArgs a = args;
  const Dims& D = a.D;
  const int blocks = (a.n_q * D.G + 15) / 16;
  a.n_splits = a.part && a.even_flags ? attend_f32_splits(D.G, D.Hkv, a.seq_count, a.n_q, n_ctx) : 1;
  const dim3 grid(blocks * a.n_splits, D.Hkv, a.seq_count);
  if (D.d == 64) attend_f32_kernel<64><<<grid, 64 * F32_WAVES, 0, s>>>(a);
  else           attend_f32_kernel<128><<<grid, 64 * F32_WAVES, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace ltri
