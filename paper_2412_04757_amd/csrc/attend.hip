// Step 3 on the device (Sec. 3.4 third step): exact attention of the query chunk over
// initial | retrieved | window tokens (read through the context token list built by step 2)
// and the chunk's own tokens (causal), plus the standalone gather of that context set.
//
// bf16 kernel: flash-style streaming over 64-key tiles on the matrix cores. A workgroup is
// eight wavefronts that share every K/V tile through LDS: the query heads of one KV head's
// group (GQA) times two 32-row sub-tiles, or one sub-tile and two groups of keys, each wavefront
// with its 32 query rows in registers.
// Scores are computed transposed (S^T = K Q^T) so that one lane owns one query: the softmax
// statistics need a single cross-lane exchange and the probabilities are already laid out as
// the B operand of O^T = V^T P^T. The same kernel also attends over a part of the context
// only (the two parts of a step that overlaps steps 1 and 2), and its key range can be split over
// workgroups (attend_shape). One-token chunks (decode) have a kernel without LDS staging
// further down; fp32 contexts have attend_f32.hip.
#include <hip/hip_ext.h>
#include "device_common.h"
#include "attend_args.h"
#include "handoff.h"
#include <algorithm>
#include <array>
#include <type_traits>

namespace ltri {

// A step whose retrieved rows first have to come from host memory attends in two parts: the one that does
// not depend on the retrieval (initial and window tokens and the chunk itself) runs while the chunk is being
// segmented, its spans scored and the rows fetched; the retrieved tokens follow, and that launch folds the first part's result
// (already in `out`, with its log-sum-exp) into its own when it writes.
enum : int { ATT_ALL = 0, ATT_LOCAL = 1, ATT_RETRIEVED = 2 };

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Partial results of a split key range: rows [seq][head][split][query row] of 128 unnormalised fp32 sums, then as
// many (running maximum in the log2 domain, sum) pairs.
__device__ __forceinline__ size_t part_row(const AttArgs& a, int bi, int head, int split, int qi) {
  return (((size_t)bi * a.D.Hq + head) * a.n_splits + split) * a.n_q + qi;
}
__device__ __forceinline__ float2* part_ml(const AttArgs& a) {
  return reinterpret_cast<float2*>(a.part + (size_t)a.seq_count * a.D.Hq * a.n_splits * a.n_q * 128);
}

// two fp32 -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  f32x2_t v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}

// ---- bf16 kernel ----
// K and V tiles go from global memory straight into LDS (global_load_lds, 16 bytes per lane, no
// registers in between) through a ring of NS stages, so NS - 1 tiles are in flight while one is
// being consumed and a single barrier per tile suffices. Both tiles keep the row-major [key][d]
// layout of the arena; inside a 256-byte row the sixteen 16-byte pieces are permuted (XOR with a
// function of the row) so that the fragment reads are free of bank conflicts; the permutation is
// applied by choosing which piece each lane fetches. V^T fragments (A operand of
// O^T = V^T P^T) are read with the transposing LDS load: lane j of a 16-lane group passes the
// address of 4 consecutive d-columns of key row0 + j / 4, lane i receives column i of keys
// row0 .. row0 + 3.
// The DMA is issued through inline assembly because the compiler would otherwise wait for ALL
// outstanding DMA before any LDS read; completion is awaited by hand with s_waitcnt vmcnt(n),
// n = DMA loads requested later than the tile about to be used. Every wavefront issues the same
// number of requests in every iteration (its rows of one stage's K/V tiles and the token ids of its rows
// of a later stage; past the last tile the requests fetch the chunk's last row into a free stage),
// so n is one constant.
// The K fragments of a tile are requested together by hand (the compiler would serialise them
// once registers are tight) and consumed in four groups; the DMA requests of a later tile are
// issued between the groups, under the matrix products. The rescale of O is skipped when no
// lane's running maximum moves.
// The tile loop is cut into segments (context tiles, the ragged last context tile, chunk tiles
// below the diagonal, chunk tiles on the diagonal, tiles this wavefront cannot see) so that the
// body of each segment is straight-line code, with the masks compiled in or out.
typedef short s16x4_t __attribute__((ext_vector_type(4)));

constexpr int TILE_BYTES = 16384;               // one 64-key tile of K or V
constexpr int TOK_SLOTS = 8;                    // ring of token-id tiles (> tokens-ahead distance)
constexpr int att_lds_bytes(int ks, int ns) { return ks * (ns * 2 * TILE_BYTES + TOK_SLOTS * 256); }

// 16 bytes per lane from base + off into LDS at lds_wave_base + 16 * lane. The idle cycle between the write of
// M0 and the load that uses it is the wait state the instruction set asks for; inside an assembly block the
// compiler does not add it.
__device__ __forceinline__ void dma16(const void* base, uint32_t off, uint32_t lds_wave_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_wave_base), "v"(off), "s"(base) : "m0");
}
// 4 bytes per lane
__device__ __forceinline__ void dma4(const void* base, uint32_t off, uint32_t lds_wave_base) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_wave_base), "v"(off), "s"(base) : "m0");
}

enum : int { MASK_NONE = 0, MASK_LIST_END = 1, MASK_CAUSAL = 2 };

// max of three. This file is compiled with -fno-honor-nans (scores are never NaN here), so fmaxf() carries no
// NaN-quieting copies and the compiler folds the pair into one v_max3_f32; being the compiler's own
// instruction, it gets the wait states it needs after matrix-core results and before lane permutes.
__device__ __forceinline__ float max3(float a, float b, float c) { return fmaxf(fmaxf(a, b), c); }

// acc + lo + hi of a packed bf16 pair (one v_dot2c_f32_bf16)
__device__ __forceinline__ float pair_sum(uint32_t packed, float acc) {
  const bf16x2_t one = {(__bf16)1.0f, (__bf16)1.0f};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, packed), one, acc, false);
}

// max over lanes l and l ^ 32 without an LDS round trip: the swap leaves the low half of v in
// both halves of r[0] and the high half in both halves of r[1]
__device__ __forceinline__ float pair_max(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// 16-byte LDS read issued by hand; LDS reads return in order, and the loop holds no scalar loads
// that could disturb the count awaited below
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
template <int OFF>
__device__ __forceinline__ u32x4_t lds_read16(uint32_t addr) {
  u32x4_t r;
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
  return r;
}
// at most N LDS reads still outstanding; ties the four fragments about to be used to the wait
template <int N>
__device__ __forceinline__ void lds_wait(u32x4_t& a, u32x4_t& b, u32x4_t& c, u32x4_t& d) {
  asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N));
}

// ---- even shares (attend_even) ----
// The stages of all blocks (a block: the query rows and heads of one workgroup of an ordinary launch) are strung together and
// cut into equal shares, one per compute unit, wherever the cuts fall. Workgroup ids go round the eight dies, so die x takes
// the ids x, x + 8, ...: it gets an eighth of the blocks (whole ones, KV heads together) and its workgroups, in the order of
// their ids, consecutive shares of it. A share that ends inside a block leaves the partial result of that piece in a place
// of its own; the workgroup whose share holds the block's last stage folds in those of the shares before it. A workgroup takes
// its pieces from the last to the first: the piece that others wait for is its first, the one that waits for others
// its last, so that the wait is short; and as it waits only for lower ids, which were dispatched before it and never wait
// before they have written, it ends whatever else runs on the chip (and is bounded besides).
constexpr int ATT_EVEN_SPINS = 1 << 22;         // polls of a partial result that does not come (some seconds): an error is raised

struct EvenFlag {
  int32_t* p;
  __device__ __forceinline__ int load() const { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ __forceinline__ void store(int v) const { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ __forceinline__ int add(int v) const { return __hip_atomic_fetch_add(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
  __device__ __forceinline__ void pause() const { __builtin_amdgcn_s_sleep(4); }
};

struct EvenShare {
  int xcd, k, per, b0, m;                       // the die's place, this workgroup's among its `per`; first block, blocks
  int u0, u1, lo, hi;                           // stages [u0, u1) of the die's, in its blocks lo .. hi
};

// Stages of one block: those of its context list and of the chunk tiles that its rows see (KS tiles each).
template <int KS>
__device__ __forceinline__ int even_stages(const AttArgs& a, int block, int n_rb) {
  const Dims& D = a.D;
  const int gpk = D.G / (D.G < 4 ? D.G : 4), RS = ATT_NW / KS / (D.G < 4 ? D.G : 4);
  const int sidx = block / n_rb, yb = block - sidx * n_rb, hk = sidx / a.seq_count, bi = sidx - hk * a.seq_count;
  const int slot = slot_of(D, a.layer, a.bp.seq[bi], hk / gpk);
  const int list_len = a.st.meta[(size_t)slot * META_WORDS + META_LIST_LEN];
  const int rb_end = RS == 1 ? min(a.n_q, (n_rb - yb) * 32) : min(a.n_q, (n_rb * RS - yb * (RS / 2)) * 32);
  return ((list_len + 63) / 64 + (rb_end + 63) / 64 + KS - 1) / KS;
}

// The workgroup's share; pre[0 .. m]: first stage of each of the die's blocks, and their sum. All 512 threads.
template <int KS>
__device__ __forceinline__ EvenShare even_share(const AttArgs& a, int n_blocks, int n_rb, int* pre) {
  static_assert(64 * ATT_NW >= ATT_EVEN_BLOCKS, "a block per thread");
  __shared__ int wtot[ATT_NW], edge[2];
  EvenShare e;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  e.xcd = (int)blockIdx.x & 7;
  e.k = (int)blockIdx.x >> 3;
  e.per = (int)gridDim.x >> 3;
  e.b0 = (int)((long long)n_blocks * e.xcd / 8);
  e.m = (int)((long long)n_blocks * (e.xcd + 1) / 8) - e.b0;
  const int own = tid < e.m ? even_stages<KS>(a, e.b0 + tid, n_rb) : 0;
  int incl = wave_scan_i32(own);
  if (lane == 63) wtot[wave] = incl;
  __syncthreads();
  for (int w = 0; w < wave; ++w) incl += wtot[w];
  if (tid < e.m) pre[tid + 1] = incl;
  if (tid == 0) pre[0] = 0;
  __syncthreads();
  const int total = __builtin_amdgcn_readfirstlane(pre[e.m]);
  e.u0 = (int)((long long)total * e.k / e.per);
  e.u1 = (int)((long long)total * (e.k + 1) / e.per);
  if (tid < e.m && pre[tid] <= e.u0 && e.u0 < pre[tid + 1]) edge[0] = tid;
  if (tid < e.m && pre[tid] < e.u1 && e.u1 <= pre[tid + 1]) edge[1] = tid;
  __syncthreads();
  e.lo = e.u0 < e.u1 ? __builtin_amdgcn_readfirstlane(edge[0]) : 1;
  e.hi = e.u0 < e.u1 ? __builtin_amdgcn_readfirstlane(edge[1]) : 0;
  return e;
}

// Partial results from this size on are stored past the caches. 355 split launches (2 to 1024 rows, 1 to 12 sequences), past them
// against through them: up to 1 MB 4 % slower in the mean (two rows of 16 / 1 heads 12.3 us against 11.4), 1 to 3 MB 2 %, 3 to 6 MB
// the same, 6 to 24 MB 2 to 4 % faster.
constexpr size_t ATT_FAR_BYTES = (size_t)4 << 20;

// KS groups of ATT_NW / KS wavefronts, each wavefront with 32 query rows of one head; a ring stage holds KS tiles of
// 64 keys, one per group. NS ring stages. FORM: a block per workgroup, even shares, or a split of a block per workgroup, stored
// through or past the caches. One kernel each: the launches of a stream of ragged chunks (32 / 8 heads, up to 700 tokens, 1 in 26
// in splits) took 55.9 us each from one kernel that can also split, 56.6 from one with both kinds of stores, 54.1 from one per form.
enum : int { ATT_WHOLE = 0, ATT_EVEN = 1, ATT_SPLIT = 2, ATT_SPLIT_FAR = 3 };
template <int KS, int NS, int FORM>
__global__ __launch_bounds__(64 * ATT_NW) void attend_bf16_kernel(AttArgs a) {
  constexpr int NW = ATT_NW, NWQ = NW / KS;         // wavefronts in all, and per group (they cover the workgroup's rows)
  constexpr int TOK_AHEAD = 2 * (NS - 1) + 1;       // token ids of stage t + TOK_AHEAD are requested in iteration t
  constexpr int NI = 16 * KS / NW;                  // DMA row groups per wave and stage
  constexpr int LPT = 2 * NI;                       // K/V requests per lane and stage
  constexpr int IN_FLIGHT = (NS - 2) * (LPT + 1);   // requests that may be pending when a stage is used
  constexpr int TPW = 64 * KS / NW;                 // token ids a wave fetches per stage (those of its own rows)
  constexpr bool EVEN = FORM == ATT_EVEN, SPLIT = FORM >= ATT_SPLIT;
  constexpr int STAGE_BYTES = KS * 2 * TILE_BYTES, TOK_SLOT_BYTES = KS * 256;
  static_assert(NS >= 2 && NS <= 4 && TOK_AHEAD < TOK_SLOTS && (NI == 2 || NI == 4), "request pattern");
  extern __shared__ __attribute__((aligned(16))) unsigned char ring[];
  const Dims& D = a.D;
  const int HG = D.G < 4 ? D.G : 4;                 // heads of the group handled by this block
  const int RS = NWQ / HG;                          // row sub-tiles per block
  const int RPB = 32 * RS;                          // query rows per block
  const int gpk = D.G / HG;                         // blocks per KV head
  // KV head along x: consecutive workgroup ids go to different XCDs, so all query tiles of one
  // KV head run on one XCD and share its K/V rows in that XCD's L2
  // (even shares give each die consecutive blocks, and these are numbered by KV head first)
  const int L = a.n_q, d = 128;
  const int n_splits = SPLIT ? a.n_splits : 1;
  const int n_rb = EVEN ? (L + RPB - 1) / RPB : (int)gridDim.y / n_splits;       // row blocks
  __shared__ int pre[EVEN ? ATT_EVEN_BLOCKS + 1 : 1];
  EvenShare share{};
  if constexpr (EVEN) share = even_share<KS>(a, D.Hkv * gpk * a.seq_count * n_rb, n_rb, pre);
  for (int blk = EVEN ? share.hi : 0; blk >= (EVEN ? share.lo : 0); --blk) {
  int bi = blockIdx.z, hk = blockIdx.x, yb = (int)blockIdx.y / n_splits;
  if constexpr (EVEN) {
    const int block = share.b0 + blk, sidx = block / n_rb;
    yb = block - sidx * n_rb;
    hk = sidx / a.seq_count;
    bi = sidx - hk * a.seq_count;
    if (blk != share.hi) __syncthreads();           // the piece before is done with the ring
  }
  const int h = hk / gpk, gsub = hk - h * gpk;
  const int seq = a.bp.seq[bi], c0 = a.bp.c0[bi];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NWQ, wq = wave % NWQ;       // the wave's key group, and its place among the group's waves
  const int l32 = lane & 31, hf = lane >> 5;
  const int head = h * D.G + gsub * HG + (wq % HG);
  const int split = SPLIT ? (int)blockIdx.y % n_splits : 0;
  // Query rows of the workgroup. The chunk's rows are cut into sub-tiles of 32; workgroup y takes RS / 2 of them
  // from the low end and RS / 2 from the high end (sub-tiles y RS / 2 .. and their mirror images), so that under
  // the causal mask every workgroup has about the same number of (sub-tile, chunk tile) pairs to compute: the
  // low sub-tiles stop early at their diagonal, the high ones walk on alone. With one sub-tile per workgroup
  // (RS == 1) the last rows, which walk furthest, start first.
  const int nsub = n_rb * RS;                       // sub-tiles, padded to whole workgroups
  const int rs = wq / HG;
  const int sub = (RS == 1) ? n_rb - 1 - yb : (rs < RS / 2 ? yb * (RS / 2) + rs : nsub - (yb + 1) * (RS / 2) + (rs - RS / 2));
  const int r0 = sub * 32;                          // first row of this wave
  const int rb_end = (RS == 1) ? min(L, r0 + 32) : min(L, (nsub - yb * (RS / 2)) * 32);   // past the last row of the workgroup
  const int slot = slot_of(D, a.layer, seq, h);
  const unsigned char* Kb = reinterpret_cast<const unsigned char*>(a.k_arena) + arena_off(D, slot) * 2;
  const unsigned char* Vb = reinterpret_cast<const unsigned char*>(a.v_arena) + arena_off(D, slot) * 2;
  const int32_t* meta = a.st.meta + (size_t)slot * META_WORDS;
  // the context list is initial | retrieved | window; the two parts of a two-part step read
  // initial | window from a list of their own, or the retrieved slice of the full list
  const int n_init = min(D.n_sink, c0), n_win = c0 - max(n_init, c0 - D.window);
  int list_len = meta[META_LIST_LEN];
  const int32_t* list = a.st.row_list + (size_t)slot * D.list_cap;
  if (a.part_mode == ATT_LOCAL) {
    list_len = n_init + n_win;
    list = a.loclist + (size_t)bi * a.loc_cap;
  } else if (a.part_mode == ATT_RETRIEVED) {
    list_len = max(list_len - n_init - n_win, 0);
    list += n_init;
  }
  const int n_ctx_tiles = (list_len + 63) / 64;
  const int crow0 = chunk_tok_row(D, c0, c0);       // row of the chunk's first token (the chunk's rows are consecutive)
  const int n_chunk_tiles = a.part_mode == ATT_RETRIEVED ? 0 : (rb_end + 63) / 64;
  const int n_tiles = n_ctx_tiles + n_chunk_tiles;
  // stages of KS tiles; with splits, this workgroup takes the stages [st0, st1) of context and chunk
  const int n_st = (n_tiles + KS - 1) / KS;
  const int first_st = EVEN ? __builtin_amdgcn_readfirstlane(pre[blk]) : 0;       // (of the block, among the die's)
  const int st0 = EVEN ? max(share.u0 - first_st, 0) : (int)((long long)split * n_st / n_splits);
  const int st1 = EVEN ? min(share.u1 - first_st, n_st) : (int)((long long)(split + 1) * n_st / n_splits);
  const uint32_t ring0 = (uint32_t)(uintptr_t)ring;
  const uint32_t tok0 = ring0 + NS * STAGE_BYTES + (uint32_t)wave * (TPW * 4);       // this wave's ids of slot 0
  const int32_t* tokring = reinterpret_cast<const int32_t*>(ring + NS * STAGE_BYTES) + wave * TPW;

  // ---- requests ----
  // A wavefront fetches rows 4 NW i + 4 wave + lq (i < NI, lq = lane / 16) of every stage, lane
  // piece lp = lane % 16 of the row. The token ids of its own rows travel through LDS the
  // same way (lanes 0 .. TPW - 1, id j = 4 i + lq), TOK_AHEAD stages ahead; no other wave reads them, so
  // the wave's own wait makes them visible. Tiles past the list read a dummy entry.
  auto request_tokens = [&](int u) {
    if (lane < TPW) {
      const int row = 4 * NW * (lane >> 2) + 4 * wave + (lane & 3), t = KS * u + (row >> 6);
      dma4(list, (uint32_t)((t < n_ctx_tiles ? t * 64 : 0) + (row & 63)) * 4u, tok0 + (uint32_t)(u % TOK_SLOTS) * TOK_SLOT_BYTES);
    }
  };
  const int lq = lane >> 4, lp = lane & 15;
  // 16-byte pieces of a row that this lane fetches (the row's place in groups of 16 does not depend on i)
  const int prow = 4 * wave + lq;
  const uint32_t kpiece = (uint32_t)((lp ^ (prow & 15)) << 4);
  // V: LDS piece p' of a row holds global piece swap13(p' ^ ((row & 3) << 1)), swap13 = exchange of bits 1 and 3
  const int vp = lp ^ ((prow & 3) << 1);
  const uint32_t vpiece = (uint32_t)(((vp & 5) | ((vp & 2) << 2) | ((vp & 8) >> 2)) << 4);
  // tokens of the rows this lane fetches for stage u (list padding is token 0, masked by position;
  // past the last tile: the chunk's last token)
  auto stage_tokens = [&](int u, int (&tok)[NI]) {
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const int t = KS * u + k;
      if (t < n_ctx_tiles) {
#pragma unroll
        for (int i = k * (NI / KS); i < (k + 1) * (NI / KS); ++i) tok[i] = tokring[(u % TOK_SLOTS) * (TOK_SLOT_BYTES / 4) + 4 * i + lq];
      } else {
#pragma unroll
        for (int i = k * (NI / KS); i < (k + 1) * (NI / KS); ++i)
          tok[i] = crow0 + min((t - n_ctx_tiles) * 64 + 4 * NW * i - 64 * k + prow, L - 1);
      }
    }
  };
  auto request_rows = [&](int u, int i, int tok) {
    const uint32_t dst = ring0 + (uint32_t)(u % NS) * STAGE_BYTES + (uint32_t)(4 * NW * i + 4 * wave) * 256;
    dma16(Kb, ((uint32_t)tok << 8) + kpiece, dst);
    dma16(Vb, ((uint32_t)tok << 8) + vpiece, dst + KS * TILE_BYTES);
  };

  // ---- query fragments: B operand of S^T = K Q^T; lane (l32, hf) holds Q[row l32][16 kk + 8 hf ..] ----
  uint4 qf[8];
  {
    const uint16_t* Qb = reinterpret_cast<const uint16_t*>(a.q) + (size_t)bi * L * D.Hq * d;
    const int row = min(r0 + l32, L - 1);
    const uint16_t* qrow = Qb + ((size_t)row * D.Hq + head) * d;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qf[kk] = *reinterpret_cast<const uint4*>(qrow + kk * 16 + hf * 8);
  }
  // The fragments are "used" here so that the compiler's wait for these loads sits before the
  // loop: a wait for them inside the loop would also wait for every DMA request in flight.
#pragma unroll
  for (int kk = 0; kk < 8; ++kk)
    asm volatile("" ::"v"(qf[kk].x), "v"(qf[kk].y), "v"(qf[kk].z), "v"(qf[kk].w));

  f32x16_t o[4];
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[mb][v] = 0.f;
  float m_run = -1e30f, l_run = 0.f;                // running maximum (log2 domain) and sum
  const float sc = 1.4426950408889634f / sqrtf((float)d);     // log2(e) / sqrt(d)

  // per-lane parts of the fragment addresses
  // K: row l32 (+ 32 kb), piece (2 kk + hf) ^ (row & 15) = ((2 kk) ^ (row & 14)) | (hf ^ (row & 1))
  const uint32_t kbase = (uint32_t)(l32 * 256 + ((hf ^ (l32 & 1)) << 4));
  const uint32_t kswz = (uint32_t)((l32 & 14) << 4);
  uint32_t koff[8];                                 // fragment kk of rows l32 and l32 + 32 (+ 8192)
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) koff[kk] = ring0 + kg * TILE_BYTES + kbase + (kswz ^ (uint32_t)(kk << 5));
  const int vj = lane & 15, vgq = (lane >> 4) & 1;
  const int vrow_in = 4 * hf + (vj >> 2);           // key row inside a group of 8
  // V: the fragment of d-block mb needs global piece 4 mb + 2 gq + x (x = (j & 3) / 2). In LDS it sits at
  // piece swap13(.) ^ swizzle = (gq << 3 | x) | ((mb & 1) << 2 | (mb >> 1) << 1) ^ swizzle: the two
  // 16-lane groups of a half-wave read different 128-byte halves of their rows (no bank conflicts
  // between them), and the four key rows of a group are spread by the swizzle in bits 1..2.
  const uint32_t vbase = (uint32_t)(vrow_in * 256 + (((vgq << 3) | ((vj & 3) >> 1)) << 4) + (vj & 1) * 8);
  const uint32_t vswz = (uint32_t)(((vrow_in & 3) << 1) << 4);
  uint32_t voff[4];                                 // d-block mb
#pragma unroll
  for (int mb = 0; mb < 4; ++mb)
    voff[mb] = ring0 + (KS + kg) * TILE_BYTES + vbase + (vswz ^ (uint32_t)((((mb & 1) << 2) | ((mb >> 1) << 1)) << 4));

  int tokreg[NI];                                   // tokens of the rows of the next stage to request

  // ---- one iteration: wait for stage u, barrier, S^T = K Q^T of the group's tile t = KS u + kg with the requests of
  //      stage u + NS - 1 between the products, masks, online softmax (one query per lane pair), O^T += V^T P^T.
  //      compute = false: a tile this wavefront cannot see (requests, wait and barrier only) ----
  auto tile = [&](int u, auto mask_kind, auto compute_kind) {
    const int t = KS * u + kg;
    constexpr int MK = decltype(mask_kind)::value;
    constexpr bool COMPUTE = decltype(compute_kind)::value;
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(IN_FLIGHT) : "memory");
    __syncthreads();            // stage u is in LDS for every wave; stage u - 1's place is free
    const uint32_t sbase = (uint32_t)(u % NS) * STAGE_BYTES;
    int toknext[NI];
    stage_tokens(u + NS, toknext);
    f32x16_t s[2];
    if constexpr (COMPUTE) {
      // all sixteen K fragments are requested at once (index 2 kk + kb) and used in groups of four
      u32x4_t kf[16];
#pragma unroll
      for (int kk = 0; kk < 8; ++kk) {
        kf[2 * kk] = lds_read16<0>(sbase + koff[kk]);
        kf[2 * kk + 1] = lds_read16<8192>(sbase + koff[kk]);
      }
      __builtin_amdgcn_s_setprio(2);               // matrix-core phases go first when both waves of a SIMD are ready
      const f32x16_t zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
      auto group = [&](int g) {
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
          for (int kb = 0; kb < 2; ++kb)
            s[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, kf[4 * g + 2 * k2 + kb]),
                                                            __builtin_bit_cast(bf16x8_t, qf[2 * g + k2]),
                                                            (g == 0 && k2 == 0) ? zero : s[kb], 0, 0, 0);
      };
      // the scheduling barriers keep each group's products between its wait and the next one
      lds_wait<12>(kf[0], kf[1], kf[2], kf[3]);     group(0); __builtin_amdgcn_sched_barrier(0);
      request_tokens(u + TOK_AHEAD);
      request_rows(u + NS - 1, 0, tokreg[0]);
      lds_wait<8>(kf[4], kf[5], kf[6], kf[7]);      group(1); __builtin_amdgcn_sched_barrier(0);
      request_rows(u + NS - 1, 1, tokreg[1]);
      lds_wait<4>(kf[8], kf[9], kf[10], kf[11]);    group(2); __builtin_amdgcn_sched_barrier(0);
      if constexpr (NI == 4) { request_rows(u + NS - 1, 2, tokreg[2]); request_rows(u + NS - 1, 3, tokreg[3]); }
      lds_wait<0>(kf[12], kf[13], kf[14], kf[15]);  group(3);
      __builtin_amdgcn_s_setprio(0);
    } else {
      request_tokens(u + TOK_AHEAD);
#pragma unroll
      for (int i = 0; i < NI; ++i) request_rows(u + NS - 1, i, tokreg[i]);
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) tokreg[i] = toknext[i];
    if constexpr (!COMPUTE) return;
    if constexpr (MK == MASK_CAUSAL) {
      const int k0 = (t - n_ctx_tiles) * 64;
      const int qi = r0 + l32;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int kp = k0 + kb * 32 + 8 * (v >> 2) + 4 * hf + (v & 3);
          if (kp > qi) s[kb][v] = -INFINITY;
        }
    } else if constexpr (MK == MASK_LIST_END) {
      const int nvalid = list_len - t * 64;
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int kr = kb * 32 + 8 * (v >> 2) + 4 * hf + (v & 3);
          if (kr >= nvalid) s[kb][v] = -INFINITY;
        }
    }
    float m4[4];                                     // four independent max chains, then a tree
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int kb = c >> 1, v0 = (c & 1) * 8;
      m4[c] = max3(s[kb][v0], s[kb][v0 + 1], s[kb][v0 + 2]);
      m4[c] = max3(m4[c], s[kb][v0 + 3], s[kb][v0 + 4]);
      m4[c] = max3(m4[c], s[kb][v0 + 5], s[kb][v0 + 6]);
    }
    float mx = max3(max3(m4[0], s[0][7], s[0][15]), max3(m4[1], s[1][7], s[1][15]), fmaxf(m4[2], m4[3]));
    mx = pair_max(mx) * sc;
    // The reference of the exponentials is the running maximum: the probability of a key that raises it is then 1, which
    // bf16 holds exactly, and such keys carry the largest weights. A reference that lags behind it by up to 2^8 would save
    // most of the rescales (2 to 3 % of a stream), but rounds those keys' probabilities like all others: measured against
    // fp64 over 12292 keys, the error of the output 2.32e-3 -> 2.34e-3, with queries of four times the size 2.03e-3 ->
    // 2.16e-3 and of the log-sum-exp 0.9e-3 -> 1.5e-3; and the sums overflow 2^8 earlier.
    if (__any(mx > m_run)) {
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int mb = 0; mb < 4; ++mb)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[mb][v] *= alpha;
    }
    // probabilities, rounded to bf16 in B-operand order; the row sum is taken over the rounded
    // values (the ones PV multiplies), two per instruction
    uint4 pf[2][2];
    float ps = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
      float pv[16];
#pragma unroll
      for (int v = 0; v < 16; ++v) pv[v] = __builtin_amdgcn_exp2f(fmaf(s[kb][v], sc, -m_run));
#pragma unroll
      for (int a2 = 0; a2 < 2; ++a2) {
        uint4 u;
        u.x = pack_bf16x2(pv[8 * a2 + 0], pv[8 * a2 + 1]);
        u.y = pack_bf16x2(pv[8 * a2 + 2], pv[8 * a2 + 3]);
        u.z = pack_bf16x2(pv[8 * a2 + 4], pv[8 * a2 + 5]);
        u.w = pack_bf16x2(pv[8 * a2 + 6], pv[8 * a2 + 7]);
        pf[kb][a2] = u;
        ps = pair_sum(u.x, ps);
        ps = pair_sum(u.y, ps);
        ps = pair_sum(u.z, ps);
        ps = pair_sum(u.w, ps);
      }
    }
    l_run += ps;
    typedef s16x4_t __attribute__((address_space(3))) * lds_s16x4_ptr;
    // one LDS address per d-block; the (kb, a2, row group) part is a constant offset of the read
    lds_s16x4_ptr vptr[4];
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) vptr[mb] = (lds_s16x4_ptr)(uintptr_t)(sbase + voff[mb]);
#pragma unroll
    for (int kb = 0; kb < 2; ++kb)
#pragma unroll
      for (int a2 = 0; a2 < 2; ++a2)
#pragma unroll
        for (int mb = 0; mb < 4; ++mb) {
          constexpr int ROWB = 256 / 8;                       // one key row in units of s16x4
          const s16x4_t v0 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(vptr[mb] + (kb * 32 + a2 * 16) * ROWB);
          const s16x4_t v1 = __builtin_amdgcn_ds_read_tr16_b64_v4i16(vptr[mb] + (kb * 32 + a2 * 16 + 8) * ROWB);
          const uint2 u0 = __builtin_bit_cast(uint2, v0), u1 = __builtin_bit_cast(uint2, v1);
          uint4 vf;
          vf.x = u0.x; vf.y = u0.y; vf.z = u1.x; vf.w = u1.y;
          o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, vf),
                                                          __builtin_bit_cast(bf16x8_t, pf[kb][a2]), o[mb], 0, 0, 0);
        }
  };

  // ---- prologue: token ids of the first NS stages, then the steady-state request pattern
  //      (ids of stage u + TOK_AHEAD, K/V of stage u + NS - 1) for u = -(NS - 1) .. -1 ----
  for (int u = 0; u < NS; ++u) request_tokens(st0 + u);
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  for (int u = 0; u < NS - 1; ++u) {
    request_tokens(st0 + u + NS);
    stage_tokens(st0 + u, tokreg);
#pragma unroll
    for (int i = 0; i < NI; ++i) request_rows(st0 + u, i, tokreg[i]);
  }
  stage_tokens(st0 + NS - 1, tokreg);

  // ---- tile segments of this wavefront, in stages: past(x) = first stage whose tile of this group is not below x ----
  const bool active = r0 < L;
  auto past = [&](int x) { return min((x - kg + KS - 1) / KS, st1); };           // (x >= 0: the division truncates at 0)
  const int t_list_end = (list_len & 63) ? n_ctx_tiles - 1 : n_ctx_tiles;       // first masked context tile
  // chunk tile kt (keys 64 kt ..) is fully visible to the wave iff 64 kt + 63 <= r0, visible iff 64 kt <= r0 + 31
  const int t_diag = n_ctx_tiles + (active ? min(n_chunk_tiles, (r0 + 1) / 64) : 0);
  const int t_end = active ? n_ctx_tiles + min(n_chunk_tiles, (r0 + 31) / 64 + 1) : 0;
  using std::integral_constant;
  using std::true_type;
  using std::false_type;
  int u = st0;
  if (active) {
    for (; u < past(t_list_end); ++u) tile(u, integral_constant<int, MASK_NONE>{}, true_type{});
    for (; u < past(n_ctx_tiles); ++u) tile(u, integral_constant<int, MASK_LIST_END>{}, true_type{});
    for (; u < past(t_diag); ++u) tile(u, integral_constant<int, MASK_NONE>{}, true_type{});
    for (; u < past(t_end); ++u) tile(u, integral_constant<int, MASK_CAUSAL>{}, true_type{});
  }
  for (; u < st1; ++u) tile(u, integral_constant<int, MASK_NONE>{}, false_type{});
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the requests past the last stage

  // ---- epilogue ----
  float lt = l_run + __shfl_xor(l_run, 32, 64);
  constexpr int NMB = 4 / KS;                       // d-blocks this wave writes, the first one mb0
  const int mb0 = NMB * kg;
  if constexpr (KS == 2) {
    // The two groups hold the same rows over different keys: each hands the other half of its columns (and its
    // maximum and sum) through LDS and merges the half it keeps (the log-sum-exp identity).
    float4* give = reinterpret_cast<float4*>(ring) + wave * 512 + lane;
    float2* mlx = reinterpret_cast<float2*>(ring + NW * 8192) + wave * 64 + lane;
    const float4* take = reinterpret_cast<const float4*>(ring) + (wave ^ NWQ) * 512 + lane;
    __syncthreads();                                // nobody reads the ring or waits for requests into it any more
#pragma unroll
    for (int b = 0; b < NMB; ++b)
#pragma unroll
      for (int a4 = 0; a4 < 4; ++a4) {
        float g[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) g[e] = kg ? o[b][4 * a4 + e] : o[NMB + b][4 * a4 + e];
        give[(b * 4 + a4) * 64] = make_float4(g[0], g[1], g[2], g[3]);
      }
    *mlx = make_float2(m_run, lt);
    __syncthreads();
    const float2 other = reinterpret_cast<const float2*>(ring + NW * 8192)[(wave ^ NWQ) * 64 + lane];
    const float m_new = fmaxf(m_run, other.x);
    const float f0 = __builtin_amdgcn_exp2f(m_run - m_new), f1 = __builtin_amdgcn_exp2f(other.x - m_new);
    lt = lt * f0 + other.y * f1;
    m_run = m_new;
#pragma unroll
    for (int b = 0; b < NMB; ++b)
#pragma unroll
      for (int a4 = 0; a4 < 4; ++a4) {
        const float4 g = take[(b * 4 + a4) * 64];
        const float gv[4] = {g.x, g.y, g.z, g.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float mine = kg ? o[NMB + b][4 * a4 + e] : o[b][4 * a4 + e];
          o[b][4 * a4 + e] = fmaf(gv[e], f1, mine * f0);
        }
      }
  }
  const bool writes_ml = hf == 0 && kg == 0;
  const int qi = r0 + l32;
  if constexpr (EVEN) {
    // A place per workgroup: the registers of a piece as they are, and maximum and sum per lane. Stored and loaded at device
    // scope, in front of and behind a flag (see wait_for_own_stores).
    constexpr int NP = NMB * 8;                     // pairs of sums per lane
    constexpr size_t PLACE = (size_t)NW * (NP + 1) * 64;
    static_assert(PLACE * 8 == att_even_place_bytes(KS), "room of a piece");
    unsigned long long* places = reinterpret_cast<unsigned long long*>(a.part);
    auto place = [&](int k) { return places + (size_t)(share.xcd * share.per + k) * PLACE + (size_t)wave * (NP + 1) * 64 + lane; };
    int32_t* flags = a.even_flags + share.xcd * share.per;
    if (st1 < n_st) {                               // (uniform) the block goes on in the next share
      unsigned long long* pp = place(share.k);
#pragma unroll
      for (int j = 0; j < NP; ++j)
        __hip_atomic_store(pp + j * 64, ((unsigned long long)__float_as_uint(o[j >> 3][2 * (j & 7) + 1]) << 32) | __float_as_uint(o[j >> 3][2 * (j & 7)]),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(pp + NP * 64, ((unsigned long long)__float_as_uint(lt) << 32) | __float_as_uint(m_run), __ATOMIC_RELAXED,
                         __HIP_MEMORY_SCOPE_AGENT);
      wait_for_own_stores();
      __syncthreads();
      if (tid == 0) handoff_give(EvenFlag{flags + share.k});
      continue;
    }
    const long long total = __builtin_amdgcn_readfirstlane(pre[share.m]);
    __shared__ int came[2];                         // in turn: one may still be read while the next share is waited for
    int turn = 0;
    for (int k = share.k - 1; st0 > 0 && k >= 0; --k) {     // the shares before it, back to the block's first stage
      const int v0 = (int)(total * k / share.per), v1 = (int)(total * (k + 1) / share.per);
      if (v0 == v1) continue;
      if (tid == 0) {
        came[turn] = handoff_take(EvenFlag{flags + k}, ATT_EVEN_SPINS);
        if (!came[turn]) atomicCAS(&a.st.err[0], 0, LTRI_EHIP);
      }
      __syncthreads();
      const bool there = came[turn];
      turn ^= 1;
      const unsigned long long* pp = place(k);      // (requested whether it is there or not: the place is the context's)
      const unsigned long long ml = __hip_atomic_load(pp + NP * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      unsigned long long pv[NP];
#pragma unroll
      for (int j = 0; j < NP; ++j) pv[j] = __hip_atomic_load(pp + j * 64, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (!there) {                                 // (the others are still taken: their flags have to be)
        if (v0 <= first_st) break;
        continue;
      }
      const float om = __uint_as_float((uint32_t)ml), ol = __uint_as_float((uint32_t)(ml >> 32));
      const float m_new = fmaxf(m_run, om);
      const float f0 = __builtin_amdgcn_exp2f(m_run - m_new), f1 = __builtin_amdgcn_exp2f(om - m_new);
      lt = lt * f0 + ol * f1;
      m_run = m_new;
#pragma unroll
      for (int j = 0; j < NP; ++j) {
        const int b = j >> 3, v = 2 * (j & 7);
        o[b][v] = fmaf(__uint_as_float((uint32_t)pv[j]), f1, o[b][v] * f0);
        o[b][v + 1] = fmaf(__uint_as_float((uint32_t)(pv[j] >> 32)), f1, o[b][v + 1] * f0);
      }
      if (v0 <= first_st) break;
    }
  }
  auto write_rows = [&]() {
  if constexpr (SPLIT) {
    // unnormalised O, running maximum and sum of this split (the layout of part_row)
    // Many of them past the caches: the launch ends when its writes are out, and 12.6 MB (128 rows of 32 heads in six splits) went
    // out at its end, 19.4 us, now 17.8. Few of them into the caches, where the merge finds them (ATT_FAR_BYTES). (Rows put together
    // in LDS first, so that a store covers 256 bytes of a row instead of 32 of every row, on top of that: no difference.)
    const size_t row = part_row(a, bi, head, split, qi);
    float* pr = a.part + row * d + mb0 * 32 + 4 * hf;
#pragma unroll
    for (int b = 0; b < NMB; ++b)
#pragma unroll
      for (int a4 = 0; a4 < 4; ++a4) {
        const f32x4_t v = {o[b][4 * a4 + 0], o[b][4 * a4 + 1], o[b][4 * a4 + 2], o[b][4 * a4 + 3]};
        f32x4_t* to = reinterpret_cast<f32x4_t*>(pr + b * 32 + 8 * a4);
        if constexpr (FORM == ATT_SPLIT_FAR) __builtin_nontemporal_store(v, to);
        else                                 *to = v;
      }
    if (writes_ml) part_ml(a)[row] = make_float2(m_run, lt);
    return;
  }
  const size_t rh = ((size_t)bi * L + qi) * D.Hq + head;
  uint16_t* orow = reinterpret_cast<uint16_t*>(a.out) + rh * d + mb0 * 32 + 4 * hf;
  if (a.part_mode == ATT_RETRIEVED) {
    // O = (w_a O_a + w_b O_b) / (w_a + w_b) with w = 2^(lse - max lse) (the log-sum-exp identity, log2 domain);
    // O_b = o / lt and lse_b = m_run + log2(lt), so w_b / lt = 2^(m_run - max). Every lane rewrites the
    // elements of O_a it reads. Without a retrieved key the first part stands as it is.
    const float la = a.lse_a[rh];
    if (lt > 0.f) {
      const float la2 = la * 1.4426950408889634f, lb2 = m_run + log2f(lt);
      const float mx = fmaxf(la2, lb2);
      const float wa = __builtin_amdgcn_exp2f(la2 - mx), wb = __builtin_amdgcn_exp2f(lb2 - mx);
      const float inv = 1.f / (wa + wb);
      const float fa = wa * inv, fb = __builtin_amdgcn_exp2f(m_run - mx) * inv;
#pragma unroll
      for (int b = 0; b < NMB; ++b)
#pragma unroll
        for (int a4 = 0; a4 < 4; ++a4) {
          uint2* p = reinterpret_cast<uint2*>(orow + b * 32 + 8 * a4);
          const uint2 ua = *p;
          uint2 u2;
          u2.x = pack_bf16x2(fa * __uint_as_float(ua.x << 16) + fb * o[b][4 * a4 + 0],
                             fa * __uint_as_float(ua.x & 0xFFFF0000u) + fb * o[b][4 * a4 + 1]);
          u2.y = pack_bf16x2(fa * __uint_as_float(ua.y << 16) + fb * o[b][4 * a4 + 2],
                             fa * __uint_as_float(ua.y & 0xFFFF0000u) + fb * o[b][4 * a4 + 3]);
          *p = u2;
        }
      if (a.lse && writes_ml) a.lse[rh] = (mx + log2f(wa + wb)) * 0.6931471805599453f;
    } else if (a.lse && writes_ml) {
      a.lse[rh] = la;
    }
    return;
  }
  const float inv = 1.f / lt;
#pragma unroll
  for (int b = 0; b < NMB; ++b)
#pragma unroll
    for (int a4 = 0; a4 < 4; ++a4) {
      uint2 u2;
      u2.x = pack_bf16x2(o[b][4 * a4 + 0] * inv, o[b][4 * a4 + 1] * inv);
      u2.y = pack_bf16x2(o[b][4 * a4 + 2] * inv, o[b][4 * a4 + 3] * inv);
      *reinterpret_cast<uint2*>(orow + b * 32 + 8 * a4) = u2;
    }
  if (a.lse && writes_ml) a.lse[rh] = (m_run + log2f(lt)) * 0.6931471805599453f;
  };
  if (qi < L) write_rows();
  }                                                 // pieces
}

// ---- merge of the splits: O = sum_s w_s O_s / sum_s w_s l_s, w_s = 2^(m_s - max m) (the log-sum-exp identity).
//      Half a wavefront per row of (head, query row), four columns per lane; lane s of the half holds split s's maximum
//      and sum. A wavefront takes PAIRS pairs of consecutive rows and UNROLL splits of each at a time, so that
//      PAIRS * UNROLL 16-byte loads per lane are in flight. ----
template <int PAIRS, int UNROLL>
__global__ __launch_bounds__(256) void attend_merge_kernel(AttArgs a) {
  const Dims& D = a.D;
  const int L = a.n_q, ns = a.n_splits, lane = threadIdx.x & 63, hl = lane & 31, bi = blockIdx.y;
  const int rr0 = (blockIdx.x * 4 + (threadIdx.x >> 6)) * (2 * PAIRS) + (lane >> 5), n_rows = D.Hq * L;
  int head[PAIRS], qi[PAIRS];
  size_t r0[PAIRS];
  float2 ml[PAIRS];
#pragma unroll
  for (int p = 0; p < PAIRS; ++p) {
    const int rr = min(rr0 + 2 * p, n_rows - 1);
    head[p] = rr / L; qi[p] = rr - head[p] * L;
    r0[p] = part_row(a, bi, head[p], 0, qi[p]);
    ml[p] = part_ml(a)[r0[p] + (size_t)min(hl, ns - 1) * L];
  }
  const float4* po = reinterpret_cast<const float4*>(a.part) + hl;
  float4 v[PAIRS][UNROLL], acc[PAIRS];
  auto load = [&](int s0) __attribute__((always_inline)) {
#pragma unroll
    for (int p = 0; p < PAIRS; ++p)
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) v[p][u] = po[(r0[p] + (size_t)min(s0 + u, ns - 1) * L) * 32];
  };
  load(0);
  float w[PAIRS], l[PAIRS], mmax[PAIRS];
#pragma unroll
  for (int p = 0; p < PAIRS; ++p) {
    mmax[p] = ml[p].x;                                  // lanes past the last split repeat it
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) mmax[p] = fmaxf(mmax[p], __shfl_xor(mmax[p], o, 64));
    w[p] = hl < ns ? __builtin_amdgcn_exp2f(ml[p].x - mmax[p]) : 0.f;
    l[p] = w[p] * ml[p].y;
#pragma unroll
    for (int o = 16; o > 0; o >>= 1) l[p] += __shfl_xor(l[p], o, 64);
    acc[p] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  for (int s0 = 0; s0 < ns; s0 += UNROLL) {
    if (s0 > 0) load(s0);
#pragma unroll
    for (int p = 0; p < PAIRS; ++p)
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const float ws = __shfl(w[p], (lane & 32) + ((s0 + u) & 31), 64);       // 0 past the last split
        acc[p].x = fmaf(ws, v[p][u].x, acc[p].x);
        acc[p].y = fmaf(ws, v[p][u].y, acc[p].y);
        acc[p].z = fmaf(ws, v[p][u].z, acc[p].z);
        acc[p].w = fmaf(ws, v[p][u].w, acc[p].w);
      }
  }
#pragma unroll
  for (int p = 0; p < PAIRS; ++p) {
    if (rr0 + 2 * p >= n_rows) continue;
    const float inv = 1.f / l[p];
    const size_t orow = ((size_t)bi * L + qi[p]) * D.Hq + head[p];
    uint2 u;
    u.x = pack_bf16x2(acc[p].x * inv, acc[p].y * inv);
    u.y = pack_bf16x2(acc[p].z * inv, acc[p].w * inv);
    reinterpret_cast<uint2*>(a.out)[orow * 32 + hl] = u;
    if (a.lse && hl == 0) a.lse[orow] = (mmax[p] + log2f(l[p])) * 0.6931471805599453f;
  }
}

static void launch_merge(const AttArgs& a, int seq_count, hipStream_t s) {
  const int rows = a.D.Hq * a.n_q;
  // many rows: eight rows per wavefront; few (decoding): two, with eight splits of each in flight
  if (rows * seq_count >= 8192) attend_merge_kernel<4, 2><<<dim3((rows + 31) / 32, seq_count), 256, 0, s>>>(a);
  else                          attend_merge_kernel<1, 8><<<dim3((rows + 7) / 8, seq_count), 256, 0, s>>>(a);
}

// ---- one query row per sequence (decode, G <= 4): keys across wavefronts, nothing staged in LDS ----
// The step reads every K and V row of the context once and does next to no arithmetic, so the kernel is
// built to keep loads in flight: a workgroup is four wavefronts that take every n-th 16-key group of
// one (sequence, KV head, split), each on its own (no barrier in the loop); up to three workgroups fit a
// compute unit. Per group a lane fetches 16-byte pieces straight into matrix-core operand order:
//   S^T = K Q^T by v_mfma_f32_16x16x32_bf16: A = 16 keys x 32 d (lane: key lane % 16, d-piece lane / 16),
//   B = Q^T with the heads of the group in columns 0 .. G - 1 and zeros beyond; the result leaves keys
//   4 (lane / 16) + j, j < 4, of head lane % 16 in lane's four registers;
//   O += P V on the vector ALU: a lane owns 8 d-columns (lane % 16) of the 4 keys of its lane group, fetches
//   their V pieces (one 16-byte load per key) and the 4 x G probabilities from the lanes that hold them.
// The running maximum is per head (lane column); the rescale factor of every head reaches all lanes by a
// lane read. Rows of the next group and token ids of the one after are in flight while a group is used. At the
// end the four lane groups' partial O and sums are added, the four wavefronts merge through LDS, and the
// workgroup writes one partial result in the layout attend_merge_kernel reads.
// FUSED: the workgroup of a (sequence, KV head) that finishes last merges the splits itself (a ticket counter, left at zero).
// Groups dealt out in turn let the first token ids be read without waiting for the list's length, and probabilities
// reach their lanes by row broadcasts instead of the LDS crossbar: 2053 keys of 8 heads 7.1 -> 6.6 us.
constexpr int DEC_WAVES = 4;
template <int G, bool FUSED>
__global__ __launch_bounds__(64 * DEC_WAVES, 3) void attend_decode_kernel(AttArgs a) {
  constexpr int d = 128;
  __shared__ float wpart[DEC_WAVES][G][d + 2];
  const Dims& D = a.D;
  const int split = blockIdx.x, h = blockIdx.y, bi = blockIdx.z;
  const int seq = a.bp.seq[bi], c0 = a.bp.c0[bi];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kl = lane & 15, grp = lane >> 4;
  const int slot = slot_of(D, a.layer, seq, h);
  const unsigned char* Kb = reinterpret_cast<const unsigned char*>(a.k_arena) + arena_off(D, slot) * 2;
  const unsigned char* Vb = reinterpret_cast<const unsigned char*>(a.v_arena) + arena_off(D, slot) * 2;
  const int list_len = a.st.meta[(size_t)slot * META_WORDS + META_LIST_LEN];
  const int32_t* list = a.st.row_list + (size_t)slot * D.list_cap;
  const int n_keys = list_len + 1;                  // the context list and the token itself
  const int crow0 = chunk_tok_row(D, c0, c0);
  const int n_groups = (n_keys + 15) >> 4;
  const int workers = a.n_splits * DEC_WAVES, w = split * DEC_WAVES + wave;      // a worker takes every workers-th group

  // B operand: Q^T, head kl of the group in column kl
  uint4 qf[4];
  {
    const uint16_t* qrow = reinterpret_cast<const uint16_t*>(a.q) + ((size_t)bi * D.Hq + (size_t)h * G + min(kl, G - 1)) * d;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      qf[kk] = *reinterpret_cast<const uint4*>(qrow + kk * 32 + grp * 8);
      if (kl >= G) qf[kk] = make_uint4(0u, 0u, 0u, 0u);
    }
  }
  // Tokens of the keys this lane fetches in group g: its K row (key kl) and its four V rows (keys
  // 4 grp + j). Indices are clamped to the last key, so masked keys read a valid row.
  struct Toks { int k, v[4]; };
  // The entries are read without waiting for the list's length (the list has room for list_cap of them); one past the list is
  // replaced by the token's own row when the rows are requested.
  auto load_tokens = [&](int g, Toks& t) __attribute__((always_inline)) {
    t.k = list[min(g * 16 + kl, D.list_cap - 1)];
#pragma unroll
    for (int j = 0; j < 4; ++j) t.v[j] = list[min(g * 16 + 4 * grp + j, D.list_cap - 1)];
  };
  auto load_rows = [&](int g, const Toks& t, uint4 (&kf)[4], uint4 (&vf)[4]) __attribute__((always_inline)) {
    const int tk = g * 16 + kl < list_len ? t.k : crow0;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      kf[kk] = *reinterpret_cast<const uint4*>(Kb + ((size_t)tk << 8) + kk * 64 + grp * 16);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int tv = g * 16 + 4 * grp + j < list_len ? t.v[j] : crow0;
      vf[j] = *reinterpret_cast<const uint4*>(Vb + ((size_t)tv << 8) + kl * 16);
    }
  };

  float o[G][8];
#pragma unroll
  for (int hh = 0; hh < G; ++hh)
#pragma unroll
    for (int c = 0; c < 8; ++c) o[hh][c] = 0.f;
  float m_run = -1e30f, l_lane = 0.f;               // of head kl (log2 domain); the sum over this lane's keys only
  const float sc = 1.4426950408889634f / sqrtf((float)d);

  auto compute = [&](int g, const uint4 (&kf)[4], const uint4 (&vf)[4]) __attribute__((always_inline)) {
    f32x4_t s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
      s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, kf[kk]),
                                                  __builtin_bit_cast(bf16x8_t, qf[kk]), s, 0, 0, 0);
    float sv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) sv[j] = (g * 16 + 4 * grp + j < n_keys) ? s[j] * sc : -INFINITY;
    float mx = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
    mx = fmaxf(mx, __uint_as_float(lane_xor_c<16>(__float_as_uint(mx))));
    mx = pair_max(mx);
    const float m_new = fmaxf(m_run, mx);
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
    const bool moved = __any(kl < G && m_new != m_run);
    m_run = m_new;
    float pv[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) pv[j] = __builtin_amdgcn_exp2f(sv[j] - m_new);
    l_lane = l_lane * alpha + ((pv[0] + pv[1]) + (pv[2] + pv[3]));
    if (moved) {                                    // the running maxima rarely move after the first groups
      // (every row of 16 lanes has head hh's factor in its lane hh)
      auto scale = [&](auto hc) {
        constexpr int hh = decltype(hc)::value;
        const float ah = row_lane<hh>(alpha);
#pragma unroll
        for (int c = 0; c < 8; ++c) o[hh][c] *= ah;
      };
      scale(std::integral_constant<int, 0>{});
      if constexpr (G > 1) scale(std::integral_constant<int, 1>{});
      if constexpr (G > 2) { scale(std::integral_constant<int, 2>{}); scale(std::integral_constant<int, 3>{}); }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint4 u = vf[j];
      float vv[8];
      vv[0] = __uint_as_float(u.x << 16); vv[1] = __uint_as_float(u.x & 0xFFFF0000u);
      vv[2] = __uint_as_float(u.y << 16); vv[3] = __uint_as_float(u.y & 0xFFFF0000u);
      vv[4] = __uint_as_float(u.z << 16); vv[5] = __uint_as_float(u.z & 0xFFFF0000u);
      vv[6] = __uint_as_float(u.w << 16); vv[7] = __uint_as_float(u.w & 0xFFFF0000u);
      auto add = [&](auto hc) {
        constexpr int hh = decltype(hc)::value;
        const float ph = row_lane<hh>(pv[j]);                   // key 4 grp + j of head hh
#pragma unroll
        for (int c = 0; c < 8; ++c) o[hh][c] = fmaf(ph, vv[c], o[hh][c]);
      };
      add(std::integral_constant<int, 0>{});
      if constexpr (G > 1) add(std::integral_constant<int, 1>{});
      if constexpr (G > 2) { add(std::integral_constant<int, 2>{}); add(std::integral_constant<int, 3>{}); }
    }
  };

  // Rows of the next group and tokens of the one after are requested before a group is used; the two
  // row buffers alternate by name so that they stay in registers.
  uint4 ka[4], va[4], kb[4], vb[4];
  Toks t0, t1;
  int g = w;
  load_tokens(g, t0);
  load_tokens(g + workers, t1);
  if (g < n_groups) load_rows(g, t0, ka, va);
  while (g < n_groups) {
    int gn = g + workers;
    if (gn < n_groups) load_rows(gn, t1, kb, vb);
    load_tokens(gn + workers, t0);
    compute(g, ka, va);
    g = gn;
    if (g >= n_groups) break;
    gn = g + workers;
    if (gn < n_groups) load_rows(gn, t0, ka, va);
    load_tokens(gn + workers, t1);
    compute(g, kb, vb);
    g = gn;
  }
  // the four lane groups hold disjoint keys: add their partial results
  auto over_groups = [](float v) {
    v += __uint_as_float(lane_xor_c<16>(__float_as_uint(v)));
    return v + __uint_as_float(lane_xor_c<32>(__float_as_uint(v)));
  };
  l_lane = over_groups(l_lane);
#pragma unroll
  for (int hh = 0; hh < G; ++hh)
#pragma unroll
    for (int c = 0; c < 8; ++c) o[hh][c] = over_groups(o[hh][c]);
  if (grp == 0) {
#pragma unroll
    for (int hh = 0; hh < G; ++hh)
#pragma unroll
      for (int c = 0; c < 8; ++c) wpart[wave][hh][kl * 8 + c] = o[hh][c];
    if (kl < G) { wpart[wave][kl][d] = m_run; wpart[wave][kl][d + 1] = l_lane; }
  }
  __syncthreads();
  // merge of the four wavefronts; one partial result per (head, split): unnormalised O, maximum, sum
  for (int idx = threadIdx.x; idx < G * d; idx += 64 * DEC_WAVES) {
    const int hh = idx / d, c = idx - hh * d;
    float mmax = -1e30f;
#pragma unroll
    for (int ww = 0; ww < DEC_WAVES; ++ww) mmax = fmaxf(mmax, wpart[ww][hh][d]);
    float acc = 0.f, l = 0.f;
#pragma unroll
    for (int ww = 0; ww < DEC_WAVES; ++ww) {
      const float wgt = __builtin_amdgcn_exp2f(wpart[ww][hh][d] - mmax);
      acc = fmaf(wgt, wpart[ww][hh][c], acc);
      l = fmaf(wgt, wpart[ww][hh][d + 1], l);
    }
    const size_t row = part_row(a, bi, h * G + hh, split, 0);
    if constexpr (FUSED) {                            // device scope (see wait_for_own_stores)
      __hip_atomic_store(a.part + row * d + c, acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (c == 0)
        __hip_atomic_store(reinterpret_cast<unsigned long long*>(part_ml(a) + row),
                           ((unsigned long long)__float_as_uint(l) << 32) | __float_as_uint(mmax), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else {
      a.part[row * d + c] = acc;
      if (c == 0) part_ml(a)[row] = make_float2(mmax, l);
    }
  }
  if constexpr (FUSED) {
    __shared__ int s_last;
    wait_for_own_stores();
    __syncthreads();
    int32_t* ticket = a.even_flags + bi * D.Hkv + h;
    if (threadIdx.x == 0) s_last = atomicAdd(ticket, 1) == a.n_splits - 1;
    __syncthreads();
    if (!s_last) return;
    if (threadIdx.x == 0) *ticket = 0;
    // a wavefront per head, two columns per lane; lane s holds split s's maximum and sum (the merge kernel's formula)
    static_assert(G <= DEC_WAVES && ATT_MAX_SPLITS <= 16, "a wavefront per head");
    if (wave >= G) return;
    const int head = h * G + wave, ns = a.n_splits;
    const size_t r0 = part_row(a, bi, head, 0, 0);
    const unsigned long long* po = reinterpret_cast<const unsigned long long*>(a.part + r0 * d) + lane;
    unsigned long long v[ATT_MAX_SPLITS];
    const unsigned long long ml = __hip_atomic_load(reinterpret_cast<const unsigned long long*>(part_ml(a) + r0) + min(lane, ns - 1),
                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int s = 0; s < ATT_MAX_SPLITS; ++s)
      v[s] = s < ns ? __hip_atomic_load(po + (size_t)s * (d / 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
    const float m = __uint_as_float((uint32_t)ml), mmax = lanes_max<16>(m);      // (lanes past the last split repeat it)
    const float wl = lane < ns ? __builtin_amdgcn_exp2f(m - mmax) : 0.f;
    float l = wl * __uint_as_float((uint32_t)(ml >> 32)), x = 0.f, y = 0.f;
    l += __uint_as_float(lane_xor_c<8>(__float_as_uint(l)));
    l += __uint_as_float(lane_xor_c<4>(__float_as_uint(l)));
    l += __uint_as_float(lane_xor_c<2>(__float_as_uint(l)));
    l += __uint_as_float(lane_xor_c<1>(__float_as_uint(l)));
    l = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(l)));
    const float top = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)__float_as_uint(mmax)));
#pragma unroll
    for (int s = 0; s < ATT_MAX_SPLITS; ++s) {
      const float ws = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(wl), s));       // 0 past the last split
      x = fmaf(ws, __uint_as_float((uint32_t)v[s]), x);
      y = fmaf(ws, __uint_as_float((uint32_t)(v[s] >> 32)), y);
    }
    const float inv = 1.f / l;
    const size_t orow = (size_t)bi * D.Hq + head;
    reinterpret_cast<uint32_t*>(a.out)[orow * (d / 2) + lane] = pack_bf16x2(x * inv, y * inv);
    if (a.lse && lane == 0) a.lse[orow] = (top + log2f(l)) * 0.6931471805599453f;
  }
}

// ---- first part of a two-part step: its token list ----
// initial | window tokens of every sequence of the batch, padded with token 0 to whole tiles
__global__ __launch_bounds__(256) void local_list_kernel(Dims D, BatchPos bp, int32_t* loclist, int loc_cap) {
  const int bi = blockIdx.y, c0 = bp.c0[bi];
  const int n_init = min(D.n_sink, c0), w0 = max(n_init, c0 - D.window), len = n_init + c0 - w0;
  const int r = blockIdx.x * 256 + threadIdx.x;
  if (r < loc_cap) loclist[(size_t)bi * loc_cap + r] = r < n_init ? r : (r < len ? window_tok_row(D, w0 + r - n_init) : 0);
}

// ---- standalone gather: K/V rows of the context list into packed buffers ----
struct GatherArgs { Dims D; DevState st; const void* k_arena; const void* v_arena; int layer, seq;
                    void* k_packed; void* v_packed; int32_t* n_tokens; };

constexpr int GATHER_ROWS = 4;
__global__ __launch_bounds__(256) void gather_pack_kernel(GatherArgs a) {
  const Dims& D = a.D;
  const int h = blockIdx.y;
  const int slot = slot_of(D, a.layer, a.seq, h);
  const int32_t* meta = a.st.meta + (size_t)slot * META_WORDS;
  const int list_len = meta[META_LIST_LEN];
  const int32_t* list = a.st.row_list + (size_t)slot * D.list_cap;
  const int row16 = D.d * D.elt / 16;                        // 16-byte pieces per row
  const int rows_per_pass = 256 / row16;
  const int r_in = threadIdx.x / row16, piece = threadIdx.x - r_in * row16;
  typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
  const u32x4* Kb = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(a.k_arena) + arena_off(D, slot) * D.elt);
  const u32x4* Vb = reinterpret_cast<const u32x4*>(reinterpret_cast<const char*>(a.v_arena) + arena_off(D, slot) * D.elt);
  u32x4* Kp = reinterpret_cast<u32x4*>(a.k_packed) + (size_t)h * D.list_cap * row16;
  u32x4* Vp = reinterpret_cast<u32x4*>(a.v_packed) + (size_t)h * D.list_cap * row16;
  // GATHER_ROWS rows per thread and trip: the token ids first, then all the row pieces (2 x GATHER_ROWS independent
  // 16-byte loads in flight per lane), then the stores, which nothing reads again soon (non-temporal)
  const int stride = gridDim.x * rows_per_pass;
  for (int r0 = blockIdx.x * rows_per_pass + r_in; r0 < list_len; r0 += GATHER_ROWS * stride) {
    int tok[GATHER_ROWS];
#pragma unroll
    for (int u = 0; u < GATHER_ROWS; ++u) tok[u] = list[min(r0 + u * stride, list_len - 1)];
    u32x4 kv[GATHER_ROWS], vv[GATHER_ROWS];
#pragma unroll
    for (int u = 0; u < GATHER_ROWS; ++u) {
      kv[u] = Kb[(size_t)tok[u] * row16 + piece];
      vv[u] = Vb[(size_t)tok[u] * row16 + piece];
    }
#pragma unroll
    for (int u = 0; u < GATHER_ROWS; ++u) {
      const int r = r0 + u * stride;
      if (r < list_len) {
        __builtin_nontemporal_store(kv[u], Kp + (size_t)r * row16 + piece);
        __builtin_nontemporal_store(vv[u], Vp + (size_t)r * row16 + piece);
      }
    }
  }
  if (a.n_tokens && blockIdx.x == 0 && threadIdx.x == 0) a.n_tokens[h] = list_len;
}

// ---- how a launch splits the key range of a short query block, and what its partial results need ----
// kind: 0 = no short block, 1 = the one-token kernel, 2 = the matrix-core kernel with splits
static int attend_split_count(const Dims& D, int seq_count, int n_q, int n_cus, int* kind) {
  *kind = 0;
  if (!attend_on_matrix_cores(D) || n_q > ATT_SPLIT_MAX_ROWS) return 1;
  if (n_q == 1 && D.G <= 4) {
    // decode: two workgroups per compute unit (measured best at 16 sequences x 8 KV heads: 67 us against
    // 70 .. 81 us with 3 .. 16 splits; the step runs at the rate of a plain copy either way)
    const int slots = D.Hkv * seq_count;
    const int ns = (2 * n_cus) / slots;
    *kind = 1;
    return ns > ATT_MAX_SPLITS ? ATT_MAX_SPLITS : (ns < 1 ? 1 : ns);
  }
  // a short query block on few workgroups: split the key range so that every compute unit streams a
  // share of it; the partial results are merged by a second kernel
  const int HG = D.G < 4 ? D.G : 4;
  const int blocks = D.Hkv * (D.G / HG) * seq_count;
  if (blocks >= 256) return 1;
  const int ns = 256 / blocks;
  if (ns <= 1) return 1;
  *kind = 2;
  return ns > ATT_MAX_SPLITS ? ATT_MAX_SPLITS : ns;
}

// Context tokens that a chunk behind c0 tokens is expected to attend (the lists themselves are on the device): initial and
// window tokens, and retrieved ones.
static long long near_tokens(const Dims& D, long long c0) { return std::min<long long>(c0, (long long)D.n_sink + D.window); }
static long long far_tokens(const Dims& D, long long c0) {
  const long long far = D.budget ? D.budget : D.k_max ? (long long)D.k_max * 256 : c0;
  return std::min(far, c0);
}

// Rows of partial results a context's scratch has room for: short query blocks at any batch, and as many as a launch of
// longer ones takes within the context's limits (on 256 compute units).
size_t attend_part_rows(const Dims& D) {
  if (!attend_on_matrix_cores(D)) return attend_f32_part_rows();
  const long long max_ctx = std::min(D.max_tokens, near_tokens(D, D.max_tokens) + far_tokens(D, D.max_tokens));
  const size_t short_rows = (size_t)D.n_seqs * D.Hq * ATT_MAX_SPLITS * ATT_SPLIT_MAX_ROWS;
  const int seqs = std::min(D.n_seqs, LTRI_MAX_BATCH);
  const size_t row = (size_t)(D.d + 2) * sizeof(float);
  const size_t even = (attend_most_even_bytes(D.Hq, D.Hkv, seqs, D.chunk_max, 256) + row - 1) / row;
  return std::max(std::max(short_rows, even), attend_most_part_rows(D.Hq, D.Hkv, seqs, D.chunk_max, max_ctx, 256));
}

static hipError_t device_cus(int* n_cus) {
  static int cached = 0;
  if (cached == 0) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cached, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) { cached = 0; return e; }
  }
  *n_cus = cached;
  return hipSuccess;
}

size_t attend_partial_bytes(const Dims& D, int seq_count, int n_q, int n_cus) {
  int kind = 0;
  const int ns = attend_split_count(D, seq_count, n_q, n_cus, &kind);
  if (kind == 0) return 0;
  return (size_t)seq_count * D.Hq * ns * (kind == 1 ? 1 : n_q) * (D.d + 2) * sizeof(float);
}

// ---- partial results for callers that bring no buffer ----
// One array per GPU, held from the moment the library is loaded until the process ends. In host code the
// array's name is only a handle for hipGetSymbolAddress; the address the kernels get is the one that call
// returns, looked up once per device with that device current.
static __device__ __align__(256) unsigned char scratch[ATT_STATIC_SCRATCH_BYTES];

hipError_t attend_static_scratch(float** ptr) {
  constexpr int MAX_DEVICES = 64;
  static void* per_device[MAX_DEVICES] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
  if (!per_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    per_device[dev] = p;
  }
  *ptr = static_cast<float*>(per_device[dev]);
  return hipSuccess;
}

hipError_t launch_attend(const Dims& D, const DevState& st, const void* k_arena, const void* v_arena,
                         const void* q, int layer, const BatchPos& bp, int seq_count, int n_q,
                         void* out, float* lse, int stages, float* part, int32_t* even_flags, int part_mode,
                         const int32_t* loclist, int loc_cap, const float* lse_a, hipStream_t s, hipEvent_t t_begin, hipEvent_t t_end) {
  if ((t_begin == nullptr) != (t_end == nullptr)) return hipErrorInvalidValue;
  AttArgs a;
  a.D = D; a.st = st; a.k_arena = k_arena; a.v_arena = v_arena; a.q = q; a.out = out; a.lse = lse;
  a.layer = layer; a.seq_count = seq_count; a.n_q = n_q; a.bp = bp;
  a.n_splits = 1; a.part = part; a.even_flags = even_flags;
  a.part_mode = part_mode; a.loclist = loclist; a.loc_cap = loc_cap; a.lse_a = lse_a;
  if (part_mode == ATT_RETRIEVED && !lse_a) return hipErrorInvalidValue;
  const bool mfma_ok = attend_on_matrix_cores(D);
  if (part_mode != ATT_ALL && (!mfma_ok || n_q <= ATT_SPLIT_MAX_ROWS)) return hipErrorInvalidValue;
  int n_cus = 0, kind = 0;
  if (hipError_t e = device_cus(&n_cus); e != hipSuccess) return e;
  const int ns_short = (part && part_mode == ATT_ALL) ? attend_split_count(D, seq_count, n_q, n_cus, &kind) : 1;
  if (kind == 1) {
    a.n_splits = ns_short;
    dim3 g(a.n_splits, D.Hkv, seq_count);
    if (t_begin) { if (hipError_t e = hipEventRecord(t_begin, s); e != hipSuccess) return e; }
    // The last workgroup of a head merges, where the caller has tickets for it: a launch less. 16 sequences over 128K tokens
    // (retrieve and attend) 84.9 -> 83.6 us, one over 16K 18.6 -> 17.4, a token of eight sequences 33.1 -> 31.6.
    const bool fused = even_flags != nullptr;
    auto decode = [&](auto gc) {
      constexpr int G = decltype(gc)::value;
      if (fused) attend_decode_kernel<G, true><<<g, 64 * DEC_WAVES, 0, s>>>(a);
      else       attend_decode_kernel<G, false><<<g, 64 * DEC_WAVES, 0, s>>>(a);
    };
    if (D.G == 4)      decode(std::integral_constant<int, 4>{});
    else if (D.G == 2) decode(std::integral_constant<int, 2>{});
    else               decode(std::integral_constant<int, 1>{});
    if (!fused) launch_merge(a, seq_count, s);
    if (t_end) { if (hipError_t e = hipEventRecord(t_end, s); e != hipSuccess) return e; }
    return hipGetLastError();
  }
  long long c0 = 0;
  for (int i = 0; i < seq_count; ++i) c0 = bp.c0[i] > c0 ? bp.c0[i] : c0;
  const long long near = near_tokens(D, c0), far = far_tokens(D, c0);
  if (mfma_ok) {
    const long long n_ctx = part_mode == ATT_LOCAL ? near : part_mode == ATT_RETRIEVED ? far : std::min(near + far, c0);
    const size_t room = std::min((size_t)D.att_part_rows, ATT_PART_MAX_ROWS);
    const int even = part && part_mode == ATT_ALL && n_q > ATT_SPLIT_MAX_ROWS && even_flags && n_cus <= ATT_EVEN_WGS
                         ? attend_even(D.Hq, D.Hkv, seq_count, n_q, (int)n_ctx, (size_t)D.att_part_rows * (D.d + 2) * sizeof(float), room, n_cus) : 0;
    AttShape shape = attend_shape(D.Hq, D.Hkv, seq_count, n_q, (int)n_ctx, part_mode == ATT_RETRIEVED ? 0 : n_q,
                                  part && part_mode == ATT_ALL ? room : 0, n_cus);
    if (n_q <= ATT_SPLIT_MAX_ROWS) shape = AttShape{2, ns_short};
    if (even) shape = AttShape{even, 1};
    const int ks = shape.ks, ns = shape.ns;
    const int HG = D.G < 4 ? D.G : 4;
    const int gpk = D.G / HG;
    const int RPB = 32 * (ATT_NW / ks / HG);
    a.n_splits = ns;
    dim3 g(D.Hkv * gpk, (n_q + RPB - 1) / RPB * ns, seq_count);
    if (even) g = dim3(n_cus);
    static bool attr_set = false;
    if (!attr_set) {
      auto of = [](auto ksc, auto nsc) {
        constexpr int KS = decltype(ksc)::value, NS = decltype(nsc)::value;
        return std::array<const void*, 4>{reinterpret_cast<const void*>(&attend_bf16_kernel<KS, NS, ATT_WHOLE>),
                                          reinterpret_cast<const void*>(&attend_bf16_kernel<KS, NS, ATT_EVEN>),
                                          reinterpret_cast<const void*>(&attend_bf16_kernel<KS, NS, ATT_SPLIT>),
                                          reinterpret_cast<const void*>(&attend_bf16_kernel<KS, NS, ATT_SPLIT_FAR>)};
      };
      using std::integral_constant;
      for (const auto& forms : {of(integral_constant<int, 1>{}, integral_constant<int, 4>{}), of(integral_constant<int, 1>{}, integral_constant<int, 3>{}),
                                of(integral_constant<int, 2>{}, integral_constant<int, 2>{})})
        for (const void* f : forms) {
          const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, att_lds_bytes(2, 2));
          if (e != hipSuccess) return e;
        }
      attr_set = true;
    }
    auto launch = [&](auto ksc, auto nsc, auto formc) {
      constexpr int KS = decltype(ksc)::value, NS = decltype(nsc)::value, FORM = decltype(formc)::value;
      constexpr int lds = att_lds_bytes(KS, NS);
      // the events ride in the kernel's own dispatch; with a merge behind it the end is recorded after that
      if (t_begin)
        hipExtLaunchKernelGGL((attend_bf16_kernel<KS, NS, FORM>), g, dim3(64 * ATT_NW), (uint32_t)lds, s, t_begin, ns > 1 ? nullptr : t_end, 0, a);
      else
        attend_bf16_kernel<KS, NS, FORM><<<g, 64 * ATT_NW, lds, s>>>(a);
    };
    using std::integral_constant;
    auto form = [&](auto ksc, auto nsc) {
      if (even)                                  launch(ksc, nsc, integral_constant<int, ATT_EVEN>{});
      else if (ns == 1)                          launch(ksc, nsc, integral_constant<int, ATT_WHOLE>{});
      else if ((size_t)seq_count * n_q * D.Hq * ns * D.d * sizeof(float) < ATT_FAR_BYTES)
                                                 launch(ksc, nsc, integral_constant<int, ATT_SPLIT>{});
      else                                       launch(ksc, nsc, integral_constant<int, ATT_SPLIT_FAR>{});
    };
    if (ks == 2)          form(integral_constant<int, 2>{}, integral_constant<int, 2>{});
    else if (stages == 3) form(integral_constant<int, 1>{}, integral_constant<int, 3>{});
    else                  form(integral_constant<int, 1>{}, integral_constant<int, 4>{});
    if (ns > 1) {
      launch_merge(a, seq_count, s);
      if (t_end) { if (hipError_t e = hipEventRecord(t_end, s); e != hipSuccess) return e; }
    }
  } else {
    if (t_begin) { if (hipError_t e = hipEventRecord(t_begin, s); e != hipSuccess) return e; }
    if (hipError_t e = launch_attend_f32(a, std::min(near + far, c0), s); e != hipSuccess) return e;
    if (t_end) { if (hipError_t e = hipEventRecord(t_end, s); e != hipSuccess) return e; }
  }
  return hipGetLastError();
}

bool attend_on_matrix_cores(const Dims& D) {
  return D.dtype == LTRI_BF16 && D.d == 128 && (D.G == 1 || D.G == 2 || D.G % 4 == 0);
}

hipError_t launch_local_list(const Dims& D, const BatchPos& bp, int seq_count, int32_t* loclist, int loc_cap,
                             hipStream_t s) {
  local_list_kernel<<<dim3((loc_cap + 255) / 256, seq_count), 256, 0, s>>>(D, bp, loclist, loc_cap);
  return hipGetLastError();
}

hipError_t launch_gather_pack(const Dims& D, const DevState& st, const void* k_arena, const void* v_arena,
                              int layer, int seq, void* k_packed, void* v_packed, int32_t* n_tokens,
                              hipStream_t s) {
  GatherArgs a{D, st, k_arena, v_arena, layer, seq, k_packed, v_packed, n_tokens};
  const int row16 = D.d * D.elt / 16;
  const int rows_per_pass = 256 / row16;
  int gx = (D.list_cap + rows_per_pass * GATHER_ROWS - 1) / (rows_per_pass * GATHER_ROWS);
  if (gx < 1) gx = 1;
  dim3 g(gx, D.Hkv);
  gather_pack_kernel<<<g, 256, 0, s>>>(a);
  return hipGetLastError();
}

}  // namespace ltri
