// Step 1 of a chunk of up to SEG_SHORT tokens in one launch: one workgroup per (sequence, KV head) keeps the chunk's map (at
// most three 64 x 64 tiles, fp64) in LDS from the products to the index vectors. Included by seg.hip, whose tile layout,
// arithmetic and order of additions it shares.
// What bounds it: the latency of one chain on one compute unit (rows -> products -> row statistics -> percentile ->
// cumulative sums -> selection -> votes -> key sums), whatever the number of problems up to the number of compute units. The
// general path runs the same chain as up to thirteen launches, each with its own start, round trips and recomputed tile;
// a chunk of 128 tokens at the paper's settings (softmax map, percentile theta, index vectors): 83 us in eleven launches and the
// gaps between them -> 36 in one (rows and products 4.3, log-sum-exp 4.2, percentile 6.6, sums 4.9, selection 4.0, index
// tokens 5, key sums 3.8).
// 12 wavefronts, four per tile: with the chunk's 128 rows on two tiles a side there is no fourth tile.
#pragma once

namespace ltri {

constexpr int SEG_SHORT = 128;
constexpr int SHORT_NT = 768;                              // threads: 256 per tile
constexpr int SHORT_COPIES = 4;                            // interleaved histograms of the percentile's digits
constexpr int SHORT_FEW = 256;                             // keys that are ranked by comparing them all

struct SegShortShared {
  __attribute__((aligned(16))) double Ms[3][64 * 65];      // tiles (0, 0), (1, 0), (1, 1); operands before, key sums after
  double a4[3][4][64], b4[3][4][64];                       // shares of a row or column by its four threads
  double lse[SEG_SHORT];
  double pscore[3][128];
  double dyn[3][SEG_SHORT];                                // votes, row sums inside the span, whole row sums
  int8_t px[3][128];
  uint32_t hist[QUANT_BINS * SHORT_COPIES];
  unsigned long long few[SHORT_FEW];
  unsigned long long rank, count, key, wtop[SHORT_NT / 64];
  uint32_t wtot[8], bin;
  uint32_t n_few;
  int cut[SEG_SHORT + 1];
  int8_t tokspan[SEG_SHORT];
  uint32_t cutbit[8];                                      // token positions 0 .. L where a span starts or the chunk ends
  uint32_t mask[8];                                        // index tokens
  int cnt[SEG_SHORT];                                      // Eq. 7 counts of the chunk's spans
  uint64_t vkey[SEG_SHORT];
};

// 128 rows x 256 bytes (the kc-th 256-byte piece of every row), as stage_rows does it for 64.
template <typename T>
__device__ __forceinline__ void short_stage(unsigned char* dst, const T* base, size_t row_stride, int L, int kc) {
#pragma unroll
  for (int i = 0; i < (SEG_SHORT * 16 + SHORT_NT - 1) / SHORT_NT; ++i) {
    const int q = threadIdx.x + SHORT_NT * i;
    if (q >= SEG_SHORT * 16) break;
    const int row = q >> 4, piece = q & 15;
    const int grow = min(row, L - 1);                      // clamped; masked by the caller
    const uint4 v = *(reinterpret_cast<const uint4*>(reinterpret_cast<const unsigned char*>(base + (size_t)grow * row_stride) + kc * 256) + piece);
    *reinterpret_cast<uint4*>(dst + row * 256 + ((piece ^ (row & 15)) << 4)) = v;
  }
}

// Adds every thread's bins b[v] (v set in `use`) to the histogram; neighbouring cells often share one, and runs are added at
// once. Then the bin that holds the rank: S.bin, S.count its cells, S.rank the rank among them. All threads.
__device__ __forceinline__ void short_pick(const uint32_t (&b)[16], uint32_t use, unsigned long long rank, SegShortShared& S) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  uint32_t run_bin = 0u, run = 0;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    if (!((use >> v) & 1u)) continue;
    if (b[v] != run_bin) {
      if (run) atomicAdd(&S.hist[run_bin * SHORT_COPIES + (lane & (SHORT_COPIES - 1))], run);
      run_bin = b[v]; run = 0;
    }
    ++run;
  }
  if (run) atomicAdd(&S.hist[run_bin * SHORT_COPIES + (lane & (SHORT_COPIES - 1))], run);
  __syncthreads();
  // the first 512 threads hold four bins each
  uint32_t cnt[4] = {0u, 0u, 0u, 0u}, own = 0u, incl = 0u;
  if (tid < 512) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint4 h = *reinterpret_cast<const uint4*>(&S.hist[(4 * tid + e) * SHORT_COPIES]);
      static_assert(SHORT_COPIES == 4 && QUANT_BINS == 4 * 512, "a bin is one 16-byte piece");
      cnt[e] = (h.x + h.y) + (h.z + h.w);
      own += cnt[e];
    }
    incl = (uint32_t)wave_scan_i32((int)own);
    if (lane == 63) S.wtot[wave] = incl;
  }
  __syncthreads();
  if (tid < 512) {
    for (int w = 0; w < wave; ++w) incl += (uint32_t)S.wtot[w];
    const uint32_t excl = incl - own;
    if (rank >= excl && rank < incl) {                     // one thread: the counts add up to more than the rank
      uint32_t below = excl;
      int at = 3;
      uint32_t c = cnt[3];
      bool open = true;
#pragma unroll
      for (int e = 0; e < 3; ++e) {
        const bool here = open && below + cnt[e] > rank;
        if (here) { at = e; c = cnt[e]; open = false; }
        if (open) below += cnt[e];
      }
      S.bin = (uint32_t)(4 * tid + at);
      S.rank = rank - below;
      S.count = c;
    }
  }
  __syncthreads();
}

// The cell of rank a.quant_rank of the chunk's map, whose cells the threads hold: m[v] where valid bit v is set. Order keys as
// in quant_pick_step, in registers. The first histogram takes the distance below the largest key in steps of 2^-6 of an octave,
// 32 octaves: its bin has few cells unless many are equal or far below the largest one, and they are compared. Else the digits
// of quant_pick_step, 11 bits each, until at most SHORT_FEW are left. (By digits from the start: 8 us of the kernel, the first
// one being sign and exponent, which most cells share; like this 6.6.)
__device__ __forceinline__ double short_quantile(const SegArgs& a, const double (&m)[16], uint32_t valid, SegShortShared& S) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto clear = [&]() {
    for (int i = tid; i < QUANT_BINS * SHORT_COPIES / 4; i += SHORT_NT) reinterpret_cast<uint4*>(S.hist)[i] = make_uint4(0u, 0u, 0u, 0u);
  };
  auto collect = [&](uint32_t use) {                       // the marked cells' keys to S.few
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      if (!((use >> v) & 1u)) continue;
      const uint32_t at = atomicAdd(&S.n_few, 1u);
      if (at < (uint32_t)SHORT_FEW) S.few[at] = ascending_key(m[v]);
    }
    __syncthreads();
  };
  uint64_t top = 0ull;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const uint64_t k = ascending_key(m[v]);
    if (((valid >> v) & 1u) && k > top) top = k;
  }
  auto larger = [&](auto mc) {
    constexpr int M = decltype(mc)::value;
    const uint64_t o = ((uint64_t)lane_xor_c<M>((uint32_t)(top >> 32)) << 32) | lane_xor_c<M>((uint32_t)top);
    top = o > top ? o : top;
  };
  larger(std::integral_constant<int, 1>{}); larger(std::integral_constant<int, 2>{}); larger(std::integral_constant<int, 4>{});
  larger(std::integral_constant<int, 8>{}); larger(std::integral_constant<int, 16>{}); larger(std::integral_constant<int, 32>{});
  if (lane == 0) S.wtop[wave] = top;
  if (tid == 0) S.n_few = 0u;
  clear();
  __syncthreads();
#pragma unroll
  for (int w = 0; w < SHORT_NT / 64; ++w) top = S.wtop[w] > top ? S.wtop[w] : top;
  uint32_t b[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const uint64_t step = (top - ascending_key(m[v])) >> 46;
    b[v] = step < (uint64_t)QUANT_BINS ? (uint32_t)step : (uint32_t)QUANT_BINS - 1u;
  }
  short_pick(b, valid, a.quant_cells - 1ull - a.quant_rank, S);        // (counted from the largest cell down)
  if (S.count <= (unsigned long long)SHORT_FEW) {          // uniform
    const uint32_t bin = S.bin;
    uint32_t use = 0u;
#pragma unroll
    for (int v = 0; v < 16; ++v) use |= (b[v] == bin) ? (valid & (1u << v)) : 0u;
    collect(use);
    const int n = (int)min(S.n_few, (uint32_t)SHORT_FEW);
    if (tid < n) {
      const unsigned long long k = S.few[tid], rank = S.rank;
      int above = 0, same = 0;
#pragma unroll 4
      for (int j = 0; j < n; ++j) { above += S.few[j] > k; same += S.few[j] == k; }
      // equal keys all pass this test and write the same value
      if ((unsigned long long)above <= rank && rank < (unsigned long long)(above + same)) S.key = k;
    }
    __syncthreads();
    return key_to_double(S.key);
  }
  unsigned long long left = a.quant_cells, rank = a.quant_rank, prefix = 0ull;
  int digit = 0;
  auto matching = [&](int hi) {                            // cells that share the prefix down to bit hi
    uint32_t use = 0u;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const uint64_t k = ascending_key(m[v]);
      use |= (hi >= 64 || (k >> hi) == (prefix >> hi)) ? (valid & (1u << v)) : 0u;
    }
    return use;
  };
  for (; digit < QUANT_PASSES && left > (unsigned long long)SHORT_FEW; ++digit) {
    __syncthreads();                                       // the state is read
    clear();
    __syncthreads();
    const int shift = quant_shift(digit), width = quant_width(digit);
#pragma unroll
    for (int v = 0; v < 16; ++v) b[v] = (uint32_t)(ascending_key(m[v]) >> shift) & ((1u << width) - 1u);
    short_pick(b, matching(64 - QUANT_BITS * digit), rank, S);
    prefix |= (uint64_t)S.bin << shift;
    rank = S.rank;
    left = S.count;
  }
  if (digit == QUANT_PASSES) return key_to_double(prefix);
  collect(matching(64 - QUANT_BITS * digit));
  const int n = (int)min(S.n_few, (uint32_t)SHORT_FEW);
  if (tid < n) {
    const unsigned long long k = S.few[tid];
    int below = 0, same = 0;
    for (int j = 0; j < n; ++j) { below += S.few[j] < k; same += S.few[j] == k; }
    if ((unsigned long long)below <= rank && rank < (unsigned long long)(below + same)) S.key = k;
  }
  __syncthreads();
  return key_to_double(S.key);
}

template <int DT, int KIND>
__global__ __launch_bounds__(SHORT_NT) void seg_short_kernel(SegArgs a) {
  typedef typename Elt<DT>::type T;
  __shared__ SegShortShared S;
  const Dims& D = a.D;
  const int p = blockIdx.x, sl = p / D.Hkv, h = p - sl * D.Hkv, bi = a.batch_off + sl;
  if (blockIdx.y > 0) {
    copy_chunk_rows(D, a.src, a.layer, a.bp, bi, h, a.n_new, (int)blockIdx.y - 1, a.copy_wgs);
    return;
  }
  const int c0 = a.bp.c0[bi], slot = slot_of(D, a.layer, a.bp.seq[bi], h);
  const int L = a.n_new, d = D.d, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = __builtin_amdgcn_readfirstlane(tid >> 8);      // the thread's tile
  const int I = grp > 0, J = grp > 1, t = tid & 255, li = t & 63, part = t >> 6;
  const int wi = part >> 1, wj = part & 1, hf = lane >> 5, l32 = lane & 31;
  const bool live = grp == 0 || L > 64;
  const bool whole = I > J && L == SEG_SHORT;
  int32_t* meta = a.st.meta + (size_t)slot * META_WORDS;
  const int base = meta[META_N_SPANS];
  const T* Kc = chunk_keys<T>(a, bi, h);
  const T* Qb = a.q_seg ? reinterpret_cast<const T*>(a.q_seg) + (size_t)bi * L * D.Hq * d + (size_t)h * D.G * d : nullptr;
  const int n_h = a.q_seg ? D.G : 1;
  const int nkc = d * (int)sizeof(T) / 256;                // 256-byte pieces per row
  const double scale = 1.0 / sqrt((double)d);
  constexpr bool logit = KIND == LTRI_MAP_LOGIT;
  unsigned char* kbuf = reinterpret_cast<unsigned char*>(S.Ms);
  unsigned char* qbuf = Qb ? kbuf + SEG_SHORT * 256 : kbuf;
  double* Ms = S.Ms[grp];
  const int i0 = I * 64 + wi * 32 + 4 * hf, jcol = J * 64 + wj * 32 + l32;     // cell v: row i0 + 8 (v / 4) + v % 4, column jcol
  uint32_t valid = 0;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const int i = i0 + 8 * (v >> 2) + (v & 3);
    valid |= (live && jcol <= i && i < L) ? 1u << v : 0u;
  }
  auto cell = [&](int v) -> double& { return Ms[(wi * 32 + 8 * (v >> 2) + 4 * hf + (v & 3)) * 65 + wj * 32 + l32]; };

  // ---- the map (compute_tile; softmax maps with their row log-sum-exp, as lse_tile_kernel and lse_reduce_kernel take it) ----
  double m[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) m[v] = 0.0;
  f32x16_t acc = {0};
  for (int g = 0; g < n_h; ++g) {
    if constexpr (!logit) {
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    }
    for (int kc = 0; kc < nkc; ++kc) {
      short_stage<T>(kbuf, Kc, (size_t)d, L, kc);
      if (Qb) short_stage<T>(qbuf, Qb + (size_t)g * d, (size_t)D.Hq * d, L, kc);
      __syncthreads();
      if (live) TileDot<DT>::run(qbuf + I * 64 * 256, kbuf + J * 64 * 256, wi * 32, wj * 32, l32, hf, acc);
      __syncthreads();
    }
    if constexpr (!logit) {
#pragma unroll
      for (int v = 0; v < 16; ++v) cell(v) = ((valid >> v) & 1u) ? (double)acc[v] * scale : -INFINITY;
      __syncthreads();
      double z[16], mx = -INFINITY;
#pragma unroll
      for (int c = 0; c < 16; ++c) { z[c] = Ms[li * 65 + part * 16 + c]; mx = fmax(mx, z[c]); }
      S.a4[grp][part][li] = mx;
      __syncthreads();
      mx = fmax(fmax(S.a4[grp][0][li], S.a4[grp][1][li]), fmax(S.a4[grp][2][li], S.a4[grp][3][li]));
      double sm = 0.0;
      if (mx > -INFINITY) {
#pragma unroll
        for (int c = 0; c < 16; ++c) sm += (double)exp2_f32(z[c] - mx);
      }
      S.b4[grp][part][li] = sm;
      __syncthreads();
      if (tid < SEG_SHORT) {
        const int g0 = tid < 64 ? 0 : 1, g1 = tid < 64 ? 0 : 2;
        double mt[2], st[2], mr = -INFINITY, sr = 0.0;
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const int gg = e ? g1 : g0;
          mt[e] = fmax(fmax(S.a4[gg][0][lane], S.a4[gg][1][lane]), fmax(S.a4[gg][2][lane], S.a4[gg][3][lane]));
          st[e] = ((S.b4[gg][0][lane] + S.b4[gg][1][lane]) + S.b4[gg][2][lane]) + S.b4[gg][3][lane];
        }
        mr = tid < 64 ? mt[0] : fmax(mt[0], mt[1]);
        if (mt[0] > -INFINITY) sr += st[0] * exp(mt[0] - mr);
        if (tid >= 64 && mt[1] > -INFINITY) sr += st[1] * exp(mt[1] - mr);
        S.lse[tid] = tid < L ? mr + log(sr) : 0.0;
      }
      __syncthreads();
#pragma unroll
      for (int v = 0; v < 16; ++v) m[v] += (double)exp2_f32((double)acc[v] * scale - S.lse[min(i0 + 8 * (v >> 2) + (v & 3), L - 1)]);
    }
  }
  if constexpr (logit) {
#pragma unroll
    for (int v = 0; v < 16; ++v) m[v] = (double)acc[v] * scale;
  }
  auto store_map = [&]() {
#pragma unroll
    for (int v = 0; v < 16; ++v) cell(v) = ((valid >> v) & 1u) ? m[v] : 0.0;
  };
  store_map();
  // Eq. 5's theta per head, times the heads summed; a percentile of the map is already per summed cell
  double th = (double)D.theta * (double)n_h;
  if (a.quant_cells) {
    th = short_quantile(a, m, valid, S);
    if (tid == 0) qstore(a.sc.qstate + (size_t)p * QUANT_STATE_WORDS + 2, (unsigned long long)__double_as_longlong(th));
  }
  if (tid < 8) { S.cutbit[tid] = 0u; S.mask[tid] = 0u; }
  __syncthreads();

  // ---- the cumulative sums and the anti-diagonals (seg_tile_scan_kernel) ----
  {
    double v[16], s = 0.0;
#pragma unroll
    for (int c = 0; c < 16; ++c) { v[c] = Ms[li * 65 + part * 16 + c]; s += v[c]; }
    S.a4[grp][part][li] = s;
    __syncthreads();
    // row carry of tile (1, 0): the row's sum over tile (1, 1)
    double run = (grp == 1 && live) ? ((S.a4[2][0][li] + S.a4[2][1][li]) + S.a4[2][2][li]) + S.a4[2][3][li] : 0.0;
    for (int q2 = 3; q2 > part; --q2) run += S.a4[grp][q2][li];
#pragma unroll
    for (int c = 15; c >= 0; --c) { run += v[c]; Ms[li * 65 + part * 16 + c] = run; }
  }
  __syncthreads();
  {
    double w[16], s = 0.0;
#pragma unroll
    for (int r = 0; r < 16; ++r) { w[r] = Ms[(part * 16 + r) * 65 + li]; s += w[r]; }
    S.b4[grp][part][li] = s;
    __syncthreads();
    // column carry of tile (1, 0): the column's suffix sums over the rows of tile (0, 0)
    double run = grp == 1 ? ((S.b4[0][0][li] + S.b4[0][1][li]) + S.b4[0][2][li]) + S.b4[0][3][li] : 0.0;
    for (int q2 = 0; q2 < part; ++q2) run += S.b4[grp][q2][li];
    const int x = J * 64 + li, n0 = I * 64 + part * 16 - x;
    double nd = (double)n0, tri = (double)(n0 * (n0 + 1) / 2);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rl = part * 16 + r, y = I * 64 + rl;
      run += w[r];
      nd += 1.0;
      tri += nd;
      Ms[rl * 65 + li] = (live && x <= y && y < L) ? run - th * tri : -INFINITY;      // Eq. 5
    }
  }
  __syncthreads();
  {
    double v[16], bestA = -INFINITY, bestB = -INFINITY;
    int xA = -1, xB = -1;
#pragma unroll
    for (int j = 0; j < 16; ++j) { const int xl = 16 * part + j; v[j] = Ms[((li - xl) & 63) * 65 + xl]; }
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int xl = 16 * part + j;
      const bool first = xl <= li, ok = whole || v[j] > -INFINITY;
      const bool upA = first && ok && v[j] >= bestA, upB = !first && ok && v[j] >= bestB;
      bestA = upA ? v[j] : bestA; xA = upA ? xl : xA;
      bestB = upB ? v[j] : bestB; xB = upB ? xl : xB;
    }
    double* hb = Ms;                                       // the tile is consumed: [2][4][64] partial maxima, then their columns
    int* hx = reinterpret_cast<int*>(hb + 512);
    __syncthreads();
    hb[part * 64 + li] = bestA; hb[256 + part * 64 + li] = bestB;
    hx[part * 64 + li] = xA;    hx[256 + part * 64 + li] = xB;
    __syncthreads();
    if (t < 128) {
      const int o = (t >> 6) * 256 + li;
      double best = hb[o];
      int bx = hx[o];
#pragma unroll
      for (int k = 1; k < 4; ++k) {
        const double ob = hb[o + 64 * k];
        const int ox = hx[o + 64 * k];
        if (ox >= 0 && (bx < 0 || ob >= best)) { best = ob; bx = ox; }
      }
      S.pscore[grp][t] = best;
      S.px[grp][t] = (int8_t)bx;
    }
  }
  __syncthreads();

  // ---- merge, greedy NMS (seg_select_kernel) by one wavefront, four anti-diagonals per lane: no barriers ----
  if (wave == 0) {
    uint64_t key[4];
    uint32_t xy[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int s = 4 * lane + r, b = s >> 6;
      double best = -INFINITY;
      int bx = -1;
#pragma unroll
      for (int w = 0; w < 2; ++w) {                        // tile bb lies on block anti-diagonal bb
        const int bb = b - w, bc = min(max(bb, 0), 2), sloc = s - 64 * bc;
        const int xl = S.px[bc][sloc & 127], x = (bc > 1 ? 64 : 0) + xl;
        const double v = S.pscore[bc][sloc & 127];
        if (bb == bc && (bc == 0 || L > 64) && xl >= 0 && (v > best || (v == best && x > bx))) { best = v; bx = x; }
      }
      const bool is_cand = s < 2 * L - 1 && bx >= 0 && best > 0.0;
      key[r] = is_cand ? ~(uint64_t)__double_as_longlong(best) : ~0ull;
      xy[r] = is_cand ? (((uint32_t)bx << 16) | (uint32_t)(s - bx)) : 0xFFFFFFFFu;
    }
    int nkept = 0;
    for (;;) {
      uint64_t b1 = key[0];
      uint32_t b2 = xy[0];
#pragma unroll
      for (int r = 1; r < 4; ++r)
        if (key_less(key[r], xy[r], b1, b2)) { b1 = key[r]; b2 = xy[r]; }
      if (__ballot(b1 != ~0ull) == 0ull) break;            // nothing alive
      uint32_t top = (uint32_t)(b1 >> 32);
      const uint32_t mine = top;
      top = min(top, lane_xor_c<1>(top)); top = min(top, lane_xor_c<2>(top)); top = min(top, lane_xor_c<4>(top));
      top = min(top, lane_xor_c<8>(top)); top = min(top, lane_xor_c<16>(top)); top = min(top, lane_xor_c<32>(top));
      const uint64_t tie = __ballot(mine == top);
      if (__popcll(tie) == 1) {
        b2 = (uint32_t)__builtin_amdgcn_readlane((int)b2, __ffsll((long long)tie) - 1);
      } else {
        auto step = [&](auto mc) {
          constexpr int M = decltype(mc)::value;
          const uint64_t o1 = ((uint64_t)lane_xor_c<M>((uint32_t)(b1 >> 32)) << 32) | lane_xor_c<M>((uint32_t)b1);
          const uint32_t o2 = lane_xor_c<M>(b2);
          if (key_less(o1, o2, b1, b2)) { b1 = o1; b2 = o2; }
        };
        step(std::integral_constant<int, 1>{}); step(std::integral_constant<int, 2>{}); step(std::integral_constant<int, 4>{});
        step(std::integral_constant<int, 8>{}); step(std::integral_constant<int, 16>{}); step(std::integral_constant<int, 32>{});
      }
      const int kx = (int)(b2 >> 16), ky = (int)(b2 & 0xFFFFu);
      if (lane == 0) {
        atomicOr(&S.cutbit[kx >> 5], 1u << (kx & 31));
        atomicOr(&S.cutbit[(ky + 1) >> 5], 1u << ((ky + 1) & 31));
      }
      ++nkept;
      if (D.max_keep > 0 && nkept >= D.max_keep) break;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int x = (int)(xy[r] >> 16), y = (int)(xy[r] & 0xFFFFu);
        const int inter = min(y, ky) - max(x, kx) + 1;
        const int uni = (y - x + 1) + (ky - kx + 1) - inter;
        const bool kill = (xy[r] == b2) | ((inter > 0) & ((float)inter > __fmul_rn(D.phi, (float)uni)));
        key[r] = kill ? ~0ull : key[r];
      }
    }
  }
  __syncthreads();
  // ---- cuts: 0, L, both ends of every kept interval, every unit edge; the span table ----
  for (int i = tid; i <= L; i += SHORT_NT)
    if (i == 0 || i == L || (D.unit > 0 && (c0 + i) % D.unit == 0)) atomicOr(&S.cutbit[i >> 5], 1u << (i & 31));
  __syncthreads();
  auto cuts_before = [&](int i) {                          // cuts at positions < i
    int c = 0;
#pragma unroll
    for (int w = 0; w < (SEG_SHORT >> 5) + 1; ++w) {
      const int bits = min(max(i - 32 * w, 0), 32);
      c += __popc(bits == 32 ? S.cutbit[w] : S.cutbit[w] & ((1u << bits) - 1u));
    }
    return c;
  };
  const int nsp = cuts_before(L);                          // (a cut stands at L)
  if (tid <= L && ((S.cutbit[tid >> 5] >> (tid & 31)) & 1u)) S.cut[cuts_before(tid)] = tid;
  if (tid < SEG_SHORT) S.tokspan[tid] = (int8_t)(cuts_before(tid + 1) - 1);      // (past the chunk: anything)
  __syncthreads();
  const bool fits = base + nsp <= D.max_spans;
  if (fits && tid < nsp) {
    a.st.span_start[(size_t)slot * D.max_spans + base + tid] = c0 + S.cut[tid];
    a.st.span_len[(size_t)slot * D.max_spans + base + tid] = S.cut[tid + 1] - S.cut[tid];
  }
  if (tid == 0) {
    if (!fits) atomicCAS(&a.st.err[0], 0, LTRI_ECAPACITY);
    meta[META_N_SPANS] = fits ? base + nsp : base;         // (see append_spans)
    meta[META_CHUNK_FIRST] = base;
    meta[META_CHUNK_NSP] = fits ? nsp : 0;
    meta[META_CHUNK_START] = c0;
    meta[META_CHUNK_LEN] = L;
  }

  // ---- dynamic index vectors (the dyn_* kernels): the map again, votes and row sums, counts, index tokens ----
  const bool dynamic = D.rep_mode == LTRI_REP_DYNAMIC;
  if constexpr (!logit) {
    if (dynamic) {
      store_map();                                         // (pscore and px are not in the tiles)
      __syncthreads();
      {
        const int mine = S.tokspan[I * 64 + li];
        double s = 0.0, sin = 0.0;
#pragma unroll
        for (int c = 0; c < 16; ++c) {
          const double v = Ms[li * 65 + part * 16 + c];
          s += v;
          sin += S.tokspan[J * 64 + part * 16 + c] == mine ? v : 0.0;
        }
        S.a4[grp][part][li] = s;
        S.b4[grp][part][li] = sin;
      }
      double cs = 0.0;
#pragma unroll
      for (int r = 0; r < 16; ++r) cs += Ms[(part * 16 + r) * 65 + li];
      __syncthreads();
      auto sum4 = [&](const double (&q)[3][4][64], int gg, int l) { return ((q[gg][0][l] + q[gg][1][l]) + q[gg][2][l]) + q[gg][3][l]; };
      if (tid < SEG_SHORT) {
        S.dyn[1][tid] = tid < 64 ? sum4(S.b4, 0, lane) : sum4(S.b4, 1, lane) + sum4(S.b4, 2, lane);
        S.dyn[2][tid] = tid < 64 ? sum4(S.a4, 0, lane) : sum4(S.a4, 1, lane) + sum4(S.a4, 2, lane);
      }
      __syncthreads();
      S.a4[grp][part][li] = cs;
      __syncthreads();
      if (tid < SEG_SHORT) {
        const double v = tid < 64 ? sum4(S.a4, 0, lane) + (L > 64 ? sum4(S.a4, 1, lane) : 0.0) : sum4(S.a4, 2, lane);
        S.dyn[0][tid] = v;
        S.vkey[tid] = vote_key(v);
      }
      __syncthreads();
      for (int q = wave; q < nsp; q += SHORT_NT / 64) {    // Eq. 7, one wavefront per span
        const int s0 = S.cut[q], len = S.cut[q + 1] - s0;
        double v0 = 0.0, v1 = 0.0, v2 = 0.0;
        for (int u = lane; u < len; u += 64) { v0 += S.dyn[0][s0 + u]; v1 += S.dyn[1][s0 + u]; v2 += S.dyn[2][s0 + u]; }
        v0 = wave_sum_f64(v0); v1 = wave_sum_f64(v1); v2 = wave_sum_f64(v2);
        const int n = index_count(D, len, v0, v1, v2);
        if (lane == 0) S.cnt[q] = n;
      }
      __syncthreads();
      for (int q = wave; q < nsp; q += SHORT_NT / 64) {
        const int s0 = S.cut[q], len = S.cut[q + 1] - s0;
        int count = S.cnt[q];
        if (D.index_block_max > 0) {                       // a budget per memory block, shared over its spans
          const int blk = (c0 + s0) / D.unit;
          uint64_t in[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int mq = lane + 64 * e;
            in[e] = __ballot(mq < nsp && (c0 + S.cut[min(mq, nsp - 1)]) / D.unit == blk);
          }
          const int mlo = in[0] ? __ffsll((long long)in[0]) - 1 : 63 + __ffsll((long long)in[1]);
          count = block_share(S.cnt + mlo, __popcll(in[0]) + __popcll(in[1]), q - mlo, D.index_block_max);
        }
        for (int u = lane; u < len; u += 64) {
          const uint64_t ku = S.vkey[s0 + u];
          int rank = 0;
#pragma unroll 4
          for (int w = 0; w < len; ++w) {
            const uint64_t kw = S.vkey[s0 + w];
            rank += (kw < ku || (kw == ku && w < u)) ? 1 : 0;
          }
          if (rank < count) atomicOr(&S.mask[(s0 + u) >> 5], 1u << ((s0 + u) & 31));
        }
      }
      __syncthreads();
      if (tid < IDX_MASK_WORDS) a.st.idx_mask[(size_t)slot * IDX_MASK_WORDS + tid] = tid < 8 && fits ? S.mask[tid] : 0u;
    }
  }
  if (!fits || (logit && dynamic)) return;                 // (LOGIT maps with index vectors: the dyn_* kernels follow)
  // ---- stored vectors: means of the spans' keys, or sums over their index tokens ----
  __syncthreads();
  static_assert(sizeof(S.Ms) >= short_sums_lds(128), "place of the key sums");
  T* rep = reinterpret_cast<T*>(a.st.krep) + ((size_t)slot * D.max_spans + base) * d;
  short_span_sums<DT, SHORT_NT / 64>(Kc, (size_t)d, 1, L, d, nsp, [&](int q) { return S.cut[q]; }, dynamic ? S.mask : nullptr,
                                     reinterpret_cast<unsigned char*>(S.Ms), [&](int q, int c, double v, int n) {
                                       rep[(size_t)q * d + c] = Elt<DT>::from_f64(dynamic ? v : v / (double)n);
                                     });
}

}  // namespace ltri
