// gfx950 kernels of the target verification step, one launch per
// operation (prefill chunks and passes the persistent step kernel does not
// take).  The per-tile work lives in tiles.h and is shared with step.hip.
//
// Every row's arithmetic is independent of how many rows share the pass:
// GEMM k-splits depend only on the matrix shape, attention splits the key
// axis at fixed 32-key boundaries and merges them in order, and arg-max is
// exact.  A verification call over root + k candidates therefore computes,
// bit for bit, the logits and cache rows of k + 1 sequential target-only
// steps (the pathwise-equivalence requirement of Appendix C.4, met here
// numerically and not only up to masks).
#include "attn.h"

namespace as2d {

// ---------------------------------------------------------------------------
// Weight packing: row-major [N][K] -> 1 KiB tiles in the order one wave
// streams them.  Tile pair tp holds 32 output columns as two 16-column
// tiles j; per k-step kt the pair's two tiles are adjacent:
//   index ((tp * KT + kt) * 2 + j) * 64 + lane
// and lane l holds matrix row n(tp, j, l % 16) at elements
// [kt * KE + (l / 16) * PER16, + PER16) (the MFMA B operand of column l % 16).
// The column order n(tp, j, c) is the PackMap of kernels.h: gate/up puts
// gate unit u and up unit u in the same pair, RoPE pairs put dimensions i
// and i + d/2 of a head in the same pair, so the fused epilogues find both
// operands in one workgroup.

__device__ __forceinline__ int packed_row(int map, int arg, int tp, int j, int c) {
  if (map == PACK_GATE_UP) return j * arg + 16 * tp + c;
  if (map == PACK_ROPE_PAIRS) {
    const int d = arg, ppd = d / kPairCols;
    const int head = tp / ppd, q = tp % ppd;
    return head * d + j * (d / 2) + 16 * q + c;
  }
  return tp * kPairCols + 16 * j + c;
}

template <bool BF>
__global__ void pack_kernel(const typename ET<BF>::T* __restrict__ src, uint4* __restrict__ dst,
                            int N, int K, int map, int arg) {
  constexpr int PER16 = ET<BF>::PER16;
  constexpr int KE = 4 * PER16;
  const int KT = K / KE;
  const long long total = (long long)(N / 16) * KT * 64;  // 64 lanes x 16 B per 16-row tile
  for (long long idx = blockIdx.x * (long long)blockDim.x + threadIdx.x; idx < total;
       idx += (long long)gridDim.x * blockDim.x) {
    const int lane = (int)(idx & 63);
    const long long t = idx >> 6;
    const int j = (int)(t & 1);
    const long long u = t >> 1;
    const int kt = (int)(u % KT);
    const int tp = (int)(u / KT);
    const int row = packed_row(map, arg, tp, j, lane & 15);
    const int k0 = kt * KE + (lane >> 4) * PER16;
    dst[idx] = *reinterpret_cast<const uint4*>(src + (size_t)row * K + k0);
  }
}

hipError_t launch_pack(bool bf16, const void* src, uint4* dst, int N, int K, int map, int arg,
                       hipStream_t s) {
  const int threads = 256, blocks = 4096;
  if (N % kPairCols || (map == PACK_GATE_UP && N != 2 * arg) ||
      (map == PACK_ROPE_PAIRS && (arg % kPairCols || N % arg)))
    return hipErrorInvalidValue;
  if (bf16)
    pack_kernel<true><<<blocks, threads, 0, s>>>((const uint16_t*)src, dst, N, K, map, arg);
  else
    pack_kernel<false><<<blocks, threads, 0, s>>>((const float*)src, dst, N, K, map, arg);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Embedding gather (embed_row), one workgroup per row.  With `put` set, the
// descriptors are read from the host's pinned memory and written to the
// device arrays the later kernels of the pass read: a verification pass then
// needs no copy before its first kernel (two 16-byte reads per row, about
// 2 us, against about 10 us for two copies in the stream).

template <bool BF>
__global__ __launch_bounds__(256) void embed_kernel(const RowDesc* rows, const PassDesc put,
                                                    const typename ET<BF>::T* __restrict__ embed,
                                                    const typename ET<BF>::T* __restrict__ audio,
                                                    int H, const float* __restrict__ gain,
                                                    float* __restrict__ x, float* __restrict__ sumsq,
                                                    void* __restrict__ xg, long long xg_plane) {
  const int m = blockIdx.x;
  RowDesc rd;
  if (put.rows) {
    const u32x4* src = reinterpret_cast<const u32x4*>(rows + m);
    const u32x4 a = __builtin_nontemporal_load(src), b = __builtin_nontemporal_load(src + 1);
    rd = RowDesc{(int32_t)a.x, (int32_t)a.y, (int32_t)a.z, (int32_t)a.w, (int32_t)b.x, {0, 0, 0}};
    if (threadIdx.x == 0) put.rows[m] = rd;
    if (m == 0)
      for (int i = threadIdx.x; i < put.n_att + put.n_fin; i += 256) {
        const int r = i < put.n_att ? i : put.fin0 + i - put.n_att;
        reinterpret_cast<u32x4*>(put.reqs)[r] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(put.reqs_in) + r);
      }
  } else {
    rd = load_invariant(rows + m);
  }
  embed_row<BF, false>(rd, m, embed, audio, H, gain, x, sumsq, xg, xg_plane);
}

hipError_t launch_embed(bool bf16, const RowDesc* rows, const PassDesc& put, int M, const void* embed, const void* audio,
                        int H, const float* gain, float* x, float* sumsq, void* xg, long long xg_plane,
                        hipStream_t s) {
  if (H > 256 * 8 * 4 || H % 128) return hipErrorInvalidValue;
  if (bf16)
    embed_kernel<true><<<M, 256, 0, s>>>(rows, put, (const uint16_t*)embed, (const uint16_t*)audio, H, gain,
                                           x, sumsq, xg, xg_plane);
  else
    embed_kernel<false><<<M, 256, 0, s>>>(rows, put, (const float*)embed, (const float*)audio, H, gain, x,
                                            sumsq, xg, xg_plane);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Weight-streaming GEMM  Y[M][N] = A[M][K] * W[N][K]^T  for small M
// (tiles.h).  Up to 32 rows (direct path): one workgroup per (np tile
// pairs, k-split), its four waves streaming the ns slices of the split,
// each k-step's 1 KiB weight tiles (fully coalesced, non-temporal) and the
// activation fragments issued 2 to 4 k-steps ahead of their use.  The
// streaming must reach every compute unit (each keeps a bounded amount of
// memory traffic in flight), so narrow matrices are split along k.  More rows:
// the wide path (wide.h) for bf16 models; the staged path for float32 models,
// one workgroup per (4 or 8 tile pairs, k-split, row group), activations
// staged through LDS.  All paths add every element in the same
// order, so a row's result does not depend on M.  With KS > 1 each split writes a
// float32 partial and the last workgroup of the tile (device-scope
// counter) sums the partials in split order and runs the fused epilogue.

template <bool BF, int MT, int NP, int NW, int AM, int EPI, bool SPLIT>
__global__ __launch_bounds__(NW * 64, MT == 1 && NP == 1 ? 5 : 4) void gemm_direct_kernel(const GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float s_scale[kMaxRows];
  __shared__ int s_flag;
  const int tile = blockIdx.x / p.KS, split = blockIdx.x - tile * p.KS;
  gemm_tile_direct<BF, MT, NP, NW, false, AM, EPI, false, SPLIT>(p, p.M, tile, split, smem, s_scale, &s_flag,
                                                                 [] {});
}

template <bool BF, int MT, int NP, int NW, int AM, int EPI>
static void launch_direct(const GemmArgs& a, hipStream_t s) {
  const dim3 grid((a.N / kPairCols / NP) * a.KS), block(NW * 64);
  const int lds = gemm_direct_lds_bytes<MT, NP>(a.ns);
  if (a.KS > 1) gemm_direct_kernel<BF, MT, NP, NW, AM, EPI, true><<<grid, block, lds, s>>>(a);
  else gemm_direct_kernel<BF, MT, NP, NW, AM, EPI, false><<<grid, block, lds, s>>>(a);
}

// Balanced direct path: one workgroup per compute unit (the dynamic LDS
// is at least kRangeMinLds, so two never share one), each streaming an
// equal share of the (pair, split) units.  SL > 0: the variant with the
// activation slice in registers (KS = 1, KT = 4 SL; range_ra_slice).

template <bool BF, int MT, int SL, int AM, int EPI>
__global__ __launch_bounds__(256, 1) void gemm_range_kernel(const GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float s_scale[kMaxRows];
  __shared__ int s_flags[kMaxUnits];
  if constexpr (SL == 0) {
    gemm_range_direct<BF, MT, kRangePrefetch, AM, EPI, false>(p, p.M, smem, s_scale, s_flags, [] {});
  } else {
    constexpr int P = SL % kRangePrefetch == 0 ? kRangePrefetch : SL;
    gemm_range_direct_ra<BF, MT, P, SL, AM, EPI, false>(p, p.M, smem, s_scale, s_flags, [] {});
  }
}

bool range_plan_ok(const GemmArgs& a) {
  const int U = (a.N / kPairCols) * a.KS;
  const int last = a.KT - (a.KS - 1) * a.ktps;   // k-steps of the last split
  return a.G >= 1 && a.G <= U && (U + a.G - 1) / a.G <= kMaxUnits && a.ktps >= kWaves && last >= kWaves &&
         a.KS <= kMaxSplits && a.ns == kWaves && a.MT >= 1 && a.MT <= kDirectMT;
}

template <bool BF, int AM, int EPI>
static hipError_t launch_range(const GemmArgs& a, hipStream_t s) {
  if (!range_plan_ok(a)) return hipErrorInvalidValue;
  const int U = (a.N / kPairCols) * a.KS;
  int lds = gemm_range_lds_bytes(a.MT, (U + a.G - 1) / a.G);
  if (lds < kRangeMinLds) lds = kRangeMinLds;
  const int sl = range_ra_slice<BF>(AM, EPI, a.MT, a.KS, a.KT);
  if constexpr (AM == A_NORM && (EPI == EPI_SWIGLU || EPI == EPI_ARGMAX)) {
    auto run = [&](auto c) {
      constexpr int SL = decltype(c)::value;
      if constexpr (BF)
        if (a.MT == 2) {
          gemm_range_kernel<BF, 2, SL, AM, EPI><<<a.G, 256, lds, s>>>(a);
          return;
        }
      gemm_range_kernel<BF, 1, SL, AM, EPI><<<a.G, 256, lds, s>>>(a);
    };
    if (sl == kRangeSL<BF>[0]) run(std::integral_constant<int, kRangeSL<BF>[0]>());
    else if (sl == kRangeSL<BF>[1]) run(std::integral_constant<int, kRangeSL<BF>[1]>());
    else if (sl == kRangeSL<BF>[2]) run(std::integral_constant<int, kRangeSL<BF>[2]>());
  }
  if (!sl) {
    if (a.MT == 1) gemm_range_kernel<BF, 1, 0, AM, EPI><<<a.G, 256, lds, s>>>(a);
    else gemm_range_kernel<BF, 2, 0, AM, EPI><<<a.G, 256, lds, s>>>(a);
  }
  return hipGetLastError();
}

// Most row tiles per row group when a staged GEMM would otherwise leave
// compute units idle.
constexpr int kStagedGroupMT = 3;

// Staged path: work item v = (pair group, split, row group), the row group
// fastest; RG row groups of MT row tiles each (RG = 1: all the pass's rows).
// With row groups, the RG blocks of one (pair group, split) run on one XCD
// at about the same time (xcd_contiguous), so its weight tiles come from
// memory once and from that XCD's L2 for the other row groups.
// Row groups (up to three row tiles) fit four workgroups per compute unit,
// or two with two pairs per wave (NPW = 2: a pair group of 8 pairs); more
// rows need the whole register file.
template <int MT, int AM, int EPI, int NPW = 1>
__global__ __launch_bounds__(256, NPW > 1 ? 2 : MT <= kStagedGroupMT ? 4 : 1) void gemm_staged_kernel(const GemmArgs p,
                                                                                                    const int RG) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float s_scale[kMaxRows];
  __shared__ int s_flag;
  const int v = RG > 1 ? xcd_contiguous(blockIdx.x, gridDim.x) : (int)blockIdx.x;
  const int rg = v % RG, t = v / RG;
  const int group = t / p.KS, split = t - group * p.KS;
  gemm_tile_staged<MT, AM, EPI, (MT <= kStagedGroupMT), NPW>(p, p.M, group, split, smem, s_scale, &s_flag, rg * MT,
                                                             group * RG + rg);
}

template <int AM, int EPI>
static hipError_t launch_staged(const GemmArgs& a, hipStream_t s) {
  const int pairs = a.N / kPairCols;
  if (pairs % kPairsS) return hipErrorInvalidValue;
  const int base = (pairs / kPairsS) * a.KS;
  // matrices with fewer than two workgroups per compute unit: row groups of
  // g <= kStagedGroupMT tiles, the largest g whose grid reaches rg_grid
  // workgroups (else one tile), so that each compute unit keeps several
  // workgroups' loads in flight.  Each group reads the weights again (from
  // its XCD's L2: xcd_contiguous).  The counters (group * RG + rg) cover
  // (pairs / kPairsS) * kMaxMTiles tiles.
  if (base < 512 && a.MT > kStagedGroupMT) {
    int g = kStagedGroupMT;
    while (g > 1 && base * ((a.MT + g - 1) / g) < a.rg_grid) --g;
    const int RG = (a.MT + g - 1) / g;
    if (RG > kMaxMTiles) return hipErrorInvalidValue;
    if (g == 3 && pairs % (2 * kPairsS) == 0) {
      // two pairs per wave: each staged activation fragment feeds twice the
      // weights, half the workgroups
      gemm_staged_kernel<3, AM, EPI, 2>
          <<<base / 2 * RG, 256, gemm_staged_lds_bytes<3, 2>(), s>>>(a, RG);
    } else if (g == 3) gemm_staged_kernel<3, AM, EPI><<<base * RG, 256, gemm_staged_lds_bytes<3>(), s>>>(a, RG);
    else if (g == 2) gemm_staged_kernel<2, AM, EPI><<<base * RG, 256, gemm_staged_lds_bytes<2>(), s>>>(a, RG);
    else gemm_staged_kernel<1, AM, EPI><<<base * RG, 256, gemm_staged_lds_bytes<1>(), s>>>(a, RG);
    return hipGetLastError();
  }
  const dim3 grid(base), block(256);
  switch (a.MT) {
#define AS2D_MT(mt) \
  case mt: gemm_staged_kernel<mt, AM, EPI><<<grid, block, gemm_staged_lds_bytes<mt>(), s>>>(a, 1); break;
    AS2D_MT(3) AS2D_MT(4) AS2D_MT(5) AS2D_MT(6) AS2D_MT(7) AS2D_MT(8) AS2D_MT(9)
#undef AS2D_MT
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <bool BF, int AM, int EPI>
static hipError_t gemm_dispatch(const GemmArgs& a, hipStream_t s) {
  const int pairs = a.N / kPairCols;
  if (a.MT <= kDirectMT && a.G > 0) return launch_range<BF, AM, EPI>(a, s);
  if (a.MT <= kDirectMT) {
    if ((a.np != 1 && (a.np != 2 || pairs % 2)) || a.ns < kWaves || a.ns > kMaxSlices || a.ns % kWaves)
      return hipErrorInvalidValue;
    if (a.MT == 1) {
      if (a.np == 1) launch_direct<BF, 1, 1, kWaves, AM, EPI>(a, s);
      else launch_direct<BF, 1, 2, kWaves, AM, EPI>(a, s);
    } else {
      if (a.np == 1) launch_direct<BF, 2, 1, kWaves, AM, EPI>(a, s);
      else launch_direct<BF, 2, 2, kWaves, AM, EPI>(a, s);
    }
    return hipGetLastError();
  }
  if constexpr (BF) {
    return launch_wide(AM, EPI, a, s);
  } else {
    return launch_staged<AM, EPI>(a, s);
  }
}

hipError_t launch_gemm(bool bf16, int amode, int epi, const GemmArgs& a, hipStream_t s) {
#define AS2D_G(bf, am, ep) \
  if (bf16 == bf && amode == am && epi == ep) return gemm_dispatch<bf, am, ep>(a, s);
  AS2D_G(true, A_NORM, EPI_QKV) AS2D_G(true, A_PLAIN, EPI_RESID) AS2D_G(true, A_NORM, EPI_SWIGLU)
  AS2D_G(true, A_NORM, EPI_ARGMAX) AS2D_G(true, A_PLAIN, EPI_DOWN)
  AS2D_G(false, A_NORM, EPI_QKV) AS2D_G(false, A_PLAIN, EPI_RESID) AS2D_G(false, A_NORM, EPI_SWIGLU)
  AS2D_G(false, A_NORM, EPI_ARGMAX) AS2D_G(false, A_PLAIN, EPI_DOWN)
#undef AS2D_G
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Block-causal grouped-query attention (attn.h).
//
// Verification passes.  attn_group_kernel: work items (request, run of
// 128-key spans, KV head, row block), a row block being up to 16 RT rows of
// the query heads that share the KV head (their rows of the request, head by
// head), so each span's keys and values are read once per block; the blocks
// of one (run, KV head) are adjacent and dealt to one XCD.  A fixed grid of
// workgroups takes the items in turn, so the grid does not depend on the
// cache length; each item stores its rows' span states.  The states of a
// row are folded in order, for caches of up to 16 spans by the last item of
// the block to finish (one quarter wave per row and head), else by
// attn_merge_kernel (one wave per row and head).
//
// Prefill passes (one request) of float32 models: one workgroup per (query
// head, 16 rows) walks the spans in ascending order and merges them as it
// goes, with the same arithmetic, so no partials go through memory
// (attn_prefill.hip does so for bf16 models).

// The items of a launch with blocks of RT row tiles.  LOWREG (RT = 1): a
// workgroup within half the register file (two per compute unit), one span
// buffer, the values fetched once the span's scores are formed.
template <bool BF, int D, int RT, bool LOWREG = false>
__device__ __forceinline__ void attn_group_items(const AttnArgs& p, int n_reqs, unsigned char* smem) {
  static_assert(!LOWREG || RT == 1, "one row tile");
  constexpr int KS = D / AttnFmt<BF>::KE;
  constexpr int BR = 16 * RT;   // rows of a block
  const int G = gridDim.x;
  const int hpg = p.n_q / p.n_kv;   // query heads per KV head
  auto blocks = [&](const ReqDesc& rq) { return (hpg * rq.W + BR - 1) / BR; };
  // an item covers a run of up to R consecutive spans: the least R whose
  // items fit the grid (one span each while they do; long caches take
  // several per workgroup)
  const auto items = [&](const ReqDesc& rq, int R) {
    const int ns = (rq.L0 + rq.W - 1) / kAttnSpanKeys + 1;
    return p.n_kv * blocks(rq) * ((ns + R - 1) / R);
  };
  int R, total;
  attn_run_length(p.reqs, n_reqs, G, items, [&](const ReqDesc& rq) { return p.n_kv * blocks(rq); }, R, total);
  for (int t = xcd_contiguous(blockIdx.x, G); t < total; t += G) {
    // item t: request r, then run j, KV head g, row block b
    int u = t;
    const int r = n_reqs == 1 ? 0 : find_request(p.reqs, n_reqs, u, [&](const ReqDesc& q) { return items(q, R); });
    const ReqDesc rq = load_invariant(p.reqs + r);
    const int ns = (rq.L0 + rq.W - 1) / kAttnSpanKeys + 1, nb = blocks(rq);
    const int j = u / (p.n_kv * nb);
    const int v = u - j * p.n_kv * nb;
    const int g = v / nb, b = v - g * nb;
    const AttnRows rows{g * hpg, rq.W, hpg * rq.W, b * BR};
    const int sp0 = j * R, sp1 = min(sp0 + R, ns);
    // the first span's keys and values, then the queries, all in flight at once
    AttnRaw<BF, D> ka;
    if constexpr (LOWREG) attn_fetch_k<BF, D>(p, rq, g, sp0, ka);
    else attn_fetch<BF, D>(p, rq, g, sp0, ka);
    Op2 q[RT][KS];
    attn_load_q<BF, D, RT>(p, rq, rows, q);
    auto run = [&](int sp, const AttnRaw<BF, D>& raw) {
      AttnState<RT, D / 64> state;
      attn_span_state<BF, D, RT>(p, rq, rows, sp, q, raw, smem, state);
      attn_store_span<D, RT>(p, rq, rows, sp, state);
      lds_sync();   // the LDS is written again next (a prefetch stays in flight)
    };
    if constexpr (LOWREG) {
      // once a span's scores are formed its keys' registers take the next
      // span's keys, requested right after the span's values
      for (int sp = sp0; sp < sp1; ++sp) {
        AttnState<1, D / 64> state;
        attn_span_chunks<BF, D, 1>(p, rq, rows, sp, q, ka, smem, [&] {
          attn_fetch_v<BF, D>(p, rq, g, sp, ka);
          if (sp + 1 < sp1) attn_fetch_k<BF, D>(p, rq, g, sp + 1, ka);
        });
        attn_merge_chunks<BF, D, 1>(smem, state);
        attn_store_span<D, 1>(p, rq, rows, sp, state);
        lds_sync();   // the LDS is written again next
      }
    } else if constexpr (RT == 1) {
      // two chunk buffers taken in turn, a buffer refilled right after its
      // span's state is stored: the wait for a buffer's data (inserted by
      // the compiler) then leaves the later span's stores in flight
      AttnRaw<BF, D> kb;
      if (sp0 + 1 < sp1) attn_fetch<BF, D>(p, rq, g, sp0 + 1, kb);
      for (int sp = sp0; sp < sp1; sp += 2) {
        run(sp, ka);
        if (sp + 2 < sp1) attn_fetch<BF, D>(p, rq, g, sp + 2, ka);
        if (sp + 1 >= sp1) break;
        run(sp + 1, kb);
        if (sp + 3 < sp1) attn_fetch<BF, D>(p, rq, g, sp + 3, kb);
      }
    } else {   // two row tiles: one buffer (two would not fit the registers)
      for (int sp = sp0; sp < sp1; ++sp) {
        if (sp > sp0) attn_fetch<BF, D>(p, rq, g, sp, ka);
        run(sp, ka);
      }
    }
    if (p.merge_last) {
      // the last item of the block to finish (agent-scope counter) merges
      // its rows, one quarter wave per (row, head)
      __shared__ int s_last;
      wait_vmem();
      __syncthreads();   // every wave's span stores are performed
      const int done = sp1 - sp0;
      int* cnt = p.attn_cnt + (r * p.n_kv + g) * 2 * hpg + b;
      if (threadIdx.x == 0) s_last = counter_add(cnt, done) == ns - done;
      __syncthreads();
      if (s_last) {
        if (threadIdx.x == 0) st<true>(cnt, 0);   // ready for the next launch
        const int nv = min(BR, rows.n - rows.u0);
        for (int k = threadIdx.x >> 4; k < nv; k += 16) attn_merge_row<BF, D, false>(p, rq, rows.row(k), rows.head(k));
      }
      __syncthreads();   // s_last is reused by the next item
    }
  }
}

// Blocks of one row tile while each (span, KV head, block) can have a
// workgroup of its own, or while two-tile blocks would not cut the items by
// a third (requests of few rows: the second tile would be padding); else
// of two (half the reads of the keys and values per row, fewer runs of
// spans per workgroup).  An attn_rt of 1 or 2 fixes it.
template <bool BF, int D>
__global__ __launch_bounds__(256) void attn_group_kernel(const AttnArgs p, int n_reqs) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  int rt = p.attn_rt;
  if (rt != 1 && rt != 2) {
    const int hpg = p.n_q / p.n_kv;
    // items with one-tile and two-tile blocks, one span each
    const auto items = [&](const ReqDesc& rq, int rows) {
      return p.n_kv * ((hpg * rq.W + rows - 1) / rows) * ((rq.L0 + rq.W - 1) / kAttnSpanKeys + 1);
    };
    const auto n_items = [&](int rows) {
      if (n_reqs == 1) return items(load_invariant(p.reqs), rows);
      return sum_requests(p.reqs, n_reqs, [&](const ReqDesc& rq) { return items(rq, rows); });
    };
    const int n1 = n_items(16), n2 = n_items(32);
    rt = n1 <= (int)gridDim.x || 2 * n1 < 3 * n2 ? 1 : 2;
  }
  if (rt == 1) attn_group_items<BF, D, 1>(p, n_reqs, smem);
  else attn_group_items<BF, D, 2>(p, n_reqs, smem);
}

// Slots whose one-tile items outnumber the compute units: one-tile blocks
// on two workgroups per compute unit, each overlapping the other's waits.
template <bool BF, int D>
__global__ __launch_bounds__(256, 2) void attn_group2_kernel(const AttnArgs p, int n_reqs) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  attn_group_items<BF, D, 1, true>(p, n_reqs, smem);
}

// One wave per (request row, query head), heads of a row adjacent.
template <bool BF, int D>
__global__ __launch_bounds__(64) void attn_merge_kernel(const AttnArgs p, int n_reqs) {
  int u = blockIdx.x, r = 0;
  if (n_reqs > 1) r = find_request(p.reqs, n_reqs, u, [&](const ReqDesc& q) { return q.W * p.n_q; });
  if (r < 0) return;
  const ReqDesc rq = load_invariant(p.reqs + r);
  if (u >= rq.W * p.n_q) return;
  const int i = u / p.n_q;
  attn_merge_wave<BF, D>(p, rq, i, u - i * p.n_q);
}

// Prefill attention of float32 models (bf16: attn_prefill.hip): one workgroup
// per (query head, 16-row tile) runs
// the tile's spans two at a time with eight waves, group 0 (waves 0-3) on
// spans 0, 2, 4, ..., group 1 on spans 1, 3, 5, ...,
// each group on its own LDS span buffer and with one chunk buffer in
// registers (a span's keys give way to the group's next span's keys once
// its scores are formed, its values to the next values once its products
// are), so that two waves share each SIMD.  The running state
// stays in group 0, which merges the spans in order: its own span, then
// group 1's state handed over through the LDS; the same arithmetic as one
// span at a time.  Group 1 runs the last span again when the count is odd
// (its state is not merged) so that both groups reach the same barriers.
template <int D> __host__ __device__ constexpr int attn_prefill_lds_bytes() {
  return 2 * attn_span_lds_bytes<false, D, 1>() + kWaves * (2 + D / 64) * 64 * 16;
}

template <int D>
__global__ __launch_bounds__(512) void attn_prefill_kernel(const AttnArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr bool BF = false;
  constexpr int KS = D / AttnFmt<BF>::KE;
  constexpr int DTW = D / 64;
  const int h = blockIdx.x, r0 = blockIdx.y * 16;
  const ReqDesc full = load_invariant(p.reqs);
  if (r0 >= full.W) return;
  const ReqDesc rq{full.row_start + r0, min(full.W - r0, 16), full.L0 + r0, full.slot};
  const int lane = threadIdx.x & 63, grp = threadIdx.x >> 8, wave = attn_wave();
  unsigned char* mine = smem + grp * attn_span_lds_bytes<BF, D, 1>();
  // group 1's span state for group 0: [wave][M, L, A tiles][lane]
  f4* X = reinterpret_cast<f4*>(smem + 2 * attn_span_lds_bytes<BF, D, 1>()) + wave * (2 + DTW) * 64 + lane;
  const AttnRows rows = attn_rows_of_head(h, rq.W);
  const int g = attn_kv_head(p, rows);
  const int ns = (rq.L0 + rq.W - 1) / kAttnSpanKeys + 1;
  const auto span_of = [&](int j) { return min(j + grp, ns - 1); };
  AttnRaw<BF, D> raw;
  attn_fetch<BF, D>(p, rq, g, span_of(0), raw);
  Op2 q[1][KS];
  attn_load_q<BF, D, 1>(p, rq, rows, q);
  AttnState<1, DTW> all;
  const auto take = [&](int sp) {
    return [&, sp](int, int i) { return rq.L0 + min(4 * (lane >> 4) + i, rq.W - 1) >= sp * kAttnSpanKeys; };
  };
  for (int j = 0; j < ns; j += 2) {
    const int sp = span_of(j);
    AttnState<1, DTW> st;
    attn_span_chunks<BF, D, 1>(p, rq, rows, sp, q, raw, mine, [&] {
      if (j + 2 < ns) attn_fetch_k<BF, D>(p, rq, g, span_of(j + 2), raw);
    });
    if (j + 2 < ns) attn_fetch_v<BF, D>(p, rq, g, span_of(j + 2), raw);
    attn_merge_chunks<BF, D, 1>(mine, st);
    if (grp) {
      X[0] = f4{st.M[0][0], st.M[0][1], st.M[0][2], st.M[0][3]};
      X[64] = f4{st.L[0][0], st.L[0][1], st.L[0][2], st.L[0][3]};
#pragma unroll
      for (int t = 0; t < DTW; ++t) X[(2 + t) * 64] = f4{st.A[0][t][0], st.A[0][t][1], st.A[0][t][2], st.A[0][t][3]};
    } else {
      attn_state_merge<1, DTW>(all, st.M, st.L, st.A, j == 0, take(j));
    }
    lds_sync();   // group 1's state is in the LDS; the span buffers are free
    if (!grp && j + 1 < ns) {
      const f4 m = X[0], l = X[64];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        st.M[0][i] = m[i];
        st.L[0][i] = l[i];
      }
#pragma unroll
      for (int t = 0; t < DTW; ++t) {
        const f4 a = X[(2 + t) * 64];
#pragma unroll
        for (int i = 0; i < 4; ++i) st.A[0][t][i] = a[i];
      }
      attn_state_merge<1, DTW>(all, st.M, st.L, st.A, false, take(j + 1));
    }
  }
  if (grp) return;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = 4 * (lane >> 4) + i;
    if (r < rq.W)
#pragma unroll
      for (int t = 0; t < DTW; ++t)
        store_act<BF, false>(p.out, p.out_plane,
                             frag_index<BF>(rq.row_start + r, h * D + 16 * (wave * DTW + t) + (lane & 15), p.n_q * D),
                             all.A[0][t][i] / all.L[0][i]);
  }
}

template <bool BF, int D>
static hipError_t attn_dispatch(const AttnArgs& a, int n_reqs, int max_blocks, bool prefill, hipStream_t s) {
  if (max_blocks > kMaxBlocks || n_reqs < 1) return hipErrorInvalidValue;
  if (prefill) {
    if (n_reqs != 1) return hipErrorInvalidValue;
    if constexpr (BF) return launch_attn_prefill(a, s);
    else attn_prefill_kernel<D><<<dim3(a.n_q, (a.M + 15) / 16), 512, attn_prefill_lds_bytes<D>(), s>>>(a);
    return hipGetLastError();
  }
  // items of one-tile blocks at the slot capacity, from the most rows a
  // request of the pass can have (so that one captured graph serves every
  // pass of M rows and n_reqs requests)
  const int hpg = a.n_q / a.n_kv;
  const long long rows = (long long)hpg * (a.M - n_reqs + 1);
  const long long items = (long long)n_reqs * a.n_kv * ((rows + 15) / 16) * ((max_blocks + kAttnSpan - 1) / kAttnSpan);
  const int cus = a.cus > 0 ? std::min(a.cus, kAttnGrid) : kAttnGrid;
  if (BF && a.wave_tiles) {
    const hipError_t e = launch_attn_spans(a, n_reqs, 2 * cus, s);
    if (e != hipSuccess) return e;
  } else if (items > cus && a.attn_rt == 0) {
    const int grid2 = (int)std::min<long long>(2 * cus, (items + 7) / 8 * 8);
    attn_group2_kernel<BF, D><<<grid2, 256, attn_span_lds_bytes<BF, D, 1>(), s>>>(a, n_reqs);
  } else {
    const int grid = (int)std::min<long long>(cus, (items + 7) / 8 * 8);
    attn_group_kernel<BF, D><<<grid, 256, attn_span_lds_bytes<BF, D, 2>(), s>>>(a, n_reqs);
  }
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.merge_last) return e;
  attn_merge_kernel<BF, D><<<a.M * a.n_q, 64, 0, s>>>(a, n_reqs);
  return hipGetLastError();
}

// Kernels whose dynamic LDS may exceed the default 64 KiB limit.
template <bool BF, int AM, int EPI>
static hipError_t prepare_range() {
  const int bytes = gemm_range_lds_bytes(kDirectMT, kMaxUnits);
  auto allow = [bytes](const void* k) { return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); };
  hipError_t e = allow(reinterpret_cast<const void*>(&gemm_range_kernel<BF, 1, 0, AM, EPI>));
  if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(&gemm_range_kernel<BF, 2, 0, AM, EPI>));
  if constexpr (AM == A_NORM && (EPI == EPI_SWIGLU || EPI == EPI_ARGMAX)) {
#define AS2D_R(mt, i) \
  if (e == hipSuccess) e = allow(reinterpret_cast<const void*>(&gemm_range_kernel<BF, mt, kRangeSL<BF>[i], AM, EPI>));
    AS2D_R(1, 0) AS2D_R(1, 1) AS2D_R(1, 2)
    if constexpr (BF) {
      AS2D_R(2, 0) AS2D_R(2, 1) AS2D_R(2, 2)
    }
#undef AS2D_R
  }
  return e;
}

template <int AM, int EPI>
static hipError_t prepare_staged() {
  hipError_t e = hipSuccess;
  auto allow = [&](const void* k, int bytes) {
    if (e == hipSuccess) e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  };
#define AS2D_S(mt) \
  allow(reinterpret_cast<const void*>(&gemm_staged_kernel<mt, AM, EPI>), gemm_staged_lds_bytes<mt>());
  AS2D_S(1) AS2D_S(2) AS2D_S(3) AS2D_S(4) AS2D_S(5) AS2D_S(6) AS2D_S(7) AS2D_S(8) AS2D_S(9)
#undef AS2D_S
  return e;
}

// Attention kernels: two row tiles of 128 dimensions exchange 64 KiB of
// chunk sums plus their statistics; the prefill kernel's two span groups
// 81 KiB with the handed-over states.
template <bool BF, int D>
static hipError_t prepare_attention() {
  auto allow = [](const void* k, int bytes) { return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); };
  hipError_t e = allow(reinterpret_cast<const void*>(&attn_group_kernel<BF, D>), attn_span_lds_bytes<BF, D, 2>());
  if constexpr (!BF)
    if (e == hipSuccess)
      e = allow(reinterpret_cast<const void*>(&attn_prefill_kernel<D>), attn_prefill_lds_bytes<D>());
  return e;
}

hipError_t prepare_kernels() {
  hipError_t e = prepare_step_kernels();
  if (e == hipSuccess) e = prepare_attention<true, 128>();
  if (e == hipSuccess) e = prepare_attention<true, 64>();
  if (e == hipSuccess) e = prepare_attention<false, 128>();
  if (e == hipSuccess) e = prepare_attention<false, 64>();
#define AS2D_P(bf, am, ep) \
  if (e == hipSuccess) e = prepare_range<bf, am, ep>(); \
  if (e == hipSuccess && !bf) e = prepare_staged<am, ep>();
  AS2D_P(true, A_NORM, EPI_QKV) AS2D_P(true, A_PLAIN, EPI_RESID) AS2D_P(true, A_NORM, EPI_SWIGLU)
  AS2D_P(true, A_NORM, EPI_ARGMAX) AS2D_P(true, A_PLAIN, EPI_DOWN)
  AS2D_P(false, A_NORM, EPI_QKV) AS2D_P(false, A_PLAIN, EPI_RESID) AS2D_P(false, A_NORM, EPI_SWIGLU)
  AS2D_P(false, A_NORM, EPI_ARGMAX) AS2D_P(false, A_PLAIN, EPI_DOWN)
#undef AS2D_P
  if (e == hipSuccess) e = prepare_wide();
  if (e == hipSuccess) e = prepare_attn_prefill();
  return e;
}

hipError_t launch_attention(bool bf16, const AttnArgs& a, int n_reqs, int max_blocks, bool prefill, hipStream_t s) {
  if (a.head_dim == 128) return bf16 ? attn_dispatch<true, 128>(a, n_reqs, max_blocks, prefill, s)
                                     : attn_dispatch<false, 128>(a, n_reqs, max_blocks, prefill, s);
  if (a.head_dim == 64) return bf16 ? attn_dispatch<true, 64>(a, n_reqs, max_blocks, prefill, s)
                                    : attn_dispatch<false, 64>(a, n_reqs, max_blocks, prefill, s);
  return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------------
// Final arg-max over the LM head's per-pair partials, one workgroup per
// verified row, then greedy verification by the last row of each request
// to finish (device-scope counter per request).  The results go straight to
// the host's pinned memory (a few words per row, visible when the stream has
// been waited for), so no copies follow the pass.

__global__ __launch_bounds__(256) void finish_kernel(const RowDesc* __restrict__ rows,
                                                     const ReqDesc* __restrict__ reqs, int n_reqs,
                                                     const float* __restrict__ amax_val,
                                                     const float* __restrict__ amax_val2,
                                                     const int* __restrict__ amax_idx, int n_pairs,
                                                     int* __restrict__ row_tok, int* __restrict__ row_bad,
                                                     int* __restrict__ counters, const HostOut out) {
  __shared__ float s4f[4], s4s[4];
  __shared__ int s4i[4];
  __shared__ int s_tok, s_bad;
  __shared__ float s_margin;
  int r = 0, i = blockIdx.x;   // the grid is the sum of the requests' rows
  if (n_reqs > 1) r = find_request(reqs, n_reqs, i, [](const ReqDesc& q) { return q.W; });
  if (r < 0) return;
  const ReqDesc rq = reqs[r];
  const int row = rq.row_start + i;
  argmax_row<false>(amax_val, amax_val2, amax_idx, n_pairs, row, &s_tok, &s_bad, &s_margin, s4f, s4s, s4i);
  if (threadIdx.x == 0) {
    st<true>(row_tok + row, s_tok);
    st<true>(row_bad + row, s_bad);
    out.tok[row] = s_tok;   // read by the host after the pass
    out.margin[row] = s_margin;
    wait_vmem();
    if (counter_add(&counters[r], 1) == rq.W - 1) {
      counters[r] = 0;  // ready for the next launch
      int bad = 0;
      for (int q = 0; q < rq.W; ++q) bad |= ld_coherent(row_bad + rq.row_start + q);
      out.req[r] = verify_request(rows, rq, [&](int rr) { return ld_coherent(row_tok + rr); }, bad);
    }
  }
}

hipError_t launch_finish(const RowDesc* rows, const ReqDesc* reqs, int n_reqs, int n_rows,
                         const float* amax_val, const float* amax_val2, const int* amax_idx, int n_pairs,
                         int* row_tok, int* row_bad, int* counters, const HostOut& out, hipStream_t s) {
  finish_kernel<<<n_rows, 256, 0, s>>>(rows, reqs, n_reqs, amax_val, amax_val2, amax_idx, n_pairs, row_tok,
                                       row_bad, counters, out);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Zero fill.

__global__ void fill_zero_kernel(int* __restrict__ p, int n) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) p[i] = 0;
}

hipError_t launch_fill_zero(int* p, int n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  fill_zero_kernel<<<min((n + 255) / 256, 1024), 256, 0, s>>>(p, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Read-bandwidth reference: wave w of the grid streams its contiguous
// segment of `per_wave` 16-byte units, 8 loads (8 KiB per wave) in flight.

__global__ __launch_bounds__(256) void stream_read_kernel(const uint4* __restrict__ buf, long long per_wave,
                                                          unsigned* __restrict__ out) {
  constexpr int D = 8;
  const int lane = threadIdx.x & 63;
  const long long wave = (long long)blockIdx.x * 4 + (threadIdx.x >> 6);
  const u32x4* p = reinterpret_cast<const u32x4*>(buf + wave * per_wave + lane);
  const int steps = (int)(per_wave / 64);
  u32x4 r[D];
  unsigned acc = 0;
#pragma unroll
  for (int u = 0; u < D; ++u) r[u] = __builtin_nontemporal_load(p + u * 64);
  for (int i = 0; i + D < steps; i += D) {
#pragma unroll
    for (int u = 0; u < D; ++u) {
      acc ^= r[u].x ^ r[u].y ^ r[u].z ^ r[u].w;
      r[u] = __builtin_nontemporal_load(p + (long long)(i + D + u) * 64);
    }
  }
#pragma unroll
  for (int u = 0; u < D; ++u) acc ^= r[u].x ^ r[u].y ^ r[u].z ^ r[u].w;
  if (acc == 0x9e3779b9u) out[wave] = acc;   // keeps the loads; never true for a zeroed buffer
}

hipError_t launch_stream_read(const uint4* buf, long long n16, int grid, unsigned* out, hipStream_t s) {
  const long long waves = (long long)grid * 4;
  const long long per_wave = n16 / waves;
  if (grid < 1 || per_wave < 64 * 8 || per_wave % (64 * 8)) return hipErrorInvalidValue;
  stream_read_kernel<<<grid, 256, 0, s>>>(buf, per_wave, out);
  return hipGetLastError();
}

}  // namespace as2d
