// Prefill attention of bf16 models: one request's rows of a pass, block
// causal, with the arithmetic of attn.h.
//
// A workgroup of eight waves serves one KV head: each wave owns one tile of
// 16 rows of one of its query heads and walks the keys chunk by chunk (32
// keys) in ascending order, so the fold over chunks and spans stays in its
// registers.  The chunk's keys and values are read once per workgroup into
// LDS (three key buffers, two of values), the next keys two chunks ahead, the
// next values one.  Tiles are numbered row tile first, query head second, so a
// workgroup's tiles see about the same keys; the rows with the most keys
// start first.
//
// Both products are formed transposed (s: keys x rows, A: dimensions x
// rows), so a lane holds values of one query row only: the row's maximum
// and sum need the two cross-row swaps, and the fold's coefficients are the
// lane's own.
//
// What bounds it: a wave's chain of dependent steps per chunk (24 products,
// softmax, 24 products, fold: about 3,900 cycles alone, 4,500 with the two
// waves of a SIMD; a third of it waits, 35 % matrix-core busy).  Measured at
// the 7B shape, one layer: rows 5,673-7,563 of a prefill 0.79 ms, all 7,564
// rows 1.45 ms (passes of 144 rows by a workgroup per head and 16 rows, each
// reading its keys itself: 5.4 ms).  Four waves per workgroup, two
// workgroups per compute unit: 1.59 ms (twice the reads); the next chunk's
// scores issued among the softmax: 1.71 ms; all of a chunk's LDS reads at
// once instead of in groups: 1.54 ms.
#include "attn.h"

namespace as2d {

constexpr int kPrefillWaves = 8;
constexpr int kSpanWaves = 4;   // of the verification kernel below: two workgroups per compute unit

// LDS: three buffers of a chunk's keys [32][4 D bytes] (a chunk's first keys
// are read at the end of the chunk before) and two of its values [32 D 4
// bytes].  Keys: unit u (16 bytes) of key k at u ^ (k % 16), so that the 16
// keys a fragment read takes at one u lie in 16 different bank groups, and
// so do the units of one key.  Values: fragment order (block of 16
// dimensions and one part, lane).
template <int D> __host__ __device__ constexpr int attn_wide_units() { return 8 * D; }   // 16-byte units, keys or values
template <int D> __host__ __device__ constexpr int attn_wide_lds_bytes() { return (3 + 2) * attn_wide_units<D>() * 16; }

// attn_merge_coef for states that may be empty (M = -inf, L = 0, A = 0: the
// identity): 2^(-inf - 0) = 0.
__device__ __forceinline__ MergeCoef attn_coef0(float& M, float& L, float m, float l) {
#pragma clang fp contract(off)
  const float Mn = fmaxf(M, m), ref = Mn == -INFINITY ? 0.0f : Mn;
  const MergeCoef k{exp2_hw(M - ref), exp2_hw(m - ref)};
  L = __builtin_fmaf(L, k.a, l * k.c);
  M = Mn;
  return k;
}

// Chunks [c_first, c_end) (c_first the first of a span) of KV head g for the
// NW waves' row tiles.  This lane's row sits at position pos and its queries
// come from load_q once the first keys are requested; p0: a position no row
// of the tile is before; last: the last key any of the workgroup's rows sees.
// on_span(span, M, S, A) gets each span's state: A[t][i] is dimension
// 16 t + 4 (lane / 16) + i.  Ends with the workgroup's barrier.
template <int D, int NW, class LoadQ, class OnSpan>
__device__ __forceinline__ void attn_walk(const AttnArgs& p, const ReqDesc& rq, int g, int p0, int pos, int last,
                                          int c_first, int c_end, unsigned char* smem, LoadQ&& load_q, OnSpan&& on_span) {
#pragma clang fp contract(off)
  constexpr int KS = D / 32, DT = D / 16, U = attn_wide_units<D>(), NV = U / (64 * NW);
  constexpr int KU = D / 4;   // units of a key: hi, lo
  static_assert(NV >= 1, "whole units per thread");
  const int tid = threadIdx.x, lane = tid & 63, lg = lane >> 4, lr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const size_t head = (size_t)rq.slot * p.slot_stride + (size_t)g * p.kv_cap * D;   // float32 units
  const uint4* kb = reinterpret_cast<const uint4*>(p.k_cache + head);
  const uint4* vb = reinterpret_cast<const uint4*>(p.v_cache + head);
  u32x4* L = reinterpret_cast<u32x4*>(smem);   // keys [3][U], values [2][U]

  // this thread's units of a chunk: NV of its keys, NV of its values
  uint4 kr[NV], vr[NV];
  auto request_k = [&](int c, uint4(&kr)[NV]) {
#pragma unroll
    for (int i = 0; i < NV; ++i) kr[i] = ldg(kb + (size_t)c * U + tid + i * 64 * NW);
  };
  auto request_v = [&](int c) {
#pragma unroll
    for (int i = 0; i < NV; ++i)
      vr[i] = ldg(vb + (size_t)c * U + (wave * 64 + i * 64 * NW) + frag_lane_unit(lane));
  };
  auto stage_k = [&](int buf, const uint4(&kr)[NV]) {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int u = tid + i * 64 * NW, key = u / KU, ku = u % KU;
      L[buf * U + key * KU + (ku ^ (key & 15))] = __builtin_bit_cast(u32x4, kr[i]);
    }
  };
  // to buffer c % 2; values past the workgroup's last row (never written, or left by an
  // earlier request) are set to zero: their p is 0
  auto stage_v = [&](int c) {
    const int kc = c * kAttnChunk;
    if (kc + kAttnChunk > last + 1) {
      const int n0 = min(max(last + 1 - (kc + 4 * lg), 0), 4), n1 = min(max(last + 1 - (kc + 16 + 4 * lg), 0), 4);
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const uint4 a = keep_first<true>(make_uint4(vr[i].x, vr[i].y, 0, 0), n0);
        const uint4 b = keep_first<true>(make_uint4(vr[i].z, vr[i].w, 0, 0), n1);
        vr[i] = make_uint4(a.x, a.y, b.x, b.y);
      }
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) L[(3 + (c & 1)) * U + tid + i * 64 * NW] = __builtin_bit_cast(u32x4, vr[i]);
  };
  int k0 = 0, k1 = 1, k2 = 2;   // key buffers of this chunk, the next one and the one after
  Op2 q[KS];
  {
    uint4 kn[NV];   // the second chunk's keys
    const int c1 = min(c_first + 1, c_end - 1);
    request_k(c_first, kr);
    request_v(c_first);
    request_k(c1, kn);
    load_q(q);
    stage_k(k0, kr);
    stage_v(c_first);
    stage_k(k1, kn);
  }
  lds_sync();

  float Ms, Ss, As[DT][4];   // the span's maximum, sum and p v
  // A chunk's operands from the LDS in groups of two: KS groups of keys (the
  // two 16-key tiles of a k-step), then DT / 2 groups of values (two
  // dimension tiles).  Group n sits in slot n % 4 of f and is requested AHEAD
  // groups before its products, across chunks, so that the LDS serves the
  // eight waves evenly while the matrix cores work.
  constexpr int NG = KS + DT / 2, AHEAD = 2;
  static_assert(NG % 4 == 0 && AHEAD <= KS, "slots repeat every chunk; only keys are requested across chunks");
  Op2 f[4][2];
  auto load = [&](int c, int n) {   // group n < NG of chunk c, or group n - NG of the next one
    const int kbuf = n >= NG ? k1 : k0;
    if (n >= NG) n -= NG;   // keys: AHEAD <= KS
    if (n < KS) {
      const u32x4* K = L + kbuf * U + lr * KU;
#pragma unroll
      for (int j = 0; j < 2; ++j)
        f[n & 3][j] = Op2{__builtin_bit_cast(uint4, K[16 * j * KU + ((4 * n + lg) ^ lr)]),
                          __builtin_bit_cast(uint4, K[16 * j * KU + ((KU / 2 + 4 * n + lg) ^ lr)])};
    } else {
      const u32x4* V = L + (3 + (c & 1)) * U + lane;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int t = 2 * (n - KS) + j;
        f[n & 3][j] = Op2{__builtin_bit_cast(uint4, V[t * 64]), __builtin_bit_cast(uint4, V[(DT + t) * 64])};
      }
    }
  };
  // chunk c, whose first AHEAD groups are requested, into the span's state;
  // requests those of the next chunk (past the last: whatever the buffers
  // hold, unused).  The sched_barriers keep the order.
  auto chunk = [&](int c) {
    const int kc = c * kAttnChunk;
    // scores, transposed: lane l holds keys kc + 16 kt + 4 (l / 16) + i of row l % 16
    f4 sa[2] = {f4{0.f, 0.f, 0.f, 0.f}, f4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      load(c, ks + AHEAD);
      __builtin_amdgcn_sched_barrier(0);
      const Op2(&k)[2] = f[ks & 3];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) sa[kt] = mma_step<true>(k[kt].h, q[ks].h, sa[kt]);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) sa[kt] = mma_step<true>(k[kt].h, q[ks].l, sa[kt]);
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) sa[kt] = mma_step<true>(k[kt].l, q[ks].h, sa[kt]);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (kc + kAttnChunk > p0 + 1) {   // keys after the row are hidden
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (kc + 16 * kt + 4 * lg + i > pos) sa[kt][i] = -INFINITY;
    }
    float s[2][4];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 4; ++i) s[kt][i] = sa[kt][i] * p.scale;
    float mx = s[0][0];
#pragma unroll
    for (int e = 1; e < 8; ++e) mx = fmaxf(mx, s[e >> 2][e & 3]);
    mx = swap_combine<false>(mx, FMax{});
    mx = swap_combine<true>(mx, FMax{});
    // a chunk with no visible key: 2^(-inf - 0) = 0
    const float ref = mx == -INFINITY ? 0.0f : mx;
    float pj[2][4];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 4; ++i) pj[kt][i] = exp2_hw(s[kt][i] - ref);
    float sm = (((pj[0][0] + pj[0][1]) + pj[0][2]) + pj[0][3]) + (((pj[1][0] + pj[1][1]) + pj[1][2]) + pj[1][3]);
    sm = swap_combine<false>(sm, FAdd{});
    sm = swap_combine<true>(sm, FAdd{});
    uint32_t hw[4], lw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {   // keys 2 (e % 2), 2 (e % 2) + 1 of tile e / 2
      const float v0 = pj[e >> 1][2 * (e & 1)], v1 = pj[e >> 1][2 * (e & 1) + 1];
      hw[e] = f2bf2(v0, v1);
      lw[e] = f2bf2(v0 - bf2f(hw[e]), v1 - __uint_as_float(hw[e] & 0xffff0000u));
    }
    const Op2 pp{make_uint4(hw[0], hw[1], hw[2], hw[3]), make_uint4(lw[0], lw[1], lw[2], lw[3])};
    const MergeCoef k = attn_coef0(Ms, Ss, mx, sm);
    __builtin_amdgcn_sched_barrier(0);
    // p v transposed (lane l: dimensions 16 t + 4 (l / 16) + i of row l % 16),
    // folded into the span's state one group late: p_hi v_hi, p_hi v_lo, p_lo v_hi
    f4 acc[2][2];
    auto fold = [&](int n) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int i = 0; i < 4; ++i) As[2 * n + j][i] = attn_merge_acc(As[2 * n + j][i], acc[n & 1][j][i], k);
    };
#pragma unroll
    for (int n = 0; n < DT / 2; ++n) {
      load(c, KS + n + AHEAD);
      __builtin_amdgcn_sched_barrier(0);
      const Op2(&v)[2] = f[(KS + n) & 3];
      f4(&o)[2] = acc[n & 1];
#pragma unroll
      for (int j = 0; j < 2; ++j) o[j] = mma_step<true>(v[j].h, pp.h, f4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
      for (int j = 0; j < 2; ++j) o[j] = mma_step<true>(v[j].l, pp.h, o[j]);
#pragma unroll
      for (int j = 0; j < 2; ++j) o[j] = mma_step<true>(v[j].h, pp.l, o[j]);
      if (n) fold(n - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    fold(DT / 2 - 1);
  };
#pragma unroll
  for (int n = 0; n < AHEAD; ++n) load(c_first, n);
  for (int c0 = c_first; c0 < c_end; c0 += kAttnSpanKeys / kAttnChunk) {
    Ms = -INFINITY;
    Ss = 0.f;
#pragma unroll
    for (int t = 0; t < DT; ++t)
#pragma unroll
      for (int i = 0; i < 4; ++i) As[t][i] = 0.f;
    const int c1 = min(c0 + kAttnSpanKeys / kAttnChunk, c_end);
    for (int c = c0; c < c1; ++c) {
      if (c + 2 < c_end) request_k(c + 2, kr);
      if (c + 1 < c_end) request_v(c + 1);
      chunk(c);   // past a tile's last key: every key hidden, the state unchanged
      // these buffers were last read in the chunk before, which every wave
      // has left
      if (c + 2 < c_end) stage_k(k2, kr);
      if (c + 1 < c_end) stage_v(c + 1);
      lds_sync();
      const int k = k0;
      k0 = k1;
      k1 = k2;
      k2 = k;
    }
    on_span(c0 / (kAttnSpanKeys / kAttnChunk), Ms, Ss, As);
  }
}

// The operands of one query row and head: this lane's share of every k-step.
template <int D> __device__ __forceinline__ void attn_load_row(const AttnArgs& p, int row, int h, Op2 (&q)[D / 32]) {
  const float4* src = reinterpret_cast<const float4*>(p.q + (size_t)row * p.n_q * D + h * D + 8 * ((threadIdx.x & 63) >> 4));
#pragma unroll
  for (int ks = 0; ks < D / 32; ++ks) {
    const float4 v[2] = {ldg(src + 8 * ks), ldg(src + 8 * ks + 1)};
    q[ks] = split_op<true>(v);
  }
}

template <int D>
__global__ __launch_bounds__(64 * kPrefillWaves, 2) void attn_prefill_wide_kernel(const AttnArgs p) {
#pragma clang fp contract(off)
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int DT = D / 16;
  const ReqDesc rq = load_invariant(p.reqs);
  const int lane = threadIdx.x & 63, lg = lane >> 4, lr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int hpg = p.n_q / p.n_kv;
  const int tiles = (rq.W + 15) / 16 * hpg, nw = (tiles + kPrefillWaves - 1) / kPrefillWaves;
  const int g = blockIdx.x % p.n_kv, w = nw - 1 - blockIdx.x / p.n_kv;
  const int T = min(w * kPrefillWaves + wave, tiles - 1);
  const bool mine = w * kPrefillWaves + wave < tiles;
  const int rt = T / hpg, h = g * hpg + (T - rt * hpg);
  const int p0 = rq.L0 + rt * 16;                                 // position of the tile's first row
  const int last = rq.L0 + min(rt * 16 + 15, rq.W - 1);           // ... and of its last one
  const int pos = min(p0 + lr, last);                             // this lane's row (past the last: the last again)
  const int last_all = rq.L0 + min(min((w + 1) * kPrefillWaves - 1, tiles - 1) / hpg * 16 + 15, rq.W - 1);

  // the state of all spans so far (an empty one joins as the identity)
  float M = -INFINITY, S = 0.f, A[DT][4];
#pragma unroll
  for (int t = 0; t < DT; ++t)
#pragma unroll
    for (int i = 0; i < 4; ++i) A[t][i] = 0.f;
  const int row = rq.row_start + pos - rq.L0;
  attn_walk<D, kPrefillWaves>(
      p, rq, g, p0, pos, last_all, 0, last_all / kAttnChunk + 1, smem, [&](Op2(&q)[D / 32]) { attn_load_row<D>(p, row, h, q); },
      [&](int, float Ms, float Ss, const float(&As)[DT][4]) {
        // a row that does not reach the span: unchanged
        const MergeCoef ka = attn_coef0(M, S, Ms, Ss);
#pragma unroll
        for (int t = 0; t < DT; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) A[t][i] = attn_merge_acc(A[t][i], As[t][i], ka);
      });
  if (!mine || p0 + lr > last) return;
#pragma unroll
  for (int t = 0; t < DT; ++t) {
    float o[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = A[t][i] / S;
    store_act_run<true, false, 4>(p.out, p.out_plane, frag_index<true>(row, h * D + 16 * t + 4 * lg, p.n_q * D), o);
  }
}

// Verification passes over long caches: work items (request, run of spans,
// KV head, group of four row tiles), the rows of the query heads that share
// the KV head packed head by head as in attn_group_kernel.  Each wave owns a
// tile, so a run's keys and values are read once for up to 64 rows and a
// span needs no exchange between waves (attn_group2_kernel: once per 16
// rows, its four waves meeting twice per span).  Span states go to memory
// for attn_merge_kernel.  A fixed grid takes the items in turn.
template <int D>
__global__ __launch_bounds__(64 * kSpanWaves, 2) void attn_spans_wide_kernel(const AttnArgs p, int n_reqs) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int DT = D / 16, kRows = 16 * kSpanWaves, kChunks = kAttnSpanKeys / kAttnChunk;
  const int lane = threadIdx.x & 63, lg = lane >> 4, lr = lane & 15;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int G = gridDim.x, hpg = p.n_q / p.n_kv;
  const auto spans = [](const ReqDesc& rq) { return (rq.L0 + rq.W - 1) / kAttnSpanKeys + 1; };
  const auto groups = [&](const ReqDesc& rq) { return p.n_kv * ((hpg * rq.W + kRows - 1) / kRows); };
  const auto items = [&](const ReqDesc& rq, int R) { return groups(rq) * ((spans(rq) + R - 1) / R); };
  int R, total;
  attn_run_length(p.reqs, n_reqs, G, items, groups, R, total);
  for (int t = xcd_contiguous(blockIdx.x, G); t < total; t += G) {
    int u = t;
    const int r = n_reqs == 1 ? 0 : find_request(p.reqs, n_reqs, u, [&](const ReqDesc& q) { return items(q, R); });
    const ReqDesc rq = load_invariant(p.reqs + r);
    const int ng = groups(rq), j = u / ng, v = u - j * ng;   // run j
    const int per = ng / p.n_kv, g = v / per, b = v - g * per;
    const AttnRows rows{g * hpg, rq.W, hpg * rq.W, b * kRows};
    const int rr = 16 * wave + lr, i = rows.row(rr), h = rows.head(rr), row = rq.row_start + i;
    const int last = rq.L0 + rq.W - 1, pos = rq.L0 + i;
    const int c_first = j * R * kChunks, c_end = min(c_first + R * kChunks, last / kAttnChunk + 1);
    attn_walk<D, kSpanWaves>(
        p, rq, g, rq.L0, pos, last, c_first, c_end, smem, [&](Op2(&q)[D / 32]) { attn_load_row<D>(p, row, h, q); },
        [&](int sp, float Ms, float Ss, const float(&As)[DT][4]) {
          if (!rows.valid(rr) || pos < sp * kAttnSpanKeys) return;
          const size_t o = ((size_t)row * p.n_q + h) * p.part_spans + sp;
#pragma unroll
          for (int t = 0; t < DT; ++t)
            *gmem(reinterpret_cast<f4*>(p.pacc + o * D + 16 * t + 4 * lg)) = f4{As[t][0], As[t][1], As[t][2], As[t][3]};
          if (lg == 0) *gmem(reinterpret_cast<f2*>(p.pml + o * 2)) = f2{Ms, Ss};
        });
  }
}

hipError_t prepare_attn_prefill() {
  auto allow = [](const void* k) {
    return hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, attn_wide_lds_bytes<128>());
  };
  const hipError_t e = allow(reinterpret_cast<const void*>(&attn_prefill_wide_kernel<128>));
  return e == hipSuccess ? allow(reinterpret_cast<const void*>(&attn_spans_wide_kernel<128>)) : e;
}

hipError_t launch_attn_spans(const AttnArgs& a, int n_reqs, int grid, hipStream_t s) {
  if (a.head_dim == 128) attn_spans_wide_kernel<128><<<grid, 64 * kSpanWaves, attn_wide_lds_bytes<128>(), s>>>(a, n_reqs);
  else if (a.head_dim == 64) attn_spans_wide_kernel<64><<<grid, 64 * kSpanWaves, attn_wide_lds_bytes<64>(), s>>>(a, n_reqs);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_attn_prefill(const AttnArgs& a, hipStream_t s) {
  const int hpg = a.n_q / a.n_kv, tiles = (a.M + 15) / 16 * hpg;
  const int grid = (tiles + kPrefillWaves - 1) / kPrefillWaves * a.n_kv;
  if (a.head_dim == 128) attn_prefill_wide_kernel<128><<<grid, 64 * kPrefillWaves, attn_wide_lds_bytes<128>(), s>>>(a);
  else if (a.head_dim == 64) attn_prefill_wide_kernel<64><<<grid, 64 * kPrefillWaves, attn_wide_lds_bytes<64>(), s>>>(a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace as2d
