// Wide GEMM tiles of bf16 models: passes of more rows than the direct path
// takes (prefill and fused batches), on matrix cores.
//
// A workgroup of four waves owns TM row tiles x 4 TN column tiles (16 x 16
// each) of Y = A W^T.  Wave w owns the column tiles [w TN, (w + 1) TN) for
// all TM row tiles.  A wave's weights are its own: they go straight from
// memory to registers, AH k-steps ahead.  The activation fragments
// (hi and lo planes) are shared by the four waves: staged through LDS two
// k-steps at a time in three buffers, one barrier per stage, with the next
// k-step's first fragment read before the current one ends.
//
// Sums.  The order is that of every GEMM path (tiles.h): a slice is
// accumulated over its k-steps by MFMA from zero, the slices of a split are
// added in order, then the splits in order.  The k-steps of consecutive
// slices and splits are consecutive, so a workgroup walks them as one run;
// at a slice's first k-step the finished sums are added to S while the
// matrix cores start the new ones from zero.  S starts at -0, which leaves
// the first addend as it is.
//
// A unit covers spu slices: all of them (the workgroup ends with the
// output; finished splits are kept in memory, T), the four of one split, or
// one slice.  In the last two cases each unit writes its sums as one record
// and the last unit of the tile to arrive adds the records in order.
//
// What bounds it: matrix-core issue and the loads' latency, hidden by two
// workgroups per compute unit (4 x 4 tiles: 1.1 PFLOP/s of (hi, lo) products
// at 1,904 rows, about the rate of a plain 8192^3 library product on this
// device; one workgroup of 8 x 4 tiles per unit, with half the reads per
// product, reached 0.7).  The 4 x 4 tiles fill the 256 registers that two
// workgroups leave them and spill 4 to 6 (20 to 28 bytes per lane).  782 rows of the 7B shape, against passes of 144
// rows through the staged path it replaces: gate/up 780 -> 432 us, down
// 640 -> 240, QKV 354 -> 88, O 198 -> 69 us; at 84 rows (a fused batch)
// 115 -> 90, 106 -> 61, 48 -> 27, 33 -> 21 us.  (QKV and O were 77 and 55,
// 24 and 20 us with the three and two k-splits they had before the direct
// path's plan left them whole; the direct path gained more than that.)
#pragma once
#include "tiles.h"

namespace as2d {

constexpr int kWideStages = 3;    // LDS buffers of two k-steps
constexpr int kWideFRows = 64;    // rows per epilogue pass

template <int TM> __host__ __device__ constexpr int wide_stage_units() { return 4 * TM * 64; }   // 16-byte units
template <int TN> __host__ __device__ constexpr int wide_fstride() { return kWaves * TN * 16 + 4; }
template <int TM> __host__ __device__ constexpr int wide_frows() { return TM * 16 < kWideFRows ? TM * 16 : kWideFRows; }
template <int TM, int TN> __host__ __device__ constexpr int wide_lds_bytes() {
  constexpr int a = kWideStages * wide_stage_units<TM>() * 16, f = wide_frows<TM>() * wide_fstride<TN>() * 4;
  return a > f ? a : f;
}

// Row scales of rows [r0, r1) into s_scale[0 ..): the sums of row_scales.
template <int RPW>
__device__ __forceinline__ void wide_row_scales(const GemmArgs& p, int r0, int r1, float* s_scale) {
  constexpr int kR = 8, kT = 4;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int np = p.n_norm_pairs;
#pragma unroll 1
  for (int b = 0; b < RPW; b += kR) {
    float v[kR][kT];
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const int m = min(r0 + wave + kWaves * (b + r), r1 - 1);
#pragma unroll
      for (int t = 0; t < kT; ++t) {
        const int i = lane + 64 * t;
        v[r][t] = 64 * t < np ? ldg(p.sumsq + (size_t)m * np + (i < np ? i : 0)) : 0.0f;
      }
    }
#pragma unroll
    for (int r = 0; r < kR; ++r) {
      const int m = r0 + wave + kWaves * (b + r);
      float s = 0.0f;
#pragma unroll
      for (int t = 0; t < kT; ++t)
        if (lane + 64 * t < np) s += v[r][t];
      const float tot = wave_sum(s);
      if (lane == 0 && m < r1) s_scale[m - r0] = 1.0f / sqrtf(tot / (float)p.K + p.eps);
    }
  }
}

// Epilogue of rows [r0, r1) (r1 - r0 <= FR) of the workgroup's C = 64 TN
// columns from pair pair0, with epilogue_rows' results: `put` writes the
// finished sums to F (row stride FS).  A thread takes eight consecutive
// columns of a row (QKV: and the eight that rotate with them), FR / RP rows
// RP apart.  What it reads from memory (residual, rotation angles, row
// descriptors) is requested for all its rows before the sums are put, so a
// chunk pays for one round trip; everything but the V cache is stored 16
// bytes at a time.
template <int TN, int FR, int EPI, class Put>
__device__ __forceinline__ void wide_epilogue(const GemmArgs& p, float* F, int pair0, int r0, int r1, Put&& put) {
  constexpr int C = 64 * TN, FS = wide_fstride<TN>();
  const int tid = threadIdx.x;
  auto load8 = [](const float* q, float(&v)[8]) {
    const float4 a = ldg(reinterpret_cast<const float4*>(q)), b = ldg(reinterpret_cast<const float4*>(q) + 1);
    v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
    v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
  };
  auto store8 = [](float* q, const float(&v)[8]) {
    *gmem(reinterpret_cast<f4*>(q)) = f4{v[0], v[1], v[2], v[3]};
    *gmem(reinterpret_cast<f4*>(q) + 1) = f4{v[4], v[5], v[6], v[7]};
  };
  auto lds8 = [&](int row, int c, float(&v)[8]) {
    const f4* q = reinterpret_cast<const f4*>(F + row * FS + c);
    const f4 a = q[0], b = q[1];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      v[t] = a[t];
      v[4 + t] = b[t];
    }
  };
  // the (hi, lo) pairs of eight values at o and o + plane
  auto store_pairs = [](uint16_t* o, long long plane, const BfPair(&v)[8]) {
    u32x4 h, l;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      h[t] = v[2 * t].hi | ((uint32_t)v[2 * t + 1].hi << 16);
      l[t] = v[2 * t].lo | ((uint32_t)v[2 * t + 1].lo << 16);
    }
    *gmem(reinterpret_cast<u32x4*>(o)) = h;
    *gmem(reinterpret_cast<u32x4*>(o + plane)) = l;
  };
  if constexpr (EPI == EPI_RESID || EPI == EPI_DOWN) {
    constexpr int U = C / 8, RP = 256 / U, NR = FR / RP;
    const int c = (tid % U) * 8, n = pair0 * kPairCols + c, rr = tid / U, N = p.N;
    float x[NR][8], gain[8];
    load8(p.gain_next + n, gain);
#pragma unroll
    for (int i = 0; i < NR; ++i) load8(p.x + (size_t)min(r0 + rr + RP * i, r1 - 1) * N + n, x[i]);
    put();
    lds_sync();
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int m = r0 + rr + RP * i;
      float v[8];
      BfPair o[8];
      lds8(rr + RP * i, c, v);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        v[t] = x[i][t] + v[t];
        o[t] = split_mul(v[t], gain[t]);
      }
      float s = sumsq8(v);   // four neighbours hold a pair
      s = s + dpp_get<kDppXor1>(s);
      s = s + dpp_get<kDppXor2>(s);
      if (m < r1) {
        store8(p.x_out + (size_t)m * N + n, v);
        store_pairs(static_cast<uint16_t*>(p.out) + frag_index<true>(m, n, N), p.out_plane, o);
        if ((tid & 3) == 0) *gmem(p.sumsq_out + (size_t)m * (N / kPairCols) + n / kPairCols) = s;
      }
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    constexpr int U = C / 16, RP = 256 / U, NR = (FR + RP - 1) / RP;
    const int u = tid % U, c = (u >> 1) * kPairCols + (u & 1) * 8, n = pair0 * 16 + u * 8, rr = tid / U, F2 = p.N / 2;
    put();
    lds_sync();
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int m = r0 + rr + RP * i;
      if (FR % RP && rr + RP * i >= FR) break;
      float g[8], up[8];
      BfPair o[8];
      lds8(rr + RP * i, c, g);
      lds8(rr + RP * i, c + 16, up);
#pragma unroll
      for (int t = 0; t < 8; ++t) o[t] = split_mul(silu(g[t]), up[t]);
      if (m < r1) store_pairs(static_cast<uint16_t*>(p.out) + frag_index<true>(m, n, F2), p.out_plane, o);
    }
  } else if constexpr (EPI == EPI_QKV) {
    // PACK_ROPE_PAIRS: columns c + t and c + 16 + t of a pair are dimensions
    // i0 + t and d / 2 + i0 + t of its head
    constexpr int U = C / 16, RP = 256 / U, NR = (FR + RP - 1) / RP;
    const int u = tid % U, c = (u >> 1) * kPairCols + (u & 1) * 8, rr = tid / U;
    const int d = p.head_dim, half = d >> 1, ppd = d / kPairCols;
    const int pair = pair0 + (u >> 1), head = pair / ppd, i0 = 16 * (pair - head * ppd) + (u & 1) * 8;
    const bool rotated = head < p.n_q + p.n_kv;
    const int n = head * d + i0;
    int pos[NR], slot[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const RowDesc* r = p.rows + min(r0 + rr + RP * i, r1 - 1);
      pos[i] = ldg(&r->pos);
      slot[i] = ldg(&r->slot);
    }
    float b0[8] = {}, b1[8] = {};
    if (p.bias) {
      load8(p.bias + n, b0);
      load8(p.bias + n + half, b1);
    }
    put();
    lds_sync();
    // (cos, sin) of the eight angles
    float cs[NR][2][8];
#pragma unroll
    for (int i = 0; i < NR; ++i)
      if (rotated) {
        const float* q = p.rope_cs + ((size_t)pos[i] * half + i0) * 2;
        load8(q, cs[i][0]);
        load8(q + 8, cs[i][1]);
      }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int m = r0 + rr + RP * i;
      if (m >= r1 || (FR % RP && rr + RP * i >= FR)) break;
      float v0[8], v1[8];
      lds8(rr + RP * i, c, v0);
      lds8(rr + RP * i, c + 16, v1);
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        v0[t] += b0[t];
        v1[t] += b1[t];
      }
      if (rotated) {
        float o0[8], o1[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const float co = cs[i][t >> 2][2 * (t & 3)], si = cs[i][t >> 2][2 * (t & 3) + 1];
          o0[t] = rope(v0[t], -v1[t], co, si);
          o1[t] = rope(v1[t], v0[t], co, si);
        }
        if (head < p.n_q) {
          float* q = p.q_out + (size_t)m * p.n_q * d + n;
          store8(q, o0);
          store8(q + half, o1);
        } else {
          float* kb = p.k_cache + (size_t)slot[i] * p.slot_stride + (size_t)(head - p.n_q) * p.kv_cap * d;
          uint16_t* k16 = reinterpret_cast<uint16_t*>(kb) + (size_t)pos[i] * 2 * d + i0;
          BfPair h0[8], h1[8];
#pragma unroll
          for (int t = 0; t < 8; ++t) {
            h0[t] = split_val(o0[t]);
            h1[t] = split_val(o1[t]);
          }
          store_pairs(k16, d, h0);
          store_pairs(k16 + half, d, h1);
        }
      } else {
        float* vb = p.v_cache + (size_t)slot[i] * p.slot_stride + (size_t)(head - p.n_q - p.n_kv) * p.kv_cap * d;
        uint16_t* v16 = reinterpret_cast<uint16_t*>(vb);
#pragma unroll
        for (int t = 0; t < 16; ++t) {
          const BfPair h = split_val(t < 8 ? v0[t & 7] : v1[t & 7]);
          const int dd = (t < 8 ? 0 : half) + i0 + (t & 7);
          *gmem(v16 + v_elem(pos[i], 0, dd, d, true)) = h.hi;
          *gmem(v16 + v_elem(pos[i], 1, dd, d, true)) = h.lo;
        }
      }
    }
  } else {
    put();
    lds_sync();
    epilogue_rows<true, EPI, false>(p, F, FS, pair0, C / kPairCols, r0, r1);
  }
}

template <int TM, int TN, int AH, int AM, int EPI>
__device__ __forceinline__ void gemm_wide_tile(const GemmArgs& p, int rb, int cb, int unit, unsigned char* smem,
                                               float* s_scale, int* s_flag) {
  constexpr int STG = wide_stage_units<TM>();
  constexpr int NP = TN / 2;                     // tile pairs per wave
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int KT = p.KT, ns = p.ns, spu = p.spu, n_slices = p.KS * ns;
  const int M = p.M;
  // first k-step of slice g (g = n_slices: past the last)
  auto slice_at = [&](int g) {
    if (g >= n_slices) return KT;
    const int s = g / ns, kt0 = s * p.ktps, n = min(KT, kt0 + p.ktps) - kt0;
    return slice_start(kt0, n, g - s * ns, ns);
  };
  const int g0 = unit * spu, g1 = g0 + spu;
  const int k0 = slice_at(g0), k1 = slice_at(g1);
  const int mt0 = rb * TM, mt_last = (M - 1) >> 4;
  const int pair0 = (cb * kWaves + wave) * NP;
  u32x4* la = reinterpret_cast<u32x4*>(smem);

  // weights: column tile j of this wave at k-step kt
  const uint4* wp = p.W + (size_t)pair0 * KT * 128;
  auto load_w = [&](int kt, uint4(&w)[TN]) {
    const uint4* o = wp + (size_t)min(kt, k1 - 1) * 128;
#pragma unroll
    for (int j = 0; j < TN; ++j) w[j] = ldg(o + (size_t)(j >> 1) * KT * 128 + ((j & 1) * 64 + lane));
  };
  // activations: block b = wave + 4 i of a stage is (k-step b / 2 TM, plane
  // (b / TM) % 2, row tile b % TM); a row tile past the pass's last one
  // takes the last one (its rows are never stored)
  const uint4* ag = static_cast<const uint4*>(p.A);
  const long long lo = p.a_plane / ET<true>::PER16;
  const uint32_t lu = frag_lane_unit(lane);
  uint4 av[TM];
  auto request = [&](int kt) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int b = wave + kWaves * i, mt = b % TM;
      av[i] = ldg(ag + ((b / TM) & 1) * lo + ((size_t)min(mt0 + mt, mt_last) * KT + min(kt + b / (2 * TM), KT - 1)) * 64 + lu);
    }
  };
  auto stage = [&](int at) {   // at: 16-byte unit of the stage buffer
    u32x4* d = la + at + wave * 64 + lane;
#pragma unroll
    for (int i = 0; i < TM; ++i) d[kWaves * i * 64] = __builtin_bit_cast(u32x4, av[i]);
  };
  auto frag = [&](int at, int mt) {   // at: 16-byte unit of (stage buffer, k-step)
    const u32x4* f = la + at + lane;
    return AFrag{__builtin_bit_cast(uint4, f[mt * 64]), __builtin_bit_cast(uint4, f[(TM + mt) * 64])};
  };

  uint4 w[AH][TN];
#pragma unroll
  for (int u = 0; u < AH; ++u) load_w(k0 + u, w[u]);
  request(k0);
  if constexpr (AM == A_NORM)
    wide_row_scales<TM * 4>(p, mt0 * 16, min(M, (mt0 + TM) * 16), s_scale);
  stage(0);
  request(k0 + 2);
  lds_sync();

  f4 acc[TM][TN], S[TM][TN];
#pragma unroll
  for (int mt = 0; mt < TM; ++mt)
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      acc[mt][j] = f4{0.f, 0.f, 0.f, 0.f};
      S[mt][j] = f4{-0.f, -0.f, -0.f, -0.f};
    }
  // T: the sums of the splits before, kept by this workgroup in memory
  f4* T = reinterpret_cast<f4*>(p.part) + (size_t)(rb * p.CB + cb) * (TM * TN * 256) + tid;
  int g = g0, nb = slice_at(g0 + 1);   // current slice, first k-step of the next
  // the slices before k-step kt == nb end: their sums go to S (and T)
  auto flush = [&](int kt) {
    bool split_end = false;
    do {
      ++g;
      split_end |= g % ns == 0;
      nb = slice_at(g + 1);
    } while (nb == kt);
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int j = 0; j < TN; ++j) {
        S[mt][j] += acc[mt][j];
        acc[mt][j] = f4{0.f, 0.f, 0.f, 0.f};
      }
    if (split_end) {
      const bool add = g / ns > 1;
#pragma unroll
      for (int mt = 0; mt < TM; ++mt)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          f4* t = T + (mt * TN + j) * 256;
          *gmem(t) = add ? *gmem(t) + S[mt][j] : S[mt][j];
          S[mt][j] = f4{-0.f, -0.f, -0.f, -0.f};
        }
    }
  };
  // one k-step: fragments at `at`, those of the next k-step at `nx`; each
  // fragment is read FD row tiles before its products
  constexpr int FD = 2;
  AFrag fr[FD];
#pragma unroll
  for (int u = 0; u < FD; ++u) fr[u] = frag(0, u);
  auto kstep = [&](int kt, const uint4(&ww)[TN], int at, int nx) {
    if (kt == nb) flush(kt);
#pragma unroll
    for (int mt = 0; mt < TM; ++mt) {
      const AFrag nf = mt + FD < TM ? frag(at, mt + FD) : frag(nx, mt + FD - TM);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[mt][j] = mma_step<true>(fr[0].h, ww[j], acc[mt][j]);
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[mt][j] = mma_step<true>(fr[0].l, ww[j], acc[mt][j]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u + 1 < FD; ++u) fr[u] = fr[u + 1];
      fr[FD - 1] = nf;
    }
  };
  int cur = 0;
  for (int kt = k0; kt < k1; kt += AH) {
#pragma unroll
    for (int h = 0; h < AH / 2; ++h) {
      const int k = kt + 2 * h;
      if (k >= k1) break;
      const int nxt = cur + STG == kWideStages * STG ? 0 : cur + STG;
      kstep(k, w[2 * h], cur, cur + 2 * TM * 64);
      load_w(k + AH, w[2 * h]);
      stage(nxt);
      request(k + 4);
      lds_sync();
      if (k + 1 < k1) {
        kstep(k + 1, w[2 * h + 1], cur + 2 * TM * 64, nxt);
        load_w(k + 1 + AH, w[2 * h + 1]);
      }
      cur = nxt;
    }
  }
#pragma unroll
  for (int mt = 0; mt < TM; ++mt)
#pragma unroll
    for (int j = 0; j < TN; ++j) S[mt][j] += acc[mt][j];

  if (spu < n_slices) {
    // one record per unit, read back by the workgroup that arrives last
    // (same thread, same elements)
    const int n_rec = n_slices / spu;
    const __amdgpu_buffer_rsrc_t rec = coherent_rsrc(p.part);
    const uint32_t base = (uint32_t)(rb * p.CB + cb) * n_rec * (TM * TN * 256 * 16) + tid * 16;
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int j = 0; j < TN; ++j)
        st_coherent4(rec, base + ((uint32_t)unit * TM * TN + mt * TN + j) * 4096, S[mt][j]);
    wait_vmem();
    __syncthreads();
    int* cnt = &p.counters[rb * p.CB + cb];
    if (tid == 0) *s_flag = counter_add(cnt, 1) == n_rec - 1;
    __syncthreads();
    if (!*s_flag) return;
    if (tid == 0) st<true>(cnt, 0);   // ready for the next launch
    const int per = ns / spu;         // records per split (spu 1: 4), or one
    const int rps = per > 0 ? per : 1;
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[mt][j] = f4{-0.f, -0.f, -0.f, -0.f};
    for (int s = 0; s < p.KS; ++s) {
      for (int q = 0; q < rps; ++q)
#pragma unroll
        for (int mt = 0; mt < TM; ++mt)
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const float4 v = ld_coherent4(rec, base + ((uint32_t)(s * rps + q) * TM * TN + mt * TN + j) * 4096);
            const f4 x = f4{v.x, v.y, v.z, v.w};
            S[mt][j] = q == 0 ? x : S[mt][j] + x;
          }
#pragma unroll
      for (int mt = 0; mt < TM; ++mt)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[mt][j] += S[mt][j];
    }
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int j = 0; j < TN; ++j) S[mt][j] = acc[mt][j];
  } else if (p.KS > 1) {
#pragma unroll
    for (int mt = 0; mt < TM; ++mt)
#pragma unroll
      for (int j = 0; j < TN; ++j) S[mt][j] = *gmem(T + (mt * TN + j) * 256) + S[mt][j];
  }

  lds_sync();   // the stages are no longer read (F reuses the LDS); s_scale written
  float* F = reinterpret_cast<float*>(smem);
  constexpr int FS = wide_fstride<TN>(), FR = wide_frows<TM>();
  static_assert(TM * 16 % FR == 0, "whole chunks of rows");
  const int R0 = mt0 * 16, R1 = min(M, (mt0 + TM) * 16);
#pragma unroll
  for (int c = 0; c < TM * 16; c += FR) {
    if (R0 + c >= R1) break;
    if (c) lds_sync();   // the chunk before has been read
    wide_epilogue<TN, FR, EPI>(p, F, cb * kWaves * NP, R0 + c, min(R1, R0 + c + FR), [&] {
#pragma unroll
      for (int mt = c / 16; mt < (c + FR) / 16; ++mt)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int row = mt * 16 + (lane >> 4) * 4 + i;
          const float sc = AM == A_NORM ? s_scale[row] : 1.0f;
#pragma unroll
          for (int j = 0; j < TN; ++j)
            F[(row - c) * FS + (wave * TN + j) * 16 + (lane & 15)] = AM == A_NORM ? S[mt][j][i] * sc : S[mt][j][i];
        }
    });
  }
}

}  // namespace as2d
