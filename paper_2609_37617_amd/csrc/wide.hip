// Wide GEMMs of bf16 models (wide.h): kernels, the choice of tile and units
// for a pass, and the launcher.
#include "wide.h"

namespace as2d {

// Rows of a column block that run together: row blocks are numbered in
// groups of kWideGroup, and within a group by column block first, so that
// the workgroups that share an XCD at a time (they take consecutive
// numbers) read few column blocks' weights and few row blocks' activations.
constexpr int kWideGroup = 8;

template <int TM, int TN, int AH, int OCC, int AM, int EPI>
__global__ __launch_bounds__(256, OCC) void gemm_wide_kernel(const GemmArgs p) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float s_scale[TM * 16];
  __shared__ int s_flag;
  const int v = xcd_contiguous(blockIdx.x, gridDim.x), tiles = p.RB * p.CB;
  const int unit = v / tiles, t = v - unit * tiles;
  const int per = kWideGroup * p.CB, grp = t / per, r = t - grp * per;
  const int h = min(kWideGroup, p.RB - grp * kWideGroup);
  const int cb = r / h, rb = grp * kWideGroup + r - cb * h;
  gemm_wide_tile<TM, TN, AH, AM, EPI>(p, rb, cb, unit, smem, s_scale, &s_flag);
}

// Tiles (TM x TN sixteens per wave, AH k-steps of weights ahead, OCC
// workgroups per compute unit) and their times in microseconds, fitted to a
// sweep of the 7B, 3B and 0.5B shapes' matrices at 48 to 1,904 rows (960
// timings; the choice by this estimate is on average 1 % slower than the
// best of the sweep, at most 19 %): `lat` per k-step of a workgroup that
// waits for its own loads, `thr` per k-step and `fix` per unit of a compute
// unit's throughput.
struct WideTile {
  int tm, tn, occ;
  float lat, thr, fix;
};
constexpr WideTile kWideTiles[] = {
    {4, 4, 2, 0.594f, 0.373f, 6.4f},
    {3, 4, 2, 0.520f, 0.336f, 5.1f},
    {2, 4, 2, 0.335f, 0.303f, 2.0f},
    {2, 2, 4, 0.179f, 0.152f, 1.3f},
};
constexpr float kWideStart = 5.3f;     // launch to the first products, and the epilogue
constexpr float kWideRecord = 2e-6f;   // per float of the records of split tiles

struct WidePlan {
  int tile = -1, RB = 0, CB = 0, spu = 0, grid = 0;
};

// The tile and the slices per unit for a pass of a.M rows: the least
// estimated time over the tiles and, for each, whole tiles, splits and
// slices as units (smaller units fill the device when a narrow matrix has
// few tiles, and cost their records).  A tile's units run in rounds of
// 256 x occ workgroups.
static WidePlan wide_plan(const GemmArgs& a) {
  constexpr int kCUs = 256;
  WidePlan best;
  float best_us = 0.f;
  const int n_slices = a.KS * a.ns, last = a.KT - (a.KS - 1) * a.ktps;
  for (int i = 0; i < (int)(sizeof kWideTiles / sizeof kWideTiles[0]); ++i) {
    const WideTile& t = kWideTiles[i];
    if ((a.N / 16) % (kWaves * t.tn)) continue;
    const int RB = (a.MT + t.tm - 1) / t.tm, CB = a.N / (16 * kWaves * t.tn);
    const long long tile_floats = (long long)t.tm * t.tn * 1024;   // of one tile's sums
    for (const int spu : {n_slices, a.ns, 1}) {
      if (spu == 1 && (a.ktps < a.ns || last < a.ns)) continue;   // empty slices
      const int U = n_slices / spu;
      const long long rec = U > 1 ? (long long)RB * CB * U * tile_floats : 0;
      const long long scratch = U > 1 ? rec : a.KS > 1 ? (long long)RB * CB * tile_floats : 0;
      if (scratch * 4 > a.part_bytes || (U > 1 && RB * CB > a.n_counters)) continue;
      const long long wgs = (long long)RB * CB * U;
      if (wgs > 0x7fffffff) continue;
      const float ks = (float)a.KT / U, full = (float)wgs / kCUs;
      const long long slots = (long long)kCUs * t.occ;
      const float lat = (float)((wgs + slots - 1) / slots) * (ks * t.lat + kWideStart);
      const float thr = (full < 4.f ? ceilf(full) : full + 0.5f) * (ks * t.thr + t.fix);
      const float us = fmaxf(lat, thr) + kWideRecord * (float)rec;
      if (best.tile < 0 || us < best_us) {
        best_us = us;
        best = WidePlan{i, RB, CB, spu, (int)wgs};
      }
    }
  }
  return best;
}

template <int TM, int TN, int AH, int OCC, int AM, int EPI>
static hipError_t launch_tile(const GemmArgs& a, int grid, hipStream_t s) {
  gemm_wide_kernel<TM, TN, AH, OCC, AM, EPI><<<grid, 256, wide_lds_bytes<TM, TN>(), s>>>(a);
  return hipGetLastError();
}

template <int AM, int EPI>
static hipError_t launch_epi(GemmArgs a, hipStream_t s) {
  if (a.MT < 1 || a.ns != kWaves || a.N % 128) return hipErrorInvalidValue;
  const WidePlan w = wide_plan(a);
  a.RB = w.RB;
  a.CB = w.CB;
  a.spu = w.spu;
  switch (w.tile) {
    case 0: return launch_tile<4, 4, 2, 2, AM, EPI>(a, w.grid, s);
    case 1: return launch_tile<3, 4, 2, 2, AM, EPI>(a, w.grid, s);
    case 2: return launch_tile<2, 4, 4, 2, AM, EPI>(a, w.grid, s);
    case 3: return launch_tile<2, 2, 4, 4, AM, EPI>(a, w.grid, s);
    default: return hipErrorInvalidValue;   // the split sums' scratch is too small
  }
}

hipError_t launch_wide(int amode, int epi, const GemmArgs& a, hipStream_t s) {
#define AS2D_W(am, ep) \
  if (amode == am && epi == ep) return launch_epi<am, ep>(a, s);
  AS2D_W(A_NORM, EPI_QKV) AS2D_W(A_PLAIN, EPI_RESID) AS2D_W(A_NORM, EPI_SWIGLU)
  AS2D_W(A_NORM, EPI_ARGMAX) AS2D_W(A_PLAIN, EPI_DOWN)
#undef AS2D_W
  return hipErrorInvalidValue;
}

size_t wide_scratch_floats(int N, int rows) { return (size_t)((rows + 15) / 16 + 3) * 16 * N; }

template <int AM, int EPI>
static hipError_t prepare_epi() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_wide_kernel<4, 4, 2, 2, AM, EPI>),
                             hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds_bytes<4, 4>());
}

hipError_t prepare_wide() {
  hipError_t e = prepare_epi<A_NORM, EPI_QKV>();
  if (e == hipSuccess) e = prepare_epi<A_PLAIN, EPI_RESID>();
  if (e == hipSuccess) e = prepare_epi<A_NORM, EPI_SWIGLU>();
  if (e == hipSuccess) e = prepare_epi<A_NORM, EPI_ARGMAX>();
  if (e == hipSuccess) e = prepare_epi<A_PLAIN, EPI_DOWN>();
  return e;
}

}  // namespace as2d
