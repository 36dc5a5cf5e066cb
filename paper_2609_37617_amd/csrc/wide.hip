// Wide GEMMs of bf16 models (wide.h): kernels and launcher.  The tile and
// units of a pass are chosen by wide_plan (plan.h).
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

template <int TM, int TN, int AH, int OCC, int AM, int EPI>
static hipError_t launch_tile(const GemmArgs& a, int grid, hipStream_t s) {
  gemm_wide_kernel<TM, TN, AH, OCC, AM, EPI><<<grid, 256, wide_lds_bytes<TM, TN>(), s>>>(a);
  return hipGetLastError();
}

template <int AM, int EPI>
static hipError_t launch_epi(GemmArgs a, hipStream_t s) {
  if (a.MT < 1 || a.ns != kWaves || a.N % 128) return hipErrorInvalidValue;
  const WidePlan w = wide_plan(WideMatrix{a.N, a.KT, a.KS, a.ktps, a.ns}, a.MT, a.part_bytes, a.n_counters);
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
