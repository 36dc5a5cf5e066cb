// Sizes and splits chosen on the host, from shapes alone: tile and units of a
// wide GEMM (wide.h) and the scratch they need.  Plain C++ (no HIP), so that
// the rules can be run without a device.
#pragma once
#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace as2d {

constexpr int kWaves = 4;               // waves per workgroup
constexpr int kPairCols = 32;           // columns of a tile pair
constexpr int kMaxMTiles = 9;           // up to 144 rows per verification pass (and float32 prefill pass)
constexpr int kMaxRows = kMaxMTiles * 16;
constexpr int kPrefillRows = 8192;      // rows per prefill pass of bf16 models, at most
constexpr int kDirectMT = 2;            // row tiles of the direct path (up to 32 rows)
constexpr long long kWideSplitBytes = 128ll << 20;   // records the wide path may split tiles into, whatever the model

// ---------------------------------------------------------------------------
// Wide GEMMs

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
// Bytes of records a launch can address: the kernel reaches them by 32-bit
// offsets through a buffer descriptor of this range (coherent_rsrc), which
// drops stores past its end.
constexpr long long kWideMaxRecords = 0x7fffffff;

struct WideMatrix {
  int N, KT, KS, ktps, ns;   // columns, k-steps, splits, k-steps per split, slices per split
};
struct WidePlan {
  int tile = -1, RB = 0, CB = 0, spu = 0, grid = 0;
  long long scratch = 0;   // bytes of records, or of the sums kept by whole tiles of a matrix with k-splits
};

// Bytes that whole tiles of an N-column matrix with k-splits keep their sums
// in, for passes of up to `rows` rows.
inline size_t wide_scratch(int N, int rows) { return (size_t)((rows + 15) / 16 + 3) * 16 * N * 4; }

// The tile and the slices per unit for a pass of MT row tiles: the least
// estimated time over the tiles and, for each, whole tiles, splits and
// slices as units (smaller units fill the device when a narrow matrix has
// few tiles, and cost their records).  A tile's units run in rounds of
// 256 x occ workgroups.  part_bytes and n_counters bound the units a tile can
// be split into.
inline WidePlan wide_plan(const WideMatrix& a, int MT, long long part_bytes, int n_counters) {
  constexpr int kCUs = 256;
  WidePlan best;
  float best_us = 0.f;
  const int n_slices = a.KS * a.ns, last = a.KT - (a.KS - 1) * a.ktps;
  for (int i = 0; i < (int)(sizeof kWideTiles / sizeof kWideTiles[0]); ++i) {
    const WideTile& t = kWideTiles[i];
    if ((a.N / 16) % (kWaves * t.tn)) continue;
    const int RB = (MT + t.tm - 1) / t.tm, CB = a.N / (16 * kWaves * t.tn);
    const long long tile_floats = (long long)t.tm * t.tn * 1024;   // of one tile's sums
    for (const int spu : {n_slices, a.ns, 1}) {
      if (spu == 1 && (a.ktps < a.ns || last < a.ns)) continue;   // empty slices
      const int U = n_slices / spu;
      const long long rec = U > 1 ? (long long)RB * CB * U * tile_floats : 0;
      const long long scratch = U > 1 ? rec : a.KS > 1 ? (long long)RB * CB * tile_floats : 0;
      if (scratch * 4 > part_bytes || rec * 4 > kWideMaxRecords || (U > 1 && RB * CB > n_counters)) continue;
      const long long wgs = (long long)RB * CB * U;
      if (wgs > 0x7fffffff) continue;
      const float ks = (float)a.KT / U, full = (float)wgs / kCUs;
      const long long slots = (long long)kCUs * t.occ;
      const float lat = (float)((wgs + slots - 1) / slots) * (ks * t.lat + kWideStart);
      const float thr = (full < 4.f ? std::ceil(full) : full + 0.5f) * (ks * t.thr + t.fix);
      const float us = std::fmax(lat, thr) + kWideRecord * (float)rec;
      if (best.tile < 0 || us < best_us) {
        best_us = us;
        best = WidePlan{i, RB, CB, spu, (int)wgs, scratch * 4};
      }
    }
  }
  return best;
}

// ---------------------------------------------------------------------------
// Pass buffers

// A matrix and the rows of the passes that read it, at most.
struct PassMatrix {
  WideMatrix w;
  int rows;
};

// Bytes of split sums that the passes of a bf16 model need: what the direct
// path's k-splits and the wide path's chosen plans write.  The plans are
// chosen within kWideSplitBytes, or what whole tiles take if that is more;
// a launch that is given the result as its bound chooses the same ones.
inline long long pass_part_bytes(const PassMatrix* m, int n, int n_counters) {
  long long limit = kWideSplitBytes, need = 0;
  for (int i = 0; i < n; ++i)
    if (m[i].w.KS > 1) {
      need = std::max(need, (long long)m[i].w.KS * kDirectMT * 16 * m[i].w.N * 4);
      limit = std::max(limit, (long long)wide_scratch(m[i].w.N, m[i].rows));
    }
  for (int i = 0; i < n; ++i)
    for (int MT = kDirectMT + 1; MT <= (m[i].rows + 15) / 16; ++MT)
      need = std::max(need, wide_plan(m[i].w, MT, limit, n_counters).scratch);
  return need;
}

// Rows of each pass but the last of a prefill of `total` rows in passes of up
// to `most` (whole row tiles): passes of about the same size, but full ones
// where float32 models then leave the last pass to the direct path.  Equal
// passes against full ones, 0.5B widths in float32 (3 layers): 145, 161, 290,
// 320, 433 rows 774, 820, 1,338, 1,415, 1,916 / 676, 726, 1,189, 1,275,
// 1,716 us (the tiny model the same way); 177 rows, which leave 33 to the
// staged path, 857 / 1,035, 3B widths 225 and 512 rows (81 and 80 left) 1,397
// and 2,918 / 1,516 and 3,223.
inline int pass_rows(int total, int most, bool bf16) {
  const int left = total % most;
  if (!bf16 && total > most && left > 0 && left <= kDirectMT * 16) return most;
  const int passes = (total + most - 1) / most;
  return ((total + passes - 1) / passes + 15) / 16 * 16;
}

// Rows per pass for which fits(rows) holds: `rows`, or else half as many at a
// time (whole row tiles), down to `least`.  0: not even that.
template <class Fits> inline int rows_that_fit(int rows, int least, Fits&& fits) {
  for (;;) {
    if (fits(rows)) return rows;
    if (rows <= least) return 0;
    rows = std::max(least, (rows / 2 + 15) / 16 * 16);
  }
}

}  // namespace as2d
