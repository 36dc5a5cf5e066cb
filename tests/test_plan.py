"""The host's rules for pass sizes and wide GEMM units (csrc/plan.h), run
without a device: a small C++ shim built with the host compiler exports them.

Wide GEMM units write their sums as records that the kernel reaches by 32-bit
byte offsets below 2^31: no plan may need more, whatever the scratch.  The
scratch a context reserves is what the chosen plans write, and no plan changes
for it; where the memory is short, passes get smaller instead of the load
failing."""
import ctypes
import os
import random
import subprocess

import pytest

from workload import QWEN3B, QWEN7B, QWEN05B, TINY_BF16

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r"""
#include "plan.h"
using namespace as2d;
extern "C" void plan(const int* m, int MT, long long part_bytes, int n_counters, long long* out) {
  const WideMatrix w{m[0], m[1], m[2], m[3], m[4]};
  const WidePlan p = wide_plan(w, MT, part_bytes, n_counters);
  out[0] = p.tile < 0 ? 0 : kWideTiles[p.tile].tm;
  out[1] = p.tile < 0 ? 0 : kWideTiles[p.tile].tn;
  out[2] = p.RB; out[3] = p.CB; out[4] = p.spu; out[5] = p.grid; out[6] = p.scratch;
}
extern "C" long long part_bytes(const int* m, int n, int n_counters) {   // n matrices: a WideMatrix and its rows
  PassMatrix a[8];
  for (int i = 0; i < n; ++i, m += 6) a[i] = PassMatrix{WideMatrix{m[0], m[1], m[2], m[3], m[4]}, m[5]};
  return pass_part_bytes(a, n, n_counters);
}
extern "C" int rows_per_pass(int total, int most, int bf16) { return pass_rows(total, most, bf16); }
extern "C" int fit(int rows, int least, int most, int* tried) {
  int n = 0;
  const int r = rows_that_fit(rows, least, [&](int x) { tried[n++] = x; return x <= most; });
  tried[n] = 0;
  return r;
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2609_37617_amd", "csrc"), str(d / "shim.cpp"), "-o", str(d / "shim.so")],
                   check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.part_bytes.restype = ctypes.c_longlong
    return lib


def wide(lib, matrix, MT, part_bytes, n_counters):
    out = (ctypes.c_longlong * 7)()
    lib.plan((ctypes.c_int * 5)(*matrix), MT, ctypes.c_longlong(part_bytes), n_counters, out)
    return dict(zip(("tm", "tn", "RB", "CB", "spu", "grid", "scratch"), out))


def matrix(N, K, KS):
    KT = K // 32
    return N, KT, KS, (KT + KS - 1) // KS, 4


def check(p, m, MT):
    """A plan covers the matrix, and its records are addressable."""
    N, KT, KS, _, ns = m
    U = KS * ns // p["spu"]
    assert p["RB"] * p["tm"] >= MT and p["CB"] * p["tn"] * 64 == N
    assert p["grid"] == p["RB"] * p["CB"] * U
    per_tile = p["tm"] * p["tn"] * 1024 * 4
    assert p["scratch"] == p["RB"] * p["CB"] * per_tile * (U if U > 1 else int(KS > 1))
    if U > 1:
        assert p["RB"] * p["CB"] * U * per_tile <= 0x7fffffff


# columns, inner dimension, splits: narrow matrices whose tiles need splitting at few rows,
# and wide ones whose records would pass 2 GiB at many (the longer the inner
# dimension, the more the estimate prefers small units)
@pytest.mark.parametrize("N,K,KS", [(256, 8192, 16), (4096, 8192, 16), (16384, 32768, 16), (65536, 65536, 16),
                                    (131072, 8192, 1), (131072, 1 << 20, 16), (65536, 1 << 21, 16)])
def test_records_stay_below_2_gib(lib, N, K, KS):
    m = matrix(N, K, KS)
    split = 0
    for MT in list(range(1, 20)) + [64, 128, 250, 512]:
        p = wide(lib, m, MT, 1 << 40, 1 << 30)
        check(p, m, MT)
        split += p["spu"] < KS * 4
    if N <= 16384:
        assert split   # the rule still splits where it pays


def test_plans_of_the_models(lib):
    rng = random.Random(1)
    for s in (TINY_BF16, QWEN05B, QWEN3B, QWEN7B):
        for N, K in ((s.qkv_out, s.hidden), (s.hidden, s.n_q_heads * s.head_dim), (2 * s.ffn, s.hidden),
                     (s.hidden, s.ffn), (s.vocab, s.hidden)):
            for KS in (1, 2, 4, 5):
                for MT in [3, 4, 5, 9] + [rng.randint(3, 512) for _ in range(8)]:
                    m = matrix(N, K, KS)
                    check(wide(lib, m, MT, 128 << 20 if KS == 1 else 1 << 33, N * 17), m, MT)


def matrices(s, splits, rows):
    """The five matrices of a model with the given k-splits; the head's passes have up to 144 rows."""
    dims = ((s.qkv_out, s.hidden), (s.hidden, s.n_q_heads * s.head_dim), (2 * s.ffn, s.hidden),
            (s.hidden, s.ffn), (s.vocab, s.hidden))
    return [matrix(N, K, KS) + (rows if i < 4 else 144,) for i, ((N, K), KS) in enumerate(zip(dims, splits))]


@pytest.mark.parametrize("shape,splits", [(TINY_BF16, (1, 1, 1, 1, 1)), (QWEN05B, (1, 1, 1, 5, 1)),
                                          (QWEN3B, (1, 1, 1, 4, 1)), (QWEN7B, (1, 1, 1, 2, 1)), (QWEN7B, (3, 2, 1, 2, 4))],
                         ids=lambda v: getattr(v, "name", str(v)))
@pytest.mark.parametrize("rows", [144, 800, 8192])
def test_split_scratch_is_what_the_plans_write(lib, shape, splits, rows):
    ms = matrices(shape, splits, rows)
    n_counters = max(N // 128 * max(9, (rows + 31) // 32) for N, *_ in ms)
    flat = [v for m in ms for v in m]
    part = lib.part_bytes((ctypes.c_int * len(flat))(*flat), len(ms), n_counters)
    limit = max([128 << 20] + [((m[5] + 15) // 16 + 3) * 64 * m[0] for m in ms if m[2] > 1])
    used = max([m[2] * 32 * m[0] * 4 for m in ms if m[2] > 1], default=0)
    for m in ms:
        for MT in range(3, (m[5] + 15) // 16 + 1):
            p = wide(lib, m[:5], MT, limit, n_counters)
            assert p == wide(lib, m[:5], MT, part, n_counters)   # the same plan within what is reserved
            used = max(used, p["scratch"])
    assert part == used <= limit


def test_passes_shrink_to_the_memory(lib):
    def fit(rows, least, most):
        tried = (ctypes.c_int * 32)()
        r = lib.fit(rows, least, most, tried)
        return r, list(tried)[:list(tried).index(0)]
    assert fit(8192, 144, 8192) == (8192, [8192])
    assert fit(8192, 144, 3000) == (2048, [8192, 4096, 2048])
    assert fit(8192, 144, 150) == (144, [8192, 4096, 2048, 1024, 512, 256, 144])
    assert fit(1040, 144, 300) == (272, [1040, 528, 272])
    assert fit(144, 144, 143) == (0, [144])
    assert fit(8192, 144, 100)[0] == 0


@pytest.mark.parametrize("bf16,mosts", [(0, (144, 48, 16)), (1, (8192, 2048, 144, 16))])
def test_passes_of_a_prefill(lib, bf16, mosts):
    """Whole row tiles of at most `most` rows, as few passes as it allows, and
    none without rows."""
    for most in mosts:
        for total in list(range(1, 700)) + [2047, 2048, 2049, 8191, 8192, 8193, 16032, 32767, 32768]:
            rows = lib.rows_per_pass(total, most, bf16)
            assert 0 < rows <= most and rows % 16 == 0
            assert -(-total // rows) == -(-total // most), (total, most)


def test_float32_passes_leave_a_few_rows_to_the_direct_path(lib):
    # a remainder of up to 32 rows stays the last pass (145 rows: 144 and 1, not 80 and 65)
    assert [lib.rows_per_pass(n, 144, 0) for n in (144, 145, 176, 177, 289, 320, 321, 433)] == [144, 144, 144, 96, 144, 144, 112, 144]
    assert [lib.rows_per_pass(n, 8192, 1) for n in (145, 8192, 8193, 8413)] == [160, 8192, 4112, 4208]
