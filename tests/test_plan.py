"""The host's rules for pass sizes and wide GEMM units (csrc/plan.h), run
without a device: a small C++ shim built with the host compiler exports them.

Wide GEMM units write their sums as records that the kernel reaches by 32-bit
byte offsets below 2^31: no plan may need more, whatever the scratch."""
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
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2609_37617_amd", "csrc"), str(d / "shim.cpp"), "-o", str(d / "shim.so")],
                   check=True)
    return ctypes.CDLL(str(d / "shim.so"))


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
