"""Verification attention over long caches with a row tile per wave gives the
bits of the kernels whose four waves share a tile (AS2D_ATTN_RT=1), for
requests of one to many row tiles, alone and in ragged batches, with caches
that end inside, at and just past a 128-key span.

A pass takes a row tile per wave once its (span, KV head, row tile) items
outnumber the workgroups, two per compute unit: the requests of EDGES have as
many items as workgroups and one span more, and a budget of few compute units
takes every batch past the line."""
import os
from dataclasses import replace

import numpy as np
import pytest

from tests.harness import make_pair, prefix
from workload import QWEN7B, QWEN05B

pytestmark = pytest.mark.gpu

# (prefix, candidates) per request: caches of 1 to 18 spans in slots of 36
BATCHES = [[(300, 31)], [(2300, 2)], [(1151, 15)], [(120, 7), (2047, 31), (129, 0), (640, 8), (2200, 17)],
           [(100 + 37 * i, (0, 4, 8)[i % 3]) for i in range(12)]]


# one request of 17 rows by KV heads: 8 row tiles x KV heads x spans = 512, then one span more
EDGES = {4: [[(2031, 16)], [(2032, 16)]], 2: [[(4079, 16)], [(4080, 16)]]}


def run(shape, rt, batches=BATCHES, cus=0):
    old = os.environ.pop("AS2D_ATTN_RT", None)
    if rt:
        os.environ["AS2D_ATTN_RT"] = str(rt)
    try:
        _, gpu = make_pair(shape, seed=9, max_requests=12, max_kv_len=4608, max_k=31, oracle=False)
    finally:
        os.environ.pop("AS2D_ATTN_RT", None)
        if old is not None:
            os.environ["AS2D_ATTN_RT"] = old
    out = []
    try:
        gpu.set_keep_logits(True)
        gpu.set_cu_budget(cus)
        for b, batch in enumerate(batches):
            print(f"{shape.name}: AS2D_ATTN_RT={rt} budget {cus} batch {b}", flush=True)
            for r, (n, _) in enumerate(batch):
                _, audio, instr = prefix(shape, n - 8, 8, 9, r)
                gpu.prefill(r, audio, instr)
            rng = np.random.default_rng(b)
            cands = [[int(t) for t in rng.integers(0, shape.vocab, k)] for _, k in batch]
            res = gpu.verify_batch(list(range(len(batch))), cands)
            out.append((res, [gpu.logits(r) for r in range(len(batch))]))
    finally:
        gpu.close()
    return out


@pytest.mark.parametrize("shape", [QWEN7B, QWEN05B], ids=lambda s: s.name)
def test_tile_per_wave_equals_shared_tile(shape):
    shape = replace(shape.with_layers(2), vocab=4096)
    same(run(shape, 0), run(shape, 1))


@pytest.mark.parametrize("shape", [QWEN7B, QWEN05B], ids=lambda s: s.name)
def test_both_sides_of_the_rule(shape):
    shape = replace(shape.with_layers(2), vocab=4096)
    edges = EDGES[shape.n_kv_heads]
    for (n, k), items in zip((b[0] for b in edges), (512, 512 + 8 * shape.n_kv_heads)):
        tiles = -(-(shape.n_q_heads // shape.n_kv_heads * (k + 1)) // 16)
        assert shape.n_kv_heads * tiles * -(-(n + k + 1) // 128) == items
    same(run(shape, 0, edges), run(shape, 1, edges))


@pytest.mark.parametrize("shape", [QWEN7B, QWEN05B], ids=lambda s: s.name)
def test_tile_per_wave_on_few_compute_units(shape):
    shape = replace(shape.with_layers(2), vocab=4096)
    same(run(shape, 0, cus=16), run(shape, 1))


def same(a, b):
    for i, ((ra, la), (rb, lb)) in enumerate(zip(a, b)):
        assert ra == rb, f"batch {i}"
        for r, (x, y) in enumerate(zip(la, lb)):
            assert np.array_equal(x, y), f"batch {i} request {r}"
