"""Verification attention over long caches with a row tile per wave gives the
bits of the kernels whose four waves share a tile (AS2D_ATTN_RT=1), for
requests of one to many row tiles, alone and in ragged batches, with caches
that end inside, at and just past a 128-key span."""
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


def run(shape, rt):
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
        for b, batch in enumerate(BATCHES):
            print(f"{shape.name}: AS2D_ATTN_RT={rt} batch {b}", flush=True)
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
    for b, ((ra, la), (rb, lb)) in enumerate(zip(run(shape, 0), run(shape, 1))):
        assert ra == rb, f"batch {b}"
        for r, (x, y) in enumerate(zip(la, lb)):
            assert np.array_equal(x, y), f"batch {b} request {r}"
