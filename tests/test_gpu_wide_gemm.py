"""The wide GEMM path (prefill passes of more than 32 rows) gives the bits of
the one-row path: a reply is decoded one token at a time, then its prefix is
prefilled afresh, each time in one pass, at lengths around the tiles' edges;
every key and value and the next token must be the same.  (Several passes:
test_gpu_prefill_passes.py.)"""
from dataclasses import replace

import numpy as np
import pytest

from tests.harness import make_pair, prefix
from workload import QWEN3B, QWEN7B, QWEN05B, TINY_BF16

pytestmark = pytest.mark.gpu

# 16-row tiles 3 and up, tile heights of 2, 3 and 4 row tiles and one row more,
# and passes of many row blocks, whole (2,048 rows) and ragged
LENGTHS = (33, 48, 49, 64, 65, 97, 128, 129, 193, 290, 511, 782, 1297, 2048, 2060)


@pytest.mark.parametrize("shape", [TINY_BF16, QWEN05B, QWEN3B, QWEN7B], ids=lambda s: s.name)
def test_fresh_prefill_equals_one_row_decoding(shape):
    shape = replace(shape.with_layers(2), vocab=4096)
    n_audio, n_instr, total = 24, 8, max(LENGTHS)
    _, gpu = make_pair(shape, seed=5, max_requests=2, max_kv_len=total + 8, max_k=4, oracle=False)
    try:
        _, audio, instr = prefix(shape, n_audio, n_instr, 5, 0)
        first, n = gpu.prefill(0, audio, instr)
        tokens = list(instr) + [first]
        while n < total:
            r = gpu.decode_one(0)
            n = r["kv_len"]
            tokens.append(r["correction_token"])
        kv = [gpu.read_kv(0, layer, total) for layer in range(shape.n_layers)]
        for length in LENGTHS:
            print(f"{shape.name}: prefill of {length} rows", flush=True)
            nxt, got = gpu.prefill(1, audio, np.array(tokens[:length - n_audio], dtype=np.int32))
            assert got == length and nxt == tokens[length - n_audio]
            for layer in range(shape.n_layers):
                k, v = gpu.read_kv(1, layer, length)
                assert np.array_equal(k, kv[layer][0][:, :length]), f"layer {layer} keys at {length} rows"
                assert np.array_equal(v, kv[layer][1][:, :length]), f"layer {layer} values at {length} rows"
    finally:
        gpu.close()
