"""Verification passes of two row tiles (17 to 32 rows) at the slice lengths
that keep activations in registers: 3B widths hold both tiles, 7B widths the
first and stream the second, the tiny shape has slices of two k-steps; the
edges of the second tile (one row, a middle, all sixteen).  The pass of
W = k + 1 rows has to give, row by row, the logits of W decoding steps of one
row each, bit for bit, and to accept all k candidates that those steps
committed; the appended keys and values are the same too."""
import numpy as np
import pytest

from tests.harness import make_pair, prefix
from workload import QWEN3B, QWEN7B, TINY_BF16

pytestmark = pytest.mark.gpu

SHAPES = {"7b": QWEN7B.with_layers(1), "3b": QWEN3B.with_layers(1), "tiny-bf16": TINY_BF16}
WIDTHS = (17, 25, 32)


@pytest.fixture(scope="module", params=sorted(SHAPES))
def sequential(request):
    """A model with one prefix in every slot, and max(WIDTHS) decoding steps
    of slot 0: (name, model, prefix length, tokens, logits by step, KV)."""
    shape, n_audio = SHAPES[request.param], 100
    _, gpu = make_pair(shape, max_requests=1 + len(WIDTHS), max_kv_len=256, max_k=31, oracle=False)
    gpu.set_keep_logits(True)
    _, a_dev, instr = prefix(shape, n_audio, 16)
    for slot in range(1 + len(WIDTHS)):
        gpu.prefill(slot, a_dev, instr)
    tokens, logits = [], []
    for _ in range(max(WIDTHS)):
        tokens.append(gpu.decode_one(0)["correction_token"])
        logits.append(gpu.logits(0, 1)[0].copy())
    L = n_audio + 16
    yield request.param, gpu, L, tokens, logits, gpu.read_kv(0, shape.n_layers - 1, L + max(WIDTHS))
    gpu.close()


@pytest.mark.parametrize("width", WIDTHS)
def test_rows_of_two_tiles_equal_single_rows(sequential, width):
    name, gpu, L, tokens, logits, kv = sequential
    print(f"{name}: {width} rows", flush=True)
    slot = 1 + WIDTHS.index(width)
    out = gpu.verify(slot, tokens[:width - 1])
    assert out["accepted_len"] == width - 1 and out["correction_token"] == tokens[width - 1]
    got = gpu.logits(slot, width)
    for r in range(width):
        assert np.array_equal(got[r], logits[r]), r
    mine = gpu.read_kv(slot, SHAPES[name].n_layers - 1, L + width)
    for a, b in zip(mine, kv):   # [KV head][position][dimension]
        assert np.array_equal(a, b[:, :L + width])
