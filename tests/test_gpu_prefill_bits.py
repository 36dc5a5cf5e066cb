"""A prefilled cache equals the incrementally built one bit for bit, with
prefixes of several spans.

Commit-and-repair (Appendix C.4): after verification rounds with rejections,
a fresh prefill of the committed prefix must reproduce the retained cache.
The second layer's keys and values depend on the first layer's attention
output, so they compare the two attention paths: verification stores every
span's state and merges them in order; a bf16 prefill (7B shape) walks all
spans chunk by chunk in one pass; a float32 prefill (3B and 0.5B widths, for
both head sizes) runs its spans two at a time, the second group of four waves
handing its span state to the first, in passes of at most 144 rows. Prefixes
of 256 and 300 rows (two and three spans) are extended by the verification
rounds and prefilled again, so the row tiles see even and odd span counts,
and one whose last span is the second group's span run again.
"""
from dataclasses import replace

import numpy as np
import pytest

from tests.harness import make_pair, prefix
from workload import QWEN3B, QWEN7B, QWEN05B
from workload.configs import F32

pytestmark = pytest.mark.gpu

SHAPES = [QWEN7B.with_layers(2)] + [replace(s.with_layers(2), name=s.name + "-f32", dtype=F32, vocab=4096)
                                    for s in (QWEN3B, QWEN05B)]


@pytest.mark.parametrize("SHAPE", SHAPES, ids=lambda s: s.name)
@pytest.mark.parametrize("n_audio,n_instr", [(240, 16), (284, 16)])
def test_prefill_equals_incremental_several_spans(SHAPE, n_audio, n_instr):
    print(f"{SHAPE.name}, prefix {n_audio} + {n_instr}", flush=True)
    _, gpu = make_pair(SHAPE, seed=11, max_requests=2, max_kv_len=1024, max_k=8, oracle=False)
    try:
        _, a_dev, instr = prefix(SHAPE, n_audio, n_instr, 11, 0)
        first, L = gpu.prefill(0, a_dev, instr)
        rng = np.random.default_rng(11)
        committed = [first]
        for _ in range(10):
            c = [int(t) for t in rng.integers(0, SHAPE.vocab, 3)]
            r = gpu.verify(0, c)
            committed += c[:r["accepted_len"]] + [r["correction_token"]]
        kv, root, _ = gpu.state(0)
        assert kv > L
        processed = np.array(list(instr) + committed[:-1], dtype=np.int32)
        first2, kv2 = gpu.prefill(1, a_dev, processed)
        assert kv2 == kv and first2 == root
        for layer in range(SHAPE.n_layers):
            k1, v1 = gpu.read_kv(0, layer, kv)
            k2, v2 = gpu.read_kv(1, layer, kv)
            assert np.array_equal(k1, k2) and np.array_equal(v1, v2), f"layer {layer}"
    finally:
        gpu.close()
