"""A bf16 prefill in several passes gives the bits of one pass.

The rows of a pass are bounded by a load-time setting and by the device's
memory.  The same prefix is prefilled in one pass and in several (later passes
start inside the prefix: their rows attend to keys of the passes before; the
last one is ragged), and every key and value, the first token, the logits
after the prefix and a verification call must be the same.  Passes of 32 rows
and fewer take the direct GEMMs, longer ones the wide ones."""
from dataclasses import replace

import numpy as np
import pytest

from tests.harness import ensure_built, prefix
from workload import QWEN7B, QWEN05B, gen

pytestmark = pytest.mark.gpu

N_AUDIO, N_INSTR, CAP = 2200, 23, 2304   # 2,223 rows: 18 spans, the last row tile of 15 rows


def run(shape, weights, n_audio=N_AUDIO, cap=CAP, n_layers=2):
    from paper_2609_37617_amd import as2d
    m = as2d.Model(shape, weights, max_requests=1, max_kv_len=cap, max_k=4)
    try:
        m.set_keep_logits(True)
        _, audio, instr = prefix(shape, n_audio, N_INSTR, 3)
        first, n = m.prefill(0, audio, instr)
        lg = m.logits(0).copy()
        kv = [m.read_kv(0, layer, n) for layer in range(n_layers)]
        out = m.verify(0, [1, 2, 3])
        return first, n, lg, kv, out, m.logits(0).copy()
    finally:
        m.close()


def check_same(got, ref):
    assert got[:2] == ref[:2] and got[4] == ref[4]
    assert np.array_equal(got[2], ref[2]) and np.array_equal(got[5], ref[5])
    for layer, (a, b) in enumerate(zip(got[3], ref[3])):
        assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1]), f"layer {layer}"


@pytest.mark.parametrize("shape", [QWEN05B, QWEN7B], ids=lambda s: s.name)
def test_several_passes_equal_one(shape, monkeypatch):
    shape = replace(shape.with_layers(2), vocab=4096)
    ensure_built()
    weights = gen.make_weights(shape, 3, fmt="device")
    ref = run(shape, weights)
    # 2 passes of 1,120 and 1,103 rows; 3 of 752, 752, 719; 16 of 144 (the last of 63); 70 of 32 (the last of 15)
    for rows in (2208, 800, 144, 32):
        print(f"{shape.name}: passes of up to {rows} rows", flush=True)
        monkeypatch.setenv("AS2D_PREFILL_ROWS", str(rows))   # read when the model is created
        check_same(run(shape, weights), ref)


def test_two_passes_past_8192_rows(monkeypatch):
    """The split of the default setting: 8,413 rows are two passes of 4,208 and 4,205."""
    shape = replace(QWEN05B.with_layers(2), vocab=4096)
    ensure_built()
    weights = gen.make_weights(shape, 4, fmt="device")
    got = run(shape, weights, 8390, 8448)
    monkeypatch.setenv("AS2D_PREFILL_ROWS", "640")
    check_same(got, run(shape, weights, 8390, 8448))


def test_short_memory_shrinks_the_passes():
    """A context whose memory does not hold the buffers of its largest pass
    loads with smaller passes.  7B attention widths and a wide MLP, one layer:
    0.8 GB of weights (1.3 GB while they are packed) and 0.2 GB of other
    buffers, 1.7 GB for passes of 8,192 rows; 2 GB are left free."""
    import ctypes
    from paper_2609_37617_amd import as2d
    shape = replace(QWEN7B.with_layers(1), name="wide-mlp", ffn=32768, vocab=4096)
    ensure_built()
    weights = gen.make_weights(shape, 5, fmt="device")
    ref = run(shape, weights, 8000, 8192, 1)
    hip = as2d.load_library()   # its HIP runtime
    left, held = 2 * 10 ** 9, []
    free, total = ctypes.c_size_t(), ctypes.c_size_t()
    try:
        for _ in range(4):
            assert hip.hipMemGetInfo(ctypes.byref(free), ctypes.byref(total)) == 0
            if free.value - left > 64 << 20:
                p = ctypes.c_void_p()
                assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(free.value - left)) == 0
                held.append(p)
        print(f"{free.value / 1e9:.2f} of {total.value / 1e9:.2f} GB free", flush=True)
        got = run(shape, weights, 8000, 8192, 1)
    finally:
        for p in held:
            hip.hipFree(p)
    check_same(got, ref)
