"""Prefill of a float32 model through the staged GEMMs gives the same bits
whatever the row grouping (float32 models keep the staged path above 32
rows; bf16 models take the wide tiles): groups of 3 row tiles, groups of 2
for gate/up, the default, and single tiles everywhere.  0.5B widths in
float32, two layers, 290 rows (passes of 112, 112 and 66 rows: seven tiles,
so that the last group of three holds one, and a ragged five)."""
from dataclasses import replace

import numpy as np
import pytest

from tests.harness import ensure_built, prefix
from workload import QWEN05B, gen
from workload.configs import F32

pytestmark = pytest.mark.gpu

SHAPE = replace(QWEN05B.with_layers(2), name="0.5b-widths-f32", dtype=F32, vocab=4096)


@pytest.fixture(scope="module")
def weights():
    ensure_built()
    return gen.make_weights(SHAPE, 0, fmt="device")


def run(weights, rg_grid, monkeypatch):
    from paper_2609_37617_amd import as2d
    monkeypatch.setenv("AS2D_RG_GRID", str(rg_grid))   # read when the model is created
    m = as2d.Model(SHAPE, weights, max_requests=1, max_kv_len=512, max_k=8)
    try:
        m.set_keep_logits(True)
        _, a_dev, instr = prefix(SHAPE, 274, 16)
        first, L = m.prefill(0, a_dev, instr)
        kv = [m.read_kv(0, layer, L) for layer in range(SHAPE.n_layers)]
        out = m.decode_one(0)
        return first, L, kv, out, m.logits(0, 1).copy()
    finally:
        m.close()


@pytest.fixture(scope="module")
def single_tiles(weights):
    with pytest.MonkeyPatch.context() as mp:
        return run(weights, 100000, mp)


@pytest.mark.parametrize("rg_grid", [0, 250, 700])
def test_float32_prefill_bits_independent_of_row_groups(weights, single_tiles, rg_grid, monkeypatch):
    print(f"row-group grid threshold {rg_grid}", flush=True)
    first, L, kv, out, lg = run(weights, rg_grid, monkeypatch)
    assert (first, L) == single_tiles[:2]
    for layer in range(SHAPE.n_layers):
        assert np.array_equal(kv[layer][0], single_tiles[2][layer][0]), layer
        assert np.array_equal(kv[layer][1], single_tiles[2][layer][1]), layer
    assert out == single_tiles[3]
    assert np.array_equal(lg, single_tiles[4])
