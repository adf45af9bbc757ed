"""Steps of 129 to 1024 rows at the shapes and row counts where the choice of
their GEMM kernels turns: products split over K (192-row and 256-row tiles,
the eight-wave kernel below 193 rows, exactly half a round of tiles), a
gate-up product split over K, and SwiGLU rows past the last whole tile."""

from __future__ import annotations

import numpy as np
import pytest

from paper_2606_18600_amd import synth
from tests.gpu_pair import Pair, log
from tests.helpers import rel_l2, strong_weights

pytestmark = pytest.mark.gpu


def _shape(name, hidden, nq, nkv, d, ffn):
    return synth.ModelShape(name, hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=ffn,
                            rms_eps=1e-5, rope_theta=1e4)


SPLIT = _shape("split", 2048, 8, 2, 128, 256)       # every product split, gate-up included
HALF = _shape("half-round", 8192, 2, 1, 64, 128)    # 128 tiles of 256 x 256 at 769..1024 rows
HALF_LONG = _shape("half-round-long-k", 8192, 2, 1, 64, 3584)  # ... and a K that is split there
LONG = _shape("long-k", 4352, 2, 1, 64, 8192)      # K ranges of 1024 and more, 136 blocks
WIDE = _shape("wide-ffn", 128, 2, 1, 64, 32768)     # 256 column tiles of gate-up


@pytest.mark.parametrize("shape,rows", [
    (SPLIT, 129), (SPLIT, 192), (SPLIT, 193), (SPLIT, 257), (SPLIT, 385), (SPLIT, 513),
    (HALF, 769), (HALF, 1024), (HALF_LONG, 769),
    (LONG, 129), (LONG, 160), (LONG, 161), (LONG, 192),
    (WIDE, 129), (WIDE, 176), (WIDE, 177), (WIDE, 257), (WIDE, 400), (WIDE, 432), (WIDE, 433),
], ids=lambda v: v.name if isinstance(v, synth.ModelShape) else str(v))
def test_rows_around_the_turns(shape, rows):
    """One layer against the exact oracle, 1e-2 on output, branch and cache
    as elsewhere for one layer in bf16."""
    _against_oracle(shape, rows, 1, 1e-2)


@pytest.mark.parametrize("shape,rows", [(HALF_LONG, 769), (SPLIT, 129), (HALF, 769)],
                         ids=["down-split-only", "all-split", "none-split"])
def test_second_layer(shape, rows):
    """Two layers: the planes that one layer's down product leaves are added
    once, whether or not the next layer's O product leaves planes too. Each
    layer rounds as one layer does, and its input carries the first one's
    error: twice the limit of one."""
    _against_oracle(shape, rows, 2, 2e-2)


def _against_oracle(shape, rows, layers, limit):
    seed = rows
    pair = Pair(shape, "bf16", layers, 80, 1024, 4, seed,
                host_weights=[strong_weights(shape, seed, l) for l in range(layers)])
    a = rows // 3
    lens = np.array([a, rows - a], np.int32)
    bt = synth.make_block_tables(lens, 64, synth.BlockAllocator(80, seed))
    try:
        y, yr, x = pair.prefill(lens, np.zeros(2, np.int32), bt,
                                synth.hidden_states(seed, 1, rows, shape.hidden))
        e, eb, ek = rel_l2(y, yr), rel_l2(y - x, yr - x), pair.kv_errors()
        last = rel_l2((y - x)[-1], (yr - x)[-1])
        log(f"{shape.name} rows={rows}: output {e:.2e} branch {eb:.2e} last row {last:.2e} kv {ek:.2e}")
        assert e <= limit and eb <= limit and last <= 2 * limit and ek <= limit
    finally:
        pair.close()
