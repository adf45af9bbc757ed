"""Steps of at most 128 rows at the shapes and row counts where the choice of
their GEMM kernel turns: half and whole weight groups with K split inside the
block (up to 32 rows), and SwiGLU on two groups to a block."""

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


SHAPES = [
    _shape("halves-odd-k", 256, 4, 2, 64, 704),       # every product in half groups; K = 704
    _shape("o-whole-groups", 8192, 4, 2, 128, 64),    # O: 128 groups, two K ranges of 256
    _shape("gate-up-130-groups", 256, 2, 1, 128, 4160),   # SwiGLU on whole groups
    _shape("gate-up-258-groups", 384, 2, 1, 128, 8256),   # SwiGLU, two groups to a block
    _shape("gate-up-514-groups", 128, 2, 1, 64, 16448),   # SwiGLU, four groups to a block
]


@pytest.mark.parametrize("rows", [1, 16, 17, 32, 33, 65, 128])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: s.name)
def test_rows_around_the_turns(shape, rows):
    """One layer against the exact oracle. bf16 storage (inputs of the four
    products, K, V, P) rounds by 2^-9 at about six points of a layer with
    O(1) branches: 1e-2 on the branch is twice what that gives."""
    seed = rows
    pair = Pair(shape, "bf16", 1, 16, 128, 4, seed, host_weights=[strong_weights(shape, seed, 0)])
    lens = np.array([rows], np.int32)
    bt = synth.make_block_tables(lens, 8, synth.BlockAllocator(16, seed))
    try:
        y, yr, x = pair.prefill(lens, np.zeros(1, np.int32), bt,
                                synth.hidden_states(seed, 1, rows, shape.hidden))
        e, eb, ek = rel_l2(y, yr), rel_l2(y - x, yr - x), pair.kv_errors()
        log(f"{shape.name} rows={rows}: output {e:.2e} branch {eb:.2e} kv {ek:.2e}")
        assert e <= 1e-2 and eb <= 1e-2 and ek <= 1e-2
    finally:
        pair.close()
