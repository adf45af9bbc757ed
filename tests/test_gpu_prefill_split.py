"""Prefill chunks with few work items behind long prefixes: their keys are
shared by several blocks and combined. Chunk starts on both sides of a stage
and part boundary, one part next to many in a step, several group sizes, and
decodes in the same step."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2606_18600_amd import synth
from tests.gpu_pair import Pair, gpu_kv_to_oracle_layout, log
from tests.helpers import rel_l2, strong_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nq,nkv,d,chunks,decodes", [
    (8, 1, 128, [(1, 4000)], 0),
    (8, 1, 128, [(17, 1023), (3, 0), (40, 2048)], 0),     # starts next to a part boundary
    (8, 1, 128, [(33, 1025), (16, 63), (16, 64), (16, 4097)], 3),
    (4, 4, 64, [(150, 1500), (129, 900)], 0),             # group 1: items of 128 positions
    (16, 1, 64, [(20, 3000), (1, 767), (1, 768), (1, 769)], 2),
    (8, 2, 128, [(64, 6000)], 0),
])
def test_chunks_behind_prefixes(nq, nkv, d, chunks, decodes):
    """One layer against the exact oracle over a random cache: 1e-2 on the
    branch, as elsewhere for one layer in bf16."""
    shape = synth.ModelShape("s", hidden=256, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=128,
                             rms_eps=1e-5, rope_theta=1e4)
    seed = nq + d + len(chunks)
    q = np.array([a for a, _ in chunks], np.int32)
    c = np.array([b for _, b in chunks], np.int32)
    dctx = np.arange(100, 100 + 700 * decodes, 700).astype(np.int32)
    ends = np.concatenate([c + q, dctx + 1])
    nblk = (ends + 15) // 16
    blocks = int(nblk.sum()) + 1
    pair = Pair(shape, "bf16", 1, blocks, 512, 16, seed, host_weights=[strong_weights(shape, seed, 0)])
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pair.gpu.kv_pool.normal_(0.0, 1.0, generator=g)
    pair.okv = gpu_kv_to_oracle_layout(pair.gpu.kv_view())
    bt = synth.make_block_tables(ends, int(nblk.max()), synth.BlockAllocator(blocks, seed))
    pbt, dbt = bt[:len(q)].copy(), bt[len(q):].copy()
    T = int(q.sum()) + decodes
    x = synth.hidden_states(seed, 1, T, shape.hidden)
    try:
        if decodes:
            y, yr, x = pair.mixed(q, c, pbt, dctx, dbt, x)
        else:
            y, yr, x = pair.prefill(q, c, pbt, x)
        rows = [rel_l2(a, b) for a, b in zip(y - x, yr - x)]
        log(f"g{nq // nkv} kv{nkv} d{d} {chunks}: worst row's branch {max(rows):.2e}")
        assert rel_l2(y - x, yr - x) <= 1e-2 and max(rows) <= 2e-2
    finally:
        pair.close()
