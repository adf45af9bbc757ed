"""Decode attention over key splits: tokens with one split (written by the
attention kernel itself) next to tokens with many, at batch sizes on both
sides of each choice of the merge kernel's waves per token, for several group
sizes; steps whose contexts are all too short to be split; and steps whose
tokens are each taken whole by the waves of one workgroup."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2606_18600_amd import synth
from tests.gpu_pair import Pair, gpu_kv_to_oracle_layout, log
from tests.helpers import rel_l2, strong_weights

pytestmark = pytest.mark.gpu


def _shape(nq, nkv, d):
    return synth.ModelShape(f"g{nq // nkv}-kv{nkv}-d{d}", hidden=256, n_q_heads=nq, n_kv_heads=nkv,
                            head_dim=d, ffn=128, rms_eps=1e-5, rope_theta=1e4)


@pytest.mark.parametrize("nq,nkv,d,seqs,longest", [
    (8, 1, 128, 3, 1500),    # 8 waves per token, up to 24 splits
    (8, 1, 128, 1, 6000),    # one token, 32 splits
    (8, 1, 128, 1, 8000),    # one token, 48 splits
    (16, 1, 128, 5, 900),    # group 16: 4 waves
    (4, 4, 64, 32, 1100),    # 128 (token, kv head) pairs: 8 waves
    (8, 4, 64, 33, 1100),    # 132: 4 waves
    (8, 2, 128, 128, 1100),  # 256: 4 waves
    (4, 4, 64, 129, 300),    # 516: 1 wave
    (2, 2, 128, 7, 127),     # at most 8 blocks: unsplit, one wave per token
    (4, 2, 64, 7, 128),      # 9 blocks: whole tokens, 8 waves each
    (8, 1, 128, 5, 511),     # 32 blocks: whole
    (8, 1, 128, 5, 512),     # 33 blocks on few pairs: split
    (8, 4, 64, 32, 1023),    # 64 blocks on 128 pairs: whole
    (16, 1, 128, 130, 200),  # group 16, whole
    (4, 4, 128, 128, 200),   # 512 pairs: whole
])
def test_decode_over_splits(nq, nkv, d, seqs, longest):
    """One layer against the exact oracle over a random cache. The decode
    path rounds its inputs, P and its output to bf16 (2^-9 each): 1e-2 on
    the branch, as elsewhere for one layer."""
    shape, seed = _shape(nq, nkv, d), nq + d + seqs
    r = np.random.default_rng(seed)
    ctx = r.integers(0, longest + 1, size=seqs).astype(np.int32)
    ctx[0], ctx[-1] = longest, longest if seqs == 1 else 0
    nblk = (ctx + 16) // 16
    blocks = int(nblk.sum()) + 1
    pair = Pair(shape, "bf16", 1, blocks, 256, max(seqs, 16), seed,
                host_weights=[strong_weights(shape, seed, 0)])
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    pair.gpu.kv_pool.normal_(0.0, 1.0, generator=g)
    pair.okv = gpu_kv_to_oracle_layout(pair.gpu.kv_view())
    bt = synth.make_block_tables(ctx + 1, int(nblk.max()), synth.BlockAllocator(blocks, seed))
    try:
        y, yr, x = pair.decode(ctx, bt, synth.hidden_states(seed, 1, seqs, shape.hidden))
        rows = [rel_l2(a, b) for a, b in zip(y - x, yr - x)]
        log(f"{shape.name} {seqs} tokens, contexts <= {longest}: worst row's branch {max(rows):.2e}")
        assert rel_l2(y - x, yr - x) <= 1e-2 and max(rows) <= 2e-2
    finally:
        pair.close()
