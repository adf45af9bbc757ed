"""bf16 steps in which one request's rows are NaN: the other requests' rows
are bit for bit what they are without it, whichever kernels the step takes
(decode attention on whole tokens, single splits and merged splits, prefill
attention with its keys split, products of few and of mid rows)."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2606_18600_amd import synth
from paper_2606_18600_amd.harness import DeviceStage, upload_weights
from tests.helpers import strong_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("nan"), float("inf")], ids=["nan", "inf"])
@pytest.mark.parametrize("nq,nkv,d,chunks,decodes", [
    (8, 1, 128, [], [100, 30, 77, 127]),           # single splits of at most 8 blocks
    (4, 2, 64, [], [200, 500, 300]),               # whole tokens, 8 waves each
    (8, 2, 128, [], [1500, 40, 3000, 900]),        # merged splits, 8 waves; one split next to many
    (16, 1, 128, [], [4000, 2500]),                # ... 4 waves
    (8, 1, 128, [], [600] * 31),                   # 31 rows
    (8, 1, 128, [(17, 1023), (3, 0), (40, 2048)], []),      # keys split
    (4, 4, 64, [(100, 900), (60, 1500)], [50, 800]),        # ... of 162 rows, with decodes
    (4, 2, 64, [(130, 0), (260, 0)], []),
])
def test_one_request_does_not_reach_another(nq, nkv, d, chunks, decodes, value):
    shape = synth.ModelShape("i", hidden=256, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=320,
                             rms_eps=1e-5, rope_theta=1e4)
    seed = nq + d + len(decodes)
    q = np.array([a for a, _ in chunks], np.int32)
    c = np.array([b for _, b in chunks], np.int32)
    dc = np.array(decodes, np.int32)
    ends = np.concatenate([c + q, dc + 1])
    nblk = (ends + 15) // 16
    blocks = int(nblk.sum())
    bt = torch.from_numpy(synth.make_block_tables(ends, int(nblk.max()),
                                                  synth.BlockAllocator(blocks, seed))).cuda()
    pbt, dbt = bt[:len(q)].contiguous(), bt[len(q):].contiguous()
    rows = np.concatenate([q, np.ones(len(dc), np.int32)])
    first = np.concatenate([[0], np.cumsum(rows)])
    x = torch.from_numpy(synth.hidden_states(seed, 1, int(first[-1]), shape.hidden)).cuda().bfloat16()
    w = [upload_weights(strong_weights(shape, seed, l), "bf16") for l in range(2)]
    st = DeviceStage(shape, "bf16", 0, w, blocks, 512, 40)
    g = torch.Generator(device="cuda")

    def step(xi):
        g.manual_seed(seed)
        st.kv_pool.normal_(0.0, 1.0, generator=g)
        if len(q) and len(dc):
            y = st.mixed(q, c, pbt, dc, dbt, xi)
        elif len(q):
            y = st.prefill(q, c, pbt, xi)
        else:
            y = st.decode(dc, dbt, xi)
        torch.cuda.synchronize()
        return y.clone()

    try:
        plain = step(x)
        assert torch.isfinite(plain.float()).all()
        for i in sorted({0, len(rows) // 2, len(rows) - 1}):
            bad = x.clone()
            bad[first[i]:first[i + 1]] = value
            y = step(bad)
            keep = torch.ones(len(x), dtype=torch.bool, device="cuda")
            keep[first[i]:first[i + 1]] = False
            assert torch.equal(y[keep], plain[keep]), i
            assert not torch.isfinite(y[~keep].float()).any(), i
    finally:
        st.close()
