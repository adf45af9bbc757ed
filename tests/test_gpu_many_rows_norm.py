"""The input norm of many rows (eight rows per block): selected rows, a last
block that is not full, and inputs that are not 16-byte aligned (one row per
block), against float64."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2606_18600_amd import synth
from paper_2606_18600_amd.harness import DeviceStage, pack_lm_head, upload_weights

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rows,offset,H", [(1023, 0, 8192), (1024, 0, 8192), (1030, 0, 8192),
                                             (1030, 4, 8192), (1030, 0, 7168)])
def test_selected_rows(n_rows, offset, H):
    """logits of shuffled rows: norm outputs and weights are bf16 (2^-9), K
    products of random sign: 1e-2 of the largest is far above that error and
    far below a misplaced row's."""
    vocab = 128
    shape = synth.ModelShape("h", hidden=H, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=128,
                             rms_eps=1e-5, rope_theta=1e4)
    st = DeviceStage(shape, "bf16", 0, [upload_weights(synth.host_layer_weights(shape, 1, 0), "bf16")],
                     4, 2048, 4)
    try:
        g = torch.Generator(device="cuda")
        g.manual_seed(n_rows + offset)
        flat = torch.randn(1500 * H + offset, generator=g, device="cuda").to(torch.bfloat16)
        x = flat[offset:].view(1500, H)  # offset 4: 8 bytes past a 16-byte multiple
        w = torch.randn((vocab, H), generator=g, device="cuda").to(torch.bfloat16)
        gain = (torch.rand(H, generator=g, device="cuda") + 0.5).to(torch.bfloat16)
        rows = np.random.default_rng(n_rows).permutation(1500)[:n_rows].astype(np.int32)
        y = st.lm_head(gain, pack_lm_head(st.cfg, w), x, rows=rows)
        torch.cuda.synchronize()
        xd = x[torch.from_numpy(rows.astype(np.int64)).cuda()].double()
        h = xd / torch.sqrt((xd * xd).mean(-1, keepdim=True) + 1e-5) * gain.double()
        ref = h @ w.double().T
        assert (y.double() - ref).abs().max() <= 1e-2 * ref.abs().max()
        assert torch.linalg.norm(y.double() - ref) <= 5e-3 * torch.linalg.norm(ref)
    finally:
        st.close()
