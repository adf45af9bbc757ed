"""The fp32 mode's matrix-core kernels at the sizes where their dispatch
turns: GEMM tiles of 128, 64, 32 and 16 (the plain store through the LM head,
whose vocabulary and row count are free in the fp32 mode; SwiGLU and residual
add through layers), attention blocks that hold tokens of several sequences,
and buffers that are aligned to 4 bytes only."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2606_18600_amd import synth
from paper_2606_18600_amd.harness import DeviceStage, upload_weights
from tests.gpu_pair import Pair, log
from tests.helpers import rel_l2, strong_weights

pytestmark = pytest.mark.gpu

G1 = synth.ModelShape("g1-d64", hidden=256, n_q_heads=4, n_kv_heads=4, head_dim=64, ffn=512,
                      rms_eps=1e-5, rope_theta=1e4)
G2 = synth.ModelShape("g2-d128", hidden=512, n_q_heads=4, n_kv_heads=2, head_dim=128, ffn=576,
                      rms_eps=1e-5, rope_theta=1e4)


def _stage(shape, seed, blocks=128, max_tokens=512, max_seqs=24, fill=0.0):
    w = [upload_weights({k: v.astype(np.float32) for k, v in strong_weights(shape, seed, l).items()},
                        "f32") for l in range(2)]
    st = DeviceStage(shape, "f32", 0, w, blocks, max_tokens, max_seqs)
    st.kv_pool.fill_(fill)
    return st


@pytest.mark.parametrize("hidden", [256, 640])
@pytest.mark.parametrize("rows,vocab", [(8, 131), (9, 1), (9, 131), (31, 33), (32, 32), (33, 65),
                                        (64, 4096), (65, 4129), (129, 16384), (256, 16500),
                                        (300, 515), (128, 1024), (128, 1025), (17, 15)])
def test_lm_head_tiles(hidden, rows, vocab):
    """logits against float64 on the same stored values. A dot product of
    K <= 640 terms in fp32, in any order, is within K * 2^-24 of the sum of
    its terms' magnitudes; the normalised row adds a few ulps: 6e-5 relative
    to that sum would already be a wrong kernel."""
    shape = synth.ModelShape("h", hidden=hidden, n_q_heads=4, n_kv_heads=2, head_dim=64, ffn=128,
                             rms_eps=1e-5, rope_theta=1e4)
    st = _stage(shape, 3)
    try:
        g = torch.Generator(device="cuda")
        g.manual_seed(rows * 131 + vocab)
        x = torch.randn((rows, hidden), generator=g, device="cuda")
        w = torch.randn((vocab, hidden), generator=g, device="cuda")
        gain = torch.rand(hidden, generator=g, device="cuda") + 0.5
        y = st.lm_head(gain, w, x)
        torch.cuda.synchronize()
        xd = x.double()
        h = xd / torch.sqrt((xd * xd).mean(-1, keepdim=True) + 1e-5) * gain.double()
        ref, mag = h @ w.double().T, h.abs() @ w.double().abs().T
        assert torch.all((y.double() - ref).abs() <= (hidden * 2.0 ** -24 + 1e-6) * mag)
    finally:
        st.close()


@pytest.mark.parametrize("shape", [G1, G2], ids=lambda s: s.name)
@pytest.mark.parametrize("lens,decodes", [([1, 1, 2, 3, 5, 7, 9, 200], 0), ([37, 3], 17),
                                          ([5], 3)])
def test_tokens_of_several_sequences_in_one_block(shape, lens, decodes):
    seed = 11
    pair = Pair(shape, "f32", 2, 256, 1024, 32, seed,
                host_weights=[strong_weights(shape, seed, l) for l in range(2)])
    lens = np.array(lens, np.int32)
    dctx = synth.uniform_lengths(seed, 4, max(1, decodes), 1, 90)[:decodes]
    alloc = synth.BlockAllocator(256, seed)
    bt = synth.make_block_tables(lens, 16, alloc)
    dbt = synth.make_block_tables(dctx + 1, 16, alloc) if decodes else None
    try:
        if decodes:
            pair.prefill(dctx, np.zeros(decodes, np.int32), dbt,
                         synth.hidden_states(seed, 1, int(dctx.sum()), shape.hidden))
            x = synth.hidden_states(seed, 2, int(lens.sum()) + decodes, shape.hidden)
            y, yr, _ = pair.mixed(lens, np.zeros(len(lens), np.int32), bt, dctx, dbt, x)
        else:
            x = synth.hidden_states(seed, 2, int(lens.sum()), shape.hidden)
            y, yr, _ = pair.prefill(lens, np.zeros(len(lens), np.int32), bt, x)
        e = rel_l2(y, yr)
        log(f"{shape.name} lens={lens.tolist()} decodes={decodes}: {e:.2e}")
        assert e <= 1e-5  # measured ~1e-6 here; a misplaced key moves it by tens of percent
    finally:
        pair.close()


@pytest.mark.parametrize("shape", [G1, G2], ids=lambda s: s.name)
def test_other_requests_and_unwritten_slots_stay_out(shape):
    """Rows of one request are bit for bit the same whether another request's
    rows (in the same attention block) are finite or NaN, earlier tokens of a
    request do not see its later ones, and unwritten cache slots do not
    enter."""
    seed = 5
    lens = np.array([3, 6, 21], np.int32)
    bt = torch.from_numpy(synth.make_block_tables(lens, 2, synth.BlockAllocator(8, seed))).cuda()
    x = torch.from_numpy(synth.hidden_states(seed, 1, 30, shape.hidden)).cuda()
    out = {}
    for kind in ("plain", "nan rows", "nan pool"):
        st = _stage(shape, seed, blocks=8, fill=float("nan") if kind == "nan pool" else 0.0)
        xi = x.clone()
        if kind == "nan rows":
            xi[3:9] = float("nan")  # the second request
            xi[28] = float("inf")   # the third request's last but one token
        out[kind] = st.prefill(lens, [0, 0, 0], bt, xi).clone()
        torch.cuda.synchronize()
        st.close()
    assert torch.isfinite(out["plain"]).all()
    assert torch.equal(out["plain"], out["nan pool"])
    keep = [0, 1, 2, *range(9, 28)]
    assert torch.equal(out["plain"][keep], out["nan rows"][keep])


WIDE_FFN = synth.ModelShape("wide-ffn", hidden=256, n_q_heads=4, n_kv_heads=2, head_dim=64,
                            ffn=8256, rms_eps=1e-5, rope_theta=1e4)
WIDE_HIDDEN = synth.ModelShape("wide-hidden", hidden=8192, n_q_heads=2, n_kv_heads=1, head_dim=64,
                               ffn=192, rms_eps=1e-5, rope_theta=1e4)


@pytest.mark.parametrize("shape,rows", [
    (WIDE_FFN, 100), (WIDE_FFN, 128),        # SwiGLU on 64-row tiles: 129 columns of them
    (WIDE_FFN, 129), (WIDE_FFN, 300),        # ... on 128-row tiles
    (WIDE_HIDDEN, 129), (WIDE_HIDDEN, 383),  # residual add on 64 x 64 tiles
    (WIDE_HIDDEN, 450),                      # ... on 128 x 128 tiles
], ids=lambda v: v.name if isinstance(v, synth.ModelShape) else str(v))
def test_layer_tiles(shape, rows):
    """One layer against the exact oracle, output, branch and each row's
    branch: fp32 sums of at most 8256 terms of random sign, about 1e-6 as in
    the other layers here; a misplaced row or column moves a row by tens of
    percent."""
    seed = rows
    pair = Pair(shape, "f32", 1, 40, 512, 4, seed, host_weights=[strong_weights(shape, seed, 0)])
    lens = np.array([rows], np.int32)
    bt = synth.make_block_tables(lens, 40, synth.BlockAllocator(40, seed))
    try:
        y, yr, x = pair.prefill(lens, np.zeros(1, np.int32), bt,
                                synth.hidden_states(seed, 1, rows, shape.hidden))
        e, worst = rel_l2(y - x, yr - x), max(rel_l2(a, b) for a, b in zip(y - x, yr - x))
        log(f"{shape.name} rows={rows}: branch {e:.2e} worst row {worst:.2e}")
        assert rel_l2(y, yr) <= 1e-5 and e <= 1e-5 and worst <= 1e-4
    finally:
        pair.close()


def _shifted(t):
    """A copy of t that starts 4 bytes past a 16-byte multiple."""
    flat = torch.empty(t.numel() + 4, dtype=t.dtype, device="cuda")[1:1 + t.numel()]
    assert flat.data_ptr() % 16 == 4
    return flat.view(t.shape).copy_(t)


@pytest.mark.parametrize("shape", [G1, G2], ids=lambda s: s.name)
def test_buffers_aligned_to_four_bytes(shape):
    """Weights, KV pool and hidden rows may lie at any multiple of 4 bytes in
    the fp32 mode: a prefill and a decode give the same bits there."""
    seed = 7
    lens = np.array([3, 37], np.int32)
    bt = torch.from_numpy(synth.make_block_tables(lens + 1, 3, synth.BlockAllocator(8, seed))).cuda()
    x = torch.from_numpy(synth.hidden_states(seed, 1, 40, shape.hidden)).cuda()
    xd = torch.from_numpy(synth.hidden_states(seed, 2, 2, shape.hidden)).cuda()
    host = [{k: v.astype(np.float32) for k, v in strong_weights(shape, seed, l).items()}
            for l in range(2)]
    out = []
    for place in (lambda t: t, _shifted):
        w = [{k: place(v) for k, v in upload_weights(h, "f32").items()} for h in host]
        pool = place(torch.zeros(2 * 8 * shape.n_kv_heads * 2 * 16 * shape.head_dim, device="cuda"))
        # (fp32 weights are stored row-major: packing them is a copy)
        st = DeviceStage(shape, "f32", 0, w, 8, 64, 4, kv_pool=pool, packed=True)
        try:
            y = st.prefill(lens, [0, 0], bt, place(x), place(torch.empty_like(x)))
            yd = st.decode(lens, bt, place(xd), place(torch.empty_like(xd)))
            torch.cuda.synchronize()
            out.append((y.clone(), yd.clone(), pool.clone()))
        finally:
            st.close()
    assert torch.isfinite(out[0][0]).all() and torch.isfinite(out[0][1]).all()
    for a, b in zip(*out):
        assert torch.equal(a, b)


def test_workspace_without_unused_planes():
    """Only steps of at most 8 rows keep the gate and up columns in memory."""
    shape = synth.ModelShape("f", hidden=128, n_q_heads=2, n_kv_heads=2, head_dim=64, ffn=16384,
                             rms_eps=1e-5, rope_theta=1e4)
    st = DeviceStage(shape, "f32", 0, [upload_weights(synth.host_layer_weights(shape, 1, 0), "f32")],
                     4, 1024, 4, max_position=64)
    try:
        # the FFN activations, padded to whole 192-row tiles (1152 rows), the
        # gate and up columns of 8 rows, and room for 8 regions as wide as the
        # residual: 81 MB (the gate and up columns of every row: 134 MB more)
        limit = 4 * 1152 * (shape.ffn + 8 * shape.hidden) + 4 * 8 * 2 * shape.ffn
        assert st.workspace.numel() < limit
    finally:
        st.close()
