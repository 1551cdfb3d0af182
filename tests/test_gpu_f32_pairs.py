"""Float32 projections that finish their pairs themselves: gate/up with the SiLU-multiply, QKV with bias and rotation, in every
tile (32, 64, 128 rows and columns; test_tile_forms_cpu.py holds the sizes to it) and with rows and columns that end inside one."""
import numpy as np
import pytest

import helpers as H
from paper_2505_07203_amd import inputs as I

pytestmark = pytest.mark.gpu


# F: less than half a tile, ends inside half a tile, whole ones; the last sizes take tiles of 64 and of 128
GATE_UP = [(1, 4, 64), (33, 36, 104), (257, 688, 256), (70, 88, 72), (500, 2052, 128), (1500, 6148, 96)]


@pytest.mark.parametrize("M,F,K", GATE_UP)
def test_gate_up_against_float64(M, F, K):
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(M + F)
    a, wg, wu = (torch.randn(*s, generator=g, device="cuda") * 0.3 for s in ((M, K), (F, K), (F, K)))
    h = B.po_op_gate_up_silu(a, B.po_op_pack_gate_up(wg, wu)).double()
    x, y = a.double() @ wg.double().t(), a.double() @ wu.double().t()
    ref = x * torch.sigmoid(x) * y
    # K sequential float32 additions each; d(silu)/dx is at most 1.1, silu(x) at most |x|; a few roundings of the result
    ex, ey = (K * 2.0 ** -24 * (a.double().abs() @ w.double().abs().t()) for w in (wg, wu))
    assert bool(((h - ref).abs() <= 1.1 * ex * (y.abs() + ey) + x.abs() * ey + 2.0 ** -20 * ref.abs() + 1e-12).all())


def _config(hd, hq, hkv, d):
    return I.ModelConfig(n_layers=2, d_model=d, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, ffn_dim=344, vocab_size=512,
                         rms_eps=1e-5, rope_theta=10000.0, dtype=I.F32, qkv_bias=1)


@pytest.mark.parametrize("hd,hq,hkv,d,n", [(64, 4, 2, 256, 150), (128, 3, 1, 256, 100), (64, 3, 3, 192, 1), (128, 8, 2, 512, 700)])
def test_whole_path_with_bias_against_oracle(hd, hq, hkv, d, n):
    from paper_2505_07203_amd import binding as B
    cfg = _config(hd, hq, hkv, d)
    tokens = I.make_tokens(cfg, 7, n)
    z_ref, _ = H.oracle_prefill(cfg, 1001, tokens, cand=I.label_ids(cfg))
    ctx = B.Context(cfg, 2 * n + 70, 64, device="cuda:0")
    try:
        ctx.load_synthetic(1001, threads=2)
        z, _ = ctx.po_prefill(tokens, I.label_ids(cfg))
        assert np.max(np.abs(z - z_ref)) <= 1e-4
        packed = ctx.po_prefill_packed([tokens, tokens], I.label_ids(cfg), want_logits=True)[0]
        assert np.array_equal(packed[0], z) and np.array_equal(packed[1], z)
    finally:
        ctx.po_destroy()


# (head dimension, query and K/V heads, width, length of a request): QKV of one request and of two packed ones in one launch
# each, and in launches of QKV_CHUNK rows, which take the 32-row tile that the test above compares with the oracle
QKV_CHUNK = 64
QKV = [(64, 4, 2, 256, 2011), (128, 4, 2, 256, 2011), (128, 3, 1, 192, 1931)]


@pytest.mark.parametrize("hd,hq,hkv,d,n", QKV)
def test_qkv_in_large_tiles_is_the_bits_of_small_ones(hd, hq, hkv, d, n):
    from paper_2505_07203_amd import binding as B
    cfg = _config(hd, hq, hkv, d)
    one, two = I.make_tokens(cfg, 7, n), I.make_tokens(cfg, 8, n)
    z = {}
    for chunk in (QKV_CHUNK, 2 * n):
        ctx = B.Context(cfg, 2 * n, chunk, device="cuda:0")
        try:
            ctx.load_synthetic(1001, threads=2)
            z[chunk] = [ctx.po_prefill(t, I.label_ids(cfg))[0] for t in (one, two)]
            packed = ctx.po_prefill_packed([one, two], I.label_ids(cfg), want_logits=True)[0]
            assert all(np.array_equal(a, b) for a, b in zip(packed, z[chunk])), chunk
        finally:
            ctx.po_destroy()
    assert all(np.isfinite(a).all() and np.array_equal(a, b) for a, b in zip(z[QKV_CHUNK], z[2 * n]))


def test_qkv_in_two_launches_is_the_bits_of_one():
    """256 rows of 3072 columns fill one round of 32-row tiles and half of a second, with K long enough to make Q a launch by itself"""
    from paper_2505_07203_amd import binding as B
    cfg = _config(128, 32, 8, 2048)
    tokens = I.make_tokens(cfg, 7, 256)
    z = []
    for chunk in (QKV_CHUNK, 256):
        ctx = B.Context(cfg, 256, chunk, device="cuda:0")
        try:
            ctx.load_synthetic(1001, threads=4)
            z.append(ctx.po_prefill(tokens, I.label_ids(cfg))[0])
        finally:
            ctx.po_destroy()
    assert np.isfinite(z[0]).all() and np.array_equal(z[0], z[1])
