"""Attention rows whose scores leave the range of the fast form: their bits depend on the row and its keys alone, whatever the
launch they are computed in (tiles of 128 or 256 rows, few workgroups or many, starting in the middle of a tile) and whatever the
rows beside them are."""
import math

import numpy as np
import pytest

from paper_2505_07203_amd import inputs as I

pytestmark = pytest.mark.gpu
HQ, HKV, HD = 32, 8, 128


def _inputs(n, std, seed):
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return ((rnd(n, HQ, HD) * std * B.attention_q_scale(HD)).to(torch.bfloat16), (rnd(n, HKV, HD) * std).to(torch.bfloat16),
            rnd(n, HKV, HD).to(torch.bfloat16))


def _share_out_of_range(q, k, rows):
    """of these rows (all heads), the share whose sum of 2^score is not within 2^-60 .. 2^100"""
    import torch
    s = torch.matmul(q[rows].float().transpose(0, 1),
                     k.float().repeat_interleave(HQ // HKV, 1).permute(1, 2, 0).contiguous())          # [Hq, rows, n]
    s.masked_fill_(torch.arange(k.shape[0], device="cuda")[None, None] > rows[None, :, None], -math.inf)
    top = torch.logsumexp(s.double() * math.log(2.0), -1) / math.log(2.0)
    return float(((top < -60) | (top >= 100)).double().mean())


def test_rows_are_the_bits_of_a_longer_sequence():
    import torch
    from paper_2505_07203_amd import binding as B
    q, k, v = _inputs(4700, 5.0, 3)
    share = _share_out_of_range(q, k, torch.arange(0, 4700, 47, device="cuda"))
    assert 0.1 < share < 0.9, share
    whole = B.po_op_attention(q, k, v, q_prescaled=True)
    for n in (1, 31, 70, 129, 200, 300, 1000, 1931, 2048, 2049, 2300, 4000, 4096, 4097, 4500):
        o = B.po_op_attention(q[:n].contiguous(), k[:n].contiguous(), v[:n].contiguous(), q_prescaled=True)
        assert torch.equal(o, whole[:n]), n


@pytest.mark.parametrize("n", [900, 2100, 4700])
def test_rows_do_not_see_their_neighbours(n):
    """every other row turned into one that leaves the range, or back"""
    import torch
    from paper_2505_07203_amd import binding as B
    q, k, v = _inputs(n, 1.3, n)
    o = B.po_op_attention(q, k, v, q_prescaled=True)
    k[:, :, 0] = 8.0
    tame, wild = q.clone(), q.clone()
    tame[:, :, 0] = 0.0
    wild[:, :, 0] = 25.0                                  # 200 powers of two up
    mixed = torch.where((torch.arange(n, device="cuda") % 3 == 0)[:, None, None], wild, tame)
    a, b, c = (B.po_op_attention(x, k, v, q_prescaled=True) for x in (tame, wild, mixed))
    assert torch.isfinite(a).all() and torch.isfinite(b).all() and not torch.equal(a, o)
    assert torch.equal(c[0::3], b[0::3]) and torch.equal(c[1::3], a[1::3]) and torch.equal(c[2::3], a[2::3])


@pytest.fixture(scope="module")
def wide_scores():
    """two layers of 32 heads whose scores spread over some tens of powers of two"""
    import torch
    from paper_2505_07203_amd import binding as B
    cfg = I.ModelConfig(n_layers=2, d_model=256, n_q_heads=HQ, n_kv_heads=HKV, head_dim=HD, ffn_dim=256, vocab_size=512,
                        rms_eps=1e-5, rope_theta=10000.0, dtype=I.BF16)
    ctx = B.Context(cfg, 4700, 4096, device="cuda:0")
    ctx.load_synthetic(1001, threads=2)
    g = torch.Generator().manual_seed(5)
    for l in range(cfg.n_layers):
        for kind, rows in ((I.KIND_WQ, cfg.q_dim), (I.KIND_WK, cfg.kv_dim)):
            w = (torch.randn(rows, cfg.d_model, generator=g) * 0.3).to(torch.bfloat16)
            ctx.po_load_tensor(kind, l, w.view(torch.uint16).numpy())
    yield cfg, ctx
    ctx.po_destroy()


@pytest.mark.parametrize("n", [2000, 2300, 4500])
def test_whole_path_keeps_its_bits(wide_scores, n):
    """the last layer's shortcut on and off; cached prefixes that end inside a tile"""
    cfg, ctx = wide_scores
    tokens, cand = I.make_tokens(cfg, 17, n), I.label_ids(cfg)
    ctx.po_set_lazy_last_layer(False)
    z, lp = ctx.po_prefill(tokens, cand)
    assert np.isfinite(z).all()
    ctx.po_set_lazy_last_layer(True)
    for _ in range(2):                                    # (the second time over what the first one left in the buffers)
        z1, lp1 = ctx.po_prefill(tokens, cand)
        assert np.array_equal(z, z1) and np.array_equal(lp, lp1)
    for cached in (n - 1, n - 70, n - 300, n - 1100, 1000):
        ctx.po_attach_kv_cache(cached)
        ctx.po_prefill_prefix(tokens[:cached], cached, cand)
        z1, lp1, reused = ctx.po_prefill_prefix(tokens, 0, cand)
        assert reused == cached and np.array_equal(z, z1) and np.array_equal(lp, lp1), cached
