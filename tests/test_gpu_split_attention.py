"""Few-rows attention with prescaled queries (head dimension 128): pieces of the keys, all query heads of a KV head in one
workgroup, cached prefix read in place.  Against the default path on the same tokens, which other tests hold to the oracle."""
import numpy as np
import pytest

from paper_2505_07203_amd import inputs as I
import helpers as H

pytestmark = pytest.mark.gpu


def _cfg(hq, hkv):
    return I.ModelConfig(n_layers=2, d_model=512, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, ffn_dim=512, vocab_size=512,
                         rms_eps=1e-5, rope_theta=10000.0, dtype=I.BF16)


def _context(cfg, n, gain=1.0):
    from paper_2505_07203_amd import binding as B
    ctx = B.Context(cfg, n, 1024)
    for kind, layer, arr in I.iter_model_tensors(cfg, 77):
        if kind == I.KIND_ATTN_NORM and gain != 1.0:
            import torch
            t = torch.from_numpy(arr.view(np.int16)).view(torch.bfloat16).float() * gain
            arr = t.to(torch.bfloat16).view(torch.int16).numpy().view(np.uint16)
        ctx.po_load_tensor(kind, layer, arr)
    return ctx


def _compare(cfg, total, cached, gain, tol):
    ctx = _context(cfg, total, gain)
    try:
        tokens = I.make_tokens(cfg, 5, total)
        z0, _ = ctx.po_prefill(tokens)
        ctx.po_set_few_rows_split(True)
        if cached:
            ctx.po_attach_kv_cache(cached)
            ctx.po_set_few_rows_split(False)
            ctx.po_prefill_prefix(tokens[:cached], cached)
            ctx.po_set_few_rows_split(True)
            z1, _, reused = ctx.po_prefill_prefix(tokens, 0)
            z2, _, _ = ctx.po_prefill_prefix(tokens, 0)
            assert reused == cached
        else:
            (z1, _), (z2, _) = ctx.po_prefill(tokens), ctx.po_prefill(tokens)
        assert ctx.po_get_stats()["split_launches"] > 0
        assert np.array_equal(z1, z2) and np.all(np.isfinite(z1))
        rel = H.normalised_max_rel(z1, z0)
        assert rel <= tol, rel
    finally:
        ctx.po_destroy()


@pytest.mark.parametrize("hq,hkv", [(8, 2), (5, 1), (8, 8), (10, 2)])
@pytest.mark.parametrize("total,cached", [(257, 0), (640, 0), (641, 640), (700, 511), (1000, 100), (3137, 2987), (4200, 3900)])
def test_split_attention_agrees_with_the_default_path(hq, hkv, total, cached):
    # two roundings of the same bf16 model apart: the bar other tests put between the two modes
    _compare(_cfg(hq, hkv), total, cached, 1.0, 1e-2)


@pytest.mark.parametrize("total,cached", [(300, 0), (1500, 1400)])
def test_scores_far_outside_the_exponent_range(total, cached):
    """A norm gain that puts scores hundreds of nats apart: rows whose sums leave the float range are formed again with a
    running maximum, from the cached and the fresh keys.  One rounding of a query value moves a score by up to 0.1 nats
    here, hence the wider bar."""
    _compare(_cfg(8, 2), total, cached, 30.0, 6e-2)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 200])
def test_value_transpose_aligned_and_unaligned(n):
    """V at a 16-byte boundary and two bytes off it take different kernels to the same transposed copy."""
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn(n, h, 128, generator=g, device="cuda").to(torch.bfloat16) for h in (4, 2, 2))
    off = torch.empty(v.numel() + 1, dtype=torch.bfloat16, device="cuda")[1:].view(v.shape)
    off.copy_(v)
    assert off.data_ptr() % 16 == 2 and v.data_ptr() % 16 == 0
    assert torch.equal(B.po_op_attention(q, k, off), B.po_op_attention(q, k, v))
