"""bf16 GEMM launches of up to 16 rows, which are worked on in strips of 16 columns, and row tiles that take turns at fetching
weights: the bits of every other launch."""
import pytest

from paper_2505_07203_amd import inputs as I

pytestmark = pytest.mark.gpu


def _rnd(seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)


# K: less than a block of 256, whole blocks, a block and a remainder of 1 .. 3 slices; more blocks than the ring holds
@pytest.mark.parametrize("N,K", [(64, 64), (320, 256), (4096, 448), (128, 832), (16384, 1344), (16448, 128), (4096, 2752)])
def test_few_rows_are_the_bits_of_a_larger_launch(N, K):
    import torch
    from paper_2505_07203_amd import binding as B
    rnd = _rnd(N + K)
    a, r, w = rnd(40, K), rnd(40, N), rnd(N, K) * 0.05
    whole = B.po_op_linear(a, w), B.po_op_linear(a, w, residual=r), B.po_op_gate_up_silu(a, w)
    ref = a.double() @ w.double().t()
    assert bool(((whole[0].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + K * 2.0 ** -22 * (a.double().abs() @ w.double().abs().t())).all())
    for m in (1, 2, 3, 9, 15, 16, 17):
        x = a[:m].contiguous()
        assert torch.equal(B.po_op_linear(x, w), whole[0][:m]), m
        assert torch.equal(B.po_op_linear(x, w, residual=r[:m].contiguous()), whole[1][:m]), m
        assert torch.equal(B.po_op_gate_up_silu(x, w), whole[2][:m]), m


@pytest.mark.parametrize("bias", [True, False])
@pytest.mark.parametrize("cfg,K", [(I.LLAMA8B, 704), (I.TINY, 256)])
def test_few_qkv_rows_are_the_bits_of_a_larger_launch(cfg, K, bias):
    import torch
    from paper_2505_07203_amd import binding as B
    hq, hkv, hd = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim
    rnd = _rnd(K)
    a, w = rnd(40, K), rnd((hq + 2 * hkv) * hd, K) * 0.05
    b = rnd((hq + 2 * hkv) * hd) if bias else None
    cos, sin = B.po_op_rope_table(40, hd, cfg.rope_theta)
    scale = B.attention_q_scale(hd)
    q, k, vt = B.po_op_qkv_rope(a, w, b, cos, sin, hq, hkv, hd, q_scale=scale)
    for m in (1, 2, 3, 16):
        q1, k1, vt1 = B.po_op_qkv_rope(a[:m].contiguous(), w, b, cos, sin, hq, hkv, hd, q_scale=scale)
        assert torch.equal(q1, q[:m]) and torch.equal(k1, k[:m]) and torch.equal(vt1[:, :m], vt[:, :m]), m


@pytest.mark.parametrize("N,K", [(4096, 128), (4096, 192), (4096, 1088), (2112, 4096)])
def test_turns_are_the_bits_of_a_launch_without(N, K):
    """Heights whose row tiles take turns: fewer slices than a turn is ahead, odd numbers of slices, a last column tile of 64."""
    import torch
    from paper_2505_07203_amd import binding as B
    rnd = _rnd(N * K)
    a, r, w = rnd(8192, K), rnd(8192, N), rnd(N, K) * 0.05
    whole = B.po_op_linear(a, w, residual=r)
    ref, size = a.double() @ w.double().t() + r.double(), a.double().abs() @ w.double().abs().t()
    assert bool(((whole.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + K * 2.0 ** -22 * size).all())
    for m in (64, 129, 160, 300, 471, 540, 1000, 1024, 1100, 1280, 1800, 2000):
        assert torch.equal(B.po_op_linear(a[:m].contiguous(), w, residual=r[:m].contiguous()), whole[:m]), m


@pytest.mark.parametrize("N,K", [(4096, 128), (4096, 384), (4096, 1152), (2112, 4096)])
def test_fp8_turns_are_the_bits_of_a_launch_without(N, K):
    import torch
    from paper_2505_07203_amd import binding as B
    rnd = _rnd(N * K + 1)
    r = rnd(8192, N)
    (qa, sa), (qw, sw) = B.po_op_quantize_rows(rnd(8192, K)), B.po_op_quantize_rows(rnd(N, K) * 0.05)
    whole = B.po_op_linear_fp8(qa, sa, qw, sw, residual=r)
    for m in (64, 200, 300, 400, 471, 512, 600, 768, 1000, 1024):
        x, s = qa[:m].contiguous(), sa[:m].contiguous()
        assert torch.equal(B.po_op_linear_fp8(x, s, qw, sw, residual=r[:m].contiguous()), whole[:m]), m
