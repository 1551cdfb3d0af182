"""bf16 GEMM launches of up to 16 rows, which are worked on in strips of 16 columns, and row tiles that take turns at fetching
weights: the bits of every other launch."""
import pytest

import test_gpu_small_tiles as T
from paper_2505_07203_amd import inputs as I

pytestmark = pytest.mark.gpu


def _rnd(seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)


# K: less than a block of 256, whole blocks, a block and a remainder of 1 .. 3 slices; more blocks than the ring holds; more strips
# than the compute units hold at once
@pytest.mark.parametrize("N,K", [(64, 64), (320, 256), (4096, 448), (128, 832), (16384, 1344), (16448, 128), (4096, 2752), (14336, 4160)])
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


@pytest.mark.parametrize("ffn,splits", [(4096, False), (8192, False), (16384, True)])
def test_few_rows_mode_splits_where_strips_leave_compute_units_idle(ffn, splits):
    import numpy as np
    from paper_2505_07203_amd import binding as B
    cfg = I.LLAMA8B.replace(dtype=I.BF16, d_model=512, n_q_heads=4, n_kv_heads=2, ffn_dim=ffn, n_layers=2, vocab_size=512)
    ctx = B.Context(cfg, 64, 64, device="cuda:0")
    try:
        ctx.load_synthetic(3, threads=2)
        tokens, cand = I.make_tokens(cfg, 5, 12), I.label_ids(cfg)
        whole = ctx.po_prefill(tokens, cand)[0]
        ctx.po_set_few_rows_split(True)
        z = ctx.po_prefill(tokens, cand)[0]
        assert (ctx.po_get_stats()["split_launches"] > 0) == splits
        assert np.array_equal(z, whole) or splits and np.max(np.abs(z - whole)) <= 1e-2 * np.max(np.abs(whole))
    finally:
        ctx.po_destroy()


# Launches whose row tiles take turns: odd numbers of slices, of which the short ones (11 and 17 of 64, 9 of 128) end within
# the first turns; a last column tile of 64.  test_tile_forms_cpu.py holds them to reaching every tile that takes turns.
TURNS_TOP = 8192                # rows of the launch they are compared with, which takes none
TURNS_ROWS = (81, 150, 170, 250, 300, 384, 471, 512, 540, 620, 780, 840, 1000, 1100, 1240, 1400, 1600, 1800, 2000, 2200)
TURNS_BF16 = [(4096, 704), (4096, 1088), (2112, 4160)]
TURNS_QKV = [(I.LLAMA8B, 704), (I.LLAMA8B, 4160)]
TURNS_FP8 = [(4096, 1152), (4096, 5248), (2112, 5248)]
TURNS_FP8_QKV = (I.LLAMA8B, 5248)
# ... and launches that end before the first touch, or of an even number of slices; whole numbers of tiles
TURNS_BF16_SHORT, TURNS_FP8_SHORT = [(4096, 128), (4096, 192), (2112, 4096)], [(4096, 128), (4096, 384), (2112, 4096)]
TURNS_WHOLE_ROWS = (64, 129, 160, 200, 400, 600, 768, 1024, 1280)
TURNS_SPLIT = [(81, 320, 4224), (162, 320, 1408), (465, 2112, 4224), (381, 2112, 2816), (450, 2112, 14336), (771, 1024, 14336)]
TURNS_FP8_SPLIT = [(273, 320, 10496), (705, 1024, 14336)]


@pytest.mark.parametrize("N,K", TURNS_BF16 + TURNS_BF16_SHORT)
def test_turns_are_the_bits_of_a_launch_without(N, K):
    import torch
    from paper_2505_07203_amd import binding as B
    rnd = _rnd(N * K)
    a, r, w = rnd(TURNS_TOP, K), rnd(TURNS_TOP, N), rnd(N, K) * 0.05
    whole = B.po_op_linear(a, w, residual=r), B.po_op_gate_up_silu(a, w)
    ref, size = a.double() @ w.double().t() + r.double(), a.double().abs() @ w.double().abs().t()
    assert bool(((whole[0].double() - ref).abs() <= 2.0 ** -8 * ref.abs() + K * 2.0 ** -22 * size).all())
    for m in TURNS_ROWS + TURNS_WHOLE_ROWS:
        x = a[:m].contiguous()
        assert torch.equal(B.po_op_linear(x, w, residual=r[:m].contiguous()), whole[0][:m]), m
        assert torch.equal(B.po_op_gate_up_silu(x, w), whole[1][:m]), m


@pytest.mark.parametrize("cfg,K", TURNS_QKV)
def test_qkv_turns_are_the_bits_of_a_launch_without(cfg, K):
    import torch
    from paper_2505_07203_amd import binding as B
    hq, hkv, hd = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim
    rnd = _rnd(K + 1)
    a, w, b = rnd(TURNS_TOP, K), rnd((hq + 2 * hkv) * hd, K) * 0.05, rnd((hq + 2 * hkv) * hd)
    cos, sin = B.po_op_rope_table(TURNS_TOP, hd, cfg.rope_theta)
    q, k, vt = B.po_op_qkv_rope(a, w, b, cos, sin, hq, hkv, hd)
    for m in TURNS_ROWS:
        q1, k1, vt1 = B.po_op_qkv_rope(a[:m].contiguous(), w, b, cos, sin, hq, hkv, hd)
        assert torch.equal(q1, q[:m]) and torch.equal(k1, k[:m]) and torch.equal(vt1[:, :m], vt[:, :m]), m


@pytest.mark.parametrize("N,K", TURNS_FP8 + TURNS_FP8_SHORT)
def test_fp8_turns_are_the_bits_of_a_launch_without(N, K):
    import torch
    from paper_2505_07203_amd import binding as B
    rnd = _rnd(N * K + 1)
    r = rnd(TURNS_TOP, N)
    (qa, sa), (qw, sw) = B.po_op_quantize_rows(rnd(TURNS_TOP, K)), B.po_op_quantize_rows(rnd(N, K) * 0.05)
    whole = B.po_op_linear_fp8(qa, sa, qw, sw, residual=r), B.po_op_linear_fp8(qa, sa, qw, sw, silu_mul=True)
    for m in TURNS_ROWS + TURNS_WHOLE_ROWS:
        x, s = qa[:m].contiguous(), sa[:m].contiguous()
        assert torch.equal(B.po_op_linear_fp8(x, s, qw, sw, residual=r[:m].contiguous()), whole[0][:m]), m
        assert torch.equal(B.po_op_linear_fp8(x, s, qw, sw, silu_mul=True), whole[1][:m]), m


def test_fp8_qkv_turns_are_the_bits_of_a_launch_without():
    import torch
    from paper_2505_07203_amd import binding as B
    cfg, K = TURNS_FP8_QKV
    hq, hkv, hd = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim
    rnd = _rnd(K + 2)
    (qa, sa), (qw, sw) = B.po_op_quantize_rows(rnd(TURNS_TOP, K)), B.po_op_quantize_rows(rnd((hq + 2 * hkv) * hd, K) * 0.05)
    cos, sin = B.po_op_rope_table(TURNS_TOP, hd, cfg.rope_theta)
    q, k, vt = B.po_op_qkv_rope_fp8(qa, sa, qw, sw, None, cos, sin, hq, hkv, hd)
    for m in TURNS_ROWS:
        q1, k1, vt1 = B.po_op_qkv_rope_fp8(qa[:m].contiguous(), sa[:m].contiguous(), qw, sw, None, cos, sin, hq, hkv, hd)
        assert torch.equal(q1, q[:m]) and torch.equal(k1, k[:m]) and torch.equal(vt1[:, :m], vt[:, :m]), m


@pytest.mark.parametrize("M,N,K,fp8", [(*x, False) for x in TURNS_SPLIT] + [(*x, True) for x in TURNS_FP8_SPLIT])
def test_split_sums_with_turns_against_float64(M, N, K, fp8):
    T.test_split_sums_in_every_tile_against_float64(M, N, K, fp8)
