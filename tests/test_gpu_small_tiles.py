"""Small block tiles of the bf16 GEMM: the tile a launch takes depends on its rows and columns, the bits must not."""
import numpy as np
import pytest

from paper_2505_07203_amd import inputs as I

pytestmark = pytest.mark.gpu

# heights at which the tiles of 32 .. 256 rows x 128 columns and 192 or 256 x 256 come in, one row off whole tiles among
# them; test_tile_forms_cpu.py holds them to taking every tile with the sizes below
ROWS = (1, 31, 33, 191, 193, 200, 257, 471, 640, 700, 901, 1025, 1281, 1537, 1931, 2300, 2700, 3500)
TOP = 4300
BF16_SHAPES = [(4096, 64), (4096, 448), (4096, 1024), (320, 128), (64, 832), (6144, 512)]
BF16_QKV = [(I.LLAMA8B, 512, True), (I.LLAMA8B, 4096, False), (I.TINY, 192, False)]
FP8_SHAPES = [(4096, 128), (4096, 896), (6144, 2048), (320, 640), (64, 1024)]
FP8_QKV_K = 4096
BF16_SPLIT = [(m, 4096, 14336) for m in (1, 65, 129, 161, 165, 193, 245, 321, 385)]
FP8_SPLIT = [(m, 4096, 14336) for m in (1, 65, 129, 385)] + [(577, 5120, 27648)]


@pytest.mark.parametrize("N,K", BF16_SHAPES)
def test_rows_are_the_same_bits_in_launches_of_every_height(N, K):
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    top = TOP
    a, r, w = rnd(top, K), rnd(top, N), rnd(N, K) * 0.05
    whole = {"store": B.po_op_linear(a, w), "residual": B.po_op_linear(a, w, residual=r), "silu": B.po_op_gate_up_silu(a, w)}
    # fp32 sums of K products of size |a||w|, then one bf16 rounding
    ref = (a.double() @ w.double().t()).cpu().numpy()
    tol = 2.0 ** -8 * np.abs(ref) + K * 2.0 ** -22 * (a.double().abs() @ w.double().abs().t()).cpu().numpy()
    assert np.all(np.abs(whole["store"].double().cpu().numpy() - ref) <= tol)
    for m in ROWS:
        x = a[:m].contiguous()
        assert torch.equal(B.po_op_linear(x, w), whole["store"][:m]), m
        assert torch.equal(B.po_op_linear(x, w, residual=r[:m].contiguous()), whole["residual"][:m]), m
        assert torch.equal(B.po_op_gate_up_silu(x, w), whole["silu"][:m]), m


@pytest.mark.parametrize("cfg,K,bias", BF16_QKV)
def test_qkv_rows_are_the_same_bits_in_launches_of_every_height(cfg, K, bias):
    import torch
    from paper_2505_07203_amd import binding as B
    hq, hkv, hd = cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim
    g = torch.Generator(device="cuda").manual_seed(K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    top = TOP
    a, w = rnd(top, K), rnd((hq + 2 * hkv) * hd, K) * 0.05
    b = rnd((hq + 2 * hkv) * hd) if bias else None
    cos, sin = B.po_op_rope_table(top, hd, cfg.rope_theta)
    q, k, vt = B.po_op_qkv_rope(a, w, b, cos, sin, hq, hkv, hd)
    for m in ROWS:
        q1, k1, vt1 = B.po_op_qkv_rope(a[:m].contiguous(), w, b, cos, sin, hq, hkv, hd)
        assert torch.equal(q1, q[:m]) and torch.equal(k1, k[:m]) and torch.equal(vt1[:, :m], vt[:, :m]), m


@pytest.mark.parametrize("N,K", FP8_SHAPES)
def test_fp8_rows_are_the_same_bits_in_launches_of_every_height(N, K):
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(N + K)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    top = TOP
    r = rnd(top, N)
    (qa, sa), (qw, sw) = B.po_op_quantize_rows(rnd(top, K)), B.po_op_quantize_rows(rnd(N, K) * 0.05)
    whole = {"store": B.po_op_linear_fp8(qa, sa, qw, sw), "residual": B.po_op_linear_fp8(qa, sa, qw, sw, residual=r),
             "silu": B.po_op_linear_fp8(qa, sa, qw, sw, silu_mul=True)}
    val = lambda q, s: q.view(torch.float8_e4m3fn).double() * s.double()[:, None]
    ref = (val(qa, sa) @ val(qw, sw).t()).cpu().numpy()
    tol = 2.0 ** -8 * np.abs(ref) + K * 2.0 ** -22 * (val(qa, sa).abs() @ val(qw, sw).abs().t()).cpu().numpy()
    assert np.all(np.abs(whole["store"].double().cpu().numpy() - ref) <= tol)
    for m in ROWS:
        x, s = qa[:m].contiguous(), sa[:m].contiguous()
        assert torch.equal(B.po_op_linear_fp8(x, s, qw, sw), whole["store"][:m]), m
        assert torch.equal(B.po_op_linear_fp8(x, s, qw, sw, residual=r[:m].contiguous()), whole["residual"][:m]), m
        assert torch.equal(B.po_op_linear_fp8(x, s, qw, sw, silu_mul=True), whole["silu"][:m]), m


@pytest.mark.parametrize("bias", [True, False])
def test_fp8_qkv_rows_are_the_same_bits_in_launches_of_every_height(bias):
    import torch
    from paper_2505_07203_amd import binding as B
    hq, hkv, hd, K = 32, 8, 128, FP8_QKV_K
    g = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    top = TOP
    (qa, sa), (qw, sw) = B.po_op_quantize_rows(rnd(top, K)), B.po_op_quantize_rows(rnd((hq + 2 * hkv) * hd, K) * 0.05)
    b = rnd((hq + 2 * hkv) * hd) if bias else None
    cos, sin = B.po_op_rope_table(top, hd, 500000.0)
    q, k, vt = B.po_op_qkv_rope_fp8(qa, sa, qw, sw, b, cos, sin, hq, hkv, hd)
    for m in ROWS:
        q1, k1, vt1 = B.po_op_qkv_rope_fp8(qa[:m].contiguous(), sa[:m].contiguous(), qw, sw, b, cos, sin, hq, hkv, hd)
        assert torch.equal(q1, q[:m]) and torch.equal(k1, k[:m]) and torch.equal(vt1[:, :m], vt[:, :m]), m


@pytest.mark.parametrize("M,N,K,fp8", [(*x, False) for x in BF16_SPLIT] + [(*x, True) for x in FP8_SPLIT])
def test_split_sums_in_every_tile_against_float64(M, N, K, fp8):
    """Partial sums of few-rows mode, tile by tile: against float64, and the splits and the tile the planner names."""
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(M + N)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    a, w, r = rnd(M, K), rnd(N, K) * 0.05, rnd(M, N)
    if fp8:
        qa, qw = B.po_op_quantize_rows(a), B.po_op_quantize_rows(w)
        c, splits = B.po_op_linear_fp8_split(*qa, *qw, r)
        a, w = (x.view(torch.float8_e4m3fn).double() * y.double()[:, None] for x, y in (qa, qw))
    else:
        c, splits = B.po_op_linear_split(a, w, r)
        a, w = a.double(), w.double()
    assert splits == B.po_gemm_tile(M, N, K, 0, fp8)[2] > 1
    ref = a @ w.t() + r.double()
    # fp32 sums of K products of size |a||w|, then one bf16 rounding
    tol = 2.0 ** -8 * ref.abs() + K * 2.0 ** -22 * (a.abs() @ w.abs().t())
    assert bool(((c.double() - ref).abs() <= tol).all())


def _rotated(a, b, cos, sin, first_fused):
    """(a cos - b sin, second half) in float32 with one product of each sum fused: bf16 GEMM b cos + [a sin], FP8 GEMM
    a sin + [b cos] (the bracketed product unrounded); a, b, cos, sin float32 tensors."""
    import torch
    fma = lambda x, y, z: (x.double() * y.double() + z.double()).float()
    lo = fma(a, cos, -(b * sin))
    return lo, fma(a, sin, b * cos) if first_fused else fma(b, cos, a * sin)


@pytest.mark.parametrize("m", [64, 3000])
@pytest.mark.parametrize("fp8", [False, True])
def test_rotation_keeps_its_rounding(fp8, m):
    """One-hot activations make every accumulator exact, so the stored bits show which product of the rotation is rounded:
    part of the library's results, the same in every tile form and from version to version."""
    import torch
    from paper_2505_07203_amd import binding as B
    hq, hkv, hd, K = 16, 4, 128, 128
    g = torch.Generator(device="cuda").manual_seed(m)
    scale = torch.randn(m, generator=g, device="cuda").to(torch.bfloat16)
    hot = torch.arange(m, device="cuda") % K
    codes = torch.randint(0, 0x78, ((hq + 2 * hkv) * hd, K), generator=g, device="cuda").to(torch.uint8)      # E4M3, below 2^8
    w = codes.view(torch.float8_e4m3fn).to(torch.bfloat16) if fp8 else torch.randn(codes.shape, generator=g, device="cuda").to(torch.bfloat16)
    wqkv, _ = B.po_op_pack_qkv(w[:hq * hd].contiguous(), w[hq * hd:(hq + hkv) * hd].contiguous(), w[(hq + hkv) * hd:].contiguous(),
                               hq, hkv, hd)
    cos, sin = B.po_op_rope_table(m, hd, 500000.0)
    if fp8:
        a8 = torch.zeros(m, K, dtype=torch.uint8, device="cuda")
        a8[torch.arange(m, device="cuda"), hot] = 0x38                                                  # 1.0
        w8 = wqkv.float().to(torch.float8_e4m3fn).view(torch.uint8).contiguous()
        q, k, _ = B.po_op_qkv_rope_fp8(a8, scale.float(), w8, torch.ones(w8.shape[0], device="cuda"), None, cos, sin, hq, hkv, hd)
    else:
        a = torch.zeros(m, K, dtype=torch.bfloat16, device="cuda")
        a[torch.arange(m, device="cuda"), hot] = scale
        q, k, _ = B.po_op_qkv_rope(a, wqkv, None, cos, sin, hq, hkv, hd)
    acc = (w.float()[:, hot].t() * scale.float()[:, None])[:, :(hq + hkv) * hd].view(m, hq + hkv, hd)      # exact: 16 bits
    lo, hi = _rotated(acc[..., :hd // 2], acc[..., hd // 2:], cos[:, None], sin[:, None], not fp8)
    want = torch.cat((lo, hi), -1).to(torch.bfloat16)
    got = torch.cat((q.view(m, hq, hd), k.view(m, hkv, hd)), 1)
    assert int((got != want).sum()) == 0


@pytest.mark.parametrize("N,K", [(4096, 64), (4096, 100), (1030, 688), (256, 4), (33, 1000)])
def test_f32_rows_are_the_same_bits_in_launches_of_every_height(N, K):
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(N + K)
    top = TOP
    a, r, w = (torch.randn(*s, generator=g, device="cuda") for s in ((top, K), (top, N), (N, K)))
    whole, whole_r = B.po_op_linear(a, w), B.po_op_linear(a, w, residual=r)
    ref = (a.double() @ w.double().t()).cpu().numpy()
    tol = K * 2.0 ** -24 * (a.double().abs() @ w.double().abs().t()).cpu().numpy()      # K sequential float32 additions
    assert np.all(np.abs(whole.double().cpu().numpy() - ref) <= tol + 2.0 ** -24 * np.abs(ref))
    for m in ROWS:
        x = a[:m].contiguous()
        assert torch.equal(B.po_op_linear(x, w), whole[:m]), m
        assert torch.equal(B.po_op_linear(x, w, residual=r[:m].contiguous()), whole_r[:m]), m


def test_f32_rows_of_more_than_a_million_elements():
    """Above 2^20 elements per row only the tiles whose offsets still fit are taken, not the plain kernel: right, and no
    step in time from one side of that size to the other."""
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(3)
    a, w = (torch.randn(m, 2 ** 20 + 64, generator=g, device="cuda") for m in (70, 40))
    us = {}
    for K in (2 ** 20 - 32, 2 ** 20 + 60):
        x, y = a[:, :K].contiguous(), w[:, :K].contiguous()
        ref, size = x.double() @ y.double().t(), x.double().abs() @ y.double().abs().t()
        # one running sum of K terms: its roundings add up like a walk of sqrt(K) steps (a fixed sum of K would allow 6 %)
        assert float(((B.po_op_linear(x, y).double() - ref).abs() / size).max()) <= 8 * K ** 0.5 * 2.0 ** -24
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(6)]
        for e in ev:
            B.po_op_linear(x, y)
            e.record()
        torch.cuda.synchronize()
        us[K] = min(i.elapsed_time(j) for i, j in zip(ev, ev[1:])) * 1e3
    print("70 x 40 outputs:", {k: round(v) for k, v in us.items()}, "us")
    assert max(us.values()) <= 2 * min(us.values())


@pytest.mark.parametrize("Hq,Hkv,hd,n", [(4, 2, 64, 1700), (4, 1, 128, 1200), (2, 2, 128, 33)])
def test_f32_attention_rows_do_not_depend_on_the_length(Hq, Hkv, hd, n):
    """Rows below and above the change of work split: against float64, and the same bits in a shorter sequence."""
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn(n, h, hd, generator=g, device="cuda") for h in (Hq, Hkv, Hkv))
    q = q * 2
    o = B.po_op_attention(q, k, v)
    mask = torch.ones(n, n, dtype=torch.bool, device="cuda").tril()
    for h in range(Hq):
        c = h // (Hq // Hkv)
        s = (q[:, h].double() @ k[:, c].double().t()) * hd ** -0.5
        ref = s.masked_fill(~mask, -float("inf")).softmax(-1) @ v[:, c].double()
        # float32 dot products of hd terms in the exponent, sums of n non-negative terms
        assert (o[:, h].double() - ref).abs().max().item() <= 4e-6 * v.abs().max().item()
    for m in (1, 31, 32, 33, 127, 129, 1023, 1024, 1025, 1100, 1535, 1537, 1601):
        if m < n:
            assert torch.equal(B.po_op_attention(q[:m].contiguous(), k[:m].contiguous(), v[:m].contiguous()), o[:m]), m


@pytest.mark.parametrize("hd,n", [(64, 200), (64, 1700), (128, 200), (128, 1200)])
def test_f32_attention_with_whole_tiles_at_minus_infinity(hd, n):
    """Scores whose product overflows to -inf have probability 0, also where they fill all the tiles that one of the four
    wavefronts of an early row's workgroup sees, or its first ones."""
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(n)
    q, k, v = (torch.randn(n, h, hd, generator=g, device="cuda") for h in (2, 1, 1))
    q[:, :, 0], k[:, :, 0] = 1e20, 0.0
    gone = torch.zeros(n, dtype=torch.bool, device="cuda")
    for tile in (1, 3, 5, 6, 9, 13):
        gone[32 * tile:32 * tile + 32] = True
    k[gone, :, 0] = -1e20
    o = B.po_op_attention(q, k, v)
    assert torch.isfinite(o).all()
    mask = torch.ones(n, n, dtype=torch.bool, device="cuda").tril() & ~gone[None]
    for h in range(2):
        s = (q[:, h, 1:].double() @ k[:, 0, 1:].double().t()) * hd ** -0.5
        ref = s.masked_fill(~mask, -float("inf")).softmax(-1) @ v[:, 0].double()
        assert (o[:, h].double() - ref).abs().max().item() <= 4e-6 * v.abs().max().item()


@pytest.mark.parametrize("hd,n", [(64, 100), (128, 1200)])
def test_f32_attention_four_bytes_off_a_16_byte_boundary(hd, n):
    """Keys and values are copied to LDS 16 bytes at a time from wherever they start."""
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(n)
    x = [torch.randn(n, h, hd, generator=g, device="cuda") for h in (4, 2, 2)]
    off = [torch.empty(t.numel() + 1, device="cuda")[1:].view(t.shape).copy_(t) for t in x]
    assert all(t.data_ptr() % 16 == 4 for t in off)
    assert torch.equal(B.po_op_attention(*off), B.po_op_attention(*x))
