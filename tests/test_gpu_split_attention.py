"""Few-rows attention at head dimension 128: pieces of the keys, all query heads of a KV head in one workgroup, cached prefix
read in place.  Through whole calls against the default path on the same tokens, which other tests hold to the oracle, and
as an operator of its own, every row and head against float64."""
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
    """A norm gain that puts scores hundreds of nats apart: pieces whose sums come near the end of the float range go through
    their cached and fresh keys a second time.  One rounding of a query value moves a score by up to 0.1 nats here, hence
    the wider bar."""
    _compare(_cfg(8, 2), total, cached, 30.0, 6e-2)


# ---- the operator by itself, every row and head against float64

def _operands(n, hq, hkv, hd, seed, kind="ordinary", rows=None):
    """Prescaled queries (scores in log2 units), keys, values.  Kinds that leave the range 2^-60 .. 2^100 of a row's sum of
    exponentials: "shifted" moves whole rows of some heads up or down by 140 (softmax is invariant to it), "spread" makes
    scores hundreds apart, "late" raises single late keys by 150."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    q, k, v = (torch.randn(n, h, hd, generator=g, device="cuda") for h in (hq, hkv, hkv))
    q *= 1.4 * 1.4427 * hd ** -0.5
    rows = torch.arange(n, device="cuda")[:, None]
    heads = torch.arange(hq, device="cuda")[None]
    if kind == "shifted":
        k[:, :, 0] = 8.0
        q[:, :, 0] = torch.where((rows + heads) % 3 == 0, 17.5, 0.0) - torch.where((rows + heads) % 7 == 2, 17.5, 0.0)
    elif kind == "spread":
        q *= torch.where((rows + heads) % 2 == 0, 60.0, 1.0)[..., None]
    elif kind == "late":
        k[:, :, 0] = 0.0
        k[n // 2::97, :, 0] = 8.0
        q[:, :, 0] = torch.where(heads % 2 == 0, 18.75, 0.0).expand(n, hq)
    return q.to(torch.bfloat16), k.to(torch.bfloat16), v.to(torch.bfloat16)


def _reference(q, k, v, r0):
    """Rows from r0 on in float64 -> outputs, sum p |v|, sqrt(sum p^2 v^2) (p normalised), log2 of the sums of 2^score"""
    import torch
    n, hq, hkv = q.shape[0], q.shape[1], k.shape[1]
    outs = []
    for h in range(hq):
        c = h // (hq // hkv)
        s = q[r0:, h].double() @ k[:, c].double().t()
        future = torch.arange(n, device="cuda")[None] > torch.arange(r0, n, device="cuda")[:, None]
        s = s.masked_fill(future, -float("inf")) * np.log(2.0)
        lse = torch.logsumexp(s, -1)
        p, vv = (s - lse[:, None]).exp(), v[:, c].double()
        outs.append((p @ vv, p @ vv.abs(), ((p * p) @ (vv * vv)).sqrt(), lse / np.log(2.0)))
    return [torch.stack(x, 1) for x in zip(*outs)]


def _check_rows(o, ref, r0, extra=0.0):
    """bf16 keeps 8 significant bits: a rounding is off by up to 2^-8.  Each probability is rounded once for the product with
    V (not for the sum), so a value is off by up to 2^-8 sum p |v|, and the output once more by 2^-8 of itself, which is no
    larger; float32 sums and the scores' own rounding stay below 2e-4.  That is the bound per value.  The root mean square
    over a head's dimensions, where v makes the terms as good as independent, stays below 2^-8 of sqrt(sum p^2 v^2) and of
    the output (a quarter over it for 128 samples): a missing or doubled key tile shows there."""
    want, a1, a2, _ = ref
    err = (o[r0:].double() - want).abs()
    assert float((err / a1).max()) <= 2.0 ** -7 + 2e-4 + extra
    rms = lambda x: (x * x).mean(-1).sqrt()
    assert float((rms(err) / (2.0 ** -8 * (rms(a2) + rms(want)) + (1e-5 + extra) * rms(a1))).max()) <= 1.25


SHAPES = [(8, 2), (5, 1), (3, 3), (32, 8)]


@pytest.mark.parametrize("hq,hkv", SHAPES)
@pytest.mark.parametrize("n,r0,n2", [(257, 0, 0), (300, 299, 256), (641, 577, 576), (700, 511, 448), (1003, 100, 64), (1500, 500, 0),
                                     (1411, 1408, 1408), (2200, 1500, 1472), (3137, 2987, 2944)])
def test_every_row_against_float64(n, r0, n2, hq, hkv):
    from paper_2505_07203_amd import binding as B
    q, k, v = _operands(n, hq, hkv, 128, n + hq)
    ref = _reference(q, k, v, r0)
    for prescaled in (True, False):
        x = q if prescaled else (q.float() / B.attention_q_scale(128)).to(q.dtype)
        want = ref if prescaled else _reference(x.double() * B.attention_q_scale(128), k, v, r0)
        o, pieces = _split(x, k, v, r0, n2, prescaled)
        assert pieces > 1 and not o[:r0].any()
        _check_rows(o, want, r0)


def _split(q, k, v, r0, n2, prescaled=True, **kw):
    """with the first n2 positions in a pair of their own, and poison in their place in k and v"""
    import torch
    from paper_2505_07203_amd import binding as B
    if not n2:
        return B.po_op_attention_split_prefix(q, k, v, r0, prescaled, **kw)
    n, hkv, hd = k.shape
    k2 = k[:n2].clone()
    vt2 = torch.full((hkv * hd, n2 + 128), float("nan"), dtype=v.dtype, device="cuda")
    vt2[:, :n2] = v[:n2].reshape(n2, hkv * hd).t()
    k, v = k.clone(), v.clone()
    k[:n2] = float("nan")
    v[:n2] = float("nan")
    return B.po_op_attention_split_prefix(q, k, v, r0, prescaled, k2, vt2, n2, **kw)


@pytest.mark.parametrize("kind", ["shifted", "spread", "late"])
@pytest.mark.parametrize("hq,hkv", [(8, 2), (5, 1), (3, 3)])
@pytest.mark.parametrize("n,r0,n2", [(300, 0, 0), (700, 511, 448), (2200, 2050, 2048)])
def test_rows_far_outside_the_exponent_range_against_float64(n, r0, n2, hq, hkv, kind):
    q, k, v = _operands(n, hq, hkv, 128, 7 * n + hq, kind)
    ref = _reference(q, k, v, r0)
    lse = ref[3]
    assert float(lse.max()) > 100.0 and (kind != "shifted" or float(lse.min()) < -60.0)
    assert ((lse > -60.0) & (lse < 100.0)).any()                       # and ordinary rows beside them
    o, pieces = _split(q, k, v, r0, n2)
    assert pieces > 1
    # scores of several hundred: float32 holds them to about 2e-5, their sums over 128 products to a few times that
    _check_rows(o, ref, r0, extra=2e-3 if kind == "spread" else 5e-4)


@pytest.mark.parametrize("prescaled", [True, False])
def test_sums_of_probabilities_are_not_rounded(prescaled):
    """Every 32nd key has score 0, the others -1.9945 (or -2.9945), so that their probability is 0.4 % above the bf16 value it
    is rounded to for the product with V.  V is 1 at key 0 alone, where the probability is exact: the output is one over the
    row's sum.  Rows whose exact result lies within an eighth of a bf16 step of a bf16 value, while the sum of rounded
    probabilities would give another, show which sum was formed."""
    import torch
    from paper_2505_07203_amd import binding as B
    n, r0 = 1100, 400
    q, k, v = (torch.zeros(n, h, 128, device="cuda") for h in (4, 1, 1))
    q0, k1 = (1.0, 0.0055) if prescaled else (11.75, 0.017)
    q[:, :, 0], q[:, :, 1] = q0, 1.0
    k[:, :, 0], k[:, :, 1] = -2.0, k1
    k[::32] = 0.0
    v[0] = 1.0
    q, k, v = (x.to(torch.bfloat16) for x in (q, k, v))
    score = float(-2.0 * q0 + k[1, 0, 1].double()) * (1.0 if prescaled else B.attention_q_scale(128))
    rows = torch.arange(r0, n, device="cuda", dtype=torch.float64)
    anchors = torch.floor(rows / 32) + 1
    p = torch.tensor(2.0 ** score, dtype=torch.float64, device="cuda")
    exact = 1.0 / (anchors + (rows + 1 - anchors) * p)
    other = 1.0 / (anchors + (rows + 1 - anchors) * p.to(torch.bfloat16).double())
    grid = exact.to(torch.bfloat16)
    step = 2.0 ** (torch.floor(torch.log2(exact)) - 7)
    telling = ((exact - grid.double()).abs() < step / 8) & (other.to(torch.bfloat16) != grid)
    assert int(telling.sum()) >= 5
    o, pieces = _split(q, k, v, r0, 384, prescaled)
    assert pieces > 1
    assert torch.equal(o[r0:][telling], grid[telling][:, None, None].expand(-1, 4, 128))


def test_large_values_stay_finite():
    """Scores 36 above the first key's and values near 2^95: sums of 2^score times value leave the float range (2^36 2^95),
    the averages do not."""
    q, k, v = _operands(900, 4, 1, 128, 3)
    k[:, :, 0], q[:, :, 0] = 0.0, 4.5
    k[5::7, :, 0] = 8.0
    ref = _reference(q, k, v, 700)
    o, pieces = _split(q, k, v * 2.0 ** 95, 700, 640)
    assert pieces > 1
    _check_rows(o.double() * 2.0 ** -95, ref, 700, extra=5e-4)


def _seconds(q, k, v, rows, k2=None, vt2=None, n2=0):
    """fastest of eight calls for the last `rows` rows"""
    import torch
    from paper_2505_07203_amd import binding as B
    n, hq, hd = q.shape
    vt = torch.empty(k.shape[1] * hd * ((n + 63) // 64 * 64), dtype=q.dtype, device="cuda")
    part, o = torch.empty(1 << 28, dtype=torch.uint8, device="cuda"), torch.zeros_like(q)
    splits, best = B.C.c_int32(0), 1e9
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        B.check(B.lib().po_op_attention_split_prefix(q.data_ptr(), k.data_ptr(), v.data_ptr(), o.data_ptr(), vt.data_ptr(),
                                                     part.data_ptr(), part.numel(), n, hq, k.shape[1], hd, n - rows, 1,
                                                     k2.data_ptr() if n2 else None, vt2.data_ptr() if n2 else None,
                                                     vt2.shape[1] if n2 else 0, n2, B._stream(), B.C.byref(splits)))
        b.record()
        b.synchronize()
        assert splits.value > 1
        best = min(best, a.elapsed_time(b))
    return best


@pytest.mark.parametrize("kind", ["shifted", "spread", "late"])
def test_time_does_not_depend_on_the_scores(kind):
    """A row outside the exponent range costs its workgroup another pass, not a walk over its keys one by one (which took
    hundreds of times as long): 2.5 times the work at the most, 4 leaves room for the clock."""
    ordinary, other = _seconds(*_operands(8150, 32, 8, 128, 1), 150), _seconds(*_operands(8150, 32, 8, 128, 1, kind), 150)
    print(f"150 rows behind 8000 keys: ordinary scores {ordinary * 1e3:.0f} us, {kind} {other * 1e3:.0f} us")
    assert other <= 4 * ordinary


def test_time_does_not_depend_on_where_the_prefix_lies():
    """700 rows behind 14 000 keys leave two pieces: cut at the end of the prefix one of them would be all of it."""
    q, k, v = _operands(14700, 32, 8, 128, 1)
    vt2 = v[:13952].reshape(13952, -1).t().contiguous()
    whole, pair = _seconds(q, k, v, 700), _seconds(q, k, v, 700, k, vt2, 13952)
    print(f"700 rows behind 14000 keys: {whole * 1e3:.0f} us, prefix in a pair of its own {pair * 1e3:.0f} us")
    assert pair <= 1.25 * whole


@pytest.mark.parametrize("n2", [0, 448])
def test_scratch_for_fewer_pieces(n2):
    """Scratch for two or three pieces is used as it is; for less than two nothing is computed (and the call returns)."""
    q, k, v = _operands(700, 8, 2, 128, 5)
    piece = 200 * 8 * (128 + 2) * 4
    ref = _reference(q, k, v, 500)
    for pieces in (2, 3):
        o, n = _split(q, k, v, 500, n2, part_bytes=pieces * piece + 4)
        assert n == pieces
        _check_rows(o, ref, 500)
    for part_bytes in (2 * piece - 4, piece, 64):
        o, n = _split(q, k, v, 500, n2, part_bytes=part_bytes)
        assert o is None and n <= 1


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
