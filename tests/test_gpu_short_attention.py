"""Attention of prescaled queries in tiles of 128 rows, which short sequences take: against float64, the bits of 256-row tiles
(a sequence long enough to take those starts with the same rows), and rows whose scores leave the range of the fast form."""
import math

import pytest

pytestmark = pytest.mark.gpu


def _inputs(n, hq, hkv, std, seed):
    import torch
    from paper_2505_07203_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    return ((rnd(n, hq, 128) * std * B.attention_q_scale(128)).to(torch.bfloat16), (rnd(n, hkv, 128) * std).to(torch.bfloat16),
            rnd(n, hkv, 128).to(torch.bfloat16))


def _check(o, q, k, v):
    import torch
    n, hq = q.shape[:2]
    mask = torch.ones(n, n, dtype=torch.bool, device="cuda").triu(1)
    for h in range(hq):
        c = h // (hq // k.shape[1])
        s = (q[:, h].double() @ k[:, c].double().t()) * math.log(2.0)
        p = s.masked_fill(mask, -math.inf).softmax(-1)
        # probabilities (2^-8 of each for its rounding to bf16 and that of the sum) and the result's own rounding
        tol = 2.0 ** -7 * (p @ v[:, c].double().abs()) + 1e-30
        assert bool(((o[:, h].double() - p @ v[:, c].double()).abs() <= tol).all()), h


# edges of 32-key blocks, 64-key tiles and 128-row tiles
@pytest.mark.parametrize("n", [1, 31, 33, 63, 64, 65, 96, 97, 127, 128, 129, 191, 193, 257, 511, 900])
def test_against_float64(n):
    from paper_2505_07203_amd import binding as B
    q, k, v = _inputs(n, 6, 2, 1.3, n)
    _check(B.po_op_attention(q, k, v, q_prescaled=True), q, k, v)


@pytest.mark.parametrize("hq,hkv", [(32, 8), (40, 8), (20, 4)])
def test_rows_are_the_bits_of_a_longer_sequence(hq, hkv):
    import torch
    from paper_2505_07203_amd import binding as B
    top = (256 // hq) * 256                           # rows up to which 128-row tiles are taken
    q, k, v = _inputs(top + 300, hq, hkv, 1.3, hq)
    whole = B.po_op_attention(q, k, v, q_prescaled=True)
    for n in (1, 33, 100, 128, 129, 250, 385, 1000, top - 1, top):
        o = B.po_op_attention(q[:n].contiguous(), k[:n].contiguous(), v[:n].contiguous(), q_prescaled=True)
        assert torch.equal(o, whole[:n]), n


# 700: tiles of 128 rows, 2200 rows of 40 heads: of 256, both redone in place
@pytest.mark.parametrize("n,hq,hkv", [(1, 4, 2), (130, 4, 2), (700, 8, 2), (2200, 40, 8)])
@pytest.mark.parametrize("kind", ["far above", "far below", "spread", "one row"])
def test_scores_out_of_range(n, hq, hkv, kind):
    import torch
    from paper_2505_07203_amd import binding as B
    q, k, v = _inputs(n, hq, hkv, 12.0 if kind == "spread" else 1.3, n)
    if kind != "spread":
        rows = slice(n // 2, n // 2 + 1) if kind == "one row" else slice(0, n)
        k[:, :, 0] = 8.0
        q[rows, :, 0] = 25.0 if kind != "far below" else -25.0          # 200 powers of two above or below
    o = B.po_op_attention(q, k, v, q_prescaled=True)
    assert torch.isfinite(o).all()
    heads = [0, hq - 1] if n > 1000 else list(range(hq))
    group = hq // hkv
    _check(o[:, heads], q[:, heads], k[:, [h // group for h in heads]], v[:, [h // group for h in heads]])
