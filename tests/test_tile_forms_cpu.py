"""The sizes of the GPU tests of the GEMM block tiles reach every tile that launches take (the choice is a host function of
sizes): a refit of its constants that moved a tile out of the tests' sizes fails here."""
import pytest

import test_gpu_f32_pairs as P
import test_gpu_small_tiles as T
import test_gpu_strips as S
from paper_2505_07203_amd import binding as B
from paper_2505_07203_amd import inputs as I

BF16 = {(r, 128) for r in (32, 64, 96, 128, 160, 192, 256)} | {(192, 256), (256, 256)}
STRIPS = (16, 16)
FP8 = {(r, 128) for r in (64, 128, 192, 256)} | {(256, 256)}


def qkv_columns(cfg):
    return cfg.q_dim + 2 * cfg.kv_dim


def tiles(shapes, fp8=False):
    return {B.po_gemm_tile(m, N, K, 1, fp8)[:2] for N, K in shapes for m in T.ROWS + (T.TOP,)}


def test_whole_launches():
    assert tiles(T.BF16_SHAPES) == BF16 | {STRIPS}
    assert tiles([(qkv_columns(cfg), K) for cfg, K, _ in T.BF16_QKV]) == BF16 | {STRIPS}
    assert tiles(T.FP8_SHAPES, True) == FP8
    assert tiles([(qkv_columns(I.LLAMA8B), T.FP8_QKV_K)], True) == FP8


def test_split_launches():
    for shapes, fp8, every in ((T.BF16_SPLIT, False, BF16), (T.FP8_SPLIT, True, FP8)):
        got = [B.po_gemm_tile(M, N, K, 0, fp8) for M, N, K in shapes]
        assert all(s > 1 for _, _, s in got)
        assert {(r, c) for r, c, _ in got} == every


@pytest.mark.parametrize("cfg", [I.LLAMA8B, I.QWEN32B])
def test_no_launch_of_the_models_takes_another_tile(cfg):
    d, F = cfg.d_model, cfg.ffn_dim
    for N, K in ((qkv_columns(cfg), d), (d, cfg.q_dim), (2 * F, d), (d, F)):
        for splits in (0, 1):
            assert {B.po_gemm_tile(m, N, K, splits)[:2] for m in range(1, 4400, 7)} <= BF16 | {STRIPS}
            assert {B.po_gemm_tile(m, N, K, splits, True)[:2] for m in range(1, 4400, 7)} <= FP8


def test_strips():
    tile = lambda m, N, K=4096: B.po_gemm_tile(m, N, K)[:2]
    assert {tile(m, N, K) for m in (1, 2, 3, 16) for N in (64, 4096, 8192) for K in (64, 4096)} == {STRIPS}
    # more than a round of them: only with long K
    assert {tile(16, 16384), tile(16, 8256), tile(1, 12288, 1024)} == {STRIPS}
    assert STRIPS not in {tile(3, 8256, 4032), tile(1, 12352, 1024)}
    assert STRIPS not in {tile(17, 4096), tile(16, 16448), B.po_gemm_tile(1, 4096, 4096, 2)[:2], B.po_gemm_tile(1, 4096, 4096, 1, True)[:2]}


def test_arguments():
    L, n, r, c = B.lib(), B.C.c_int32(1), B.C.c_int32(0), B.C.c_int32(0)
    ask = lambda *a: L.po_gemm_tile(*a, B.C.byref(n), B.C.byref(r), B.C.byref(c))
    assert ask(2, 1, 64, 64) == ask(0, 0, 64, 64) == B.PO_ERR_INVALID_ARG
    assert ask(0, 1, 65, 64) == ask(0, 1, 64, 96) == ask(1, 1, 64, 64) == B.PO_ERR_BAD_CONFIG
    n.value = 9
    assert ask(0, 1, 64, 1024) == B.PO_ERR_INVALID_ARG
    n.value = 2
    assert ask(0, 1, 64, 64) == B.PO_ERR_BAD_CONFIG
    assert L.po_gemm_turns(None, 2, 1, 64, 64, 1, B.C.byref(r)) == L.po_gemm_turns(None, 0, 1, 64, 64, 1, None) == B.PO_ERR_INVALID_ARG
    assert L.po_gemm_turns(None, 0, 1, 64, 64, 2, B.C.byref(r)) == B.PO_ERR_BAD_CONFIG


def test_turns_where_row_tiles_wait_for_weights():
    turns = B.po_gemm_turns
    # two row tiles, whole or as K splits, have nobody to take turns with
    for M, N, K, splits in ((50, 4096, 4096, 1), (48, 4096, 4096, 0), (100, 4096, 14336, 0), (100, 8192, 8192, 0)):
        assert not turns(M, N, K, splits), (M, N, K)
    assert not any(turns(M, N, K, 0, True) for M, N, K in ((70, 5120, 5120), (100, 4096, 14336), (130, 4096, 4096)))
    # a last row tile with few rows runs ahead of the others by itself
    assert [turns(m, 4096, 14336) for m in (900, 1000)] == [False, True]
    assert [turns(m, 5120, 27648, fp8=True) for m in (400, 471)] == [False, True]
    # whatever the pitch of the weight rows and the length of K
    for N, K in ((4096, 4096), (5120, 5120), (3072, 3072), (5120, 27648)):
        assert all(turns(m, N, K) for m in (150, 300, 471, 540)), (N, K)
    # FP8 tiles of 64 rows: from 40 slices on
    assert [turns(300, K, K, fp8=True) for K in (3072, 4096, 5120)] == [False, False, True]


def test_no_turns_in_a_model_whose_weights_stay_in_the_memory_side_cache():
    at = lambda **k: I.LLAMA8B.replace(dtype=k.pop("dtype", I.BF16), **k)
    turns = lambda cfg: B.po_gemm_turns(300, 4096, 4096, model=cfg)
    small = dict(d_model=1024, n_q_heads=8, n_kv_heads=2, ffn_dim=4096)           # 31.5 MB a layer
    assert B.po_gemm_turns(300, 4096, 4096) and turns(at())
    for vocab, layers, cached in ((4096, 7, True), (4096, 8, False), (100000, 2, False), (100000, 0, True)):
        assert turns(at(n_layers=layers, vocab_size=vocab, **small)) != cached
    fp8 = at(n_layers=12, vocab_size=4096, dtype=I.BF16_FP8, **small)
    assert not B.po_gemm_turns(471, 5120, 5120, fp8=True, model=fp8) and B.po_gemm_turns(471, 5120, 5120, fp8=True)


def test_launches_of_the_gpu_tests_take_turns_in_every_tile():
    """... and are compared with launches that do not"""
    def reached(shapes, fp8=False):
        assert not any(B.po_gemm_turns(S.TURNS_TOP, N, K, 1, fp8) for N, K in shapes)
        return {B.po_gemm_tile(m, N, K, 1, fp8)[0] for N, K in shapes for m in S.TURNS_ROWS if B.po_gemm_turns(m, N, K, 1, fp8)}

    def split(launches, fp8=False):
        assert all(B.po_gemm_turns(*x, 0, fp8) and B.po_gemm_tile(*x, 0, fp8)[2] > 1 for x in launches)
        return {B.po_gemm_tile(*x, 0, fp8)[0] for x in launches}

    low = {32, 64, 96, 128, 160, 256}
    assert reached(S.TURNS_BF16[1:2]) == reached(S.TURNS_BF16[2:] + S.TURNS_BF16[:1]) == low
    assert reached([(qkv_columns(c), K) for c, K in S.TURNS_QKV]) == split(S.TURNS_SPLIT) == low
    cfg, K = S.TURNS_FP8_QKV
    assert reached(S.TURNS_FP8, True) == reached([(qkv_columns(cfg), K)], True) == split(S.TURNS_FP8_SPLIT, True) == {64, 128}
    assert all(K // 64 % 2 for _, K in S.TURNS_BF16 + S.TURNS_QKV) and all(K // 128 % 2 for _, K in S.TURNS_FP8)


def test_float32_launches_of_the_gpu_tests_take_every_tile():
    tile = B.po_gemm_f32_tile
    assert [tile(M, 2 * F, K) for M, F, K in P.GATE_UP] == [32, 32, 32, 32, 64, 128]
    of = lambda rows: [tile(rows(n), (hq + 2 * hkv) * hd, d, hd) for hd, hq, hkv, d, n in P.QKV]
    assert of(lambda n: P.QKV_CHUNK) == [32, 32, 32]
    assert of(lambda n: n) == [64, 64, 32] and of(lambda n: 2 * n) == [64, 128, 64]
    f, t = B.lib().po_gemm_f32_tile, B.C.c_int32(0)
    assert f(0, 4, 4, 0, B.C.byref(t)) == f(1, 4, 4, 32, B.C.byref(t)) == f(1, 4, 4, 0, None) == B.PO_ERR_INVALID_ARG
    assert f(1, 4, 6, 0, B.C.byref(t)) == B.PO_ERR_BAD_CONFIG
