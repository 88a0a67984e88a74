"""The GEMM for outputs of few tiles (its waves split the reduction) and the reduction splits of
the tile configurations, bit-exact against the oracle: every variant at the edges of its tiles, with
reductions shorter than the shares, forced fold segments, several workgroups per tile, residues
and reductions over several launches."""
import numpy as np
import pytest
import torch

from oracle import gemm as oracle_gemm
from paper_2609_24519_amd import awe, inputs
from tests.gpu_helpers import device, to_dev

pytestmark = pytest.mark.gpu

TILES = {1: (128, 128), 2: (64, 128), 3: (64, 64), 4: (32, 32), 5: (32, 64), 6: (64, 32)}
ENCS = [awe.ENC_AWE6, awe.ENC_AWE4, awe.ENC_B13, awe.ENC_TERNARY, awe.ENC_FP6K3, awe.ENC_FP6P4]


def _product(enc, A, B, out, kseg=0, ldc_pad=0):
    M, K = A.shape
    N = B.shape[1]
    dA, dB = to_dev(A), to_dev(B)
    pa = torch.empty(awe.plane_bytes(enc, 0, awe.SIDE_A, M, K), dtype=torch.uint8, device=device())
    pb = torch.empty(awe.plane_bytes(enc, 0, awe.SIDE_B, N, K), dtype=torch.uint8, device=device())
    awe.encode(enc, 0, awe.SIDE_A, dA, M, K, K, pa)
    awe.encode(enc, 0, awe.SIDE_B, dB, N, K, N, pb)
    C = torch.full((M, N + ldc_pad), -7, dtype=out, device=device())
    awe.gemm_planes(enc, 0, M, N, K, pa, pb, C, N + ldc_pad, awe.I64 if out == torch.int64 else awe.I32, kseg)
    torch.cuda.synchronize()
    C = C.cpu().numpy()
    assert (C[:, N:] == -7).all()
    return C[:, :N].astype(np.int64)


def _operands(enc, M, N, K, seed):
    info = awe.get_encoding_info(enc)
    return inputs.int8_pair(M, N, K, seed, info["range_a"], info["range_b"])


@pytest.mark.parametrize("variant", sorted(TILES))
@pytest.mark.parametrize("enc", ENCS)
def test_every_variant(monkeypatch, variant, enc):
    monkeypatch.setenv("AWE_GEMM_SLICE", str(variant))
    bm, bn = TILES[variant]
    # one ragged tile with a reduction shorter than the shares; more than a tile either way, an odd
    # ldc and several items per share; whole tiles
    for M, N, K, pad, out in [(bm - 1, 1, 1, 0, torch.int32), (bm + 1, 2 * bn + 3, 1300, 2, torch.int32),
                              (2 * bm, bn, 515, 0, torch.int64)]:
        A, B = _operands(enc, M, N, K, variant * 100 + M)
        assert np.array_equal(_product(enc, A, B, out, ldc_pad=pad), oracle_gemm.gemm_i64(A, B)), (M, N, K)


@pytest.mark.parametrize("variant", [1, 3, 4])
@pytest.mark.parametrize("enc", [awe.ENC_AWE6, awe.ENC_FP6P4])
@pytest.mark.parametrize("split", ["1", "3"])
def test_fold_segments_and_split_tiles(monkeypatch, variant, enc, split):
    monkeypatch.setenv("AWE_GEMM_SLICE", str(variant))
    monkeypatch.setenv("AWE_GEMM_SLICE_SPLIT", split)
    A, B = _operands(enc, 70, 133, 2600, 5)
    ref = oracle_gemm.gemm_i64(A, B)
    for kseg in (awe.K_PAD, 2 * awe.K_PAD, 0):
        for out in (torch.int32, torch.int64):
            assert np.array_equal(_product(enc, A, B, out, kseg, 1), ref), (kseg, out)


@pytest.mark.parametrize("variant", sorted(TILES))
@pytest.mark.parametrize("m", [7, 89, 157])
def test_residues(monkeypatch, variant, m):
    monkeypatch.setenv("AWE_GEMM_SLICE", str(variant))
    for M, N, K in [(1, 1, 1), (130, 70, 1111)]:
        A, B = inputs.residue_pair(M, N, K, m)
        C = awe.matmul_mod(m, to_dev(A), to_dev(B)).cpu().numpy()
        assert np.array_equal(C, oracle_gemm.gemm_mod(m, A, B)), (M, N, K)


def test_several_launches_add_up(monkeypatch):
    # int8 launches cover 130,816 indices; the second adds into C, with and without split tiles
    A, B = inputs.int8_pair(33, 40, 150000, 9)
    ref = oracle_gemm.gemm_i64(A, B)
    for variant, split in (("4", "1"), ("3", "4"), ("1", "2")):
        monkeypatch.setenv("AWE_GEMM_SLICE", variant)
        monkeypatch.setenv("AWE_GEMM_SLICE_SPLIT", split)
        assert np.array_equal(_product(awe.ENC_AWE6, A, B, torch.int64), ref), (variant, split)


@pytest.mark.parametrize("parts", ["2", "3", "5"])
@pytest.mark.parametrize("enc,out", [(awe.ENC_AWE6, torch.int32), (awe.ENC_AWE4, torch.int64), (awe.ENC_B13, torch.int32),
                                     (awe.ENC_FP6K3, torch.int32), (awe.ENC_FP6P4, torch.int64),
                                     (awe.ENC_FP8FP4, torch.int32), (awe.ENC_FP16, torch.int64),
                                     (awe.ENC_FP16, torch.int32)])
def test_split_of_every_tile(monkeypatch, parts, enc, out):
    # fewer tiles than CUs: each tile's reduction in `parts` parts, the last one shorter
    monkeypatch.setenv("AWE_GEMM_SPLIT", parts)
    if enc == awe.ENC_FP16:  # (its parts add through the epilogue of the outer groups)
        rng = np.random.default_rng(int(parts))
        K = 2900 if out == torch.int64 else 500  # what int32 holds
        A, B = (inputs.uniform(rng, s, -2048, 2047, np.int16) for s in ((300, K), (K, 270)))
        assert np.array_equal(_product(enc, A, B, out, ldc_pad=1), oracle_gemm.gemm_i64_wide(A, B))
        return
    A, B = _operands(enc, 300, 270, 2900, int(parts))
    assert np.array_equal(_product(enc, A, B, out, ldc_pad=1), oracle_gemm.gemm_i64(A, B))


@pytest.mark.parametrize("K,parts", [(1, "2"), (257, "3"), (257, "4"), (1025, "5"), (1100, "4")])
def test_short_and_empty_parts(monkeypatch, K, parts):
    # stages of 128: one, 3 (one each; more parts than stages), 9 in 5 parts (the last has one), 9 in 4
    # (3, 3, 3 and none)
    monkeypatch.setenv("AWE_GEMM_CFG", "17")
    monkeypatch.setenv("AWE_GEMM_SPLIT", parts)
    for out in (torch.int32, torch.int64):
        A, B = _operands(awe.ENC_AWE6, 300, 270, K, int(parts))
        assert np.array_equal(_product(awe.ENC_AWE6, A, B, out, ldc_pad=1), oracle_gemm.gemm_i64(A, B))


def test_chosen_route_on_mixed_shapes():
    # the library's own choice, over shapes that take different routes
    for enc, M, N, K in [(awe.ENC_AWE6, 16, 2000, 1500), (awe.ENC_B13, 700, 130, 900), (awe.ENC_AWE6, 64, 64, 20000),
                         (awe.ENC_FP6P4, 130, 900, 700), (awe.ENC_TERNARY, 1, 5000, 300), (awe.ENC_AWE4, 2100, 1900, 300)]:
        A, B = _operands(enc, M, N, K, M)
        assert np.array_equal(_product(enc, A, B, torch.int32), oracle_gemm.gemm_i64(A, B)), (enc, M, N, K)


@pytest.mark.parametrize("enc", [awe.ENC_AWE6, awe.ENC_AWE6ALT, awe.ENC_AWE4, awe.ENC_B13, awe.ENC_TERNARY])
@pytest.mark.parametrize("K", [1, 64, 65, 255, 256, 257, 512])
def test_small_products_in_one_kernel(monkeypatch, enc, K):
    # encode, products and reconstruction in one launch (one brick per wave: 8 waves up to K = 256, 16 up
    # to 512), against the oracle and against the separate launches; unaligned rows, ldc > N, both
    # output types
    for M, N, out in [(1, 1, torch.int32), (33, 31, torch.int64), (64, 96, torch.int32)]:
        A, B = _operands(enc, M, N, K, K + M)
        ref = oracle_gemm.gemm_i64(A, B)
        dA = torch.full((M, K + 3), 127, dtype=torch.int8, device=device())
        dB = torch.full((K, N + 5), 127, dtype=torch.int8, device=device())
        dA[:, :K], dB[:, :N] = to_dev(A), to_dev(B)
        ws_n = awe.workspace_bytes(enc, 0, M, N, K)
        ws = torch.empty(max(ws_n, 1), dtype=torch.uint8, device=device())
        flag = torch.zeros(1, dtype=torch.int32, device=device())
        for direct in ("1", "0"):
            monkeypatch.setenv("AWE_GEMM_DIRECT", direct)
            C = torch.full((M, N + 2), -7, dtype=out, device=device())
            awe.gemm_exact(enc, M, N, K, dA, K + 3, dB, N + 5, C, N + 2, awe.I64 if out == torch.int64 else awe.I32,
                           ws, ws_n, flag)
            C = C.cpu().numpy()
            assert np.array_equal(C[:, :N].astype(np.int64), ref) and (C[:, N:] == -7).all(), (M, N, direct)
            assert flag.item() == 0


@pytest.mark.parametrize("m,K", [(7, 256), (89, 300), (157, 512)])
def test_small_residue_products_in_one_kernel(monkeypatch, m, K):
    monkeypatch.setenv("AWE_GEMM_DIRECT", "1")
    A, B = inputs.residue_pair(70, 45, K, m)
    assert np.array_equal(awe.matmul_mod(m, to_dev(A), to_dev(B)).cpu().numpy(), oracle_gemm.gemm_mod(m, A, B))


@pytest.mark.parametrize("side", ["a", "b"])
def test_small_product_range_flag(side):
    A, B = inputs.int8_pair(40, 50, 100, 1, (-8, 7))
    flag = torch.zeros(1, dtype=torch.int32, device=device())
    awe.matmul_exact(to_dev(A), to_dev(B), awe.ENC_AWE4, d_range_flag=flag)
    assert flag.item() == 0
    t, u = inputs.int8_pair(40, 50, 100, 1, (-1, 1))
    bad = A.copy()
    bad[39, 99] = 8  # past int4
    awe.matmul_exact(to_dev(bad if side == "a" else t), to_dev(B if side == "a" else u),
                     awe.ENC_AWE4 if side == "a" else awe.ENC_TERNARY, d_range_flag=flag)
    assert (flag.item() != 0) == (side == "a")
    flag.zero_()
    r = np.full((100, 50), 6, np.uint8)
    r[99, 49] = 7  # past the residues of 7
    awe.matmul_mod(7, to_dev(np.zeros((40, 100), np.uint8)), to_dev(r), d_range_flag=flag)
    assert flag.item() != 0


@pytest.mark.parametrize("where", ["on_a", "on_b", "tail_of_a"])
def test_small_product_written_over_an_operand(where):
    # C in an operand's memory: all of A and B is read before C is written
    M, N, K = 256, 256, 256
    A, B = _operands(awe.ENC_AWE6, M, N, K, 3)
    buf = torch.zeros(M * K + 4 * M * N, dtype=torch.uint8, device=device())
    x = A if where != "on_b" else B
    at = 0 if where != "tail_of_a" else 1024
    buf[:M * K] = to_dev(x).reshape(-1).view(torch.uint8)
    mine = buf[:M * K].view(torch.int8)
    C = buf[at:at + 4 * M * N].view(torch.int32)
    ws_n = awe.workspace_bytes(awe.ENC_AWE6, 0, M, N, K)
    ws = torch.empty(ws_n, dtype=torch.uint8, device=device())
    a, b = (mine, to_dev(B)) if where != "on_b" else (to_dev(A), mine)
    awe.gemm_exact(awe.ENC_AWE6, M, N, K, a, K, b, N, C, N, awe.I32, ws, ws_n, None)
    got = C.cpu().numpy().reshape(M, N).astype(np.int64)
    assert np.array_equal(got, oracle_gemm.gemm_i64(A, B))
