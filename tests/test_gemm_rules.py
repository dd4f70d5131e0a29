"""The rules that choose between the two copies of a matrix (csrc/gemm_rules.h), compiled for the host: which GEMMs of few token rows
read the weights as they lie."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(__file__), "..", "paper_2209_09130_amd", "csrc")


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    d = tmp_path_factory.mktemp("rules")
    (d / "rules.cpp").write_text('#include "gemm_rules.h"\n'
                                 'extern "C" int f16(long rows, int N, int K, long cus) { return samp::f16_reads_rows(rows, N, K, cus); }\n'
                                 'extern "C" int i8(long rows, int N, int K) { return samp::i8_reads_rows(rows, N, K); }\n'
                                 'extern "C" int one_packed(int i8, int packed, int S, int H) { return samp::qkv_attention_packed(i8, packed, S, H); }\n'
                                 'extern "C" int tile(long rows, int fewer, int N, int K) { return samp::stream_tile(rows, fewer, N, K); }\n'
                                 'extern "C" double cost(int t, long rows, int percent, int N, int K) {\n'
                                 '    return samp::stream_cost(samp::STREAM_TILES[t], rows, percent, N, K); }\n'
                                 'extern "C" int asks(int am, int nm, int h, int n) { samp::Asks a = samp::who_asks(am, nm, h, n);\n'
                                 '    return a.attention + 2 * a.norm1 + 4 * a.norm2_qkv + 8 * a.norm2_out; }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, "-o", str(d / "rules.so"), str(d / "rules.cpp")], check=True)
    lib = C.CDLL(str(d / "rules.so"))
    lib.f16.argtypes = [C.c_long, C.c_int, C.c_int, C.c_long]
    lib.i8.argtypes = [C.c_long, C.c_int, C.c_int]
    lib.tile.argtypes = [C.c_long, C.c_int, C.c_int, C.c_int]
    lib.cost.argtypes, lib.cost.restype = [C.c_int, C.c_long, C.c_int, C.c_int, C.c_int], C.c_double
    return lib


@pytest.mark.parametrize("H,F", [(256, 1024), (512, 2048), (768, 3072), (1024, 4096), (1280, 5120), (2048, 8192)])
def test_fp16_gemms_of_a_few_dozen_rows_spread_over_the_chip(rules, H, F):
    """A packed tile is at least 128 channels wide; up to 64 rows it would leave most CUs without a block wherever tiles of 32 channels
    fit the chip.  From 2048 rows on nothing reads rows as they lie; K without a small kernel never does."""
    for N, K in ((3 * H, H), (H, H), (F, H), (H, F)):
        for rows in (1, 8, 19, 32, 48, 64):
            small = -(-rows // 32) * (N // 32)
            assert bool(rules.f16(rows, N, K, 256)) == (small <= 512), (rows, N, K)
        assert not rules.f16(2048 * 2048 // H, N, K, 256)
        assert not rules.f16(19, N, 640, 256) and not rules.f16(19, N, 384, 256)
    # the last rows with two 32 x 32 tiles per CU and with one, the step from the one to the other, and the weights fetched ahead from 256 rows on
    assert rules.f16(96, 3072, 768, 256) and not rules.f16(97, 3072, 768, 256)
    assert rules.f16(96, 2304, 768, 256) and not rules.f16(97, 2304, 768, 256)
    assert rules.f16(128, 4096, 1024, 256) and not rules.f16(129, 4096, 1024, 256)
    assert rules.f16(320, 768, 3072, 256) and not rules.f16(321, 768, 3072, 256)
    assert rules.f16(255, 2048, 8192, 256) and not rules.f16(256, 2048, 8192, 256)
    assert rules.f16(160, 1536, 512, 256) and not rules.f16(161, 1536, 512, 256)


@pytest.mark.parametrize("H,F", [(256, 1024), (512, 2048), (640, 2560), (768, 3072), (1024, 4096), (1280, 5120), (1536, 6144), (1792, 7168), (2048, 8192)])
def test_int8_gemms_read_rows_only_where_a_kernel_splits_k(rules, H, F):
    """K has to be whole slabs of eight or six waves; where it is, a few dozen rows read the weights as they lie, up to 2048 channels, and
    thousands of rows never do."""
    for N, K in ((3 * H, H), (H, H), (F, H), (H, F)):
        exists = K % 1024 == 0 or K % 768 == 0
        for rows in (1, 19, 64, 100, 128):
            if N <= 2048: assert bool(rules.i8(rows, N, K)) == exists, (rows, N, K)
            if rows * N > 128000 and N > 2048: assert not rules.i8(rows, N, K)
        assert not rules.i8(2048, N, K)
    assert rules.i8(390, 768, 3072) and not rules.i8(391, 768, 3072)
    assert rules.i8(160, 2048, 8192) and not rules.i8(192, 2048, 8192)
    assert rules.i8(128, 2048, 2048) and not rules.i8(129, 2048, 2048)
    assert rules.i8(32, 3072, 768) and not rules.i8(42, 3072, 768)


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(1, 2304, 768), (97, 3072, 768), (224, 2304, 768), (33, 1024, 4096), (128, 4096, 1024), (255, 512, 2048)])
def test_few_rows_of_both_copies_give_the_same_bytes(M, N, K):
    import torch
    import paper_2209_09130_amd as P
    rng = np.random.default_rng(M + N)
    A = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float16)).cuda()
    W = torch.from_numpy((rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float16)).cuda()
    bias = torch.from_numpy((0.1 * rng.standard_normal(N)).astype(np.float32)).cuda()
    rows, packed = P.gemm_f16(A, W, bias, True), P.gemm_f16_packed(A, P.pack_weight_f16(W), bias, True)
    assert torch.equal(rows, packed)
    want = torch.nn.functional.gelu(A.cpu().double() @ W.cpu().double().T + bias.cpu().double())
    # one rounding to 16 bits, and 32-bit sums of K terms
    assert ((rows.cpu().double() - want).abs() <= want.abs().clamp(min=2.0 ** -14) * 2.0 ** -10 + K * 2.0 ** -24).all()


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K", [(19, 512, 512), (257, 256, 1024), (100, 1280, 5120), (70, 1280, 1280)])
def test_few_int8_rows_of_both_copies_give_the_same_codes(M, N, K):
    """Sizes on both sides of the rule; the encoder takes one of the two."""
    import torch
    import oracle
    import paper_2209_09130_amd as P
    rng = np.random.default_rng(M + K)
    A, W = (rng.integers(-127, 128, shape, dtype=np.int8) for shape in ((M, K), (N, K)))
    m, b = (0.5 + rng.random(N, dtype=np.float32)) * np.float32(40 / (5400 * np.sqrt(K))), rng.standard_normal(N).astype(np.float32)
    t = [torch.from_numpy(x).cuda() for x in (A, W, m, b)]
    want = oracle.epilogue_requant(oracle.gemm_i8_i32(A, W), m, b)
    assert np.array_equal(P.gemm_i8_requant(*t).cpu().numpy(), want)
    assert np.array_equal(P.gemm_i8_requant_packed(t[0], P.pack_weight_i8(t[1]), t[2], t[3]).cpu().numpy(), want)


def test_each_matrix_is_asked_for_by_one_kernel(rules):
    """A stack whose layers differ in whether their attention kernels can ask: where LayerNorm steps may ask, every matrix from the first layer's
    attention output on is asked for exactly once, and by the attention wherever that can."""
    for n in range(1, 6):
        for can in range(2 ** n):
            for attention_may in (0, 1):
                for norm_may in (0, 1):
                    count = {}
                    for l in range(n):
                        here, there = can >> l & 1, can >> min(l + 1, n - 1) & 1
                        a = rules.asks(attention_may, norm_may, here, there)
                        assert (a & 1) == (attention_may and here)
                        asked = [(l, "o"), (l, "f1"), (l, "f2"), (l + 1, "qkv")] if a & 1 else []
                        asked += [(l, "f1"), (l, "f2")] if a & 2 else []
                        asked += [(l + 1, "qkv")] if a & 4 else []
                        asked += [(l + 1, "o")] if a & 8 else []
                        for m in asked:
                            count[m] = count.get(m, 0) + 1
                    assert set(count.values()) <= {1}
                    if norm_may:
                        assert all((l, m) in count for l in range(n) for m in ("f1", "f2"))
                        assert all((l, m) in count for l in range(1, n) for m in ("qkv", "o"))
    for H in range(128, 2049, 128):
        for S in (49, 128, 129, 256):
            assert rules.one_packed(1, 1, S, H) == (S <= 128 and H % 256 == 0)
            assert rules.one_packed(0, 1, S, H) == (S <= 128)
            assert not rules.one_packed(0, 0, S, H) and not rules.one_packed(1, 0, S, H)


@pytest.mark.parametrize("H,F", [(256, 1024), (768, 3072), (1024, 4096), (1280, 5120)])
def test_a_tile_for_fewer_rows_costs_a_full_batch_no_more_than_it_saves_the_others(rules, H, F):
    """By the estimate, a batch with a mask and all its rows never pays more than 55, 70 and 85 % of the rows save on average; the tile of a batch
    without a mask is the best one for all rows."""
    widths = [64, 64, 128, 192, 256, 128, 192]
    for N, K in ((3 * H, H), (H, H), (F, H), (H, F)):
        for rows in [*range(1, 3000, 37), 2048, 1920, 1800, 427]:
            full, masked = rules.tile(rows, 0, N, K), rules.tile(rows, 1, N, K)
            at = lambda t, percent: rules.cost(t, rows, percent, N, K)
            assert at(full, 100) == min(at(t, 100) for t, w in enumerate(widths) if N % w == 0)
            saved = sum(at(full, p) - at(masked, p) for p in (55, 70, 85)) / 3
            assert at(masked, 100) - at(full, 100) <= saved + 1e-9
    assert rules.tile(1536, 1, 768, 768) != rules.tile(1536, 0, 768, 768)      # 12 x 128: smaller tiles also with the mask's doubt
    assert rules.tile(1920, 1, 2304, 768) == rules.tile(1920, 0, 2304, 768)    # 40 x 48: a full batch would pay five times what the others save
