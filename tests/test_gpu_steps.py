"""GPU parity of the single steps of the path against the CPU oracle (through the C ABI).

Integer results (int32 accumulators, int8 codes) must be bit-exact; fp16 results of steps whose
arithmetic is a fixed sequence of binary32 operations must be bit-exact too; fp16 GEMM and fp16
attention (binary32 accumulation in hardware order against binary64 in the oracle) are compared
with a tolerance derived from that difference.
"""
import ctypes

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def P():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2209_09130_amd as P
    P.lib()
    return P


def dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    import torch
    torch.cuda.synchronize()
    return t.cpu().numpy()


# ------------------------------------------------------------------ INT8 GEMM
@pytest.mark.parametrize("M,N,K", [(1, 128, 64), (128, 128, 64), (77, 256, 192), (300, 768, 768), (513, 128, 3072)])
def test_int8_gemm_accumulators_bit_exact(P, M, N, K):
    rng = np.random.default_rng(M + N + K)
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    got = host(P.gemm_i8_i32(dev(A), dev(W)))
    assert np.array_equal(got, oracle.gemm_i8_i32(A, W))


def test_int8_gemm_extremes_and_full_size_sampled(P):
    K = 4096
    A = np.full((130, K), 127, np.int8); A[1::2] = -127
    W = np.full((128, K), 127, np.int8); W[::3] = -127
    got = host(P.gemm_i8_i32(dev(A), dev(W)))
    assert np.array_equal(got.astype(np.int64), A.astype(np.int64) @ W.astype(np.int64).T)
    # benchmark shape (tokens 4096, FFN2: N 768, K 3072): sampled rows against the oracle, all via int64 matmul
    rng = np.random.default_rng(0)
    A = rng.integers(-127, 128, (4096, 3072), dtype=np.int8)
    W = rng.integers(-127, 128, (768, 3072), dtype=np.int8)
    got = host(P.gemm_i8_i32(dev(A), dev(W)))
    rows = np.r_[0, 127, 128, 4095, rng.integers(0, 4096, 28)]
    assert np.array_equal(got[rows], oracle.gemm_i8_i32(A[rows], W))
    assert np.array_equal(got.astype(np.int64), A.astype(np.int64) @ W.astype(np.int64).T)


def _tables(rng, N, with_bias=True):
    s_w = (rng.random(N) * 2e-4 + 5e-5).astype(np.float32)
    bias = (rng.standard_normal(N) * 0.2).astype(np.float32) if with_bias else None
    return s_w, bias


@pytest.mark.parametrize("M,N,K,with_bias", [(200, 256, 768, True), (129, 768, 128, False)])
def test_int8_gemm_requant_epilogue_bit_exact(P, M, N, K, with_bias):
    rng = np.random.default_rng(M * 7 + N)
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N, with_bias)
    m, b = oracle.fold_requant(0.037, s_w, bias, 0.021 * np.sqrt(K / 768))
    want = oracle.epilogue_requant(oracle.gemm_i8_i32(A, W), m, b)
    got = host(P.gemm_i8_requant(dev(A), dev(W), dev(m), dev(b) if with_bias else None))
    assert np.array_equal(got, want)
    assert np.abs(want).max() == 127 and (np.abs(want) < 127).mean() > 0.5      # clamp and interior both hit


@pytest.mark.parametrize("config", [-1, 0, 1, 2])
def test_every_gemm_tile_configuration_gives_the_same_results(P, config):
    """The library picks a tile configuration by problem size; force each one in turn on a problem that
    spans several tiles and a ragged last row tile, for all three INT8 epilogues and the FP16 GEMM.
    Left to itself (-1) it takes the tiles for few rows here, and 64 x 96 tiles of six waves for the raw sums and for GELU
    without a table (384 channels, few tiles)."""
    rng = np.random.default_rng(77)
    M, N, K = 333, 384, 768
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    m, b = oracle.fold_requant(0.037, s_w, bias, 0.021)
    md = oracle.fold_dequant(0.05, s_w)
    Ah = (rng.standard_normal((M, K)) * 0.5).astype(np.float16)
    Wh = (rng.standard_normal((N, K)) * 0.05).astype(np.float16)
    acc = oracle.gemm_i8_i32(A, W)
    P.set_gemm_config(config)
    try:
        raw = host(P.gemm_i8_i32(dev(A), dev(W)))
        req = host(P.gemm_i8_requant(dev(A), dev(W), dev(m), dev(b)))
        gel = host(P.gemm_i8_gelu_quant(dev(A), dev(W), dev(md), dev(bias), 0.0147))
        f16 = host(P.gemm_f16(dev(Ah), dev(Wh), dev(bias), False)).astype(np.float64)
    finally:
        P.set_gemm_config(-1)
    assert np.array_equal(raw, acc)
    assert np.array_equal(req, oracle.epilogue_requant(acc, m, b))
    assert np.array_equal(gel, oracle.epilogue_gelu_quant(acc, md, bias, 0.0147))
    want = oracle.gemm_f16(Ah, Wh, bias, False).astype(np.float64)
    assert (np.abs(f16 - want) <= np.maximum(np.abs(want), 2.0 ** -14) * 2.0 ** -10 + 1e-6).all()
    with pytest.raises(P.SampError):
        P.set_gemm_config(99)


@pytest.mark.parametrize("config", [3, 4, 5, 6, 7])
@pytest.mark.parametrize("M,N,K", [(700, 512, 768), (257, 768, 256), (1100, 768, 3072), (130, 768, 128)])
def test_large_tile_configurations_give_the_same_results(P, config, M, N, K):
    """The large block tiles (128..256 tokens x 128..256 channels, 64 x 64 .. 128 x 128 per wave, rings of 64- or
    128-byte stages, operand fragments double-buffered in registers), forced on problems with a ragged last row tile
    and with fewer K stages than the ring is deep: all INT8 epilogues bit-exact, incl. the table-lookup GELU; FP16
    within one ulp.  (A configuration whose tile width does not divide N falls back to the default choice.)"""
    rng = np.random.default_rng(M + N + K + config)
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    m, b = oracle.fold_requant(0.037, s_w, bias, 0.021 * np.sqrt(K / 768))
    md = oracle.fold_dequant(0.05 * np.sqrt(768 / K), s_w)
    s_out = 0.0147
    spec, entries = P.gelu_table_build(s_out)
    Ah = (rng.standard_normal((M, K // 2)) * 0.5).astype(np.float16)
    Wh = (rng.standard_normal((N, K // 2)) * 0.05).astype(np.float16)
    acc = oracle.gemm_i8_i32(A, W)
    P.set_gemm_config(config)
    try:
        raw = host(P.gemm_i8_i32(dev(A), dev(W)))
        req = host(P.gemm_i8_requant(dev(A), dev(W), dev(m), dev(b)))
        gel = host(P.gemm_i8_gelu_quant(dev(A), dev(W), dev(md), dev(bias), s_out))
        gel_t = host(P.gemm_i8_gelu_quant(dev(A), dev(W), dev(md), dev(bias), s_out, (spec, dev(entries))))
        f16 = host(P.gemm_f16(dev(Ah), dev(Wh), dev(bias), True)).astype(np.float64)
    finally:
        P.set_gemm_config(-1)
    assert np.array_equal(raw, acc)
    assert np.array_equal(req, oracle.epilogue_requant(acc, m, b))
    want = oracle.epilogue_gelu_quant(acc, md, bias, s_out)
    assert np.array_equal(gel, want)
    assert np.array_equal(gel_t, want)
    assert want.max() == 127 and (want < 0).any()
    wantf = oracle.gemm_f16(Ah, Wh, bias, True).astype(np.float64)
    assert (np.abs(f16 - wantf) <= np.maximum(np.abs(wantf), 2.0 ** -14) * 2.0 ** -10 + 1e-6).all()


@pytest.mark.parametrize("tile", [-1, 0, 1, 2, 3, 4, 5, 6])
@pytest.mark.parametrize("M,N,K", [(1, 768, 256), (130, 768, 768), (257, 768, 1024), (33, 768, 3072), (1100, 512, 512), (70, 128, 1280)])
def test_gemms_on_packed_weights_give_the_same_codes(P, tile, M, N, K):
    """Weights packed in the order of the matrix product and loaded straight into registers: every tile with one row, a last row tile
    that is not full, two to twenty-four stages of K, both epilogues bit-exact.  The packed bytes against the definition."""
    width = {0: 64, 1: 64, 2: 128, 3: 192, 4: 256, 5: 128, 6: 192}
    rng = np.random.default_rng(M + N + K)
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    m, b = oracle.fold_requant(0.037, s_w, bias, 0.021 * np.sqrt(K / 768))
    md = oracle.fold_dequant(0.05 * np.sqrt(768 / K), s_w)
    s_out = 0.0147
    spec, entries = P.gelu_table_build(s_out)
    packed = P.pack_weight_i8(dev(W))
    assert np.array_equal(host(packed), W.reshape(N // 16, 16, K // 64, 4, 16).transpose(0, 2, 3, 1, 4).ravel())
    if tile >= 0 and N % width[tile]:
        with pytest.raises(P.SampError):
            P.gemm_i8_requant_packed(dev(A), packed, dev(m), dev(b), tile)
        return
    acc = oracle.gemm_i8_i32(A, W)
    assert np.array_equal(host(P.gemm_i8_requant_packed(dev(A), packed, dev(m), dev(b), tile)), oracle.epilogue_requant(acc, m, b))
    assert np.array_equal(host(P.gemm_i8_requant_packed(dev(A), packed, dev(m), None, tile)),
                          oracle.epilogue_requant(acc, m, np.zeros_like(b)))
    assert np.array_equal(host(P.gemm_i8_gelu_quant_packed(dev(A), packed, dev(md), dev(bias), (spec, dev(entries)), tile)),
                          oracle.epilogue_gelu_quant(acc, md, bias, s_out))


@pytest.mark.parametrize("M,tile", [(1, -1), (70, 2), (129, 5), (257, 0), (1024, -1), (1024, 4), (1025, -1)])
@pytest.mark.parametrize("N,K", [(1024, 3072), (4096, 1024)])
def test_gemm_on_packed_weights_with_channels_outermost(P, M, tile, N, K):
    """Weights of 3 MB and more, at most 1024 rows: blocks are numbered with the channels outermost (1025 rows: as everywhere else)."""
    rng = np.random.default_rng(M + N)
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    m, b = oracle.fold_requant(0.037, s_w, bias, 0.021 * np.sqrt(K / 768))
    want = oracle.epilogue_requant(oracle.gemm_i8_i32(A, W), m, b)
    assert np.abs(want).max() > 20
    assert np.array_equal(host(P.gemm_i8_requant_packed(dev(A), P.pack_weight_i8(dev(W)), dev(m), dev(b), tile)), want)


@pytest.mark.parametrize("M,tile", [(1, -1), (70, 0), (257, 2), (1024, 3), (1025, -1)])
def test_fp16_gemm_on_packed_weights_with_channels_outermost(P, M, tile):
    rng = np.random.default_rng(M)
    N, K = 2048, 768
    A = dev(rng.standard_normal((M, K)).astype(np.float16))
    W = dev((rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float16))
    bias = dev((0.1 * rng.standard_normal(N)).astype(np.float32))
    want = host(P.gemm_f16(A, W, bias, True))                  # compared with the oracle at other sizes; the same order of sums
    assert np.abs(want).max() > 0.5
    assert np.array_equal(host(P.gemm_f16_packed(A, P.pack_weight_f16(W), bias, True, tile)), want)


@pytest.mark.parametrize("tile", [-1, 0, 1, 2, 3])
@pytest.mark.parametrize("M,N,K", [(1, 768, 128), (130, 768, 768), (257, 384, 1024), (33, 768, 3072), (1100, 512, 640)])
def test_fp16_gemm_on_packed_weights_gives_the_same_values(P, tile, M, N, K):
    """Every tile with one row, a last row tile that is not full, two to forty-eight stages of K, two and four of them in flight: the bytes
    of the row-major kernels, which add in the same order.  The packed bytes against the definition."""
    width = {0: 128, 1: 128, 2: 256, 3: 256}
    rng = np.random.default_rng(M + N + K)
    A = rng.standard_normal((M, K)).astype(np.float16)
    W = (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float16)
    bias = (0.1 * rng.standard_normal(N)).astype(np.float32)
    packed = P.pack_weight_f16(dev(W))
    assert np.array_equal(host(packed), W.reshape(N // 32, 32, K // 16, 2, 8).transpose(0, 2, 3, 1, 4).ravel())
    if tile >= 0 and N % width[tile]:
        with pytest.raises(P.SampError):
            P.gemm_f16_packed(dev(A), packed, dev(bias), True, tile)
        return
    for b, gelu in ((bias, True), (bias, False), (None, False)):
        b = None if b is None else dev(b)
        got = host(P.gemm_f16_packed(dev(A), packed, b, gelu, tile))
        assert np.array_equal(got, host(P.gemm_f16(dev(A), dev(W), b, gelu)))
        # one rounding to 16 bits, and 32-bit sums of K terms, against the oracle's
        want = oracle.gemm_f16(A, W, bias if b is not None else np.zeros(N, np.float32), gelu).astype(np.float64)
        assert (np.abs(got - want) <= np.maximum(np.abs(want), 2.0 ** -14) * 2.0 ** -10 + K * 2.0 ** -24).all()


@pytest.mark.parametrize("config", [-1, 0, 1, 2])
def test_table_lookup_gelu_epilogue_in_the_small_tile_configurations(P, config):
    rng = np.random.default_rng(5 + config)
    M, N, K = 333, 384, 768
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    md = oracle.fold_dequant(0.05, s_w)
    for s_out in (0.0147, 0.031):
        spec, entries = P.gelu_table_build(s_out)
        P.set_gemm_config(config)
        try:
            got = host(P.gemm_i8_gelu_quant(dev(A), dev(W), dev(md), dev(bias), s_out, (spec, dev(entries))))
        finally:
            P.set_gemm_config(-1)
        assert np.array_equal(got, oracle.epilogue_gelu_quant(oracle.gemm_i8_i32(A, W), md, bias, s_out))


@pytest.mark.parametrize("N", [256, 384])
def test_long_rows_with_few_tiles_take_the_deeper_ring(P, N):
    """Operand rows of 3072 bytes with at most one block per CU, ragged last row tile: raw INT8 sums run through a 3-deep stage
    ring, in 64 x 128 tiles or, where the channel count allows it, 64 x 96 tiles whose six waves do not split the stage
    loads evenly; the requantising GEMM (bit-exact) and the FP16 GEMM (within one ulp) take the tiles for few rows."""
    rng = np.random.default_rng(91 + N)
    M, K = 300, 3072
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    m, b = oracle.fold_requant(0.037, s_w, bias, 0.042)
    want = oracle.epilogue_requant(oracle.gemm_i8_i32(A, W), m, b)
    assert np.array_equal(host(P.gemm_i8_requant(dev(A), dev(W), dev(m), dev(b))), want)
    assert np.array_equal(host(P.gemm_i8_i32(dev(A), dev(W))), oracle.gemm_i8_i32(A, W))
    Ah = (rng.standard_normal((M, K // 2)) * 0.5).astype(np.float16)
    Wh = (rng.standard_normal((N, K // 2)) * 0.05).astype(np.float16)
    wantf = oracle.gemm_f16(Ah, Wh, bias, False).astype(np.float64)
    gotf = host(P.gemm_f16(dev(Ah), dev(Wh), dev(bias), False)).astype(np.float64)
    assert (np.abs(gotf - wantf) <= np.maximum(np.abs(wantf), 2.0 ** -14) * 2.0 ** -10 + 1e-6).all()


def test_int8_gemm_gelu_quant_epilogue_bit_exact(P):
    rng = np.random.default_rng(21)
    M, N, K = 260, 384, 768
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    m = oracle.fold_dequant(0.05, s_w)
    s_out = 0.0147
    want = oracle.epilogue_gelu_quant(oracle.gemm_i8_i32(A, W), m, bias, s_out)
    got = host(P.gemm_i8_gelu_quant(dev(A), dev(W), dev(m), dev(bias), s_out))
    assert np.array_equal(got, want)
    assert want.max() == 127 and (want == 0).any() and (want < 0).any()


def test_gelu_quant_decision_is_exact_and_fast_path_error_is_bounded(P):
    """The kernel takes the fast GELU value only when it cannot change the rounded code.  Check
    (a) the codes equal the oracle's on a dense sweep incl. values planted next to rounding ties,
    (b) |fast - exact| stays below half the bound the kernel assumes (8e-7 * |y|)."""
    rng = np.random.default_rng(22)
    ys = np.concatenate([
        np.linspace(-12, 12, 3_000_001, dtype=np.float64).astype(np.float32),
        (rng.standard_normal(2_000_000) * 0.6).astype(np.float32),
        np.array([0.0, -0.0, 1e-30, -1e-30, 40.0, -40.0, 1e4, -1e4], np.float32),
    ])
    for s_out in (0.0247, 0.0031, 0.25):
        codes, fast = P.gelu_quant(dev(ys), s_out, want_fast=True)
        codes, fast = host(codes), host(fast)
        exact = np.array([oracle.gelu(v) for v in ys[::997]], np.float32)
        err = np.abs(fast[::997].astype(np.float64) - exact.astype(np.float64))
        bound = 8e-7 * np.abs(ys[::997].astype(np.float64)) + 1e-37
        assert (err <= 0.5 * bound + 6e-8 * np.abs(exact)).all()
        # the oracle's epilogue with acc = 0 reduces to code(GELU(bias)): feed y as the bias vector
        want = oracle.epilogue_gelu_quant(np.zeros((1, ys.size), np.int32), np.zeros(ys.size, np.float32), ys, s_out)[0]
        assert np.array_equal(codes, want)
    # values sitting right at rounding ties of the code: y with GELU(y)/s = k + 0.5 (bisection on the oracle)
    s_out = 0.0247
    ties = []
    for k in range(0, 100, 3):
        lo, hi = 0.0, 8.0
        target = (k + 0.5) * s_out
        for _ in range(60):
            mid = (lo + hi) / 2
            if oracle.gelu(np.float32(mid)) < target:
                lo = mid
            else:
                hi = mid
        c = np.float32(lo)
        ties += [np.nextafter(c, np.float32(-9)), c, np.nextafter(c, np.float32(9))]
        for step in range(2, 6):
            ties += [np.float32(c - step * np.spacing(c)), np.float32(c + step * np.spacing(c))]
    ties = np.array(ties, np.float32)
    got = host(P.gelu_quant(dev(ties), s_out))
    want = oracle.epilogue_gelu_quant(np.zeros((1, ties.size), np.int32), np.zeros(ties.size, np.float32), ties, s_out)[0]
    assert np.array_equal(got, want)


# ------------------------------------------------------------------ FP16 GEMM
@pytest.mark.parametrize("M,N,K,bias,gelu", [(200, 256, 768, True, False), (131, 128, 96, False, False),
                                             (150, 384, 768, True, True)])
def test_fp16_gemm_within_accumulation_tolerance(P, M, N, K, bias, gelu):
    rng = np.random.default_rng(M + K)
    A = rng.standard_normal((M, K)).astype(np.float16)
    W = (rng.standard_normal((N, K)) * 0.02).astype(np.float16)
    b = (rng.standard_normal(N) * 0.1).astype(np.float32) if bias else None
    want = oracle.gemm_f16(A, W, b, gelu).astype(np.float64)
    got = host(P.gemm_f16(dev(A), dev(W), dev(b) if bias else None, gelu)).astype(np.float64)
    # binary32 accumulation error << one fp16 ulp: results differ by at most one ulp, and rarely
    ulp = np.maximum(np.abs(want), 2.0 ** -14) * 2.0 ** -10
    assert (np.abs(got - want) <= ulp + 1e-6).all()
    assert (got != want).mean() < 5e-3


# ------------------------------------------------------------------ few token rows
@pytest.mark.parametrize("K,N", [(768, 768), (1024, 2304), (1536, 256), (3072, 768), (4096, 1024)])
def test_int8_gemm_of_few_rows_bit_exact(P, K, N):
    """Row counts on either side of the edges of the small tiles (and of the steps from one tile to the next), with K split
    over six or eight waves that hold one or several slabs each; both epilogues."""
    rng = np.random.default_rng(K + N)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    m, b = oracle.fold_requant(0.037, s_w, bias, 0.021 * np.sqrt(K / 768))
    mg, s_out = oracle.fold_dequant(0.05 * np.sqrt(768 / K), s_w), 0.0147
    spec, entries = P.gelu_table_build(s_out)
    table = (spec, dev(entries.view(np.int32)))
    for M in (1, 16, 17, 31, 33, 65, 129, 257, 513):
        A = rng.integers(-127, 128, (M, K), dtype=np.int8)
        acc = oracle.gemm_i8_i32(A, W)
        assert np.array_equal(host(P.gemm_i8_requant(dev(A), dev(W), dev(m), dev(b))), oracle.epilogue_requant(acc, m, b)), M
        assert np.array_equal(host(P.gemm_i8_gelu_quant(dev(A), dev(W), dev(mg), dev(bias), s_out, table)),
                              oracle.epilogue_gelu_quant(acc, mg, bias, s_out)), M


@pytest.mark.parametrize("K,N", [(256, 128), (768, 768), (768, 2304), (3072, 768)])
def test_fp16_gemm_of_few_rows_is_the_same_bytes_as_the_large_tiles(P, K, N):
    """Sums are formed in the same order in every tile configuration, so the small tiles must give the bytes of a forced
    large one; rows past the last token are neither read nor written."""
    import torch
    rng = np.random.default_rng(K + N + 1)
    W = dev((rng.standard_normal((N, K)) * 0.05).astype(np.float16))
    bias = dev((rng.standard_normal(N) * 0.1).astype(np.float32))
    for M in (1, 31, 32, 33, 97, 256, 500):
        A = dev(rng.standard_normal((M, K)).astype(np.float16))
        for gelu in (False, True):
            got = P.gemm_f16(A, W, bias, gelu)
            P.set_gemm_config(1)
            try:
                want = P.gemm_f16(A, W, bias, gelu)
            finally:
                P.set_gemm_config(-1)
            assert torch.equal(got.view(torch.int16), want.view(torch.int16)), (M, gelu)


# ------------------------------------------------------------------ one to two thousand token rows
@pytest.mark.parametrize("M,N,K", [(1400, 768, 768), (1400, 768, 3072), (1100, 1024, 4096), (2050, 768, 768), (2050, 768, 3072),
                                   (2050, 1024, 4096)])
def test_gemms_of_one_to_two_thousand_rows(P, M, N, K):
    """Too many rows for the small tiles, too few for the wide ones: 64 x 96 (N = 768) and 64 x 128 tiles, up to one block per CU
    with the stages in flight held in registers, ragged last row tile.  Every byte is that of a forced 128 x 128 tile; INT8 rows
    around the tiles' edges against the oracle."""
    import torch
    rng = np.random.default_rng(M + N + K)
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    m, b = oracle.fold_requant(0.037, s_w, bias, 0.021 * np.sqrt(K / 768))
    Ah, Wh = dev((rng.standard_normal((M, K)) * 0.5).astype(np.float16)), dev((rng.standard_normal((N, K)) * 0.05).astype(np.float16))
    runs = [lambda: P.gemm_i8_requant(dev(A), dev(W), dev(m), dev(b)), lambda: P.gemm_f16(Ah, Wh, dev(bias), False),
            lambda: P.gemm_f16(Ah, Wh, None, True)]
    got = [run() for run in runs]
    P.set_gemm_config(1)
    try:
        want = [run() for run in runs]
    finally:
        P.set_gemm_config(-1)
    for g, w in zip(got, want):
        assert torch.equal(g.view(torch.int8), w.view(torch.int8))
    rows = np.unique(np.concatenate([np.arange(8), 64 + np.arange(-4, 4), 128 + np.arange(-4, 4), M // 64 * 64 + np.arange(-4, 4), [M - 1]]))
    rows = rows[rows < M]
    assert np.array_equal(host(got[0])[rows], oracle.epilogue_requant(oracle.gemm_i8_i32(A[rows], W), m, b))


# ------------------------------------------------------------------ attention
def _cu(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


@pytest.mark.parametrize("lens,heads", [([128], 2), ([1, 5, 32, 33, 64, 17], 3), ([200, 256, 129], 2), ([512, 300], 1)])
def test_int8_attention_bit_exact(P, lens, heads):
    rng = np.random.default_rng(sum(lens))
    H = heads * 64
    cu = _cu(lens)
    T = int(cu[-1])
    # q, k ~ N(0, 26) codes as after a real projection (|code| <= 127), v likewise
    qkv = np.clip(np.rint(rng.standard_normal((T, 3 * H)) * 26), -127, 127).astype(np.int8)
    sc = (0.0209, 0.0249, 0.021, 0.0003, 0.0021)
    want = oracle.attention_i8(qkv, cu, heads, *sc)
    got = host(P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc))
    assert np.array_equal(got, want)
    assert np.abs(want).max() > 20


@pytest.mark.parametrize("kind,n", [("int8", 500), ("int8", 2048), ("p16", 1536), ("fp16", 2047), ("fp16", 2100)])
def test_attention_of_a_sequence_with_2_to_the_31_values(P, kind, n):
    """The steps bound the tokens of a sequence and not the heads: rows times row length pass 2^31 here.  The first, a middle and the last head
    against the oracle; INT8 bit-exact, FP16 within tolerance."""
    import torch
    heads = 2 ** 31 // (3 * 64 * n) + 8
    g = torch.Generator(device="cuda").manual_seed(n)
    if kind == "fp16":
        qkv = torch.empty((n, 3, heads, 64), dtype=torch.float16, device="cuda").normal_(0, 0.6, generator=g)
    else:
        qkv = torch.randint(-60, 61, (n, 3, heads, 64), dtype=torch.int8, generator=g, device="cuda")
    cu, flat, sc = _cu([n]), qkv.view(n, -1), (0.0209, 0.0249, 0.021, 0.0003, 0.0021)
    if kind == "fp16":
        ctx = P.attention_f16(flat, dev(cu), n, heads)
    else:
        ctx = P.attention_i8(flat, dev(cu), n, heads, *sc, p_fp16=kind == "p16")
    ctx = ctx.view(n, heads, 64)
    for h in (0, heads // 2, heads - 1):
        one, got = np.ascontiguousarray(host(qkv[:, :, h])).reshape(n, -1), host(ctx[:, h])
        if kind == "fp16":
            assert np.abs(got.astype(np.float64) - oracle.attention_f16(one, cu, 1).astype(np.float64)).max() <= 2e-3
        elif kind == "p16":
            assert np.array_equal(got, oracle.attention_i8_p16(one, cu, 1, sc[0], sc[1], sc[2], sc[4]))
        else:
            assert np.array_equal(got, oracle.attention_i8(one, cu, 1, *sc))


@pytest.mark.parametrize("lens,heads,offsets", [([128, 128, 128], 2, False), ([1, 5, 32, 33, 64, 17, 128, 97], 3, True),
                                                ([96] * 4, 1, False), ([128, 2, 65], 12, True), ([31], 16, True),
                                                ([256, 256], 2, False), ([200, 129, 256, 7, 160], 3, True), ([192] * 3, 4, False)])
def test_qkv_gemm_and_attention_in_one_kernel_bit_exact(P, lens, heads, offsets):
    """The kernel that does the QKV GEMM, its requantisation and the attention of a (sequence, head) at once gives the
    oracle's requantised GEMM followed by the oracle's attention, and the bytes of the two separate kernels."""
    rng = np.random.default_rng(sum(lens) + heads)
    H = heads * 64
    cu = _cu(lens)
    T = int(cu[-1])
    x = rng.integers(-127, 128, (T, H), dtype=np.int8)
    w = rng.integers(-127, 128, (3 * H, H), dtype=np.int8)
    m = (26.0 / (73.3 * 73.3 * np.sqrt(H)) * (0.8 + 0.4 * rng.random(3 * H))).astype(np.float32)   # codes ~ N(0, 26)
    m[::17] *= 4                                                     # some channels reach the clamp
    b = (rng.standard_normal(3 * H) * 3).astype(np.float32)
    sc = (0.0209, 0.0249, 0.021, 0.0003, 0.0021)
    qkv = oracle.epilogue_requant(oracle.gemm_i8_i32(x, w), m, b)
    assert np.abs(qkv).max() == 127 and 15 < qkv.astype(np.float64).std() < 60
    want = oracle.attention_i8(qkv, cu, heads, *sc)
    cu_dev = dev(cu) if offsets else None
    got = host(P.qkv_attention_i8(dev(x), dev(w), dev(m), dev(b), cu_dev, max(lens), heads, *sc))
    assert np.array_equal(got, want)
    if (3 * H) % 128 == 0:                                           # the stand-alone GEMM wants whole 128-channel tiles
        two = host(P.attention_i8(P.gemm_i8_requant(dev(x), dev(w), dev(m), dev(b)), cu_dev, max(lens), heads, *sc))
        assert np.array_equal(two, want)
    assert np.abs(want).max() > 20
    scu = (sc[0], sc[1], sc[2], sc[3] * 0.5, sc[4])                   # unsigned softmax codes: twice the levels
    unsigned = host(P.qkv_attention_i8(dev(x), dev(w), dev(m), dev(b), cu_dev, max(lens), heads, *scu, p_unsigned=True))
    assert np.array_equal(unsigned, oracle.attention_i8(qkv, cu, heads, *scu, p_unsigned=True))
    no_bias = host(P.qkv_attention_i8(dev(x), dev(w), dev(m), None, cu_dev, max(lens), heads, *sc))
    assert np.array_equal(no_bias, oracle.attention_i8(oracle.epilogue_requant(oracle.gemm_i8_i32(x, w), m, np.zeros(3 * H, np.float32)), cu, heads, *sc))


@pytest.mark.parametrize("lens,heads", [([128, 113, 112, 64, 16, 1], 4), ([128, 128], 12), ([33, 97, 17], 16)])
@pytest.mark.parametrize("unsigned", [False, True])
def test_qkv_attention_on_packed_weights_gives_the_same_codes(P, lens, heads, unsigned):
    """Sequences on both sides of a token tile's edge and of the copy of the loop that tests for dead tiles; four, six and eight stages
    of K pairs; with and without offsets in the epilogue, with explicit sequence offsets and without."""
    rng = np.random.default_rng(heads + len(lens))
    cu = _cu(lens)
    H, T = heads * 64, int(cu[-1])
    x, w = rng.integers(-127, 128, (T, H), dtype=np.int8), rng.integers(-127, 128, (3 * H, H), dtype=np.int8)
    m = (26.0 / (73.3 * 73.3 * np.sqrt(H)) * (0.8 + 0.4 * rng.random(3 * H))).astype(np.float32)
    b = (rng.standard_normal(3 * H) * 3).astype(np.float32)
    sc = (0.0209, 0.0249, 0.021, 0.0003 * (0.5 if unsigned else 1.0), 0.0021)
    packed = P.pack_weight_i8(dev(w))
    acc = oracle.gemm_i8_i32(x, w)
    for offsets in (b, None):
        qkv = oracle.epilogue_requant(acc, m, np.zeros_like(m) if offsets is None else b)
        want = oracle.attention_i8(qkv, cu, heads, *sc, p_unsigned=unsigned)
        assert np.abs(want).max() > 20
        run = lambda c: host(P.qkv_attention_i8_packed(dev(x), packed, dev(m), None if offsets is None else dev(b), c, max(lens), heads, *sc, p_unsigned=unsigned))
        assert np.array_equal(run(dev(cu)), want)
        if len(set(lens)) == 1: assert np.array_equal(run(None), want)


@pytest.mark.parametrize("lens,heads", [([128, 113, 97, 96, 65, 64, 33, 32, 1], 4), ([128, 128], 12), ([33, 97, 17], 2), ([70], 16)])
def test_fp16_qkv_attention_on_packed_weights_gives_the_same_bytes(P, lens, heads):
    """Sequences on both sides of the edges of 32-token tiles and of the two halves of the waves; two to sixteen stages of K."""
    rng = np.random.default_rng(heads + len(lens))
    cu = _cu(lens)
    H, T = heads * 64, int(cu[-1])
    x = dev(rng.standard_normal((T, H)).astype(np.float16))
    w = (rng.standard_normal((3 * H, H)) * 0.05).astype(np.float16)
    packed, w = P.pack_weight_f16(dev(w)), dev(w)
    for bias in (dev((rng.standard_normal(3 * H) * 0.1).astype(np.float32)), None):
        want = host(P.qkv_attention_f16(x, w, bias, dev(cu), max(lens), heads))
        assert np.abs(want).max() > 0.1
        assert np.array_equal(host(P.qkv_attention_f16_packed(x, packed, bias, dev(cu), max(lens), heads)), want)
        if len(set(lens)) == 1:
            assert np.array_equal(host(P.qkv_attention_f16_packed(x, packed, bias, None, max(lens), heads)), want)


@pytest.mark.parametrize("M,N,K", [(130, 384, 384), (65, 192 * 2, 640)])
def test_tables_that_arrive_with_the_last_stage_of_an_odd_number(P, M, N, K):
    """128 x 192 tiles (configuration 6): the epilogue's tables take the ring stage that the last one but one leaves free,
    the upper one when the number of 128-byte stages is odd.  Without an offset vector they are filled with zeros."""
    rng = np.random.default_rng(M + N + K)
    A = rng.integers(-127, 128, (M, K), dtype=np.int8)
    W = rng.integers(-127, 128, (N, K), dtype=np.int8)
    s_w, bias = _tables(rng, N)
    m, b = oracle.fold_requant(0.037, s_w, bias, 0.021 * np.sqrt(K / 768))
    md = oracle.fold_dequant(0.05 * np.sqrt(768 / K), s_w)
    spec, entries = P.gelu_table_build(0.0147)
    acc = oracle.gemm_i8_i32(A, W)
    P.set_gemm_config(6)
    try:
        req = host(P.gemm_i8_requant(dev(A), dev(W), dev(m), dev(b)))
        none = host(P.gemm_i8_requant(dev(A), dev(W), dev(m), None))
        gel = host(P.gemm_i8_gelu_quant(dev(A), dev(W), dev(md), dev(bias), 0.0147, (spec, dev(entries))))
    finally:
        P.set_gemm_config(-1)
    assert np.array_equal(req, oracle.epilogue_requant(acc, m, b))
    assert np.array_equal(none, oracle.epilogue_requant(acc, m, np.zeros(N, np.float32)))
    assert np.array_equal(gel, oracle.epilogue_gelu_quant(acc, md, bias, 0.0147))


@pytest.mark.parametrize("M,N,K", [(130, 384, 192), (65, 384, 320), (130, 384, 128), (64, 768, 64)])
def test_fp16_tables_that_arrive_with_the_last_stage(P, M, N, K):
    """The same for FP16, whose stages hold 64 elements (three, five, two and one), with and without an offset vector."""
    rng = np.random.default_rng(M + N + K)
    A = (rng.standard_normal((M, K)) * 0.5).astype(np.float16)
    W = (rng.standard_normal((N, K)) * 0.05).astype(np.float16)
    for bias in ((rng.standard_normal(N) * 0.1).astype(np.float32), None):
        for gelu in (False, True):
            P.set_gemm_config(6)
            try:
                got = host(P.gemm_f16(dev(A), dev(W), None if bias is None else dev(bias), gelu)).astype(np.float64)
            finally:
                P.set_gemm_config(-1)
            want = oracle.gemm_f16(A, W, bias, gelu).astype(np.float64)
            assert (np.abs(got - want) <= np.maximum(np.abs(want), 2.0 ** -14) * 2.0 ** -10 + 1e-6).all()     # one ulp, as above


def test_qkv_attention_with_an_odd_number_of_stages(P):
    """The same in the QKV + attention kernels (INT8: three 128-byte stages for six heads, FP16: five for five heads)."""
    rng = np.random.default_rng(61)
    lens = [128, 3, 77]
    cu = _cu(lens)
    H, T = 384, int(cu[-1])
    x, w = rng.integers(-127, 128, (T, H), dtype=np.int8), rng.integers(-127, 128, (3 * H, H), dtype=np.int8)
    m = (26.0 / (73.3 * 73.3 * np.sqrt(H)) * (0.8 + 0.4 * rng.random(3 * H))).astype(np.float32)
    b = (rng.standard_normal(3 * H) * 3).astype(np.float32)
    sc = (0.0209, 0.0249, 0.021, 0.0003, 0.0021)
    got = host(P.qkv_attention_i8(dev(x), dev(w), dev(m), dev(b), dev(cu), max(lens), 6, *sc))
    assert np.array_equal(got, oracle.attention_i8(oracle.epilogue_requant(oracle.gemm_i8_i32(x, w), m, b), cu, 6, *sc))
    H = 320
    x = rng.standard_normal((T, H)).astype(np.float16)
    w = (rng.standard_normal((3 * H, H)) * 0.6 / np.sqrt(H)).astype(np.float16)
    for bias in ((rng.standard_normal(3 * H) * 0.1).astype(np.float32), None):
        got = host(P.qkv_attention_f16(dev(x), dev(w), None if bias is None else dev(bias), dev(cu), max(lens), 5)).astype(np.float64)
        zeros = np.zeros(3 * H, np.float32)
        d = np.abs(got - oracle.attention_f16(oracle.gemm_f16(x, w, zeros if bias is None else bias, False), cu, 5).astype(np.float64))
        assert d.max() <= 4e-3 and d.mean() <= 2e-4                # the bound of the test of this kernel below


@pytest.mark.parametrize("S,B,heads,unsigned", [(128, 3, 2, False), (256, 2, 1, False), (384, 2, 1, False),
                                                (512, 2, 1, False), (512, 1, 2, True), (96, 3, 1, False), (320, 2, 1, False)])
def test_int8_attention_without_sequence_offsets_bit_exact(P, S, B, heads, unsigned):
    """cu_seqlens NULL: B sequences of exactly S rows.  Same bytes as with explicit offsets, and the oracle's."""
    rng = np.random.default_rng(S + B)
    H = heads * 64
    cu = _cu([S] * B)
    qkv = np.clip(np.rint(rng.standard_normal((B * S, 3 * H)) * 26), -127, 127).astype(np.int8)
    sc = (0.0209, 0.0249, 0.021, 0.0003 * (0.5 if unsigned else 1.0), 0.0021)
    want = oracle.attention_i8(qkv, cu, heads, *sc, p_unsigned=unsigned)
    got = host(P.attention_i8(dev(qkv), None, S, heads, *sc, p_unsigned=unsigned))
    assert np.array_equal(got, want)
    with_offsets = host(P.attention_i8(dev(qkv), dev(cu), S, heads, *sc, p_unsigned=unsigned))
    assert np.array_equal(with_offsets, want)
    half = host(P.attention_f16(dev(qkv.astype(np.float16)), None, S, heads))
    assert np.array_equal(half, host(P.attention_f16(dev(qkv.astype(np.float16)), dev(cu), S, heads)))


def test_int8_attention_peaked_softmax_bit_exact(P):
    # a large score step makes the softmax peaked: codes span 0..127 and clamp
    rng = np.random.default_rng(5)
    heads, lens = 2, [96, 31]
    H = heads * 64
    cu = _cu(lens)
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * H)) * 40), -127, 127).astype(np.int8)
    sc = (0.05, 0.05, 0.021, 0.004, 0.006)
    want = oracle.attention_i8(qkv, cu, heads, *sc)
    got = host(P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc))
    assert np.array_equal(got, want)


@pytest.mark.parametrize("lens,heads", [([128], 2), ([1, 5, 32, 33, 64, 17], 3), ([300, 512, 129], 1)])
def test_int8_attention_unsigned_softmax_codes_bit_exact(P, lens, heads):
    """Codes 0..255 for the softmax output: the kernel feeds code - 128 to the signed matrix core and adds
    128 * sum(V) back; the context must equal the oracle's, which multiplies the unsigned codes directly."""
    rng = np.random.default_rng(sum(lens) + 3)
    H = heads * 64
    cu = _cu(lens)
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * H)) * 30), -127, 127).astype(np.int8)
    for sc in ((0.0209, 0.0249, 0.021, 0.00015, 0.0021), (0.05, 0.05, 0.021, 0.002, 0.006)):
        want = oracle.attention_i8(qkv, cu, heads, *sc, p_unsigned=True)
        got = host(P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc, p_unsigned=True))
        assert np.array_equal(got, want)
        assert np.abs(want).max() > 20


@pytest.mark.parametrize("lens", [[32, 1, 31], [130, 256, 97], [385, 512, 5], [513, 1100, 64], [2048, 1793]])
@pytest.mark.parametrize("unsigned", [False, True])
def test_int8_attention_where_some_rows_pass_the_calibrated_range(P, lens, unsigned):
    """Codes end at 127 (255): the kernel bounds them only where a row of the wave needs it.  Half of the sequences have scores of
    zero (no code near the end), in the others every third query sees one key far above the rest, whose code is beyond it."""
    rng = np.random.default_rng(sum(lens))
    heads = 2
    cu = _cu(lens)
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3, heads, 64)) * 30), -127, 127).astype(np.int8)
    for i in range(len(lens)):
        rows = qkv[cu[i]:cu[i + 1]]
        rows[:, 0] = 0
        if i % 2 == 0:
            rows[::3, 0], rows[lens[i] // 2, 1] = 100, 100
    qkv = qkv.reshape(int(cu[-1]), -1)
    sc = (0.02, 0.02, 0.021, 0.6 / 127, 0.0021)
    want = oracle.attention_i8(qkv, cu, heads, *sc, p_unsigned=unsigned)
    assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc, p_unsigned=unsigned)), want)


@pytest.mark.parametrize("lens,heads", [([128], 2), ([1, 5, 32, 33, 64, 17, 2], 3), ([300, 512, 129], 1), ([700, 1, 1030], 1)])
def test_int8_attention_with_binary16_softmax_output_bit_exact(P, lens, heads):
    """P rounded to binary16 times integer V, added up exactly (up to 1536 keys as two binary16 parts on the FP16 matrix core, beyond as four byte planes
    of P16 * 2^24 on the int8 one), so the context must equal the oracle's exact binary64 sum, also for
    a single key (P = 1 = 2^24 units, the largest number) and for subnormal probabilities (peaked softmax)."""
    rng = np.random.default_rng(sum(lens) + 5)
    H = heads * 64
    cu = _cu(lens)
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * H)) * 30), -127, 127).astype(np.int8)
    for s_q, s_k, s_v, s_ctx in ((0.0209, 0.0249, 0.021, 0.0021), (0.08, 0.08, 0.021, 0.02), (0.004, 0.004, 0.03, 0.001)):
        want = oracle.attention_i8_p16(qkv, cu, heads, s_q, s_k, s_v, s_ctx)
        got = host(P.attention_i8(dev(qkv), dev(cu), max(lens), heads, s_q, s_k, s_v, float("nan"), s_ctx, p_fp16=True))
        assert np.array_equal(got, want)
    assert np.abs(want).max() > 20


@pytest.mark.parametrize("low", [-127, -128])
@pytest.mark.parametrize("n", [1, 17, 31, 33, 127, 128, 129, 343, 381, 511, 513, 1024, 1191, 1425, 1536, 1537])
def test_binary16_softmax_output_at_the_bounds_of_its_exact_sum(P, n, low):
    """The kernel splits P16 into a multiple of 2^-14 and a rest and adds the products with V up in binary32, which is exact as long as
    the sums stay below 2^24 units.  Largest sums: V codes of 127 throughout, with equal probabilities (1 / n; near an odd multiple of
    2^-15 at 343, 381, 1191 and 1425, where the rests are largest) and with one key that has nearly all of it; both signs.  The step takes
    any int8, so also -128, with which the whole sum passes -2^31 units of 2^-24 wherever the probabilities add up to more than 1 (17, 33, 343 and
    1425 of them)."""
    heads = 2
    qkv = np.zeros((n, 3, heads, 64), np.int8)
    qkv[:, 2, 0, :32], qkv[:, 2, 0, 32:] = 127, low
    qkv[:, 2, 1] = np.where(np.arange(n) % 2, low, 127)[:, None]
    qkv[n // 2:, 0], qkv[n // 3, 1] = 60, 60
    qkv = qkv.reshape(n, -1)
    cu = _cu([n])
    for step in (0.02, 0.05):
        for s_ctx in (0.021, 0.021 / 64):                         # the whole range of codes; the last bits of small sums
            want = oracle.attention_i8_p16(qkv, cu, heads, step, step, 0.021, s_ctx)
            got = host(P.attention_i8(dev(qkv), dev(cu), n, heads, step, step, 0.021, float("nan"), s_ctx, p_fp16=True))
            assert np.array_equal(got, want)


def test_softmax_code_usage_histogram(P):
    """The statistic of Appendix B (how many of the 256 integers a tensor's codes use) on synthetic data: the
    kernel's count of the softmax codes equals the count of the oracle's dumped codes, and samp_code_histogram of the
    context equals numpy's bincount.  Symmetric softmax codes never use the negative half (on this input 67.6 % of
    the integers stay unused; the paper reports 67.58 % on its data), unsigned codes reach into the upper half."""
    rng = np.random.default_rng(31)
    heads, lens = 2, [7, 150]
    H = heads * 64
    cu = _cu(lens)
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * H)) * 30), -127, 127).astype(np.int8)
    used = {}
    for p_unsigned in (False, True):
        sc = (0.03, 0.03, 0.021, 0.3 / (255 if p_unsigned else 127), 0.004)
        ctx, hist = P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc, p_unsigned=p_unsigned, want_hist=True)
        want_hist = np.zeros(256, np.int64)
        for b in range(len(lens)):                           # the oracle dumps the codes of the last sequence it is given
            sl = slice(cu[b], cu[b + 1])
            _, Pq = oracle.attention_i8(qkv[sl], np.array([0, lens[b]], np.int32), heads, *sc, dump_p=True,
                                        p_unsigned=p_unsigned)
            want_hist += np.bincount(Pq.view(np.uint8).ravel(), minlength=256)
        assert np.array_equal(host(hist), want_hist)
        assert want_hist.sum() == heads * sum(n * n for n in lens)
        used[p_unsigned] = want_hist > 0
        ctx_hist = host(P.code_histogram(ctx))
        assert np.array_equal(ctx_hist, np.bincount(host(ctx).view(np.uint8).ravel(), minlength=256))
    assert not used[False][128:].any() and 0.6 < 1 - used[False].mean() < 0.75
    assert used[True][128:].any() and used[True].sum() > used[False].sum()
    odd = dev(qkv.ravel()[:12345])                              # a length that is not a multiple of 16
    assert np.array_equal(host(P.code_histogram(odd)), np.bincount(qkv.ravel()[:12345].view(np.uint8), minlength=256))


@pytest.mark.parametrize("lens,heads", [([128], 2), ([1, 5, 32, 33, 64, 17], 3), ([300, 512], 1)])
def test_fp16_attention_within_tolerance(P, lens, heads):
    rng = np.random.default_rng(sum(lens) + 1)
    H = heads * 64
    cu = _cu(lens)
    qkv = (rng.standard_normal((int(cu[-1]), 3 * H)) * 0.6).astype(np.float16)
    want = oracle.attention_f16(qkv, cu, heads).astype(np.float64)
    got = host(P.attention_f16(dev(qkv), dev(cu), max(lens), heads)).astype(np.float64)
    # P is rounded to fp16 on both sides from slightly different binary32 values (fast exp vs binary64 exp):
    # each P may differ by one fp16 ulp (2^-11 relative) -> context error << 2^-11 * max|v|
    assert np.abs(got - want).max() <= 2e-3
    assert np.abs(got - want).mean() <= 1e-4


@pytest.mark.parametrize("n", [1, 31, 33, 127, 129, 160, 257, 288, 385, 511, 512, 513, 769, 1025, 1250, 1537, 2047, 2049])
def test_fp16_attention_at_the_edges_of_its_key_tiles(P, n):
    """Every number of key tiles per wave, ends inside and between tiles (tolerances as above); the rows of the sequence behind it,
    NaN here, must not reach a sequence whose last tile overlaps them."""
    rng = np.random.default_rng(n)
    qkv = (rng.standard_normal((n + 40, 192)) * 0.6).astype(np.float16)
    want = oracle.attention_f16(qkv[:n], _cu([n]), 1).astype(np.float64)
    qkv[n:] = np.nan
    got = host(P.attention_f16(dev(qkv), dev(_cu([n, 40])), max(n, 40), 1))[:n].astype(np.float64)
    assert np.abs(got - want).max() <= 2e-3
    assert np.abs(got - want).mean() <= 1e-4


@pytest.mark.parametrize("lens,heads,offsets", [([128, 128, 128], 2, False), ([1, 5, 32, 33, 64, 17, 128, 97], 2, True),
                                                ([128, 2, 65], 12, True), ([96] * 3, 4, False),
                                                ([256, 256], 2, False), ([200, 129, 256, 7, 160], 2, True), ([192] * 3, 4, False)])
def test_fp16_qkv_gemm_and_attention_in_one_kernel(P, lens, heads, offsets):
    """The FP16 kernel that does the QKV GEMM and the attention at once: the bytes of the two separate kernels, and the
    oracle's GEMM + attention within the tolerance of those kernels."""
    rng = np.random.default_rng(sum(lens) + heads + 5)
    H = heads * 64
    cu = _cu(lens)
    T = int(cu[-1])
    x = rng.standard_normal((T, H)).astype(np.float16)
    w = (rng.standard_normal((3 * H, H)) * 0.6 / np.sqrt(H)).astype(np.float16)
    bias = (rng.standard_normal(3 * H) * 0.1).astype(np.float32)
    cu_dev = dev(cu) if offsets else None
    got = host(P.qkv_attention_f16(dev(x), dev(w), dev(bias), cu_dev, max(lens), heads))
    two = host(P.attention_f16(P.gemm_f16(dev(x), dev(w), dev(bias), False), cu_dev, max(lens), heads))
    assert np.array_equal(got.view(np.uint16), two.view(np.uint16))
    qkv = oracle.gemm_f16(x, w, bias, False)
    want = oracle.attention_f16(qkv, cu, heads).astype(np.float64)
    d = np.abs(got.astype(np.float64) - want)
    assert d.max() <= 4e-3 and d.mean() <= 2e-4                    # q, k, v may differ by an fp16 ulp on top of the attention's own bound
    assert np.abs(want).max() > 0.05
    none = host(P.qkv_attention_f16(dev(x), dev(w), None, cu_dev, max(lens), heads))
    assert np.array_equal(none.view(np.uint16),
                          host(P.attention_f16(P.gemm_f16(dev(x), dev(w), None, False), cu_dev, max(lens), heads)).view(np.uint16))


@pytest.mark.parametrize("longest,B,heads", [(96, 5, 3), (97, 5, 3), (128, 8, 1), (200, 4, 2), (301, 7, 3), (512, 2, 5), (640, 3, 3), (1100, 4, 3)])
def test_attention_of_ragged_batches_dealt_out_to_the_xcds(P, longest, B, heads):
    """From four strips of queries on, the (sequence, head) pairs of a ragged batch are dealt out: with and without pairs left over after
    whole rounds of eight, fewer than eight, and sequences that end in a block's first strip; INT8 bit-exact, FP16 within tolerance."""
    rng = np.random.default_rng(longest + B * heads)
    lens = rng.integers(1, longest + 1, B)
    lens[B // 2] = longest
    cu, H = _cu(lens), heads * 64
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * H)) * 26), -127, 127).astype(np.int8)
    sc = (0.0209, 0.0249, 0.021, 0.0003, 0.0021)
    assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), longest, heads, *sc)), oracle.attention_i8(qkv, cu, heads, *sc))
    want = oracle.attention_i8_p16(qkv, cu, heads, sc[0], sc[1], sc[2], sc[4])
    assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), longest, heads, *sc, p_fp16=True)), want)
    f = (rng.standard_normal((int(cu[-1]), 3 * H)) * 0.6).astype(np.float16)
    want = oracle.attention_f16(f, cu, heads).astype(np.float64)
    assert np.abs(host(P.attention_f16(dev(f), dev(cu), longest, heads)).astype(np.float64) - want).max() <= 2e-3


@pytest.mark.parametrize("longest,B,heads", [(1, 800, 1), (31, 384, 2), (32, 383, 2), (32, 64, 12), (33, 384, 1), (64, 130, 3), (64, 127, 3), (65, 260, 1)])
def test_attention_of_many_short_sequences(P, longest, B, heads):
    """From 768 blocks on, sequences of one or two key tiles take one or two waves: sizes on either side, ragged; INT8 in its three softmax
    forms and the clamp bit-exact, FP16 the same bytes as the same sequences in a batch of fewer blocks (four waves)."""
    rng = np.random.default_rng(longest * B)
    lens = rng.integers(1, longest + 1, B)
    lens[::7] = longest
    cu, H = _cu(lens), heads * 64
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * H)) * 30), -127, 127).astype(np.int8)
    for sc in ((0.0209, 0.0249, 0.021, 0.004, 0.0021), (0.0209, 0.0249, 0.021, 0.02, 0.0021)):
        for kw in ({}, {"p_unsigned": True}):
            want = oracle.attention_i8(qkv, cu, heads, *sc, **kw)
            assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), longest, heads, *sc, **kw)), want)
    want = oracle.attention_i8_p16(qkv, cu, heads, sc[0], sc[1], sc[2], sc[4])
    assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), longest, heads, *sc, p_fp16=True)), want)
    f = (rng.standard_normal((int(cu[-1]), 3 * H)) * 0.6).astype(np.float16)
    whole = host(P.attention_f16(dev(f), dev(cu), longest, heads)).view(np.uint16)
    step = 40
    for b in range(0, B, step):
        e = min(B, b + step)
        part = host(P.attention_f16(dev(f[cu[b]:cu[e]]), dev(cu[b:e + 1] - cu[b]), longest, heads)).view(np.uint16)
        assert np.array_equal(part, whole[cu[b]:cu[e]])


@pytest.mark.parametrize("lens,heads", [([513], 1), ([700, 31, 1024], 2), ([2048, 515], 1)])
def test_long_sequence_attention_matches_the_oracle(P, lens, heads):
    """More than 512 keys: the calls that count codes take the three-sweep kernels (row maxima, row sums, codes and P.V,
    recomputing the integer scores each time), the plain ones eight waves that keep the scores; both must give what the
    oracle's plain definition gives: int8 contexts bit-exact for signed and unsigned softmax codes, the code histogram
    exact, the fp16 flavour within its tolerance."""
    rng = np.random.default_rng(sum(lens) + 9)
    H = heads * 64
    cu = _cu(lens)
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * H)) * 26), -127, 127).astype(np.int8)
    for p_unsigned, sc in ((False, (0.0209, 0.0249, 0.021, 0.0003, 0.0021)), (True, (0.03, 0.03, 0.021, 0.0004, 0.0012)),
                           (False, (0.05, 0.05, 0.021, 0.004, 0.006))):
        want = oracle.attention_i8(qkv, cu, heads, *sc, p_unsigned=p_unsigned)
        got, hist = P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc, p_unsigned=p_unsigned, want_hist=True)
        assert np.array_equal(host(got), want)
        assert np.abs(want).max() > 10
        assert int(host(hist).sum()) == heads * sum(n * n for n in lens)
        plain = P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc, p_unsigned=p_unsigned)
        assert np.array_equal(host(plain), want)
    b = len(lens) - 1                                         # code usage of the last sequence against the oracle's dump
    sl = slice(cu[b], cu[b + 1])
    sc = (0.03, 0.03, 0.021, 0.0004, 0.0012)
    one = np.array([0, lens[b]], np.int32)
    _, Pq = oracle.attention_i8(qkv[sl], one, heads, *sc, dump_p=True, p_unsigned=True)
    _, hist = P.attention_i8(dev(qkv[sl]), dev(one), lens[b], heads, *sc, p_unsigned=True, want_hist=True)
    assert np.array_equal(host(hist), np.bincount(Pq.view(np.uint8).ravel(), minlength=256))
    f = (rng.standard_normal((int(cu[-1]), 3 * H)) * 0.6).astype(np.float16)
    want = oracle.attention_f16(f, cu, heads).astype(np.float64)
    got = host(P.attention_f16(dev(f), dev(cu), max(lens), heads)).astype(np.float64)
    assert np.abs(got - want).max() <= 2e-3
    assert np.abs(got - want).mean() <= 1e-4


def test_attention_at_the_longest_supported_sequence(P):
    """4096 tokens, the largest max_len the library takes: all three INT8 softmax-output forms bit-exact."""
    rng = np.random.default_rng(4096)
    heads, n = 1, 4096
    cu = _cu([n])
    qkv = np.clip(np.rint(rng.standard_normal((n, 3 * 64)) * 26), -127, 127).astype(np.int8)
    sc = (0.0209, 0.0249, 0.021, 0.0001, 0.0012)
    for kw in ({}, {"p_unsigned": True}):
        want = oracle.attention_i8(qkv, cu, heads, *sc, **kw)
        assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), n, heads, *sc, **kw)), want)
        assert np.abs(want).max() > 10
    want = oracle.attention_i8_p16(qkv, cu, heads, sc[0], sc[1], sc[2], sc[4])
    assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), n, heads, *sc, p_fp16=True)), want)
    with pytest.raises(P.SampError):
        P.attention_i8(dev(qkv), dev(cu), n + 1, heads, *sc)


def test_long_kernel_equals_one_pass_kernel_on_short_sequences(P):
    """A batch whose longest row exceeds 512 tokens runs every sequence, also the short ones, through the eight-wave kernel,
    beyond 2048 through the three-sweep kernel: their contexts must be the bytes the four-wave kernel writes when the same
    short sequences come alone."""
    for longest in (600, 2100):
        long_against_short(P, longest)


def long_against_short(P, longest):
    rng = np.random.default_rng(77)
    heads, lens = 2, [longest, 128, 37, 512]
    H = heads * 64
    cu = _cu(lens)
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * H)) * 26), -127, 127).astype(np.int8)
    sc = (0.0209, 0.0249, 0.021, 0.0003, 0.0021)
    mixed = host(P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc))
    short = host(P.attention_i8(dev(qkv[cu[1]:]), dev(_cu(lens[1:])), 512, heads, *sc))
    assert np.array_equal(mixed[cu[1]:], short)


@pytest.mark.parametrize("longest", [640, 641, 769, 1025, 1281, 1537, 1793, 2048])
def test_every_number_of_key_tiles_per_wave(P, longest):
    """Lengths on either side of each step of the dispatch (tiles held per wave, the V^T tiles that take turns in LDS), with
    short sequences whose later tiles do not exist: INT8 in its three softmax forms bit-exact, FP16 within tolerance."""
    rng = np.random.default_rng(longest)
    heads, lens = 1, [longest, 33, longest - 1, 1, 257]
    cu = _cu(lens)
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * 64)) * 26), -127, 127).astype(np.int8)
    sc = (0.0209, 0.0249, 0.021, 0.0003, 0.0021)
    for kw in ({}, {"p_unsigned": True}):
        want = oracle.attention_i8(qkv, cu, heads, *sc, **kw)
        assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), longest, heads, *sc, **kw)), want)
        assert np.abs(want).max() > 10
    want = oracle.attention_i8_p16(qkv, cu, heads, sc[0], sc[1], sc[2], sc[4])
    assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), longest, heads, *sc, p_fp16=True)), want)
    f = (rng.standard_normal((int(cu[-1]), 3 * 64)) * 0.6).astype(np.float16)
    want = oracle.attention_f16(f, cu, heads).astype(np.float64)
    assert np.abs(host(P.attention_f16(dev(f), dev(cu), longest, heads)).astype(np.float64) - want).max() <= 2e-3


def test_three_sweep_attention_of_ragged_sequences(P):
    """Beyond 2048 tokens (1536 with the binary16 softmax output) without a histogram: sequences of every number of key tiles per
    wave, down to one key, behind one that is too long for the registers; all three INT8 forms bit-exact."""
    rng = np.random.default_rng(2100)
    heads, lens = 1, [2100, 33, 1, 700, 1281, 128]
    cu = _cu(lens)
    qkv = np.clip(np.rint(rng.standard_normal((int(cu[-1]), 3 * 64)) * 26), -127, 127).astype(np.int8)
    sc = (0.0209, 0.0249, 0.021, 0.0002, 0.0015)
    for kw in ({}, {"p_unsigned": True}):
        want = oracle.attention_i8(qkv, cu, heads, *sc, **kw)
        assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc, **kw)), want)
        assert np.abs(want).max() > 10
    want = oracle.attention_i8_p16(qkv, cu, heads, sc[0], sc[1], sc[2], sc[4])
    assert np.array_equal(host(P.attention_i8(dev(qkv), dev(cu), max(lens), heads, *sc, p_fp16=True)), want)


def test_fp16_attention_is_the_same_bytes_in_one_pass_and_in_three_sweeps(P):
    """A batch whose longest sequence exceeds 2048 tokens takes the three-sweep kernel; its other sequences must come out as
    they do alone, where the scores of every length stay in registers."""
    rng = np.random.default_rng(5)
    heads, lens = 2, [2049, 130, 700, 390, 1500]
    cu = _cu(lens)
    f = (rng.standard_normal((int(cu[-1]), 3 * 64 * heads)) * 0.6).astype(np.float16)
    mixed = host(P.attention_f16(dev(f), dev(cu), max(lens), heads))
    for b in range(1, len(lens)):
        alone = host(P.attention_f16(dev(f[cu[b]:cu[b + 1]]), dev(_cu(lens[b:b + 1])), lens[b], heads))
        assert np.array_equal(mixed[cu[b]:cu[b + 1]].view(np.uint16), alone.view(np.uint16))


# ------------------------------------------------------------------ fused bias + residual + LayerNorm (+ quant)
@pytest.mark.parametrize("H", [128, 768, 1024])
@pytest.mark.parametrize("in8,res8,out8", [(1, 1, 1), (1, 1, 0), (0, 0, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0)])
def test_add_ln_bit_exact(P, H, in8, res8, out8):
    check_add_ln(P, 37, H, in8, res8, out8)


@pytest.mark.parametrize("M,H", [(4099, 768), (4099, 1024), (37, 512), (5, 256)])
@pytest.mark.parametrize("in8,res8,out8", [(1, 1, 1), (1, 1, 0), (0, 0, 1), (0, 0, 0), (1, 0, 1), (0, 1, 0)])
def test_add_ln_in_the_forms_that_37_rows_do_not_take(P, M, H, in8, res8, out8):
    """From 4096 rows 16 lanes share a row at every width (with a ragged last block here); widths of 256 and 512 with one wave
    per row."""
    check_add_ln(P, M, H, in8, res8, out8)


def check_add_ln(P, M, H, in8, res8, out8):
    rng = np.random.default_rng(H + in8 * 4 + res8 * 2 + out8)
    a = rng.integers(-127, 128, (M, H), dtype=np.int8) if in8 else (rng.standard_normal((M, H)) * 0.5).astype(np.float16)
    r = rng.integers(-127, 128, (M, H), dtype=np.int8) if res8 else rng.standard_normal((M, H)).astype(np.float16)
    bias = (rng.standard_normal(H) * 0.1).astype(np.float32)
    g = (1 + 0.1 * rng.standard_normal(H)).astype(np.float32)
    be = (0.1 * rng.standard_normal(H)).astype(np.float32)
    s_in, s_res, s_out, eps = 0.0105, 0.0372, 0.0369, 1e-12
    want = oracle.add_ln(a, s_in, bias, r, s_res, g, be, eps, bool(out8), s_out)
    got = host(P.add_ln(dev(a), s_in, dev(bias), dev(r), s_res, dev(g), dev(be), eps, bool(out8), s_out))
    assert np.array_equal(got.view(np.uint8 if out8 else np.uint16), want.view(np.uint8 if out8 else np.uint16))


# ------------------------------------------------------------------ create-time and entry steps
def test_weight_quantisation_bit_exact(P):
    rng = np.random.default_rng(31)
    W = (rng.standard_normal((300, 768)) * 0.02).astype(np.float16)
    W[17] = 0
    Wq, s_w = P.quantize_weight(dev(W))
    wq, sw = oracle.quantize_weight(W)
    assert np.array_equal(host(Wq), wq) and np.array_equal(host(s_w), sw)


@pytest.mark.parametrize("quant", [False, True])
def test_padding_removal_packs_valid_rows(P, quant):
    rng = np.random.default_rng(32)
    B, S, H = 5, 40, 128
    lens = np.array([40, 1, 17, 33, 8], np.int32)
    hid = rng.standard_normal((B, S, H)).astype(np.float16)
    mask = (np.arange(S)[None, :] < lens[:, None]).astype(np.int32)
    s_x = 0.0371 if quant else 0.0
    packed, cu, row_map = P.pack_rows(dev(hid), dev(mask), s_x)
    packed, cu, row_map = host(packed), host(cu), host(row_map)
    assert np.array_equal(cu, _cu(lens))
    T = int(cu[-1])
    rows = np.concatenate([hid[b, :lens[b]] for b in range(B)])
    want = oracle.quantize_f16(rows, s_x) if quant else rows
    assert np.array_equal(packed[:T], want)
    assert np.array_equal(row_map[:T], np.concatenate([b * S + np.arange(lens[b]) for b in range(B)]))


@pytest.mark.parametrize("B,S", [(1, 1), (3, 63), (63, 65), (64, 2), (65, 1023), (17, 1024), (2, 1025), (130, 1100), (5, 2048)])
def test_sequence_offsets_at_the_edges_of_pieces_and_scans(P, B, S):
    """Pieces of 1024 mask entries, sixteen waves, prefix sums of 64 sequences at a time."""
    lens = np.random.default_rng(B + S).integers(1, S + 1, B).astype(np.int32)
    lens[0], lens[-1] = S, max(1, S // 2)
    mask = (np.arange(S)[None, :] < lens[:, None]).astype(np.int32)
    _, cu, _ = P.pack_rows(dev(np.zeros((B, S, 8), np.float16)), dev(mask))
    assert np.array_equal(host(cu), _cu(lens))


# ------------------------------------------------------------------ embedding kernel
@pytest.mark.parametrize("H", [128, 768, 1024])
def test_embedding_kernel_bit_exact(P, H):
    rng = np.random.default_rng(H + 50)
    V, B, S = 97, 3, 21
    emb = {"tok": (rng.standard_normal((V, H)) * 0.5).astype(np.float16), "seg": (rng.standard_normal((2, H)) * 0.5).astype(np.float16),
           "pos": (rng.standard_normal((S + 3, H)) * 0.5).astype(np.float16),
           "gamma": (1 + 0.2 * rng.standard_normal(H)).astype(np.float32), "beta": (0.3 * rng.standard_normal(H)).astype(np.float32),
           "eps": 1e-12}
    ids = rng.integers(-3, V + 3, (B, S)).astype(np.int32)          # a few ids outside the table: clamped on both sides
    seg = rng.integers(0, 2, (B, S)).astype(np.int32)
    E = P.Embedding(emb["tok"], emb["seg"], emb["pos"], emb["gamma"], emb["beta"], emb["eps"])
    for out_i8, s_out in ((False, 1.0), (True, 0.031)):
        want = np.concatenate([oracle.embed_ln(emb, ids[b], seg[b], out_i8, s_out) for b in range(B)])
        got = host(P.embed_ln(E, dev(ids), dev(seg), out_i8, s_out))
        assert np.array_equal(got, want)
    want = np.concatenate([oracle.embed_ln(emb, ids[b], None, False) for b in range(B)])
    assert np.array_equal(host(P.embed_ln(E, dev(ids), None, False)), want)
    short = P.Embedding(emb["tok"], emb["seg"], emb["pos"][:S - 1], emb["gamma"], emb["beta"], emb["eps"])
    with pytest.raises(P.SampError):
        P.embed_ln(short, dev(ids), None, False)                    # position table shorter than the sequences


@pytest.mark.parametrize("H", [256, 768])
def test_embedding_kernel_of_many_positions(P, H):
    """From 16384 positions the lanes of a row are chosen by the bytes each writes (16 lanes at 256 and for INT8 at 768, a wave
    for FP16 at 768); the last block is a ragged one."""
    rng = np.random.default_rng(H)
    V, B, S = 97, 127, 131
    emb = {"tok": (rng.standard_normal((V, H)) * 0.5).astype(np.float16), "seg": (rng.standard_normal((2, H)) * 0.5).astype(np.float16),
           "pos": (rng.standard_normal((S, H)) * 0.5).astype(np.float16), "gamma": (1 + 0.2 * rng.standard_normal(H)).astype(np.float32),
           "beta": (0.3 * rng.standard_normal(H)).astype(np.float32), "eps": 1e-12}
    ids, seg = rng.integers(0, V, (B, S)).astype(np.int32), rng.integers(0, 2, (B, S)).astype(np.int32)
    E = P.Embedding(emb["tok"], emb["seg"], emb["pos"], emb["gamma"], emb["beta"], emb["eps"])
    for out_i8, s_out in ((False, 1.0), (True, 0.031)):
        want = np.concatenate([oracle.embed_ln(emb, ids[b], seg[b], out_i8, s_out) for b in range(B)])
        assert np.array_equal(host(P.embed_ln(E, dev(ids), dev(seg), out_i8, s_out)), want)


# ------------------------------------------------------------------ classification target
@pytest.mark.parametrize("B,S,H,Cn", [(5, 7, 128, 3), (32, 128, 768, 15), (2, 1, 1024, 119)])
def test_classification_target_within_accumulation_tolerance(P, B, S, H, Cn):
    rng = np.random.default_rng(B + H + Cn)
    hid = rng.standard_normal((B, S, H)).astype(np.float16)
    wp = (rng.standard_normal((H, H)) * 0.05).astype(np.float16)
    bp = (rng.standard_normal(H) * 0.1).astype(np.float32)
    wc = (rng.standard_normal((Cn, H)) * 0.05).astype(np.float16)
    bc = (rng.standard_normal(Cn) * 0.1).astype(np.float32)
    want = oracle.classify(hid, wp, bp, wc, bc)
    got = host(P.classify(dev(hid), dev(wp), dev(bp), dev(wc), dev(bc))).astype(np.float64)
    # binary32 accumulation over H terms and a binary32 tanh against binary64: a few 1e-6 relative
    assert np.abs(got - want).max() <= 2e-5 * max(1.0, np.abs(want).max())
    assert np.array_equal(got.argmax(axis=1), want.argmax(axis=1))


@pytest.mark.parametrize("B,S,H,Cn", [(3, 2, 8, 1), (1, 3, 776, 9), (2, 1, 4096, 8)])
def test_classification_target_at_ragged_widths(P, B, S, H, Cn):
    """Widths that leave part of the last 256-channel section (or almost all of the first) empty, and class counts on
    either side of the eight rows a wave takes at a time."""
    test_classification_target_within_accumulation_tolerance(P, B, S, H, Cn)


@pytest.mark.parametrize("B,S,H,Cn", [(1, 1, 8, 1), (3, 2, 776, 9), (4, 1, 768, 8), (5, 3, 1024, 119), (33, 2, 264, 17)])
def test_classification_target_without_a_workspace_gives_the_same_bits(P, B, S, H, Cn):
    import torch
    rng = np.random.default_rng(B + H)
    t = [dev(rng.standard_normal(shape).astype(dtype)) for shape, dtype in (((B, S, H), np.float16), ((H, H), np.float16), (H, np.float32),
                                                                           ((Cn, H), np.float16), (Cn, np.float32))]
    logits = torch.empty((B, Cn), dtype=torch.float32, device="cuda")
    ptr = [ctypes.c_void_p(x.data_ptr()) for x in t + [logits]]
    assert P.lib().samp_classify(ptr[0], B, S, H, *ptr[1:5], Cn, ptr[5], ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)) == 0
    assert np.array_equal(host(logits), host(P.classify(*t)))


@pytest.mark.parametrize("H", [8, 256, 264, 768, 1024, 1288, 4096])
def test_classification_target_adds_up_in_the_order_of_64_lanes(P, H):
    """The error of a binary32 sum follows its order: chains of one fused multiply-add per channel, one chain per eight
    channels of a 512-channel section (H / 64 products long), met in a tree of 64.  The second product is replayed in
    that order, each multiply-add in extended precision and rounded once; its input, the pooled vector, is read
    through a unit matrix first (a sum of one product and zeros is exact)."""
    rng = np.random.default_rng(H)
    Cn = 203
    hid = rng.standard_normal((1, 1, H)).astype(np.float16)
    wp = (rng.standard_normal((H, H)) * H ** -0.5).astype(np.float16)
    bp = (rng.standard_normal(H) * 0.1).astype(np.float32)
    wc = (rng.standard_normal((Cn, H)) * 0.05).astype(np.float16)
    pool = lambda w: host(P.classify(dev(hid), dev(wp), dev(bp), dev(w), dev(np.zeros(len(w), np.float32))))[0]
    pooled = pool(np.eye(H, dtype=np.float16))
    got = pool(wc)
    chains = np.zeros((Cn, 64), np.float32)
    for k in range(0, H, 8):
        lane = k // 8 % 64
        for e in range(k, k + 8):
            chains[:, lane] = (wc[:, e].astype(np.longdouble) * np.longdouble(pooled[e]) + chains[:, lane]).astype(np.float32)
    step = 32
    while step:
        chains = chains + chains[:, np.arange(64) ^ step]
        step //= 2
    assert np.array_equal(got, chains[:, 0])


def test_entry_quantiser_bit_exact(P):
    """samp_quantize_f16_i8: the un-masked entry quantiser, incl. ties, values beyond the clamp and a ragged tail of
    the grid (element count not a multiple of the block size)."""
    rng = np.random.default_rng(3)
    s_x = 0.0371
    x = (rng.standard_normal(1000 * 768 + 8) * 1.3).astype(np.float16)
    x[:16] = np.float16([0.5 * s_x, 1.5 * s_x, 2.5 * s_x, -0.5 * s_x, 127.4 * s_x, 127.6 * s_x, 400.0, -400.0,
                         0.0, -0.0, 6e-8, -6e-8, 65504.0, -65504.0, s_x, -s_x])
    got = host(P.quantize_f16_i8(dev(x), s_x))
    assert np.array_equal(got, oracle.quantize_f16(x, s_x))
    assert got.max() == 127 and got.min() == -127


def test_a_sequence_with_an_all_zero_mask_row_is_inert(P):
    """The mask is not checked on the host (no synchronisation): an empty sequence takes part in nothing, its output
    rows are zeros, and the other sequences get exactly what they get without it."""
    import torch
    import samp_workloads as W
    w = W.Workload("empty", 2, 128, 2, 256, 4, 24, (W.FULL_INT8, W.FFN_INT8), varlen=True, min_len=1, plain_params=False,
                   calib_batch=2, calib_seq=24)
    wts = W.make_weights(w)
    hid, _, _ = W.make_hidden(w)
    a = (w.layers, w.hidden, w.heads, w.ffn, w.ln_eps)
    sc = oracle.calibrate(*a, wts, W.make_calibration_batch(w))
    lens = np.array([5, 0, 24, 1], np.int32)
    mask = (np.arange(w.seq)[None, :] < lens[:, None]).astype(np.int32)
    enc = P.Encoder(*a, w.modes, wts, sc, max_batch=4, max_seq=24)
    out = host(enc.forward(dev(hid), dev(mask)))
    keep = [0, 2, 3]
    out3 = host(enc.forward(dev(hid[keep]), dev(mask[keep])))
    enc.close()
    assert not out[1].any()
    assert np.array_equal(out[keep], out3)
    for b in range(4):
        assert not out[b, lens[b]:].any()


# ------------------------------------------------------------------ measured ceilings
def test_peak_probes_return_plausible_rates(P):
    """The probes behind bench.py's `peaks_measured`: matrix-instruction issue rate, device copy, operand feed.
    Loose sanity ranges only (an MI355X is far above the lower ends); random operands never beat constant ones by much."""
    const_i8, rand_i8 = P.probe_mfma_rate(False, False, 4000), P.probe_mfma_rate(False, True, 4000)
    assert 5e14 < rand_i8 < 6e15 and 5e14 < const_i8 < 6e15 and rand_i8 < 1.1 * const_i8
    assert 2e14 < P.probe_mfma_rate(True, True, 4000) < 3e15
    assert 5e11 < P.probe_copy_rate(1 << 28, 3) < 1e13
    assert 1e12 < P.probe_feed_rate(4096, 768, 768, 5) < 2e14


def _us_per_call(f, calls=50):
    """The fastest of five runs of `calls` calls."""
    import time
    import torch
    f()
    best = np.inf
    for _ in range(5):
        torch.cuda.synchronize()
        t = time.perf_counter()
        for _ in range(calls):
            f()
        torch.cuda.synchronize()
        best = min(best, (time.perf_counter() - t) / calls * 1e6)
    return best


@pytest.mark.parametrize("B,S", [(8192, 1), (8192, 4), (1024, 64), (1023, 65), (15, 64), (16, 64), (17, 63), (257, 128), (33, 512), (33, 513), (1, 1025), (3, 4096),
                                 (1, 1), (2, 8), (16, 1), (17, 1), (5, 192), (5, 193), (4, 256), (64, 64), (65, 64), (64, 65), (1, 1024), (1, 4096), (1, 4097), (20, 192)])
def test_sequence_offsets_of_many_short_rows(P, B, S):
    """One, four or sixteen chunks of 64 entries per wave and round, over row ends and past the last row; with entries behind a zero, and other values than one."""
    rng = np.random.default_rng(B + S)
    mask = (rng.random((B, S)) < 0.7).astype(np.int32) * rng.integers(-3, 4, (B, S)).astype(np.int32)
    mask[:, 0] = 1
    _, cu, _ = P.pack_rows(dev(np.zeros((B, S, 8), np.float16)), dev(mask))
    assert np.array_equal(host(cu), np.concatenate([[0], np.cumsum((mask != 0).sum(1))]))


def test_sequence_offsets_do_not_wait_for_every_short_row(P):
    """8192 rows of four entries against 32 rows of 1024, the same number of entries: the rows' latencies overlap.  (One row or less per wave and
    round: 354 and 633 us against 25; now about 110.)"""
    run = {}
    for B, S in ((8192, 4), (32, 1024)):
        hidden, mask = dev(np.zeros((B, S, 8), np.float16)), dev(np.ones((B, S), np.int32))
        run[S] = _us_per_call(lambda: P.pack_rows(hidden, mask))
    assert run[4] < 9 * run[1024], run


def _us_in_a_graph(f, calls=50):
    """Per call, of `calls` calls in one graph: no host time between them.  The fastest of ten replays."""
    import torch
    f()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        for _ in range(calls):
            f()
    best = np.inf
    for _ in range(10):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        g.replay()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / calls)
    return best


def test_sequence_offsets_of_few_rows_take_no_longer_than_their_launch(P):
    """Offsets and packing of two rows of eight tokens against two launches that fill one value each: 3.7 against 3.3 us (4.8 where every wave
    has the loads of sixteen chunks)."""
    import torch
    from paper_2209_09130_amd import binding
    B, S, H = 2, 8, 8
    hidden, mask = dev(np.zeros((B, S, H), np.float16)), dev(np.ones((B, S), np.int32))
    packed, cu, row_map = torch.zeros_like(hidden), dev(np.zeros(B + 1, np.int32)), dev(np.zeros(B * S, np.int32))

    def pack():
        dp = binding._dp
        binding._check(P.lib().samp_pack_rows(dp(hidden), dp(mask), B, S, H, binding._f(0.0), dp(packed), dp(cu), dp(row_map), binding._stream()))

    one = torch.zeros(1, device="cuda")
    took, launches = _us_in_a_graph(pack), _us_in_a_graph(lambda: (one.zero_(), one.zero_()))
    assert took < 1.3 * launches, (took, launches)
