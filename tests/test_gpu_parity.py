"""GPU parity: every entry point of the C ABI against the CPU oracle, element by element,
on the same seeded host-generated inputs.  Integer / packed outputs must be bit-exact;
the fp32 epilogue must match within 1e-6 relative (it is in fact built to be bit-exact)."""
import ctypes
import os

import numpy as np
import pytest
import torch

import oracle
from paper_1911_04477_amd import binding as B
from paper_1911_04477_amd import inputs

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def as_u64(t):
    return host(t).view("<u8")


def assert_f32_close(got, ref):
    assert got.shape == ref.shape
    # 1e-6 relative, as the contract asks; report bit-exactness too
    assert np.allclose(got, ref, rtol=1e-6, atol=1e-30), np.abs(got - ref).max()


def kernels_of(call):
    """call()'s result and the names of the kernels it launched, in order."""
    B.prof_enable(True)
    try:
        B.prof_reset()
        out = call()
        return out, [name for name, _ in B.prof_records()]
    finally:
        B.prof_enable(False)


# ---------------------------------------------------------------- encode (a1)
@pytest.mark.parametrize("rows,K", [(1, 1), (3, 31), (5, 64), (7, 65), (64, 256), (33, 200), (2, 4097), (130, 1152),
                                     (1000, 63), (17, 1024 + 13)])
def test_encode_matches_oracle(rows, K):
    print(f"encode rows={rows} K={K}", flush=True)
    rng = np.random.default_rng(rows * 100003 + K)
    x = inputs.inject_specials(rng.standard_normal((rows, K)).astype(np.float32), K, frac=0.01)
    got = as_u64(B.bnn_encode(dev(x)))
    assert np.array_equal(got, oracle.encode_rows(x))


@pytest.mark.parametrize("rows,K,gap,dst_gap", [
    (1, 1024, 0, 0), (3, 1000, 0, 0), (5, 1030, 0, 0), (40, 64, 0, 0), (17, 128, 12, 0), (33, 960, 4, 3), (7, 2047, 1, 1),
    (2, 4032, 0, 2), (9, 1088, 0, 0), (70, 65, 0, 0), (15, 64, 0, 0), (6, 3000, 0, 0)])
def test_encode_waves_of_whole_and_partial_words(rows, K, gap, dst_gap):
    """16 words a wave: inside a row, up to its end (whole or not), over rows with and without a gap, and fewer than 16."""
    print(f"encode waves rows={rows} K={K} gaps {gap} {dst_gap}", flush=True)
    rng = np.random.default_rng(rows + K)
    x = inputs.inject_specials(rng.standard_normal((rows, K + gap)).astype(np.float32), K, frac=0.01)
    Kw = B.packed_words(K)
    dst = torch.full((rows, Kw + dst_gap), -1, dtype=torch.int64, device=DEV)
    B.bnn_encode(dev(x)[:, :K], dst[:, :Kw])
    out = as_u64(dst)
    assert np.array_equal(out[:, :Kw], oracle.encode_rows(np.ascontiguousarray(x[:, :K])))
    assert np.all(out[:, Kw:] == np.uint64(0xFFFFFFFFFFFFFFFF))


def test_encode_more_words_than_a_launch_has_threads_for():
    print("encode 2^31 + 1000 rows of one value", flush=True)
    rows = 2 ** 31 + 1000
    src = torch.empty((rows, 1), dtype=torch.float32, device=DEV).fill_(-1.0)
    at = torch.randint(0, rows, (100000,), device=DEV, generator=torch.Generator(device=DEV).manual_seed(1))
    at[:2000] = torch.arange(rows - 2000, rows, device=DEV)
    src[at] = 1.0
    dst = torch.full((rows, 1), -1, dtype=torch.int64, device=DEV)
    B.bnn_encode(src, dst)
    assert bool((dst[at] == 1).all())
    ones, step = 0, 2 ** 28
    for r in range(0, rows, step):
        part = dst[r:r + step]
        assert bool(((part == 0) | (part == 1)).all())
        ones += int(part.sum())
    assert ones == int(torch.unique(at).numel())


def test_encode_strided_src_and_dst():
    print("encode strided", flush=True)
    rng = np.random.default_rng(5)
    rows, K, sld, dld = 37, 130, 140, 5
    big = rng.standard_normal((rows, sld)).astype(np.float32)
    src = dev(big)[:, :K]
    dst = torch.full((rows, dld), -1, dtype=torch.int64, device=DEV)
    B.bnn_encode(src, dst[:, :3])
    out = as_u64(dst)
    assert np.array_equal(out[:, :3], oracle.encode_rows(big[:, :K]))
    assert np.all(out[:, 3:] == np.uint64(0xFFFFFFFFFFFFFFFF))  # words past Kw untouched


def test_encode_cfg2_weights_full_size():
    print("encode cfg2 weights 4096x4096", flush=True)
    d = inputs.cfg2()
    got = as_u64(B.bnn_encode(dev(d["wt"])))
    assert np.array_equal(got, oracle.encode_rows(d["wt"]))


# ---------------------------------------------------------------- weight packing / im2col (a2)
CONV_CASES = [
    # N, C, H, W, D, kH, kW, sH, sW, pH, pW
    (2, 64, 6, 6, 5, 3, 3, 1, 1, 1, 1),
    (2, 128, 9, 7, 33, 3, 3, 1, 1, 1, 1),
    (3, 70, 8, 8, 9, 3, 3, 2, 2, 1, 1),
    (2, 200, 10, 10, 17, 1, 1, 2, 2, 0, 0),
    (1, 3, 12, 12, 4, 5, 5, 1, 1, 2, 2),
    (2, 256, 5, 6, 70, 3, 3, 1, 1, 0, 0),
    (1, 130, 7, 9, 3, 3, 1, 1, 2, 1, 0),
    (5, 192, 4, 4, 130, 1, 1, 1, 1, 0, 0),
    (1, 512, 8, 8, 12, 3, 3, 1, 1, 1, 1),
    (2, 32, 6, 5, 6, 2, 2, 1, 1, 1, 1),
    (1, 1, 3, 3, 1, 3, 3, 1, 1, 1, 1),
]


@pytest.mark.parametrize("case", CONV_CASES)
def test_pack_weight_and_im2col_match_oracle(case):
    print(f"im2col case={case}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    rng = np.random.default_rng(sum(case))
    x = inputs.inject_specials(rng.standard_normal((N, C, H, W)).astype(np.float32), 1, frac=0.01)
    w = inputs.inject_specials(rng.standard_normal((D, C, kH, kW)).astype(np.float32), 2, frac=0.01)
    assert np.array_equal(as_u64(B.bnn_pack_conv_weight(dev(w))), oracle.pack_conv_weight(w))
    cols = as_u64(B.bnn_im2col_packed(dev(x), kH, kW, (sH, sW), (pH, pW)))
    assert np.array_equal(cols, oracle.im2col_packed(x, kH, kW, (sH, sW), (pH, pW)))


# ---------------------------------------------------------------- GEMM (a3)
# tile configurations of the GEMM (bnn_testing.h) and the kernel each runs on; 21 and 22 exist with the packed epilogue
GEMM_KERNELS = {1: "xnor_gemm", 2: "xnor_gemm_small", 3: "xnor_gemm", 4: "xnor_gemm", 6: "xnor_gemm",
                23: "xnor_gemm_fp4", 24: "xnor_gemm_fp4", 25: "xnor_gemm_fp4_split", 26: "xnor_gemm_fp4_split",
                27: "xnor_gemm_fp4_split", 28: "xnor_gemm_fp4_split"}
PACKED_KERNELS = {1: "xnor_gemm", 3: "xnor_gemm", 4: "xnor_gemm", 6: "xnor_gemm", 21: "xnor_gemm_fp4",
                  22: "xnor_gemm_fp4", **{c: k for c, k in GEMM_KERNELS.items() if c >= 23}}


def _gemm_case(M, N, K, seed, cfg=None):
    rng = np.random.default_rng(seed)
    A = inputs.inject_specials(rng.standard_normal((M, K)).astype(np.float32), seed, frac=0.002)
    Bm = inputs.inject_specials(rng.standard_normal((N, K)).astype(np.float32), seed + 1, frac=0.002)
    Ap, Bp = B.bnn_encode(dev(A)), B.bnn_encode(dev(Bm))
    C, names = kernels_of(lambda: B.bnn_xnor_gemm(Ap, Bp, K, cfg=cfg))
    assert np.array_equal(host(C), oracle.gemm_pm1(A, Bm))
    if cfg is not None:
        assert names == [GEMM_KERNELS[cfg]]


# K = 130 / 192 (three-word rows: dword-at-a-time tail), 400 / 704 (4n + 3 words: window chunk at an odd word)
@pytest.mark.parametrize("K", [1, 31, 32, 33, 63, 64, 65, 130, 192, 200, 256, 257, 400, 511, 512, 544, 704, 1152,
                               2304 + 17])
@pytest.mark.parametrize("cfg", GEMM_KERNELS)
def test_gemm_k_sweep_all_tile_configs(K, cfg):
    print(f"gemm K={K} cfg={cfg}", flush=True)
    _gemm_case(37, 150, K, seed=K * 7 + cfg, cfg=cfg)


@pytest.mark.parametrize("M,N", [(1, 1), (1, 700), (65, 513), (64, 512), (130, 1030), (257, 64), (33, 65)])
@pytest.mark.parametrize("cfg", GEMM_KERNELS)
def test_gemm_ragged_tiles(M, N, cfg):
    print(f"gemm M={M} N={N} cfg={cfg}", flush=True)
    _gemm_case(M, N, 300, seed=M * 1000 + N + cfg, cfg=cfg)


@pytest.mark.parametrize("cfg", [1, 3])
@pytest.mark.parametrize("K", [1, 63, 64, 130, 192, 200, 256, 400, 512, 704, 1152, 2304 + 17])
def test_gemm_four_columns_per_lane_tiles_k_sweep(K, cfg):
    """N a multiple of 4: the 256-column tiles take four consecutive columns per lane and store 16 bytes
    (N = 150 in the sweep above takes the one-column form); every kind of K tail, one and several tiles."""
    print(f"gemm four-column tiles K={K} cfg={cfg}", flush=True)
    _gemm_case(37, 152, K, seed=K * 11 + cfg, cfg=cfg)
    _gemm_case(70, 516, K, seed=K * 13 + cfg, cfg=cfg)


@pytest.mark.parametrize("lean", [1, 0])
@pytest.mark.parametrize("cfg", [1, 3])
@pytest.mark.parametrize("case", [(3, 128, 8, 8, 40, 3, 3, 1, 1, 1, 1), (3, 128, 10, 10, 70, 3, 3, 1, 1, 1, 1),
                                  (2, 64, 7, 9, 33, 3, 3, 1, 1, 1, 1), (5, 192, 6, 6, 130, 3, 3, 2, 2, 1, 1),
                                  (4, 128, 12, 12, 64, 1, 1, 2, 2, 0, 0), (7, 256, 6, 6, 65, 3, 3, 1, 1, 1, 1)])
def test_conv2d_four_columns_per_lane_tiles(case, cfg, lean):
    """int32 and fp32 NCHW outputs of the 256-column tiles with both gathers: maps whose pixel count is a
    multiple of 4 (16-byte stores, four-pixel groups that must not straddle images: 64, 100 and 36 pixels
    per image against 256 columns per tile) and maps where it is not (63 and 9: one column per lane)."""
    print(f"conv2d four-column tiles case={case} cfg={cfg} lean={lean}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    d = inputs.conv_inputs(inputs.ConvShape(*case), seed=sum(case) + 31)
    x = inputs.inject_specials(d["x"], 8, frac=0.01)
    xp = _u64dev(oracle.pack_nhwc(x))
    wp = B.bnn_pack_conv_weight(dev(d["w"]))
    sc, bi = dev(d["scale"]), dev(d["bias"])
    st, pd = (sH, sW), (pH, pW)
    ref = oracle.conv2d_pm1(x, d["w"], st, pd)
    assert np.array_equal(host(B.bnn_conv2d_packed(xp, wp, C, D, kH, kW, st, pd, out="i32", cfg=cfg, lean=lean)), ref)
    yref = oracle.scale_bias(ref, d["scale"], d["bias"], "nchw")
    got = host(B.bnn_conv2d_packed(xp, wp, C, D, kH, kW, st, pd, scale=sc, bias=bi, out="f32", cfg=cfg, lean=lean))
    assert np.array_equal(got, yref)
    oi, of = B.bnn_conv2d(dev(x), wp, D, kH, kW, st, pd, sc, bi, want_int=True, cfg=cfg, lean=lean)
    assert np.array_equal(host(oi), ref) and np.array_equal(host(of), yref)


@pytest.mark.parametrize("cfg", [-1, 10, 11, 12])
@pytest.mark.parametrize("M,N,K", [(37, 152, 200), (8, 4, 65), (64, 256, 256), (130, 1028, 193), (257, 516, 128),
                                   (33, 260, 100), (70, 2052, 255), (5, 64, 129)])
def test_gemm_short_rows_kernel(M, N, K, cfg):
    """Rows of two or four words with N a multiple of 4: the store-bound kernel (four consecutive
    columns per lane, 16-byte stores), 8 and 16 rows per wave, and whatever the heuristic picks;
    int32 alone, and int32 + fp32 with the channel along either axis, on padded leading dimensions."""
    print(f"gemm short rows M={M} N={N} K={K} cfg={cfg}", flush=True)
    c = None if cfg < 0 else cfg
    rng = np.random.default_rng(M * 31 + N + K)
    A = inputs.inject_specials(rng.standard_normal((M, K)).astype(np.float32), 1, frac=0.01)
    Bm = inputs.inject_specials(rng.standard_normal((N, K)).astype(np.float32), 2, frac=0.01)
    Ap, Bp = as_u64(B.bnn_encode(dev(A))).copy(), as_u64(B.bnn_encode(dev(Bm))).copy()
    tail = K % 64
    if tail:  # garbage past K in both operands must not count
        g = np.uint64((0xFFFFFFFFFFFFFFFF >> tail) << tail)
        Ap[:, -1] |= g & np.uint64(0x5A5A5A5A5A5A5A5A)
        Bp[:, -1] |= g & np.uint64(0xF0F0F0F00F0F0F0F)
    Ad, Bd = dev(Ap.view(np.int64)), dev(Bp.view(np.int64))
    ref = oracle.gemm_pm1(A, Bm)
    Cbig = torch.full((M, N + 8), -7, dtype=torch.int32, device=DEV)
    B.bnn_xnor_gemm(Ad, Bd, K, Cbig[:, :N], cfg=c)
    out = host(Cbig)
    assert np.array_equal(out[:, :N], ref) and np.all(out[:, N:] == -7)
    for axis in ("row", "col"):
        nch = M if axis == "row" else N
        sc = ((rng.random(nch) + 0.5) * rng.choice([-1.0, 1.0], nch)).astype(np.float32)
        bi = rng.standard_normal(nch).astype(np.float32)
        Ci, Y = B.bnn_xnor_gemm_epilogue(Ad, Bd, K, dev(sc), dev(bi), B.CH_ROW if axis == "row" else B.CH_COL,
                                         want_int=True, cfg=c)
        assert np.array_equal(host(Ci), ref)
        assert np.array_equal(host(Y), oracle.scale_bias(ref, sc, bi, axis))


@pytest.mark.parametrize("cfg", [-1, *range(10, 18), *range(30, 38)])
@pytest.mark.parametrize("M,N,K,pa,pb", [(1, 1, 1, 0, 0), (33, 31, 64, 0, 0), (31, 129, 63, 1, 2), (65, 64, 65, 0, 1), (64, 300, 128, 2, 2),
                                         (130, 257, 129, 0, 0), (32, 513, 191, 1, 0), (300, 36, 192, 0, 0), (513, 65, 193, 0, 0),
                                         (257, 130, 256, 0, 2)])
def test_gemm_short_rows_matrix_cores(M, N, K, pa, pb, cfg):
    """Rows of one to four words in every launch form, with one block of rows a wave and with several: edges of both block sizes, odd columns, padded operands, garbage past
    K, both maps with the channel along either axis."""
    print(f"short rows {M}x{N}x{K} +{pa} +{pb} cfg={cfg}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A, Bm = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)

    def operand(a, pad):
        w = np.concatenate([as_u64(B.bnn_encode(dev(a))), np.full((len(a), pad), 0x5A5A, np.uint64)], axis=1)
        if K % 64:
            w[:, (K - 1) // 64] |= np.uint64(0xFFFFFFFFFFFFFFFF >> (K % 64) << (K % 64)) & np.uint64(0x9669C33CA55A0FF0)
        return dev(w.view(np.int64))
    Ap, Bp, ref = operand(A, pa), operand(Bm, pb), oracle.gemm_pm1(A, Bm)
    c = None if cfg < 0 else cfg
    out, names = kernels_of(lambda: B.bnn_xnor_gemm(Ap, Bp, K, cfg=c))
    assert np.array_equal(host(out), ref)
    assert cfg < 0 or names == ["xnor_gemm_lowk"]
    for axis, ch in (("row", M), ("col", N)):
        sc, bi = rng.standard_normal(ch).astype(np.float32), rng.standard_normal(ch).astype(np.float32)
        Ci, Y = B.bnn_xnor_gemm_epilogue(Ap, Bp, K, dev(sc), dev(bi), B.CH_ROW if axis == "row" else B.CH_COL, want_int=True,
                                         cfg=c)
        assert np.array_equal(host(Ci), ref)
        assert np.array_equal(host(Y), oracle.scale_bias(ref, sc, bi, axis))


@pytest.mark.parametrize("M,N,K,pa,pb", [(1, 4, 128, 0, 0), (7, 1020, 65, 0, 2), (8, 1024, 100, 1, 1), (9, 1028, 128, 0, 1), (16, 2052, 256, 2, 0),
                                         (15, 516, 193, 1, 3), (2, 3000, 256, 0, 2)])
def test_gemm_few_short_rows(M, N, K, pa, pb):
    """At most 16 rows of two or four words: edges of the groups of rows and of the workgroup's columns, padded operands, garbage
    past K, both maps with the channel along either axis."""
    print(f"few short rows {M}x{N}x{K} +{pa} +{pb}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A, Bm = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)

    def operand(a, pad):
        w = np.concatenate([as_u64(B.bnn_encode(dev(a))), np.full((len(a), pad), 0x5A5A, np.uint64)], axis=1)
        if K % 64:
            w[:, (K - 1) // 64] |= np.uint64(0xFFFFFFFFFFFFFFFF >> (K % 64) << (K % 64)) & np.uint64(0x9669C33CA55A0FF0)
        return dev(w.view(np.int64))
    Ap, Bp, ref = operand(A, pa), operand(Bm, pb), oracle.gemm_pm1(A, Bm)
    out, names = kernels_of(lambda: B.bnn_xnor_gemm(Ap, Bp, K, cfg=18))
    assert names == ["xnor_gemm_fewrows"] and np.array_equal(host(out), ref)
    for axis, ch in (("row", M), ("col", N)):
        sc, bi = rng.standard_normal(ch).astype(np.float32), rng.standard_normal(ch).astype(np.float32)
        Ci, Y = B.bnn_xnor_gemm_epilogue(Ap, Bp, K, dev(sc), dev(bi), B.CH_ROW if axis == "row" else B.CH_COL, want_int=True, cfg=18)
        assert np.array_equal(host(Ci), ref)
        assert np.array_equal(host(Y), oracle.scale_bias(ref, sc, bi, axis))


@pytest.mark.parametrize("M,N,K,kernel", [
    (1, 32768, 128, "fewrows"), (1, 32764, 128, "lowk"), (8, 147456, 100, "fewrows"), (8, 147452, 100, "lowk"), (16, 589824, 256, "fewrows"),
    (16, 589820, 256, "lowk"), (17, 600000, 128, "lowk"), (2, 400001, 128, "fp4"), (2, 400000, 64, "lowk"), (13, 2097156, 70, "lowk"),
    (24, 400004, 100, "fp4"), (24, 300004, 100, "lowk"), (33, 400004, 100, "lowk"),                                          # rows inside half lines
    (200, 400001, 100, "fp4"), (256, 300001, 100, "fp4"), (257, 300001, 100, "lowk"), (300, 230001, 100, "lowk"), (300, 229001, 100, "fp4"),             # odd columns, 275 MB
    (5000, 15001, 100, "lowk"), (6000, 13001, 100, "fp4"), (60000, 1301, 100, "fp4"), (6001, 13999, 64, "lowk")])
def test_gemm_short_rows_rule_by_rows(M, N, K, kernel):
    """Which kernel takes short rows by their number (256 compute units), and its values against a vector-ALU tile's."""
    print(f"short rows rule by rows {M}x{N}x{K}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    r = lambda n: torch.randint(-2**63, 2**63 - 1, (n, B.packed_words(K)), dtype=torch.int64, device=DEV, generator=g)
    A, Bm = r(M), r(N)
    got, names = kernels_of(lambda: B.bnn_xnor_gemm(A, Bm, K))
    assert torch.equal(got, B.bnn_xnor_gemm(A, Bm, K, cfg=3))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert names[0].startswith("xnor_gemm_" + kernel), names


@pytest.mark.parametrize("M,N,K,short", [
    (64, 64, 256, True), (64, 64, 64, False), (64, 63, 256, False),           # small calls: even words, columns by four
    (512, 4096, 60, True), (512, 4112, 190, True), (256, 4112, 190, False),   # odd words from 300 blocks on
    (300, 20004, 128, True), (300, 20004, 64, False), (96, 40004, 128, False), # rows inside half lines
    (2048, 31264, 128, True), (2048, 31252, 50, False),                                        # beyond 256 MB
    (2048, 33573, 100, True), (2048, 33569, 100, False)])                                      # columns not by four: 275 MB
def test_gemm_short_rows_rule(M, N, K, short):
    """Which kernel takes short rows, and its values against a vector-ALU tile's."""
    print(f"short rows rule {M}x{N}x{K}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    r = lambda n: torch.randint(-2**63, 2**63 - 1, (n, B.packed_words(K)), dtype=torch.int64, device=DEV, generator=g)
    A, Bm = r(M), r(N)
    got, names = kernels_of(lambda: B.bnn_xnor_gemm(A, Bm, K))
    assert (names == ["xnor_gemm_lowk"]) == short, names
    assert torch.equal(got, B.bnn_xnor_gemm(A, Bm, K, cfg=3))


@pytest.mark.parametrize("M,N,K,pad", [(1, 1, 1, 1), (127, 129, 127, 0), (129, 132, 128, 2), (130, 255, 129, 1), (64, 300, 513, 1),
                                       (257, 128, 640, 0), (100, 260, 4097, 1),
                                       (2200, 2176, 1984, 1), (2200, 2176, 1985, 0), (2200, 2176, 2050, 1)])  # both sides of the rule
def test_gemm_bit_codes(M, N, K, pad):
    """Rows expanded to 0 / 1 and corrected by their counts: edges of the tile, of a stage (512 bits) and of a word, odd
    columns, padded rows, garbage past K, both maps with the channel along either axis; all bits set and none."""
    print(f"bit codes {M}x{N}x{K} +{pad}", flush=True)
    rng = np.random.default_rng(M + N + K)
    A, Bm = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    A[0], Bm[0] = -1, 1
    A[-1], Bm[-1] = 1, -1

    def operand(a):
        w = np.concatenate([as_u64(B.bnn_encode(dev(a))), np.full((len(a), pad), 0x5A5A, np.uint64)], axis=1)
        if K % 64:
            w[:, (K - 1) // 64] |= np.uint64(0xFFFFFFFFFFFFFFFF >> (K % 64) << (K % 64)) & np.uint64(0x9669C33CA55A0FF0)
        return dev(w.view(np.int64))
    Ap, Bp = operand(A), operand(Bm)
    ref = oracle.gemm_pm1(A, Bm) if M * N * K < 1 << 28 else host(B.bnn_xnor_gemm(Ap, Bp, K, cfg=3))
    for c in (None, 29):
        assert np.array_equal(host(B.bnn_xnor_gemm(Ap, Bp, K, cfg=c)), ref)
        for axis, ch in (("row", M), ("col", N)):
            sc, bi = rng.standard_normal(ch).astype(np.float32), rng.standard_normal(ch).astype(np.float32)
            Ci, Y = B.bnn_xnor_gemm_epilogue(Ap, Bp, K, dev(sc), dev(bi), B.CH_ROW if axis == "row" else B.CH_COL,
                                             want_int=True, cfg=c)
            assert np.array_equal(host(Ci), ref)
            assert np.array_equal(host(Y), oracle.scale_bias(ref, sc, bi, axis))


@pytest.mark.parametrize("cfg", [-1, 10, 11, 12, 3])
@pytest.mark.parametrize("case", [(3, 200, 12, 12, 70, 1, 1, 2, 2, 0, 0),    # 36 pixels per image: short-row kernel
                                  (2, 200, 10, 10, 17, 1, 1, 2, 2, 0, 0),    # 25 pixels per image: not a multiple of 4
                                  (2, 128, 8, 8, 40, 1, 1, 1, 1, 0, 0),      # rows of two words, stride 1
                                  (5, 256, 6, 4, 130, 1, 1, 1, 2, 0, 0),
                                  (2, 100, 16, 16, 9, 1, 1, 2, 2, 0, 0),
                                  (2, 250, 9, 12, 33, 1, 1, 3, 2, 0, 0)])    # odd H, stride (3, 2)
def test_conv2d_pointwise_short_rows(case, cfg):
    """1x1 / pad-0 convolutions with at most 256 channels: the encode samples the strided pixels
    (8-byte loads on even rows with column stride 2) and the GEMM is the short-row kernel where the
    image size allows it; int32 and fp32 outputs against the oracle."""
    print(f"conv2d pointwise case={case} cfg={cfg}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    shape = inputs.ConvShape(*case)
    d = inputs.conv_inputs(shape, seed=sum(case) + 21)
    x = inputs.inject_specials(d["x"], 9, frac=0.01)
    wp = B.bnn_pack_conv_weight(dev(d["w"]))
    oi, of = B.bnn_conv2d(dev(x), wp, D, 1, 1, (sH, sW), (0, 0), dev(d["scale"]), dev(d["bias"]), want_int=True,
                          cfg=None if cfg < 0 else cfg)
    ref = oracle.conv2d_pm1(x, d["w"], (sH, sW), (0, 0))
    assert np.array_equal(host(oi), ref)
    assert np.array_equal(host(of), oracle.scale_bias(ref, d["scale"], d["bias"], "nchw"))


POINTWISE_CASES = [  # N, C, H, W, D, stride, one launch
    ((1, 1, 1, 1, 1, 1), True), ((1, 7, 3, 5, 33, 1), True),          # a partial granule, a partial row tile
    ((3, 200, 12, 12, 70, 2), True), ((3, 200, 11, 9, 70, 2), True),  # 36 and 30 pixels an image: columns by four or one by one
    ((2, 64, 8, 8, 128, 1), True), ((2, 65, 8, 8, 129, 1), True),     # edges of the word and of the narrow row tile
    ((5, 256, 7, 7, 300, 1), True), ((1, 257, 9, 8, 513, 1), True),   # one chunk of the reduction and one value more
    ((2, 500, 6, 10, 256, 1), True), ((4, 1000, 4, 4, 40, 1), True),
    ((84, 5, 28, 28, 9, 1), True), ((84, 64, 28, 28, 70, 1), True),   # two pixel groups per workgroup
    ((83, 33, 29, 28, 65, 1), True),
    ((24, 128, 28, 28, 520, 1), True),                                # several passes over the channels: wide row tiles,
    ((8, 200, 28, 28, 513, 1), True), ((84, 30, 28, 28, 300, 1), True),  # narrow ones shared by workgroups, two pixel groups
    ((1, 1024, 4, 4, 12, 1), False), ((1, 2049, 3, 3, 12, 1), False),
    ((120, 33, 56, 56, 66, 1), False),                                # 150 MB, few channels into twice as many
]


@pytest.mark.parametrize("case,one", POINTWISE_CASES)
def test_conv2d_pointwise_one_launch(case, one):
    """Pointwise layers from the fp32 image: encode and multiplication in one launch, or in two by the rule; both maps and
    each alone, specials among the inputs, against the oracle (large maps: against the two-launch route)."""
    print(f"conv2d pointwise case={case}", flush=True)
    N, C, H, W, D, s = case
    shape = inputs.ConvShape(N, C, H, W, D, 1, 1, s, s, 0, 0)
    d = inputs.conv_inputs(shape, seed=sum(case) + 5)
    x = inputs.inject_specials(d["x"], 4, frac=0.01)
    wp, xd, sc, bi = B.bnn_pack_conv_weight(dev(d["w"])), dev(x), dev(d["scale"]), dev(d["bias"])
    run = lambda **kw: B.bnn_conv2d(xd, wp, D, 1, 1, (s, s), (0, 0), **kw)
    (oi, of), names = kernels_of(lambda: run(scale=sc, bias=bi))
    assert (names == ["conv_pointwise"]) == one, names
    if one:
        ref = oracle.conv2d_pm1(x, d["w"], (s, s), (0, 0))
    else:
        ref = host(run(cfg=24)[0])
    assert np.array_equal(host(oi), ref)
    assert np.array_equal(host(of), oracle.scale_bias(ref, d["scale"], d["bias"], "nchw"))
    assert np.array_equal(host(run()[0]), ref)
    assert np.array_equal(host(run(scale=sc, bias=bi, want_int=False)[1]), host(of))


@pytest.mark.parametrize("case", [c for c, _ in POINTWISE_CASES] + [(2, 200, 9, 7, 33, 1, 3)])
def test_conv2d_workspace_receives_the_packed_image(case):
    """What bnn_conv2d leaves in the workspace: the packed image, of a pointwise layer the pixels that it samples; nothing
    behind it."""
    print(f"conv2d workspace case={case}", flush=True)
    N, C, H, W, D, s, k = case if len(case) == 7 else (*case, 1)
    g = torch.Generator(device=DEV).manual_seed(sum(case))
    x = torch.randn(N, C, H, W, device=DEV, generator=g)
    wp = B.bnn_pack_conv_weight(torch.randn(D, C, k, k, device=DEV, generator=g))
    want = B.bnn_im2col_packed(x, 1, 1, (s, s) if k == 1 else (1, 1), (0, 0)).view(-1)
    ws = torch.full((max(16, B.conv2d_workspace_bytes(x.shape, k, k, (s, s), (k // 2, k // 2))) + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    B.bnn_conv2d(x, wp, D, k, k, (s, s), (k // 2, k // 2), workspace=ws)
    assert torch.equal(ws[:8 * want.numel()].view(torch.int64), want)
    assert bool((ws[8 * want.numel():] == 0x5A).all())


@pytest.mark.parametrize("case", [
    (2, 64, 9, 11, 64, 3, 3, 1, 1, 1, 1),      # one word a pixel, whole
    (3, 37, 14, 20, 70, 3, 3, 1, 1, 1, 1),     # partial granule of channels; a row tile of six channels
    (1, 5, 6, 6, 33, 3, 3, 2, 2, 1, 1),        # few channels, fewer columns than a tile
    (5, 100, 13, 12, 64, 5, 3, 2, 1, 0, 1),    # strides, windows and padding of their own; two words
    (2, 129, 11, 8, 40, 3, 3, 1, 1, 1, 1),     # three words a pixel, one channel in the third
    (2, 512, 8, 8, 96, 3, 3, 1, 1, 1, 1),      # two pieces of the encode to a wave
    (40, 200, 3, 3, 40, 3, 3, 1, 1, 1, 1),     # a tile's pixels lie in five images
    (3, 64, 8, 9, 64, 2, 2, 5, 5, 0, 0),       # rows that no window reads, between windows and behind the last
    (4, 70, 3, 5, 32, 5, 5, 2, 2, 4, 4),       # windows that lie outside the image
    (3, 130, 8, 10, 40, 1, 1, 2, 2, 1, 1), (1, 60, 1, 70, 64, 3, 3, 1, 1, 1, 1), (20, 256, 1, 1, 64, 3, 3, 1, 1, 1, 1)])
def test_conv2d_in_one_launch(case):
    """Convolutions whose tiles encode the rows that they read, forced and as an application calls them: both maps and the
    packed image in the workspace, values of every kind that the sign rule names among the inputs."""
    print(f"conv2d one launch case={case}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    rows = (ctypes.c_int64 * 3)()
    d = inputs.conv_inputs(inputs.ConvShape(*case), seed=sum(case))
    x = inputs.inject_specials(d["x"], 3, frac=0.02)
    ref = oracle.conv2d_pm1(x, d["w"], (sH, sW), (pH, pW))
    xd, wp, sc, bi = dev(x), B.bnn_pack_conv_weight(dev(d["w"])), dev(d["scale"]), dev(d["bias"])
    want = oracle.pack_nhwc(x).reshape(-1)
    nbytes = B.conv2d_workspace_bytes(x.shape, kH, kW, (sH, sW), (pH, pW))
    for cfg in (40, 41, None):
        assert B.lib().bnn_testing_conv_image(*case, 256, -1 if cfg is None else cfg - 40, 0, rows) >= 0
        ws = torch.full((max(16, nbytes) + 64,), 0x5A, dtype=torch.uint8, device=DEV)
        oi, of = B.bnn_conv2d(xd, wp, D, kH, kW, (sH, sW), (pH, pW), sc, bi, workspace=ws, cfg=cfg)
        assert np.array_equal(host(oi), ref)
        assert np.array_equal(host(of), oracle.scale_bias(ref, d["scale"], d["bias"], "nchw"))
        assert np.array_equal(as_u64(ws[:8 * want.size].view(torch.int64)), want)
        assert bool((ws[max(16, nbytes):] == 0x5A).all())


def test_gemm_table1_truth_table():
    """Table 1 of the paper through encode + GEMM with K = 1 (63 masked tail bits)."""
    print("gemm truth table", flush=True)
    vals = np.array([[-1.0], [1.0]], dtype=np.float32)
    P = B.bnn_encode(dev(vals))
    assert as_u64(P).reshape(-1).tolist() == [0, 1]
    got = host(B.bnn_xnor_gemm(P, P, 1))
    assert got.tolist() == [[1, -1], [-1, 1]]


def test_gemm_masks_garbage_past_K():
    print("gemm tail garbage", flush=True)
    rng = np.random.default_rng(11)
    for K in (1, 33, 70, 200):
        A = rng.standard_normal((9, K)).astype(np.float32)
        Bm = rng.standard_normal((70, K)).astype(np.float32)
        Ap, Bp = as_u64(B.bnn_encode(dev(A))).copy(), as_u64(B.bnn_encode(dev(Bm))).copy()
        tail = K % 64
        garbage = np.uint64((0xFFFFFFFFFFFFFFFF >> tail) << tail) if tail else np.uint64(0)
        Ap[:, -1] |= garbage & np.uint64(0xA5A5A5A5A5A5A5A5)
        Bp[:, -1] |= garbage & np.uint64(0x0F0F0F0FF0F0F0F0)
        got = host(B.bnn_xnor_gemm(dev(Ap.view(np.int64)), dev(Bp.view(np.int64)), K))
        assert np.array_equal(got, oracle.gemm_pm1(A, Bm)), K


def test_gemm_leading_dimensions():
    print("gemm ld", flush=True)
    rng = np.random.default_rng(12)
    M, N, K = 20, 90, 330
    A = rng.standard_normal((M, K)).astype(np.float32)
    Bm = rng.standard_normal((N, K)).astype(np.float32)
    Kw = B.packed_words(K)
    Abig = torch.full((M, Kw + 3), 0x5555, dtype=torch.int64, device=DEV)
    Bbig = torch.full((N, Kw + 1), 0x3333, dtype=torch.int64, device=DEV)  # odd ldb: 8-byte load path
    B.bnn_encode(dev(A), Abig[:, :Kw])
    B.bnn_encode(dev(Bm), Bbig[:, :Kw])
    Cbig = torch.full((M, N + 5), -7, dtype=torch.int32, device=DEV)
    B.bnn_xnor_gemm(Abig[:, :Kw], Bbig[:, :Kw], K, Cbig[:, :N])
    out = host(Cbig)
    assert np.array_equal(out[:, :N], oracle.gemm_pm1(A, Bm))
    assert np.all(out[:, N:] == -7)


@pytest.mark.parametrize("axis", ["row", "col"])
@pytest.mark.parametrize("cfg", [-1, *GEMM_KERNELS])
@pytest.mark.parametrize("M,N,K", [(37, 150, 300), (130, 515, 1100), (8, 64, 64), (70, 200, 4096 + 77)])
def test_gemm_fp32_epilogue_both_axes(M, N, K, cfg, axis):
    """y = fma(scale[ch], float(acc), bias[ch]) with the channel along rows or columns, with and
    without the int32 result beside it, on every tile configuration."""
    print(f"gemm epilogue M={M} N={N} K={K} cfg={cfg} axis={axis}", flush=True)
    rng = np.random.default_rng(M + N + K + cfg)
    A = rng.standard_normal((M, K)).astype(np.float32)
    Bm = rng.standard_normal((N, K)).astype(np.float32)
    nch = M if axis == "row" else N
    sc = ((rng.random(nch) + 0.5) * rng.choice([-1.0, 1.0], nch)).astype(np.float32)
    bi = rng.standard_normal(nch).astype(np.float32)
    Ap, Bp = B.bnn_encode(dev(A)), B.bnn_encode(dev(Bm))
    ref = oracle.gemm_pm1(A, Bm)
    yref = oracle.scale_bias(ref, sc, bi, axis)
    ax = B.CH_ROW if axis == "row" else B.CH_COL
    (C, Y), names = kernels_of(lambda: B.bnn_xnor_gemm_epilogue(Ap, Bp, K, dev(sc), dev(bi), ax, want_int=True, cfg=cfg))
    assert cfg < 0 or names == [GEMM_KERNELS[cfg]]
    assert np.array_equal(host(C), ref)
    assert np.array_equal(host(Y), yref)
    C, Y = B.bnn_xnor_gemm_epilogue(Ap, Bp, K, dev(sc), dev(bi), ax, want_int=False, cfg=cfg)
    assert C is None and np.array_equal(host(Y), yref)


def test_gemm_deterministic_twice():
    print("gemm determinism", flush=True)
    d = inputs.cfg1()
    Ap, Bp = B.bnn_encode(dev(d["A"])), B.bnn_encode(dev(d["B"]))
    a = host(B.bnn_xnor_gemm(Ap, Bp, inputs.CFG1.K))
    b = host(B.bnn_xnor_gemm(Ap, Bp, inputs.CFG1.K))
    assert np.array_equal(a, b)


# ---------------------------------------------------------------- the five configurations
def test_cfg1_single_gemm():
    print("cfg1", flush=True)
    d = inputs.cfg1()
    A = inputs.inject_specials(d["A"], 1)
    Bm = inputs.inject_specials(d["B"], 2)
    Ap, Bp = B.bnn_encode(dev(A)), B.bnn_encode(dev(Bm))
    assert as_u64(Ap).view("<u4").shape == (64, 8)
    assert np.array_equal(host(B.bnn_xnor_gemm(Ap, Bp, 256)), oracle.gemm_pm1(A, Bm))


def test_cfg2_fc_layer_full_size():
    print("cfg2", flush=True)
    d = inputs.cfg2()
    act = inputs.inject_specials(d["act"], 3)
    Ap, Wp = B.bnn_encode(dev(act)), B.bnn_encode(dev(d["wt"]))
    C, Y = B.bnn_xnor_gemm_epilogue(Ap, Wp, inputs.CFG2.K, dev(d["scale"]), dev(d["bias"]), B.CH_COL, want_int=True)
    ref = oracle.gemm_pm1(act, d["wt"])
    assert np.array_equal(host(C), ref)
    yref = oracle.scale_bias(ref, d["scale"], d["bias"], "col")
    got = host(Y)
    assert_f32_close(got, yref)
    assert np.array_equal(got, yref)  # single-rounded fma on both sides: bit-exact


def _conv_parity(shape, data, with_epilogue=True):
    """bnn_conv2d against the oracle's direct convolution on EVERY output: int32 bit-exact, and the
    fp32 epilogue against oracle.scale_bias (1e-6 relative by contract, bit-exact by construction)."""
    x = inputs.inject_specials(data["x"], 7, frac=1e-4)
    w = data["w"]
    xd, wd = dev(x), dev(w)
    wp = B.bnn_pack_conv_weight(wd)
    st, pd = (shape.sH, shape.sW), (shape.pH, shape.pW)
    sc, bi = dev(data["scale"]), dev(data["bias"])
    oi, of = B.bnn_conv2d(xd, wp, shape.D, shape.kH, shape.kW, st, pd, sc if with_epilogue else None,
                          bi if with_epilogue else None, want_int=True)
    got = host(oi)
    assert got.shape == (x.shape[0], shape.D, shape.OH, shape.OW)
    ref = oracle.conv2d_pm1(x, w, st, pd)
    assert np.array_equal(got, ref)
    if with_epilogue:
        yref = oracle.scale_bias(ref, data["scale"], data["bias"], "nchw")
        assert_f32_close(host(of), yref)
        assert np.array_equal(host(of), yref)


def test_cfg3_cifar_conv_full_size():
    print("cfg3", flush=True)
    _conv_parity(inputs.CFG3, inputs.cfg3())


def test_cfg5a_imagenet_conv_full_size():
    """All 51.4 M int32 outputs and the fp32 epilogue of the ImageNet-shaped 3x3 convolution."""
    print("cfg5a", flush=True)
    _conv_parity(inputs.CFG5A, inputs.cfg5a())


def test_cfg5b_ragged_k_pointwise_stride2_full_size():
    print("cfg5b", flush=True)
    _conv_parity(inputs.CFG5B, inputs.cfg5b())


@pytest.mark.parametrize("case", CONV_CASES)
def test_conv2d_small_cases(case):
    print(f"conv case={case}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    shape = inputs.ConvShape(N, C, H, W, D, kH, kW, sH, sW, pH, pW)
    _conv_parity(shape, inputs.conv_inputs(shape, seed=sum(case)))


def test_conv2d_worked_examples():
    print("conv worked examples", flush=True)
    x = torch.full((1, 1, 3, 3), -1.0, device=DEV)
    w = torch.full((1, 1, 3, 3), 1.0, device=DEV)
    oi, _ = B.bnn_conv2d(x, B.bnn_pack_conv_weight(w), 1, 3, 3, (1, 1), (1, 1))
    assert host(oi)[0, 0].tolist() == [[1, -3, 1], [-3, -9, -3], [1, -3, 1]]
    x = torch.tensor([[[[1.0, -1.0], [-1.0, 1.0]]]], device=DEV)
    w = torch.tensor([[[[1.0, -1.0, 1.0], [-1.0, 1.0, -1.0], [1.0, -1.0, 1.0]]]], device=DEV)
    oi, _ = B.bnn_conv2d(x, B.bnn_pack_conv_weight(w), 1, 3, 3, (1, 1), (1, 1))
    assert host(oi)[0, 0].tolist() == [[5, -3], [-3, 5]]


# ---------------------------------------------------------------- glue (a6) and the stack (cfg 4)
def test_maxpool_and_f32_glue():
    print("glue", flush=True)
    rng = np.random.default_rng(21)
    a = rng.integers(-1152, 1153, size=(3, 5, 8, 6)).astype(np.int32)
    sc = (rng.random(5) + 0.5).astype(np.float32)
    bi = (rng.standard_normal(5) * 0.1).astype(np.float32)
    oi, of = B.bnn_maxpool2x2(dev(a), dev(sc), dev(bi), want_int=True)
    ref = oracle.maxpool2x2_i32(a)
    assert np.array_equal(host(oi), ref)
    assert np.array_equal(host(of), oracle.scale_bias(ref, sc, bi, "nchw"))
    x = rng.standard_normal((3, 3, 9, 8)).astype(np.float32)
    w = rng.standard_normal((5, 3, 3, 3)).astype(np.float32)
    got = host(B.bnn_conv2d_f32(dev(x), dev(w), (1, 1), (1, 1), dev(sc), dev(bi)))
    assert np.array_equal(got, oracle.conv2d_f32_seq(x, w, (1, 1), (1, 1), sc, bi))
    got = host(B.bnn_conv2d_f32(dev(x), dev(w), (2, 1), (0, 1)))
    assert np.array_equal(got, oracle.conv2d_f32_seq(x, w, (2, 1), (0, 1)))
    xf = rng.standard_normal((6, 100)).astype(np.float32)
    wf = rng.standard_normal((10, 100)).astype(np.float32)
    bf = rng.standard_normal(10).astype(np.float32)
    for sgn in (False, True):
        got = host(B.bnn_fc_f32(dev(xf), dev(wf), dev(bf), sign_input=sgn))
        assert np.array_equal(got, oracle.fc_f32_seq(xf, wf, bf, sign_input=sgn))


@pytest.mark.parametrize("N,D,H,W", [(1, 1, 2, 4), (3, 5, 6, 8), (2, 3, 4, 6), (1, 7, 2, 2), (5, 67, 10, 12), (2, 130, 8, 10)])
def test_maxpool_widths(N, D, H, W):
    """Rows of a multiple of 4 values (two windows a thread) and others; both outputs, either alone."""
    print(f"maxpool {N}x{D}x{H}x{W}", flush=True)
    rng = np.random.default_rng(N + D + H + W)
    a = rng.integers(-5000, 5000, (N, D, H, W)).astype(np.int32)
    sc, bi = rng.standard_normal(D).astype(np.float32), rng.standard_normal(D).astype(np.float32)
    ref = oracle.maxpool2x2_i32(a)
    fref = oracle.scale_bias(ref, sc, bi, "nchw")
    gi, gf = B.bnn_maxpool2x2(dev(a), dev(sc), dev(bi), want_int=True)
    assert np.array_equal(host(gi), ref) and np.array_equal(host(gf), fref)
    assert np.array_equal(host(B.bnn_maxpool2x2(dev(a), dev(sc), dev(bi), want_int=False)[1]), fref)
    assert np.array_equal(host(B.bnn_maxpool2x2(dev(a), None, None, want_int=True)[0]), ref)


@pytest.mark.parametrize("M,K,N", [(256, 1024, 10), (6, 100, 10), (5, 1023, 3), (33, 2500, 37), (1, 4, 1),
                                   (4100, 64, 20), (300, 1030, 250)])
@pytest.mark.parametrize("sgn", [False, True])
def test_fc_f32_matches_oracle(M, K, N, sgn):
    """Both workgroup shapes (4 and 16 rows), rows of several LDS passes, K off the 16-byte grid,
    output counts off the group of 16; with and without bias."""
    print(f"fc_f32 M={M} K={K} N={N} sign={sgn}", flush=True)
    rng = np.random.default_rng(M * 7 + K + N)
    xf = inputs.inject_specials(rng.standard_normal((M, K)).astype(np.float32), 4, frac=0.002, with_nan=False)
    wf = rng.standard_normal((N, K)).astype(np.float32)
    bf = rng.standard_normal(N).astype(np.float32)
    got = host(B.bnn_fc_f32(dev(xf), dev(wf), dev(bf), sign_input=sgn))
    ref = oracle.fc_f32_seq(xf, wf, bf, sign_input=sgn)
    assert np.array_equal(got, ref, equal_nan=True)
    got = host(B.bnn_fc_f32(dev(xf), dev(wf), None, sign_input=sgn))
    assert np.array_equal(got, oracle.fc_f32_seq(xf, wf, None, sign_input=sgn), equal_nan=True)


@pytest.mark.parametrize("M,K,N", [(4, 4, 12), (5, 60, 13), (3, 64, 12), (9, 68, 10), (1, 124, 1), (2, 128, 16), (4, 1020, 12),
                                   (257, 1024, 17), (5, 1084, 11), (3, 1152, 13), (2100, 132, 18)])
def test_fc_f32_turns(M, K, N):
    """Rows of 0, 1, 2, 16 turns of 64 steps and what is left after them, alone and behind a full LDS pass; the staged rows of w
    that outputs do not use."""
    print(f"fc_f32 turns M={M} K={K} N={N}", flush=True)
    rng = np.random.default_rng(M + K + N)
    xf, wf = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    bf = rng.standard_normal(N).astype(np.float32)
    assert np.array_equal(host(B.bnn_fc_f32(dev(xf), dev(wf), dev(bf))), oracle.fc_f32_seq(xf, wf, bf))


@pytest.mark.parametrize("M,K,N", [(1, 1, 1), (4, 3, 12), (5, 63, 13), (3, 255, 12), (2, 257, 10), (3, 1023, 12), (6, 1025, 16),
                                   (5, 2046, 11), (2100, 131, 18), (2300, 33, 16)])
@pytest.mark.parametrize("sgn", [False, True])
def test_fc_f32_rows_off_16_bytes(M, K, N, sgn):
    """Rows of no multiple of four values, staged a value of every row at a time: every form, one to four turns of 256 values, one and
    two LDS passes, rows of x and w past the last."""
    print(f"fc_f32 odd rows M={M} K={K} N={N} sign={sgn}", flush=True)
    rng = np.random.default_rng(M + K + N)
    xf, wf = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    bf = rng.standard_normal(N).astype(np.float32)
    got = host(B.bnn_fc_f32(dev(xf), dev(wf), dev(bf), sign_input=sgn))
    assert np.array_equal(got, oracle.fc_f32_seq(xf, wf, bf, sign_input=sgn))


@pytest.mark.parametrize("reading", ["A", "B"])
def test_cfg4_stack_small_batch_every_layer(reading):
    print(f"cfg4 stack batch 4 reading {reading}", flush=True)
    from paper_1911_04477_amd.stack import VggStack
    d = inputs.cfg4(batch=4, reading=reading)
    net = VggStack(d["layers"], d["params"], batch=4, device=DEV)
    out, acts = net.forward(dev(d["x"]), keep=True)
    ref = oracle.vgg_stack(d["x"], d["layers"], d["params"])
    for i, (g, r) in enumerate(zip(acts, ref["acts"])):
        assert np.array_equal(host(g).reshape(r.shape), r), f"layer {i} ({d['layers'][i].kind})"
    assert np.array_equal(host(out), ref["out"])


@pytest.fixture(scope="module")
def cfg4_b256():
    """Config 4 at the benchmarked batch with the oracle's activations of every layer, all 256
    images (computed once for the tests that use it)."""
    d = inputs.cfg4(batch=256)
    print("oracle: cfg4 stack, 256 images", flush=True)
    ref = oracle.vgg_stack(d["x"], d["layers"], d["params"])
    return d, ref


def test_cfg4_stack_full_batch_every_layer_every_image(cfg4_b256):
    """Batch 256 as benchmarked, through bnn_conv2d and the glue kernels: the activation of every
    layer and the logits of all 256 images against the oracle, bit for bit."""
    print("cfg4 stack batch 256", flush=True)
    from paper_1911_04477_amd.stack import VggStack
    d, ref = cfg4_b256
    net = VggStack(d["layers"], d["params"], batch=256, device=DEV)
    out, acts = net.forward(dev(d["x"]), keep=True)
    for i, (g, r) in enumerate(zip(acts, ref["acts"])):
        assert np.array_equal(host(g).reshape(r.shape), r), f"layer {i} ({d['layers'][i].kind})"
    out = host(out)
    assert np.array_equal(out, ref["out"])
    del acts
    out2 = host(net.forward(dev(d["x"])))
    assert np.array_equal(out, out2)


# ---------------------------------------------------------------- calls from tensors
class _OwnCode:
    """The binding without csrc/tensorcall.cpp."""

    def __enter__(self):
        self.kept = B._t()
        B._tensors = B._Tensors(B.lib(), "/nowhere")

    def __exit__(self, *exc):
        B._tensors = self.kept


def _plain_and_odd_calls():
    """name -> call(fresh outputs) -> outputs; every entry point with outputs given, plain and in forms of their own."""
    g = torch.Generator(device=DEV).manual_seed(5)
    r = lambda *s: torch.randn(*s, device=DEV, generator=g)
    e = lambda *s, dt=torch.int32: torch.full(s, 7, dtype=dt, device=DEV)
    i64, f32 = torch.int64, torch.float32
    A, W = B.bnn_encode(r(5, 130)), B.bnn_encode(r(9, 130))
    wide = torch.zeros(10, 8, dtype=i64, device=DEV)
    wide[::2, :3] = A
    sc, bi, sc9, bi9 = r(6), r(6), r(9), r(9)
    x, xp, wp = r(2, 70, 6, 8), B.bnn_im2col_packed(r(2, 70, 6, 8), 1, 1).view(2, 6, 8, 2), B.bnn_pack_conv_weight(r(6, 70, 3, 3))
    ws = e(1 << 16, dt=torch.uint8)
    img, taps = r(2, 3, 7, 9), torch.nn.Parameter(r(6, 3, 3, 3))
    acc = torch.randint(-50, 50, (2, 6, 4, 6), device=DEV, generator=g, dtype=torch.int32)
    geo = dict(stride=(1, 1), pad=(1, 1))
    return {
        "gemm": lambda: B.bnn_xnor_gemm(A, W, 130, C=e(5, 9)),
        "gemm rows apart": lambda: B.bnn_xnor_gemm(wide[::2], W, 130, C=e(5, 20)[:, :9]),
        "gemm one row": lambda: B.bnn_xnor_gemm(A[:1], W[:1], 130, C=e(1, 1)),
        "gemm nothing": lambda: B.bnn_xnor_gemm(A[:0], W, 130, C=e(0, 9)),
        "gemm numpy K": lambda: B.bnn_xnor_gemm(A, W, np.int64(130), C=e(5, 9)),
        "epilogue columns": lambda: B.bnn_xnor_gemm_epilogue(A, W, 130, sc9, bi9, B.CH_COL, out_y=e(5, 9, dt=f32)),
        "epilogue rows": lambda: B.bnn_xnor_gemm_epilogue(A, W, 130, sc, bi, B.CH_ROW, out_y=e(5, 9, dt=f32)),
        "encode": lambda: B.bnn_encode(x.view(12, 560), e(12, 9, dt=i64)),
        "encode strided": lambda: B.bnn_encode(x.view(12, 560)[::2, :65], e(6, 4, dt=i64)[:, :2]),
        "encode one row": lambda: B.bnn_encode(x.view(1, -1), e(1, 105, dt=i64)),
        "conv2d": lambda: B.bnn_conv2d(x, wp, 6, 3, 3, (1, 1), (1, 1), workspace=ws, out_i32=e(2, 6, 6, 8)),
        "conv2d both": lambda: B.bnn_conv2d(x, wp, 6, 3, 3, (2, 1), (0, 1), sc, bi, workspace=ws, out_i32=e(2, 6, 2, 8), out_f32=e(2, 6, 2, 8, dt=f32)),
        "conv2d lists": lambda: B.bnn_conv2d(x, wp, 6, 3, 3, [1, 1], [1, 1], sc, bi, want_int=False, workspace=ws, out_f32=e(2, 6, 6, 8, dt=f32)),
        "packed": lambda: B.bnn_conv2d_packed(xp, wp, 70, 6, 3, 3, **geo, scale=sc, bias=bi, out_buf=e(2, 6, 8, 1, dt=i64)),
        "packed pool": lambda: B.bnn_conv2d_packed(xp, wp, 70, 6, 3, 3, **geo, pool=2, scale=sc, bias=bi, out_buf=e(2, 3, 4, 1, dt=i64)),
        "packed i32": lambda: B.bnn_conv2d_packed(xp, wp, 70, 6, 3, 3, **geo, out="i32", out_buf=e(2, 6, 6, 8)),
        "packed f32": lambda: B.bnn_conv2d_packed(xp, wp, 70, 6, 3, 3, **geo, out="f32", scale=sc, bias=bi, out_buf=e(2, 6, 6, 8, dt=f32)),
        "im2col": lambda: B.bnn_im2col_packed(x, 3, 3, (2, 1), (1, 0), cols=e(2 * 3 * 6, 18, dt=i64), workspace=ws),
        "f32 sign": lambda: B.bnn_conv2d_f32_sign(img, taps, sc, bi, (1, 1), (1, 1), out=e(2, 7, 9, 1, dt=i64)),
        "f32": lambda: B.bnn_conv2d_f32(img, taps, (1, 1), (1, 1), sc, bi, out=e(2, 6, 7, 9, dt=f32)),
        "f32 no affine map": lambda: B.bnn_conv2d_f32(img, taps, (2, 2), (0, 0), out=e(2, 6, 3, 4, dt=f32)),
        "pool": lambda: B.bnn_maxpool2x2(acc, sc, bi, out_i32=e(2, 6, 2, 3), out_f32=e(2, 6, 2, 3, dt=f32)),
        "pool i32": lambda: B.bnn_maxpool2x2(acc, out_i32=e(2, 6, 2, 3)),
        "fc": lambda: B.bnn_fc_f32(x.view(4, -1), r(3, 1680), r(3), sign_input=True, out=e(4, 3, dt=f32)),
        # refused, by the binding or by the library
        "no K": lambda: B.bnn_xnor_gemm(A, W, 0, C=e(5, 9)), "K beyond the rows": lambda: B.bnn_xnor_gemm(A, W, 300, C=e(5, 9)),
        "CPU": lambda: B.bnn_xnor_gemm(A.cpu(), W, 130, C=e(5, 9)), "type": lambda: B.bnn_encode(x.view(12, 560).half(), e(12, 9, dt=i64)),
        "shape of y": lambda: B.bnn_xnor_gemm_epilogue(A, W, 130, sc9, bi9, B.CH_COL, out_y=e(9, 5, dt=f32)),
        "columns apart": lambda: B.bnn_encode(x.view(12, 560)[:, ::2], e(12, 5, dt=i64)),
        "not contiguous": lambda: B.bnn_conv2d(x.transpose(2, 3), wp, 6, 3, 3, (1, 1), (1, 1), workspace=ws, out_i32=e(2, 6, 8, 6)),
        "channels": lambda: B.bnn_conv2d_packed(xp, wp, 200, 6, 3, 3, **geo, out="i32", out_buf=e(2, 6, 6, 8)),
        "workspace": lambda: B.bnn_conv2d(x, wp, 6, 3, 3, (1, 1), (1, 1), workspace=ws[:16], out_i32=e(2, 6, 6, 8)),
        "cols": lambda: B.bnn_im2col_packed(x, 3, 3, (1, 1), (1, 1), cols=e(3, 18, dt=i64), workspace=ws),
        "no scale": lambda: B.bnn_conv2d_packed(xp, wp, 70, 6, 3, 3, **geo, out_buf=e(2, 6, 8, 1, dt=i64)),
        "stride": lambda: B.bnn_conv2d_packed(xp, wp, 70, 6, 3, 3, stride=(0, 1), out="i32", out_buf=e(2, 6, 6, 8)),
        "odd map": lambda: B.bnn_maxpool2x2(acc[:, :, :3].contiguous(), out_i32=e(2, 6, 1, 3)),
        "outputs of another kind": lambda: B.bnn_conv2d_packed(xp, wp, 70, 6, 3, 3, out="u8", out_buf=e(1)),
    }


def _outcome(call):
    try:
        out = call()
    except Exception as ex:
        return type(ex), str(ex)
    out = out if isinstance(out, tuple) else (out,)
    torch.cuda.synchronize()
    return [None if t is None else t.clone() for t in out]


def test_calls_from_tensors_equal_the_bindings_own():
    """The same values, the same exceptions with the same text, with csrc/tensorcall.cpp and without."""
    print("calls from tensors", flush=True)
    assert os.path.exists(B.TENSORCALL_PATH)
    fast = {k: _outcome(c) for k, c in _plain_and_odd_calls().items()}
    with _OwnCode():
        own = {k: _outcome(c) for k, c in _plain_and_odd_calls().items()}
    for k in own:
        a, b = fast[k], own[k]
        if isinstance(a, tuple) or isinstance(b, tuple):
            assert a == b, k
        else:
            assert len(a) == len(b) and all((s is None and t is None) or torch.equal(s, t) for s, t in zip(a, b)), k
    refused = [k for k, v in own.items() if isinstance(v, tuple)]
    assert refused == list(own)[list(own).index("no K"):]


def test_calls_from_tensors_survive_what_a_call_throws(tmp_path):
    """A C++ exception out of the library (memory, a lock) is declined like anything else, with the interpreter's lock held again.
    The functions called throw before anything is launched."""
    import importlib.util
    import subprocess
    print("calls from tensors: exception", flush=True)
    (tmp_path / "throws.cpp").write_text('#include <stdexcept>\nextern "C" int throws() { throw std::runtime_error("no memory"); }\n')
    subprocess.check_call(["g++", "-shared", "-fPIC", "-o", str(tmp_path / "throws.so"), str(tmp_path / "throws.cpp")])
    path = tmp_path / "_tensorcall.so"  # a copy of its own, bound to nothing yet
    path.write_bytes(open(B.TENSORCALL_PATH, "rb").read())
    spec = importlib.util.spec_from_file_location("a_copy._tensorcall", str(path))
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    L = ctypes.CDLL(str(tmp_path / "throws.so"))
    module.bind(*[ctypes.cast(L.throws, ctypes.c_void_p).value for _ in module.names])
    A, C = torch.zeros(4, 1, dtype=torch.int64, device=DEV), torch.zeros(4, 4, dtype=torch.int32, device=DEV)
    for _ in range(3):
        assert module.gemm(A, A, 64, C) is None
    assert B.bnn_xnor_gemm(A, A, 64, C=C) is C and host(C).tolist() == [[64] * 4] * 4


def test_calls_from_tensors_follow_the_current_stream():
    """A call is ordered behind what its stream holds: on a side stream after a long product that makes its input."""
    print("calls from tensors: stream", flush=True)
    side = torch.cuda.Stream()
    big = torch.randn(4096, 4096, device=DEV)
    dst = torch.empty(4096, 64, dtype=torch.int64, device=DEV)
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        y = big
        for _ in range(8):
            y = torch.tanh(y @ big)
        B.bnn_encode(y, dst)
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(dst, B.bnn_encode(y))


# ---------------------------------------------------------------- timing hook
def test_prof_hook_records_kernels():
    print("prof hook", flush=True)
    d = inputs.cfg1()
    B.prof_enable(True)
    try:
        Ap, Bp = B.bnn_encode(dev(d["A"])), B.bnn_encode(dev(d["B"]))
        B.bnn_xnor_gemm(Ap, Bp, 256)
        rec = B.prof_records()
        assert [r[0] for r in rec] == ["encode_rows", "encode_rows", "xnor_gemm_lowk"]  # K = 256: the short-row kernel
        assert all(0.0 < r[1] < 50.0 for r in rec)
        B.prof_reset()
        assert B.prof_records() == []
    finally:
        B.prof_enable(False)


# ---------------------------------------------------------------- packed activations between layers
def _u64dev(a):
    return dev(np.ascontiguousarray(a).view(np.int64))


@pytest.mark.parametrize("case", [(2, 3, 10, 9, 128, 3, 3, 1, 1, 1, 1), (3, 3, 8, 8, 70, 3, 3, 2, 2, 1, 1),
                                  (1, 1, 6, 6, 5, 5, 5, 1, 1, 2, 2), (2, 2, 7, 7, 200, 3, 3, 1, 1, 0, 0),
                                  (2, 3, 10, 9, 200, 3, 3, 1, 1, 1, 1),    # two channel chunks, the second partial
                                  (1, 3, 40, 37, 257, 3, 3, 1, 1, 1, 1),   # five words per pixel, 24 pixel groups
                                  (3, 3, 9, 11, 31, 3, 3, 1, 2, 0, 1),     # fewer than 32 channels
                                  (2, 3, 5, 5, 1, 3, 3, 1, 1, 1, 1)])      # one channel
def test_conv2d_f32_sign_matches_oracle(case):
    print(f"conv2d_f32_sign case={case}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    shape = inputs.ConvShape(*case)
    d = inputs.conv_inputs(shape, seed=sum(case) + 1)
    x = inputs.inject_specials(d["x"], 3, frac=0.01, with_nan=False)
    got = as_u64(B.bnn_conv2d_f32_sign(dev(x), dev(d["w"]), dev(d["scale"]), dev(d["bias"]), (sH, sW), (pH, pW)))
    ref = oracle.pack_nhwc(oracle.conv2d_f32_seq(x, d["w"], (sH, sW), (pH, pW), d["scale"], d["bias"]))
    assert np.array_equal(got, ref)


PACKED_CASES = CONV_CASES + [
    (2, 128, 8, 8, 64, 3, 3, 1, 1, 1, 1),
    (3, 128, 12, 10, 130, 3, 3, 1, 1, 1, 1),
    (2, 256, 6, 6, 256, 3, 3, 1, 1, 1, 1),
    (1, 64, 4, 6, 10, 3, 3, 1, 1, 1, 1),
    (1, 320, 16, 16, 70, 3, 3, 1, 1, 1, 1),
    (2, 100, 7, 9, 33, 3, 3, 1, 1, 1, 1),     # two words per pixel, the second partial
    (1, 128, 6, 8, 16, 5, 5, 1, 1, 2, 2),     # 25 taps
    (1, 128, 10, 10, 8, 6, 6, 1, 1, 2, 2),    # 36 taps: more than the tap mask of the lean gather holds
    (2, 128, 9, 9, 20, 3, 3, 2, 2, 1, 1),     # stride 2
    (2, 128, 6, 6, 12, 1, 1, 1, 1, 0, 0),     # rows of two words: a half chunk only
    (2, 192, 6, 6, 12, 1, 1, 1, 1, 0, 0),     # rows of three words (odd: general gather)
]


@pytest.mark.parametrize("cfg", PACKED_KERNELS)
@pytest.mark.parametrize("case", PACKED_CASES[-11:] + PACKED_CASES[1:4])
def test_conv2d_packed_forced_tiles(case, cfg):
    """The binarizing epilogue on every tile shape it is written for (on the vector ALU the pooled form only
    exists for the four-column tiles; 4 and 6 fall back to the heuristic)."""
    print(f"conv2d_packed forced cfg={cfg} case={case}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    shape = inputs.ConvShape(*case)
    d = inputs.conv_inputs(shape, seed=sum(case) + 3)
    xp = _u64dev(oracle.pack_nhwc(d["x"]))
    wp = B.bnn_pack_conv_weight(dev(d["w"]))
    sc, bi = dev(d["scale"]), dev(d["bias"])
    st, pd = (sH, sW), (pH, pW)
    ref = oracle.conv2d_pm1(d["x"], d["w"], st, pd)
    run = lambda **kw: kernels_of(lambda: B.bnn_conv2d_packed(xp, wp, C, D, kH, kW, st, pd, scale=sc, bias=bi,
                                                              out="packed", cfg=cfg, **kw))
    got, names = run()
    assert np.array_equal(as_u64(got), oracle.pack_nhwc(oracle.scale_bias(ref, d["scale"], d["bias"], "nchw")))
    assert names == [PACKED_KERNELS[cfg]]
    if shape.OH % 2 == 0 and shape.OW % 2 == 0:
        pref = oracle.scale_bias(oracle.maxpool2x2_i32(ref), d["scale"], d["bias"], "nchw")
        got, names = run(pool=2)
        assert np.array_equal(as_u64(got), oracle.pack_nhwc(pref))
        assert cfg in (4, 6) or names == [PACKED_KERNELS[cfg]]
    assert np.array_equal(host(B.bnn_conv2d_packed(xp, wp, C, D, kH, kW, st, pd, out="i32", cfg=cfg)), ref)
    # the same forced tile through bnn_conv2d (fp32 image in, int32 NCHW out)
    oi, _ = B.bnn_conv2d(dev(d["x"]), wp, D, kH, kW, st, pd, want_int=True, cfg=cfg)
    assert np.array_equal(host(oi), ref)


@pytest.mark.parametrize("cfg,lean", [(None, None), (24, 1), (24, 0), (3, 1), (3, 0)])
@pytest.mark.parametrize("case", PACKED_CASES)
def test_conv2d_packed_all_output_kinds(case, cfg, lean):
    """As an application calls it, and on one staged tile of the matrix cores and one of the vector ALU with both
    gathers: lean = 0 forces the general one also where the input region (the table-driven gather) applies."""
    print(f"conv2d_packed case={case} cfg={cfg} lean={lean}", flush=True)
    _conv2d_packed_all_output_kinds(case, cfg=cfg, lean=lean)


def _conv2d_packed_all_output_kinds(case, cfg=None, lean=None):
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    shape = inputs.ConvShape(*case)
    d = inputs.conv_inputs(shape, seed=sum(case) + 2)
    x = inputs.inject_specials(d["x"], 4, frac=0.01)
    xp = _u64dev(oracle.pack_nhwc(x))
    wp = B.bnn_pack_conv_weight(dev(d["w"]))
    sc, bi = dev(d["scale"]), dev(d["bias"])
    st, pd = (sH, sW), (pH, pW)
    ref = oracle.conv2d_pm1(x, d["w"], st, pd)
    assert np.array_equal(host(B.bnn_conv2d_packed(xp, wp, C, D, kH, kW, st, pd, out="i32", cfg=cfg, lean=lean)), ref)
    yref = oracle.scale_bias(ref, d["scale"], d["bias"], "nchw")
    assert np.array_equal(host(B.bnn_conv2d_packed(xp, wp, C, D, kH, kW, st, pd, scale=sc, bias=bi, out="f32", cfg=cfg,
                                                   lean=lean)), yref)
    got = as_u64(B.bnn_conv2d_packed(xp, wp, C, D, kH, kW, st, pd, scale=sc, bias=bi, out="packed", cfg=cfg,
                                     lean=lean))
    assert np.array_equal(got, oracle.pack_nhwc(yref))
    if shape.OH % 2 == 0 and shape.OW % 2 == 0:
        pref = oracle.scale_bias(oracle.maxpool2x2_i32(ref), d["scale"], d["bias"], "nchw")
        got = as_u64(B.bnn_conv2d_packed(xp, wp, C, D, kH, kW, st, pd, pool=2, scale=sc, bias=bi, out="packed", cfg=cfg,
                                         lean=lean))
        assert np.array_equal(got, oracle.pack_nhwc(pref))


@pytest.mark.parametrize("case", [
    (2, 64, 9, 11, 64, 3, 3, 1, 1, 1, 1),      # one word, whole
    (3, 37, 14, 20, 70, 3, 3, 1, 1, 1, 1),     # one word, partial; a second row tile of six channels
    (1, 5, 6, 6, 33, 3, 3, 2, 2, 1, 1),        # fewer columns than a wave
    (2, 128, 10, 26, 130, 3, 3, 1, 1, 1, 1),   # two words, columns past one workgroup
    (5, 100, 13, 12, 64, 3, 3, 2, 1, 0, 1),    # the second partial, strides and padding of their own
    (3, 192, 16, 12, 65, 3, 3, 1, 1, 1, 1),    # three words: 512 columns a workgroup
    (2, 129, 22, 25, 32, 3, 3, 1, 1, 1, 1),    # one channel in the third
    (3, 256, 14, 14, 128, 3, 3, 1, 1, 1, 1),   # four words
    (70, 200, 3, 3, 40, 3, 3, 1, 1, 1, 1),     # 64 columns cross many images
    (4, 64, 9, 9, 96, 1, 1, 1, 1, 0, 0), (3, 130, 8, 10, 40, 1, 1, 2, 2, 0, 0), (2, 97, 7, 6, 64, 1, 1, 1, 1, 1, 1),
    (3, 250, 12, 12, 129, 1, 1, 1, 2, 0, 0),   # 1 x 1 of every number of words; padding; strides
    (1, 60, 1, 70, 64, 3, 3, 1, 1, 1, 1), (40, 256, 1, 1, 64, 3, 3, 1, 1, 1, 1)])
def test_conv_word_kernel_all_output_kinds(case):
    """The kernel whose taps go straight to the matrix cores, forced: maps in every store form, signs, pooled signs."""
    print(f"conv word kernel case={case}", flush=True)
    assert B.lib().bnn_testing_conv_word(*case, 0, 1, 256) > 0
    _conv2d_packed_all_output_kinds(case, cfg=19)


@pytest.mark.parametrize("N,C,H,W,D,k,out", [
    (17, 64, 32, 32, 64, 3, "packed"), (24, 40, 32, 32, 64, 3, "i32"), (24, 128, 16, 32, 128, 3, "packed"),
    (40, 128, 16, 33, 64, 3, "f32"), (52, 192, 32, 31, 64, 3, "packed"), (70, 256, 32, 31, 64, 3, "f32"),
    (200, 256, 32, 32, 64, 3, "packed"), (1, 64, 5, 5, 8, 1, "packed")])
def test_conv_word_rule(N, C, H, W, D, k, out):
    """Layers of every number of words that the rule takes there (on 256 compute units), as an application calls them: the
    batch repeats two images that the oracle knows."""
    print(f"conv word rule N={N} C={C} {H}x{W} D={D} {out}", flush=True)
    case = (2, C, H, W, D, k, k, 1, 1, k // 2, k // 2)
    assert B.lib().bnn_testing_conv_word(N, *case[1:], 0, out == "packed", 256) == 2
    d = inputs.conv_inputs(inputs.ConvShape(*case), seed=N)
    xp = _u64dev(oracle.pack_nhwc(d["x"])).repeat((N + 1) // 2, 1, 1, 1)[:N].contiguous()
    got = B.bnn_conv2d_packed(xp, B.bnn_pack_conv_weight(dev(d["w"])), C, D, k, k, (1, 1), (k // 2, k // 2),
                              scale=dev(d["scale"]), bias=dev(d["bias"]), out=out)
    ref = oracle.conv2d_pm1(d["x"], d["w"], (1, 1), (k // 2, k // 2))
    yref = oracle.scale_bias(ref, d["scale"], d["bias"], "nchw")
    want = {"i32": ref, "f32": yref, "packed": oracle.pack_nhwc(yref)}[out]
    got = as_u64(got) if out == "packed" else host(got)
    assert all(np.array_equal(got[n], want[n % 2]) for n in range(N))


def _random_geometries(n, seed):
    rng = np.random.default_rng(seed)
    out = []
    while len(out) < n:
        N = int(rng.integers(1, 4))
        C = int(rng.choice([1, 3, 17, 63, 64, 65, 100, 128, 129, 192, 200, 256]))
        H, W = int(rng.integers(3, 13)), int(rng.integers(3, 13))
        kH, kW = int(rng.integers(1, 6)), int(rng.integers(1, 6))
        sH, sW = int(rng.integers(1, 4)), int(rng.integers(1, 4))
        pH, pW = int(rng.integers(0, 3)), int(rng.integers(0, 3))
        D = int(rng.choice([1, 7, 31, 32, 33, 64, 65, 100, 130]))
        if H + 2 * pH < kH or W + 2 * pW < kW:
            continue
        out.append((N, C, H, W, D, kH, kW, sH, sW, pH, pW))
    return out


@pytest.mark.parametrize("case", _random_geometries(36, seed=20191104))
def test_conv_entry_points_on_random_geometries(case):
    """Seeded random shapes (kernel sizes 1..5, strides 1..3, pads 0..2, channel counts on and
    off the word grid) through bnn_conv2d, bnn_im2col_packed and every output kind of
    bnn_conv2d_packed."""
    print(f"random geometry case={case}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    shape = inputs.ConvShape(*case)
    d = inputs.conv_inputs(shape, seed=sum(case) + 11)
    _conv_parity(shape, d)
    _conv2d_packed_all_output_kinds(case)
    x = inputs.inject_specials(d["x"], 5, frac=0.01)
    cols = as_u64(B.bnn_im2col_packed(dev(x), kH, kW, (sH, sW), (pH, pW)))
    assert np.array_equal(cols, oracle.im2col_packed(x, kH, kW, (sH, sW), (pH, pW)))


def test_conv2d_packed_negative_scale_and_pool_order():
    """With a negative scale the affine map is decreasing: pooling must act on the int32
    accumulators before the affine map, not on its result."""
    print("conv2d_packed negative scale", flush=True)
    shape = inputs.ConvShape(2, 128, 8, 8, 64, 3, 3, 1, 1, 1, 1)
    d = inputs.conv_inputs(shape, seed=77)
    scale = -d["scale"]
    xp = _u64dev(oracle.pack_nhwc(d["x"]))
    wp = B.bnn_pack_conv_weight(dev(d["w"]))
    ref = oracle.maxpool2x2_i32(oracle.conv2d_pm1(d["x"], d["w"], (1, 1), (1, 1)))
    pref = oracle.pack_nhwc(oracle.scale_bias(ref, scale, d["bias"], "nchw"))
    got = as_u64(B.bnn_conv2d_packed(xp, wp, 128, 64, 3, 3, (1, 1), (1, 1), pool=2, scale=dev(scale),
                                     bias=dev(d["bias"]), out="packed"))
    assert np.array_equal(got, pref)


def test_pack_fc_weight_nhwc_matches_oracle():
    print("pack_fc_weight_nhwc", flush=True)
    rng = np.random.default_rng(41)
    for (n_out, C, H, W) in [(10, 70, 2, 3), (33, 512, 4, 4), (4, 64, 1, 1)]:
        w = rng.standard_normal((n_out, C * H * W)).astype(np.float32)
        got = as_u64(B.bnn_pack_fc_weight_nhwc(dev(w), C, H, W))
        assert np.array_equal(got, oracle.pack_fc_weight_nhwc(w, C, H, W))


@pytest.mark.parametrize("reading", ["A", "B"])
def test_cfg4_fused_stack_small_batch_every_layer(reading):
    print(f"cfg4 fused stack batch 4 reading {reading}", flush=True)
    from paper_1911_04477_amd.stack import VggStackFused
    d = inputs.cfg4(batch=4, reading=reading)
    net = VggStackFused(d["layers"], d["params"], batch=4, device=DEV)
    out, acts = net.forward(dev(d["x"]), keep=True)
    ref = oracle.vgg_stack(d["x"], d["layers"], d["params"])
    for i, (L, g, r) in enumerate(zip(d["layers"], acts, ref["acts"])):
        if L.kind in ("conv_f32", "bconv"):
            assert np.array_equal(as_u64(g), oracle.pack_nhwc(r)), f"layer {i} ({L.kind})"
        else:
            assert np.array_equal(host(g), r), f"layer {i} ({L.kind})"
    assert np.array_equal(host(out), ref["out"])


def test_cfg4_fused_stack_full_batch_is_deterministic():
    """Twenty passes at the benchmark's batch size give the same bits every time, layer by layer
    (a race between waves would show up as a difference between passes)."""
    print("cfg4 fused stack batch 256, repeated passes", flush=True)
    from paper_1911_04477_amd.stack import VggStackFused
    d = inputs.cfg4(batch=256)
    net = VggStackFused(d["layers"], d["params"], batch=256, device=DEV)
    x = dev(d["x"])
    out0, acts0 = net.forward(x, keep=True)
    torch.cuda.synchronize()
    for rep in range(20):
        out, acts = net.forward(x, keep=True)
        for i, (a, b) in enumerate(zip(acts0, acts)):
            assert torch.equal(a, b), f"pass {rep}, layer {i}"
        assert torch.equal(out0, out), f"pass {rep}"


def test_cfg4_fused_stack_graph_replays_match_oracle():
    """The fused pass captured into a HIP graph: every replay (new input contents each time,
    eager work and synchronisations of this process in between) must give the oracle's result
    for the input it ran on."""
    print("cfg4 fused stack, graph replays", flush=True)
    from paper_1911_04477_amd.stack import VggStackFused
    batch = 4
    d = inputs.cfg4(batch=batch)
    net = VggStackFused(d["layers"], d["params"], batch=batch, device=DEV)
    xbuf = dev(d["x"]).clone()
    net.capture(xbuf)
    rng = np.random.default_rng(5)
    for rep in range(4):
        x = d["x"] if rep == 0 else rng.standard_normal(d["x"].shape).astype(np.float32)
        xbuf.copy_(dev(x))
        got = host(net.replay()).copy()
        ref = oracle.vgg_stack(x, d["layers"], d["params"])["out"]
        assert np.array_equal(got, ref), f"replay {rep}"
        # eager work between replays: the same pass outside the graph, and an unrelated GEMM
        assert np.array_equal(host(net.forward(xbuf)), ref), f"eager pass after replay {rep}"
        _gemm_case(9, 70, 200, seed=rep)


def test_cfg4_fused_stack_full_batch_every_layer_every_image(cfg4_b256):
    """The benchmark's default step (packed activations between layers, batch 256): every layer's
    packed activation and the logits of all 256 images against the oracle."""
    print("cfg4 fused stack batch 256", flush=True)
    from paper_1911_04477_amd.stack import VggStackFused
    d, ref = cfg4_b256
    net = VggStackFused(d["layers"], d["params"], batch=256, device=DEV)
    out, acts = net.forward(dev(d["x"]), keep=True)
    for i, (L, g, r) in enumerate(zip(d["layers"], acts, ref["acts"])):
        if L.kind in ("conv_f32", "bconv"):
            assert np.array_equal(as_u64(g), oracle.pack_nhwc(r)), f"layer {i} ({L.kind})"
        else:
            assert np.array_equal(host(g), r), f"layer {i} ({L.kind})"
    assert np.array_equal(host(out), ref["out"])


CHAIN_CASES = [  # N, C, H, W, [(D, pool)]
    (3, 128, 8, 8, [(128, 0)]),                                    # one layer: 64 columns, half the waves idle
    (2, 128, 8, 8, [(64, 2)]),                                     # 64 channels out
    (2, 128, 32, 32, [(128, 2), (256, 0), (256, 2), (512, 0), (512, 2)]),
    (1, 128, 7, 9, [(128, 0), (64, 0)]),                           # 63 columns
    (2, 384, 12, 10, [(384, 2), (128, 0), (256, 0)]),              # six words per pixel; 30 pooled columns
    (1, 128, 2, 2, [(128, 0), (128, 2), (128, 0)]),                # down to one pixel
    (1, 512, 6, 6, [(512, 0), (512, 2), (512, 0), (64, 0)]),
    (1, 128, 33, 31, [(256, 0)]),                                  # 1023 columns
    (1, 128, 4, 4, [(128, 0)] * 8),                                # the most layers
]


@pytest.mark.parametrize("case", CHAIN_CASES)
def test_conv_chain(case):
    """Consecutive layers in one launch, bit for bit against the oracle; scales of both signs, and a layer with affine maps
    that never or always give +1, hit the boundary exactly, or are not finite."""
    print(f"conv_chain case={case}", flush=True)
    N, C, H, W, layers = case
    rng = np.random.default_rng(sum(case[:4]))
    h = rng.standard_normal((N, C, H, W)).astype(np.float32)
    xp = _u64dev(oracle.pack_nhwc(h))
    arr, keep = [], []
    for D, pool in layers:
        w = rng.standard_normal((D, C, 3, 3)).astype(np.float32)
        sc = (rng.uniform(0.5, 1.5, D) * rng.choice([-1.0, 1.0], D)).astype(np.float32)
        bi = (rng.standard_normal(D) * 20).astype(np.float32)
        for i, (s, b) in enumerate([(0.0, -0.0), (-0.0, 1.0), (np.nan, 1.0), (np.inf, 0.5), (1.0, np.inf), (-np.inf, 1.0),
                                    (1.0, -np.inf), (1e-42, 1e-43), (-3e38, 1e38), (0.25, -0.75), (-0.5, 3.0), (1.0, np.nan),
                                    (np.inf, -np.inf), (1.0, 1e9), (1.0, -1e9), (1e-45, -1e-45)]):
            sc[i], bi[i] = s, b
        acc = oracle.conv2d_pm1(h, w, (1, 1), (1, 1))
        if pool:
            acc = oracle.maxpool2x2_i32(acc)
        h = oracle.scale_bias(acc, sc, bi, "nchw")
        wc = B.bnn_pack_conv_chain_weight(B.bnn_pack_conv_weight(dev(w)), C)
        keep.append((wc, dev(sc), dev(bi)))
        arr.append((*keep[-1], D, pool))
        C = D
    ref = oracle.pack_nhwc(h)
    out = torch.zeros(ref.shape, dtype=torch.int64, device=DEV)
    for rep in range(3):
        out.fill_(-1)
        _, names = kernels_of(lambda: B.bnn_conv_chain(xp, case[1], B.conv_chain_layers(arr), out))
        assert names == ["conv_chain"]
        assert np.array_equal(as_u64(out), ref), rep


@pytest.mark.parametrize("N,C,H,W,layers", [(700, 128, 4, 4, [(128, 0), (256, 2), (64, 0)]), (513, 256, 6, 10, [(128, 2), (512, 0)]),
                                            (300, 128, 16, 16, [(128, 2), (128, 0)])])
def test_conv_chain_more_images_than_units(N, C, H, W, layers):
    """Images that start on a unit after others have ended there, and more workgroups than the shares of the filters that are
    fetched ahead: the layers one by one give the same bits, twice."""
    print(f"conv_chain {N}x{C}x{H}x{W} {layers}", flush=True)
    rng = np.random.default_rng(N)
    x = torch.randint(-2**63, 2**63 - 1, (N, H, W, C // 64), dtype=torch.int64, device=DEV, generator=torch.Generator(device=DEV).manual_seed(N))
    h, cin, arr = x, C, []
    for D, pool in layers:
        wp = B.bnn_pack_conv_weight(dev(rng.standard_normal((D, cin, 3, 3)).astype(np.float32)))
        sc = dev((rng.uniform(0.5, 1.5, D) * rng.choice([-1.0, 1.0], D)).astype(np.float32))
        bi = dev((rng.standard_normal(D) * 20).astype(np.float32))
        h = B.bnn_conv2d_packed(h, wp, cin, D, 3, 3, (1, 1), (1, 1), pool=pool, scale=sc, bias=bi)
        arr.append((B.bnn_pack_conv_chain_weight(wp, cin), sc, bi, D, pool))
        cin = D
    out = torch.empty_like(h)
    for rep in range(2):
        out.fill_(-1)
        B.bnn_conv_chain(x, C, B.conv_chain_layers(arr), out)
        assert torch.equal(out, h), rep


@pytest.mark.parametrize("pool", [0, 2])
def test_conv_chain_zero_at_negative_scale(pool):
    """A layer's affine map that is exactly 0 is +1 also where scale is negative and the boundary lies at minus twice the set
    bits of the filter row: the accumulator and the threshold are then both 0.  Filters of 0 to 15 set bits, scales of both
    signs, the boundary at each of them."""
    print(f"conv_chain zero at a negative scale, pool={pool}", flush=True)
    rng = np.random.default_rng(41 + pool)
    N, C, H, W, D = 2, 128, 16, 16, 128
    x = rng.standard_normal((N, C, H, W)).astype(np.float32)
    w = np.full((D, C * 9), -1.0, np.float32)
    ones = np.arange(D) % 16
    for d in range(D):
        w[d, rng.choice(C * 9, ones[d], replace=False)] = 1.0
    w = w.reshape(D, C, 3, 3)
    sc = np.where(np.arange(D) < D // 2, -0.5, 0.5).astype(np.float32)
    bi = (sc * 2.0 * ones).astype(np.float32)  # 0 at an accumulator of -2 * ones
    acc = oracle.conv2d_pm1(x, w, (1, 1), (1, 1))
    if pool:
        acc = oracle.maxpool2x2_i32(acc)
    y = oracle.scale_bias(acc, sc, bi, "nchw")
    zeros = (y == 0).reshape(N, D, -1).sum(axis=(0, 2))
    assert (zeros[sc < 0] > 0).sum() >= 16 and (zeros[sc > 0] > 0).sum() >= 16  # the boundary is met, not only stood beside
    ref = oracle.pack_nhwc(y)
    wc, dsc, dbi = B.bnn_pack_conv_chain_weight(B.bnn_pack_conv_weight(dev(w)), C), dev(sc), dev(bi)
    out = torch.zeros(ref.shape, dtype=torch.int64, device=DEV)
    B.bnn_conv_chain(_u64dev(oracle.pack_nhwc(x)), C, B.conv_chain_layers([(wc, dsc, dbi, D, pool)]), out)
    assert np.array_equal(as_u64(out), ref)


@pytest.mark.parametrize("batch,reading,chain", [(129, "A", True), (256, "A", True), (300, "A", False), (400, "A", True),
                                                 (256, "B", True), (400, "B", True)])
def test_fused_stack_chain_equals_layers(batch, reading, chain):
    """The stack's convolutions in one launch and one by one: the same logits, eagerly and replayed; the larger stack's first
    binarized convolution stays outside.  At 300 images a second round of a few does not pay, at 400 units take two."""
    print(f"fused stack, chain against layers, batch {batch}, reading {reading}", flush=True)
    from paper_1911_04477_amd.stack import VggStackFused
    d = inputs.cfg4(batch=batch, reading=reading)
    net = VggStackFused(d["layers"], d["params"], batch=batch, device=DEV)
    x = dev(d["x"])
    want, _ = net.forward(x, keep=True)
    want = host(want).copy()
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert (net._chain is not None) == chain
    _, names = kernels_of(lambda: net.forward(x))
    if net._chain is not None:
        assert names.count("conv_chain") == 1 and len(names) == (4 if reading == "A" else 5)
        assert len(net.conv_launches()) == (1 if reading == "A" else 2)
    else:
        assert "conv_chain" not in names and len(net.conv_launches()) == (5 if reading == "A" else 6)
    assert np.array_equal(host(net.forward(x)), want)
    net.capture(x)
    for rep in range(3):
        assert np.array_equal(host(net.replay()), want), rep
        assert np.array_equal(host(net.forward(x)), want), rep


@pytest.mark.parametrize("inference", [False, True])
def test_fused_stack_chain_follows_its_parameters(inference):
    """Parameters of layers inside the chain that are changed in place or replaced after construction count from the next
    pass on, eagerly as in the layers one by one; a captured pass reads the tensors that it was captured with."""
    print(f"fused stack, chain follows its parameters, inference mode {inference}", flush=True)
    import copy
    from paper_1911_04477_amd.stack import VggStackFused
    batch = 160
    d, e = inputs.cfg4(batch=batch), inputs.cfg4(batch=batch, seed=inputs.BASE_SEED + 77)
    x = dev(d["x"])
    with torch.inference_mode(inference):
        net = VggStackFused(d["layers"], d["params"], batch=batch, device=DEV)
        other = VggStackFused(e["layers"], e["params"], batch=batch, device=DEV)
        assert net._chain is not None
        layers = lambda: host(net.forward(x, keep=True)[0]).copy()
        i, j = net._chain.first + 1, net._chain.last
        first = layers()
        net.capture(x)

        def check(replayed):
            want = layers()
            _, names = kernels_of(lambda: net.forward(x))
            assert names.count("conv_chain") == 1
            assert np.array_equal(host(net.forward(x)), want)
            assert np.array_equal(host(net.replay()), want if replayed is None else replayed)
            return want
        assert np.array_equal(check(None), first)
        net.p[i]["wp"].copy_(other.p[i]["wp"])              # in place: the captured pass follows
        a = check(None)
        net.p[j]["scale"].neg_()
        net.p[j]["bias"][3:40] += 25.0
        b = check(None)
        net.p[j]["wp"] = other.p[j]["wp"].clone()           # another tensor: the captured pass keeps its own
        c = check(b)
        net.p[j]["scale"], net.p[j]["bias"] = net.p[j]["scale"].abs(), net.p[j]["bias"] * 2 - 1
        net.p[i] = dict(net.p[i], wp=net.p[i]["wp"].flip(0).contiguous())
        f = check(b)
        assert len({v.tobytes() for v in (first, a, b, c, f)}) == 5  # every change showed
        net._graph = net._graph_out = None
        net._graph_weights = net._graph_array = None
        twin = copy.deepcopy(net)
        assert np.array_equal(host(twin.forward(x)), f) and twin.p[j]["wp"] is not net.p[j]["wp"]


@pytest.mark.parametrize("N,C,H,W,D,k,s,pool", [
    (3000, 64, 3, 3, 300, 3, 2, 0), (258, 256, 7, 7, 1024, 3, 2, 2), (617, 192, 16, 17, 200, 3, 3, 2),  # many rows: eight waves
    (60, 192, 16, 16, 300, 3, 1, 2), (50, 128, 28, 28, 96, 3, 1, 0),                                    # few: four
    (3904, 64, 3, 3, 1024, 3, 2, 2), (1540, 192, 8, 9, 512, 3, 2, 0),                                   # two tiles a unit
    (429, 128, 11, 11, 1024, 5, 2, 2), (347, 192, 12, 12, 256, 3, 1, 0)])
def test_conv_sign_tiles_by_rows_and_words(N, C, H, W, D, k, s, pool):
    """Packed outputs on both sides of the line between four and eight waves for a 128 x 256 tile, against a vector-ALU tile."""
    print(f"sign tiles {N}x{C}x{H}x{W} -> {D} k{k} s{s} pool={pool}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(N + C + D)
    x = torch.randn(N, C, H, W, device=DEV, generator=g)
    xp = B.bnn_im2col_packed(x, 1, 1).view(N, H, W, -1)
    wp = B.bnn_pack_conv_weight(torch.randn(D, C, k, k, device=DEV, generator=g))
    sc, bi = torch.randn(D, device=DEV, generator=g), torch.randn(D, device=DEV, generator=g)
    run = lambda cfg=None: B.bnn_conv2d_packed(xp, wp, C, D, k, k, (s, s), (k // 2, k // 2), pool=pool, scale=sc, bias=bi, cfg=cfg)
    got, names = kernels_of(run)
    assert names == ["xnor_gemm_fp4"]
    assert torch.equal(got, run(cfg=3))
    for cfg in (21, 22):
        assert torch.equal(got, run(cfg=cfg)), cfg


# ---------------------------------------------------------------- MFMA ablation
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (37, 150, 300), (128, 128, 64), (130, 257, 1152), (64, 64, 256),
                                   (200, 333, 2304 + 17), (5, 700, 63),
                                   (300, 3300, 200), (513, 1650, 127)])
def test_mfma_ablation_matches_oracle(M, N, K):
    print(f"mfma M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(M * 7919 + N * 31 + K)
    A = inputs.inject_specials(rng.standard_normal((M, K)).astype(np.float32), 1, frac=0.002)
    Bm = inputs.inject_specials(rng.standard_normal((N, K)).astype(np.float32), 2, frac=0.002)
    Ap, Bp = B.bnn_encode(dev(A)), B.bnn_encode(dev(Bm))
    ref = oracle.gemm_pm1(A, Bm)
    assert np.array_equal(host(B.bnn_xnor_gemm_mfma_i8(Ap, Bp, K)), ref)
    assert np.array_equal(host(B.bnn_xnor_gemm_mfma_fp4(Ap, Bp, K)), ref)


def test_mfma_ablation_equals_valu_path_at_cfg2():
    print("mfma cfg2", flush=True)
    d = inputs.cfg2()
    Ap, Wp = B.bnn_encode(dev(d["act"])), B.bnn_encode(dev(d["wt"]))
    a = host(B.bnn_xnor_gemm_mfma_i8(Ap, Wp, inputs.CFG2.K))
    b = host(B.bnn_xnor_gemm(Ap, Wp, inputs.CFG2.K))
    assert np.array_equal(a, b)
    assert np.array_equal(host(B.bnn_xnor_gemm_mfma_fp4(Ap, Wp, inputs.CFG2.K)), b)


def _e2m1_rows(x):
    """Rows of +-1 values as 4-bit floating-point codes, written out from the format's definition:
    +1.0 is 0x2, -1.0 is 0xA, value k in nibble k % 2 (low first) of byte k / 2, rows padded with
    0.0 (0x0) to a multiple of 64 values."""
    rows, K = x.shape
    Kp = (K + 63) // 64 * 64
    codes = np.zeros((rows, Kp), dtype=np.uint8)
    codes[:, :K] = np.where(x >= 0, 0x2, 0xA)
    return (codes[:, 0::2] | (codes[:, 1::2] << 4)).astype(np.uint8)


@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (37, 150, 300), (128, 128, 64), (130, 257, 1152), (64, 64, 256),
                                   (200, 333, 2304 + 17), (5, 700, 63), (300, 3300, 200), (513, 1650, 127),
                                   (256, 1000, 128), (260, 129, 192)])
def test_mfma_fp4_expanded_ablation_matches_oracle(M, N, K):
    """Operands kept in memory as E2M1 +-1 rows: the expansion pass against the format's definition,
    the GEMM on every workgroup tile against the oracle."""
    print(f"mfma fp4 expanded M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(M * 7919 + N * 31 + K + 5)
    A = inputs.inject_specials(rng.standard_normal((M, K)).astype(np.float32), 1, frac=0.002)
    Bm = inputs.inject_specials(rng.standard_normal((N, K)).astype(np.float32), 2, frac=0.002)
    A4, B4 = B.bnn_expand_fp4(B.bnn_encode(dev(A)), K), B.bnn_expand_fp4(B.bnn_encode(dev(Bm)), K)
    assert np.array_equal(host(A4), _e2m1_rows(A))
    assert np.array_equal(host(B4), _e2m1_rows(Bm))
    ref = oracle.gemm_pm1(A, Bm)
    for tile in (None, 0, 1, 2):
        assert np.array_equal(host(B.bnn_xnor_gemm_mfma_fp4_expanded(A4, B4, K, tile=tile)), ref), f"tile {tile}"


def test_mfma_fp4_expanded_strided_operands_and_output():
    """Leading dimensions larger than the rows: operands inside wider buffers, C inside a wider matrix."""
    print("mfma fp4 expanded strided", flush=True)
    M, N, K = 70, 200, 330
    rng = np.random.default_rng(77)
    A = rng.standard_normal((M, K)).astype(np.float32)
    Bm = rng.standard_normal((N, K)).astype(np.float32)
    rb = 32 * ((K + 63) // 64)
    A4w = torch.full((M, rb + 48), 0x77, dtype=torch.uint8, device="cuda")
    B4w = torch.full((N, rb + 16), 0x77, dtype=torch.uint8, device="cuda")
    B.bnn_expand_fp4(B.bnn_encode(dev(A)), K, out=A4w[:, :rb])
    B.bnn_expand_fp4(B.bnn_encode(dev(Bm)), K, out=B4w[:, :rb])
    assert np.array_equal(host(A4w[:, :rb]), _e2m1_rows(A)) and bool((A4w[:, rb:] == 0x77).all())
    Cw = torch.full((M, N + 24), -7, dtype=torch.int32, device="cuda")
    B.bnn_xnor_gemm_mfma_fp4_expanded(A4w[:, :rb], B4w[:, :rb], K, C=Cw[:, :N])
    assert np.array_equal(host(Cw[:, :N]), oracle.gemm_pm1(A, Bm))
    assert bool((Cw[:, N:] == -7).all())


@pytest.mark.parametrize("case", [(2, 64, 9, 7, 40, 3, 3, 1, 1, 1, 1), (3, 128, 12, 12, 130, 3, 3, 1, 1, 1, 1),
                                  (2, 192, 11, 10, 70, 3, 3, 2, 2, 1, 1), (1, 64, 8, 8, 300, 1, 1, 1, 1, 0, 0),
                                  (2, 128, 9, 9, 33, 5, 3, 1, 2, 2, 0), (2, 256, 14, 14, 256, 3, 3, 1, 1, 1, 1),
                                  (5, 64, 6, 6, 17, 2, 2, 1, 1, 1, 1)])
def test_conv2d_mfma_fp4_expanded_matches_oracle(case):
    """The matrix-core ablation as a convolution: patches gathered from the 4-bit NHWC image."""
    print(f"conv2d mfma fp4 expanded case={case}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    d = inputs.conv_inputs(inputs.ConvShape(*case), seed=sum(case) + 23)
    x = inputs.inject_specials(d["x"], 7, frac=0.01)
    Cw = C // 64
    x4 = B.bnn_expand_fp4(_u64dev(oracle.pack_nhwc(x)).view(N * H * W, Cw), C).view(N, H, W, C // 2)
    assert np.array_equal(host(x4).reshape(N * H * W, C // 2), _e2m1_rows(x.transpose(0, 2, 3, 1).reshape(N * H * W, C)))
    w4 = B.bnn_expand_fp4(B.bnn_pack_conv_weight(dev(d["w"])), C * kH * kW)
    got = host(B.bnn_conv2d_mfma_fp4_expanded(x4, w4, C, D, kH, kW, (sH, sW), (pH, pW)))
    assert np.array_equal(got, oracle.conv2d_pm1(x, d["w"], (sH, sW), (pH, pW)))


# ---------------------------------------------------------------- fp32 control group (section 4.4)
@pytest.mark.parametrize("case", PACKED_CASES + [(1, 3, 5, 5, 130, 3, 3, 1, 1, 1, 1), (2, 40, 20, 20, 200, 3, 3, 2, 2, 0, 0)])
def test_control_group_conv_equals_binarized_result(case):
    """The real-valued GEMM on sign(x), sign(w) gives the same integers as the oracle (and so as
    the Xnor-Bitcount path), exactly: all partial sums are integers below 2^24."""
    print(f"control conv case={case}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    shape = inputs.ConvShape(*case)
    d = inputs.conv_inputs(shape, seed=sum(case) + 5)
    x = inputs.inject_specials(d["x"], 6, frac=0.01)
    got = host(B.bnn_control_conv2d_f32(dev(x), dev(d["w"]), (sH, sW), (pH, pW)))
    ref = oracle.conv2d_pm1(x, d["w"], (sH, sW), (pH, pW))
    assert got.dtype == np.float32 and np.array_equal(got, ref.astype(np.float32))


def test_control_group_conv_cfg3_full_size():
    print("control conv cfg3", flush=True)
    d = inputs.cfg3()
    s = inputs.CFG3
    got = host(B.bnn_control_conv2d_f32(dev(d["x"]), dev(d["w"]), (s.sH, s.sW), (s.pH, s.pW)))
    ref = oracle.conv2d_pm1(d["x"], d["w"], (s.sH, s.sW), (s.pH, s.pW))
    assert np.array_equal(got, ref.astype(np.float32))


# ---------------------------------------------------------------- sizes far off the tile grid
def _popcount_rows(a_words, b_words, K):
    """K - 2 * popcount(a xor b) for every pair of packed rows, with numpy only: the identity the
    oracle's float GEMM is pinned against, usable where K >= 2^24 puts that fp32 sum out of its
    exact range."""
    x = a_words[:, None, :] ^ b_words[None, :, :]
    cnt = np.unpackbits(x.view(np.uint8), axis=-1).sum(axis=-1, dtype=np.int64)
    return (K - 2 * cnt).astype(np.int32)


@pytest.mark.parametrize("cfg", [-1, 3, 25, 26, 27, 28])
def test_gemm_very_long_rows(cfg):
    """K = 2^24 + 77 bits: 65536 full chunks and a ragged tail per row, accumulators in the millions; beyond the
    staged matrix-core tiles' range."""
    print(f"gemm long K cfg={cfg}", flush=True)
    M, N, K = 3, 5, (1 << 24) + 77
    rng = np.random.default_rng(77)
    A = rng.standard_normal((M, K)).astype(np.float32)
    Bm = rng.standard_normal((N, K)).astype(np.float32)
    Bm[1] = A[0]            # one identical pair: C = K
    Bm[2] = -A[1]           # one opposite pair: C = -K (no zeros in a normal sample)
    Ap, Bp = B.bnn_encode(dev(A)), B.bnn_encode(dev(Bm))
    C, names = kernels_of(lambda: B.bnn_xnor_gemm(Ap, Bp, K, cfg=None if cfg < 0 else cfg))
    assert names == ["xnor_gemm_fp4_split" if cfg < 0 else GEMM_KERNELS[cfg]]
    got = host(C)
    assert got[0, 1] == K and got[1, 2] == -K
    # rows encoded by the oracle, not by the GPU
    assert np.array_equal(got, _popcount_rows(oracle.encode_rows(A), oracle.encode_rows(Bm), K))
    # the first 2^24 - 1 columns through the float oracle, the rest by the identity
    K0 = (1 << 24) - 1
    head = oracle.gemm_pm1(np.ascontiguousarray(A[:, :K0]), np.ascontiguousarray(Bm[:, :K0]))
    tail = _popcount_rows(oracle.encode_rows(np.ascontiguousarray(A[:, K0:])),
                          oracle.encode_rows(np.ascontiguousarray(Bm[:, K0:])), K - K0)
    assert np.array_equal(got, head + tail)


def test_gemm_many_columns():
    """N = 1.5 million columns (grid far beyond 65535 workgroups), K = 100 (masked tail only)."""
    print("gemm many columns", flush=True)
    M, N, K = 9, 1_500_001, 100
    rng = np.random.default_rng(5)
    A = rng.standard_normal((M, K)).astype(np.float32)
    Bm = rng.standard_normal((N, K)).astype(np.float32)
    got = host(B.bnn_xnor_gemm(B.bnn_encode(dev(A)), B.bnn_encode(dev(Bm)), K))
    assert np.array_equal(got, oracle.gemm_pm1(A, Bm))


@pytest.mark.parametrize("N,C", [(255, 128), (510, 64)])
def test_conv2d_packed_largest_images(N, C):
    """Batches at the documented limit of N*C*H*W (2^33 values): 67 / 134 million pixels, a packed input of
    1 GiB; an even (C = 128) and an odd (C = 64) number of words per pixel.  The batch
    repeats three distinct images, so every image's result is known from the oracle's three."""
    print(f"conv2d_packed largest images N={N} C={C}", flush=True)
    H, W, D, st, pd = 512, 512, 8, (1, 1), (1, 1)
    d = inputs.conv_inputs(inputs.ConvShape(3, C, H, W, D, 3, 3, 1, 1, 1, 1), seed=N)
    x = inputs.inject_specials(d["x"], 6, frac=0.001)
    ref = oracle.conv2d_pm1(x, d["w"], st, pd)
    xp = _u64dev(oracle.pack_nhwc(x)).repeat(N // 3, 1, 1, 1)
    wp = B.bnn_pack_conv_weight(dev(d["w"]))
    # one image more is beyond the range: refused, nothing launched
    with pytest.raises(B.BnnError):
        B.bnn_conv2d_packed(torch.cat([xp, xp[:3]]), wp, C, D, 3, 3, st, pd, out="i32")
    out = B.bnn_conv2d_packed(xp, wp, C, D, 3, 3, st, pd, out="i32")
    torch.cuda.synchronize()
    assert torch.equal(out.view(N // 3, 3, D, H, W), dev(ref).expand(N // 3, 3, D, H, W))
    del out
    sc, bi = dev(d["scale"]), dev(d["bias"])
    pref = oracle.pack_nhwc(oracle.scale_bias(oracle.maxpool2x2_i32(ref), d["scale"], d["bias"], "nchw"))
    got = B.bnn_conv2d_packed(xp, wp, C, D, 3, 3, st, pd, pool=2, scale=sc, bias=bi, out="packed")
    torch.cuda.synchronize()
    assert torch.equal(got.view(N // 3, 3, H // 2, W // 2, 1), _u64dev(pref).expand(N // 3, 3, H // 2, W // 2, 1))
    del xp, got
    torch.cuda.empty_cache()
    if C == 128:
        # the same batch as fp32 NCHW (34 GB) through bnn_conv2d: its encode, then the same GEMM
        xf = dev(x).repeat(N // 3, 1, 1, 1)
        oi, _ = B.bnn_conv2d(xf, wp, D, 3, 3, st, pd)
        torch.cuda.synchronize()
        assert torch.equal(oi.view(N // 3, 3, D, H, W), dev(ref).expand(N // 3, 3, D, H, W))
        del xf, oi
        torch.cuda.empty_cache()


@pytest.mark.parametrize("cfg", [None, 23, 25])
def test_conv2d_packed_rows_of_4_gib(cfg):
    """An input row of 2^29 one-word pixels (2^32 bytes) under one output column: rows 1 and 2 are 4 and 8 GiB
    into the image.  Counts from the nine pixels that the taps read."""
    print(f"conv2d_packed rows of 4 GiB cfg={cfg}", flush=True)
    W, D = 1 << 29, 40000  # enough outputs for the staged tiles
    rng = np.random.default_rng(29)
    px = rng.integers(0, 2, (3, 3))
    w = rng.standard_normal((D, 1, 3, 3)).astype(np.float32)
    xp = torch.zeros((1, 3, W, 1), dtype=torch.int64, device=DEV)
    xp[0, :, :3, 0] = torch.from_numpy(px).to(DEV)
    got = host(B.bnn_conv2d_packed(xp, B.bnn_pack_conv_weight(dev(w)), 1, D, 3, 3, (1, 1 << 30), (0, 0), out="i32",
                                   cfg=cfg))
    del xp
    torch.cuda.empty_cache()
    ref = (np.where(w[:, 0] >= 0, 1, -1) * (2 * px - 1)).sum(axis=(1, 2))
    assert np.array_equal(got[0, :, 0, 0], ref)


def _pm1_rows(packed, K):
    """Packed rows (uint64 words, element k in bit k % 64 of word k / 64, bit 1 = +1) as +-1 floats."""
    bits = np.unpackbits(np.ascontiguousarray(packed).view(np.uint8), axis=-1, bitorder="little")[:, :K]
    return np.where(bits == 1, 1.0, -1.0).astype(np.float32)


@pytest.mark.parametrize("N,K", [((1 << 31) - 257, 64), ((1 << 31) - 260, 128)])
def test_gemm_maximum_column_count(N, K):
    """The largest column count the header allows (2^31 - 257; the second case is the largest multiple of 4,
    which the short-row kernel takes): 17 / 34 GB of packed rows, 17 GB of output, checked on the first and
    last columns and on a random sample, against the oracle."""
    print(f"gemm max columns N={N} K={K}", flush=True)
    M, Kw = 2, K // 64
    g = torch.Generator(device="cuda").manual_seed(191104477)
    Bp = torch.randint(-2**63, 2**63 - 1, (N, Kw), dtype=torch.int64, device="cuda", generator=g)
    Ap = torch.randint(-2**63, 2**63 - 1, (M, Kw), dtype=torch.int64, device="cuda", generator=g)
    C = B.bnn_xnor_gemm(Ap, Bp, K)
    rng = np.random.default_rng(3)
    idx = np.unique(np.concatenate([np.arange(0, 1024), np.arange(N - 1024, N),
                                    rng.integers(0, N, size=200_000)])).astype(np.int64)
    it = torch.from_numpy(idx).cuda()
    got = host(C[:, it])
    rows = host(Bp[it]).view(np.uint64)
    ref = oracle.gemm_pm1(_pm1_rows(host(Ap).view(np.uint64), K), _pm1_rows(rows, K))
    assert np.array_equal(got, ref)
    del Bp, C
    torch.cuda.empty_cache()


def test_fused_stack_split_over_two_streams_matches_oracle():
    print("split batch over two streams", flush=True)
    from paper_1911_04477_amd.stack import SplitBatch
    d = inputs.cfg4(batch=6)
    sb = SplitBatch(d["layers"], d["params"], batch=6, parts=2, device=DEV)
    x = dev(d["x"])
    want = oracle.vgg_stack(d["x"], d["layers"], d["params"])["out"]
    for _ in range(3):  # replays reuse the per-slice buffers
        outs = sb.forward(x)
        got = np.concatenate([host(o) for o in outs], axis=0)
        assert np.array_equal(got, want)


def test_f32_glue_hand_worked_cases(golden_dir):
    """The hand-worked order / rounding cases of the real-valued layers, straight against the
    stored values (no oracle in between)."""
    import json
    import os
    with open(os.path.join(golden_dir, "f32_glue_order_examples.json")) as f:
        cases = json.load(f)
    f32 = lambda v: np.array([float(t) for t in v], dtype=np.float32)
    for c in cases["conv"]:
        print(f"conv2d_f32 hand-worked {c['name']}", flush=True)
        x, w = f32(c["x"]).reshape(c["x_shape"]), f32(c["w"]).reshape(c["w_shape"])
        args = (dev(x), dev(w), tuple(c["stride"]), tuple(c["pad"]))
        if "scale" in c:
            args += (dev(f32(c["scale"])), dev(f32(c["bias"])))
        got = host(B.bnn_conv2d_f32(*args)).ravel()
        assert np.array_equal(got, f32(c["out"]), equal_nan=True), (c["name"], got)
    for c in cases["fc"]:
        print(f"fc_f32 hand-worked {c['name']}", flush=True)
        x, w = np.array(c["x"], dtype=np.float32), np.array(c["w"], dtype=np.float32)
        got = host(B.bnn_fc_f32(dev(x), dev(w), dev(f32(c["bias"])), sign_input=c["sign_input"]))
        assert np.array_equal(got, np.array(c["out"], dtype=np.float32)), (c["name"], got)


@pytest.mark.parametrize("xs,ws", [(1e-25, 1e-15), (1e-38, 1.0), (1e18, 1e18), (1.0, 1e-44)])
def test_conv2d_f32_first_layer_chain_rounds_like_fmaf(xs, ws):
    """The 3x3x3 layer runs its (c, kh, kw) chain on the fp32 matrix cores, one reduction step
    per instruction; it must round exactly like the oracle's fmaf chain also where products or
    sums are subnormal, underflow to zero, or overflow."""
    case = (2, 3, 9, 8, 45, 3, 3, 1, 1, 1, 1)
    print(f"conv2d_f32 extreme magnitudes xs={xs} ws={ws}", flush=True)
    shape = inputs.ConvShape(*case)
    d = inputs.conv_inputs(shape, seed=77)
    x = (d["x"].astype(np.float64) * xs).astype(np.float32)
    w = (d["w"].astype(np.float64) * ws).astype(np.float32)
    got = host(B.bnn_conv2d_f32(dev(x), dev(w), (1, 1), (1, 1)))
    ref = oracle.conv2d_f32_seq(x, w, (1, 1), (1, 1))
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got.view(np.uint32)[~np.isnan(ref)], ref.view(np.uint32)[~np.isnan(ref)])
    sc = np.ones(45, np.float32)
    bi = np.zeros(45, np.float32)
    gp = as_u64(B.bnn_conv2d_f32_sign(dev(x), dev(w), dev(sc), dev(bi), (1, 1), (1, 1)))
    assert np.array_equal(gp, oracle.pack_nhwc(oracle.conv2d_f32_seq(x, w, (1, 1), (1, 1), sc, bi)))
    # an infinite filter tap: NaN wherever it meets a padding zero, on both sides
    w2 = w.copy()
    w2[0, 0, 0, 0] = np.inf
    w2[7, 2, 2, 1] = -np.inf
    got = host(B.bnn_conv2d_f32(dev(x), dev(w2), (1, 1), (1, 1)))
    ref = oracle.conv2d_f32_seq(x, w2, (1, 1), (1, 1))
    assert np.isnan(ref).any() and np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got, ref, equal_nan=True)
    gp = as_u64(B.bnn_conv2d_f32_sign(dev(x), dev(w2), dev(sc), dev(bi), (1, 1), (1, 1)))
    assert np.array_equal(gp, oracle.pack_nhwc(oracle.conv2d_f32_seq(x, w2, (1, 1), (1, 1), sc, bi)))


@pytest.mark.parametrize("case", [(2, 3, 10, 9, 128, 3, 3, 1, 1, 1, 1), (3, 3, 8, 8, 70, 3, 3, 2, 2, 1, 1),
                                  (1, 3, 7, 5, 5, 3, 3, 1, 2, 0, 1), (2, 4, 6, 6, 9, 3, 3, 1, 1, 1, 1),
                                  (2, 3, 6, 6, 9, 5, 5, 1, 1, 2, 2), (1, 3, 20, 19, 161, 3, 3, 1, 1, 1, 1)])
@pytest.mark.parametrize("affine", [True, False])
def test_conv2d_f32_real_valued_layer(case, affine):
    """fp32 convolution with fp32 output: the 3-channel 3x3 form runs on the matrix-core kernel,
    other geometries on the general one; both follow the (c, kh, kw) fma order."""
    print(f"conv2d_f32 case={case} affine={affine}", flush=True)
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    shape = inputs.ConvShape(*case)
    d = inputs.conv_inputs(shape, seed=sum(case) + 9)
    x = inputs.inject_specials(d["x"], 8, frac=0.01, with_nan=False)
    if affine:
        got = host(B.bnn_conv2d_f32(dev(x), dev(d["w"]), (sH, sW), (pH, pW), dev(d["scale"]), dev(d["bias"])))
        ref = oracle.conv2d_f32_seq(x, d["w"], (sH, sW), (pH, pW), d["scale"], d["bias"])
    else:
        got = host(B.bnn_conv2d_f32(dev(x), dev(d["w"]), (sH, sW), (pH, pW)))
        ref = oracle.conv2d_f32_seq(x, d["w"], (sH, sW), (pH, pW))
    # injected infinities of both signs meet in some sums: NaN there on both sides
    assert np.array_equal(np.isnan(got), np.isnan(ref))
    assert np.array_equal(got, ref, equal_nan=True)


# ---------------------------------------------------------------- whatever the size heuristic picks
def test_heuristic_kernel_selection_on_random_gemm_shapes():
    """Seeded random (M, N, K) on and off every grid through the entry points as an application
    calls them: the host chooses between the staged and the split-K matrix-core tiles and the short-row kernel."""
    rng = np.random.default_rng(1234)
    done = 0
    while done < 80:
        M = int(rng.choice([1, 3, 8, 31, 32, 33, 64, 100, 256, 300, 513]))
        N = int(rng.choice([1, 4, 60, 64, 68, 128, 200, 256, 1000, 1024, 4100]))
        K = int(rng.choice([1, 64, 65, 128, 200, 256, 257, 1000, 2048, 4096, 4100, 8192]))
        if M * N * K > 2e9:
            continue
        done += 1
        print(f"heuristic gemm M={M} N={N} K={K}", flush=True)
        A = rng.standard_normal((M, K)).astype(np.float32)
        Bm = rng.standard_normal((N, K)).astype(np.float32)
        sc = ((rng.random(N) + 0.5) * rng.choice([-1.0, 1.0], N)).astype(np.float32)
        bi = rng.standard_normal(N).astype(np.float32)
        C, Y = B.bnn_xnor_gemm_epilogue(B.bnn_encode(dev(A)), B.bnn_encode(dev(Bm)), K, dev(sc), dev(bi), B.CH_COL,
                                        want_int=True)
        ref = oracle.gemm_pm1(A, Bm)
        assert np.array_equal(host(C), ref), (M, N, K)
        assert np.array_equal(host(Y), oracle.scale_bias(ref, sc, bi, "col")), (M, N, K)


def test_heuristic_kernel_selection_on_random_packed_convs():
    """Seeded random layer shapes (few to many output pixels, scales of both signs) through
    bnn_conv2d_packed as the stack calls it: split-K and staged tiles, short-row kernel."""
    rng = np.random.default_rng(4321)
    for it in range(60):
        N = int(rng.integers(1, 9))
        C = int(rng.choice([64, 128, 130, 192, 256, 512]))
        H, W = int(rng.choice([4, 6, 8, 10, 16])), int(rng.choice([4, 6, 8, 12, 16]))
        D = int(rng.choice([8, 31, 32, 33, 64, 100, 128, 256]))
        k = int(rng.choice([1, 3]))
        p = k // 2
        shape = inputs.ConvShape(N, C, H, W, D, k, k, 1, 1, p, p)
        print(f"heuristic conv {shape}", flush=True)
        d = inputs.conv_inputs(shape, seed=1000 + it)
        sc = (d["scale"] * rng.choice([-1.0, 1.0], D)).astype(np.float32)
        xp = _u64dev(oracle.pack_nhwc(d["x"]))
        wp = B.bnn_pack_conv_weight(dev(d["w"]))
        ref = oracle.conv2d_pm1(d["x"], d["w"], (1, 1), (p, p))
        assert np.array_equal(host(B.bnn_conv2d_packed(xp, wp, C, D, k, k, (1, 1), (p, p), out="i32")), ref)
        got = as_u64(B.bnn_conv2d_packed(xp, wp, C, D, k, k, (1, 1), (p, p), scale=dev(sc), bias=dev(d["bias"]),
                                         out="packed"))
        assert np.array_equal(got, oracle.pack_nhwc(oracle.scale_bias(ref, sc, d["bias"], "nchw")))
        got = as_u64(B.bnn_conv2d_packed(xp, wp, C, D, k, k, (1, 1), (p, p), pool=2, scale=dev(sc),
                                         bias=dev(d["bias"]), out="packed"))
        assert np.array_equal(got, oracle.pack_nhwc(oracle.scale_bias(oracle.maxpool2x2_i32(ref), sc, d["bias"], "nchw")))


# ---------------------------------------------------------------- matrix-core GEMM on packed operands
@pytest.mark.parametrize("cfg", [23, 24, 25, 26, 27, 28])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (129, 257, 128), (128, 256, 512), (65, 300, 129), (37, 152, 640 + 33),
                                   (200, 515, 1024), (64, 1028, 2321), (257, 130, 512 * 3 + 1)])
def test_gemm_matrix_core_tiles(M, N, K, cfg):
    """Edges of tiles and of the 512-bit stages, rows that end anywhere in a 128-bit piece; int32 and both
    affine axes, padded strides.  Exact: the counts are integers below 2^24, the affine map one fma."""
    print(f"gemm matrix core M={M} N={N} K={K} cfg={cfg}", flush=True)
    _gemm_case(M, N, K, seed=M + 3 * N + 7 * K, cfg=cfg)
    rng = np.random.default_rng(M + N + K)
    A, Bm = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    ref = oracle.gemm_pm1(A, Bm)
    Kw = B.packed_words(K)
    Ap = torch.randint(-2**62, 2**62, (M, Kw + 1), dtype=torch.int64, device=DEV)  # odd or even stride, garbage past K
    Bp = torch.randint(-2**62, 2**62, (N, Kw + 3), dtype=torch.int64, device=DEV)
    Ap[:, :Kw], Bp[:, :Kw] = B.bnn_encode(dev(A)), B.bnn_encode(dev(Bm))
    for axis, n in ((B.CH_ROW, M), (B.CH_COL, N)):
        sc, bi = inputs.rand_scale(n, inputs._gen(K)), inputs.rand_bias(n, inputs._gen(K + 1))
        C, Y = B.bnn_xnor_gemm_epilogue(Ap, Bp, K, dev(sc), dev(bi), axis, want_int=True, cfg=cfg)
        assert np.array_equal(host(C), ref)
        assert np.array_equal(host(Y), oracle.scale_bias(ref, sc, bi, "row" if axis == B.CH_ROW else "col"))


@pytest.mark.parametrize("M,N,K,ldc", [
    (130, 100004, 300, 100004),   # ordinary stores
    (132, 100003, 300, 100003),   # 4-byte stores
    (130, 20004, 2500, 20012),    # rows inside half lines, non-temporal
    (130, 120016, 300, 120016),   # whole half lines, ordinary
    (130, 40016, 300, 40016),     # whole half lines, non-temporal
    (130, 40032, 300, 40064),     # whole lines
    (701, 2113, 1220, 2113),      # a last wave of 61 rows, 4-byte stores
    (701, 2116, 1220, 2116),      # ... 8-byte stores
])
def test_map_store_forms(M, N, K, ldc):
    """The forms of the matrix-core tiles' stores at full, partial and padded tiles against the vector-ALU tiles; nothing
    past the map is written."""
    print(f"map stores M={M} N={N} K={K} ldc={ldc}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    Ap = torch.randint(-2**62, 2**62, (M, B.packed_words(K)), dtype=torch.int64, device=DEV, generator=g)
    Bp = torch.randint(-2**62, 2**62, (N, B.packed_words(K)), dtype=torch.int64, device=DEV, generator=g)
    out = [torch.full((M + 8, ldc), -7, dtype=torch.int32, device=DEV) for _ in range(2)]
    for o, cfg in ((out[0], None), (out[1], 3)):
        _, names = kernels_of(lambda: B.bnn_xnor_gemm(Ap, Bp, K, o[:M, :N], cfg=cfg))
        assert names == ["xnor_gemm" if cfg else "xnor_gemm_fp4"]
    assert torch.equal(out[0], out[1])
    assert (out[0][:, N:] == -7).all() and (out[0][M:] == -7).all()
    sc, bi = torch.rand(M, device=DEV, generator=g) + 0.5, torch.randn(M, device=DEV, generator=g)
    ys = [B.bnn_xnor_gemm_epilogue(Ap, Bp, K, sc, bi, B.CH_ROW, want_int=True, cfg=cfg) for cfg in (None, 3)]
    assert torch.equal(ys[0][0], ys[1][0]) and torch.equal(ys[0][1], ys[1][1])
    assert torch.equal(ys[0][0], out[0][:M, :N])


@pytest.mark.parametrize("M,N,K,split", [
    (4, 40000, 1024, True),     # one row of tiles: nothing that a larger tile could use twice
    (32, 65536, 4096, True),
    (40000, 10, 2048, True),    # one column of tiles
    (4, 66000, 1024, False),    # more than eight 32 x 32 tiles per compute unit
    (4, 50000, 300, False),     # short rows, more than six
    (256, 4384, 576, True),     # few staged tiles, short rows
    (250, 5629, 1100, True),    # 5.5 tiles per compute unit
    (250, 5633, 1100, False),
    (250, 4385, 2100, True),    # from nine chunks on: up to eight
])
def test_gemm_few_rows_or_columns_split_the_reduction(M, N, K, split):
    """Which kernel takes a call at the edges of the rule (256 compute units), and its counts against the
    vector-ALU tiles."""
    print(f"gemm split rule M={M} N={N} K={K}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    Ap = torch.randint(-2**62, 2**62, (M, B.packed_words(K)), dtype=torch.int64, device=DEV, generator=g)
    Bp = torch.randint(-2**62, 2**62, (N, B.packed_words(K)), dtype=torch.int64, device=DEV, generator=g)
    got, names = kernels_of(lambda: B.bnn_xnor_gemm(Ap, Bp, K))
    assert torch.equal(got, B.bnn_xnor_gemm(Ap, Bp, K, cfg=3))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert names == ["xnor_gemm_fp4_split" if split else "xnor_gemm_fp4"]


@pytest.mark.parametrize("cfg", [25, 26, 27, 28])
@pytest.mark.parametrize("M,N,ldc", [(64, 64, 64), (128, 63, 63), (128, 66, 67), (70, 64, 66), (97, 61, 64), (33, 65, 65), (1, 2, 2)])
def test_split_map_store_forms(M, N, ldc, cfg):
    """Whole and partial tiles of rows, pairs of columns and single ones, maps and both affine axes, against the vector-ALU
    tiles (integers, and one fma of them: bit for bit); nothing past the map is written."""
    print(f"split map stores M={M} N={N} ldc={ldc} cfg={cfg}", flush=True)
    K = 641
    g = torch.Generator(device=DEV).manual_seed(M + N + ldc)
    A, Bm = (torch.randint(-2**62, 2**62, (n, B.packed_words(K)), dtype=torch.int64, device=DEV, generator=g) for n in (M, N))
    out = [torch.full((M + 8, ldc), -7, dtype=torch.int32, device=DEV) for _ in range(2)]
    for o, c in zip(out, (cfg, 3)):
        _, names = kernels_of(lambda: B.bnn_xnor_gemm(A, Bm, K, o[:M, :N], cfg=c))
        assert names == [GEMM_KERNELS[c]]
    assert torch.equal(out[0], out[1])
    assert (out[0][:, N:] == -7).all() and (out[0][M:] == -7).all()
    for axis, n in ((B.CH_ROW, M), (B.CH_COL, N)):
        sc, bi = torch.rand(n, device=DEV, generator=g) + 0.5, torch.randn(n, device=DEV, generator=g)
        ys = [B.bnn_xnor_gemm_epilogue(A, Bm, K, sc, bi, axis, want_int=True, cfg=c) for c in (cfg, 3)]
        assert torch.equal(ys[0][0], ys[1][0]) and torch.equal(ys[0][1], ys[1][1])
        assert torch.equal(ys[0][0], out[0][:M, :N])


MATRIX_CONV_CASES = [  # N, C, H, W, D, kH, kW, sH, sW, pH, pW
    (3, 64, 9, 7, 70, 3, 3, 1, 1, 1, 1),      # one word per pixel: the row ends in the middle of a piece
    (2, 200, 12, 12, 130, 3, 3, 1, 1, 1, 1),  # pad bits inside a tap's last word
    (40, 128, 4, 4, 128, 3, 3, 1, 1, 1, 1),   # many images per tile
    (1, 128, 40, 130, 64, 3, 3, 1, 1, 1, 1),  # rows longer than half a tile
    (2, 320, 17, 16, 65, 5, 3, 2, 1, 2, 0),   # strides and paddings that differ, odd words per pixel
    (5, 256, 10, 6, 256, 3, 3, 2, 2, 1, 1),
    (2, 128, 8, 8, 40, 1, 1, 1, 1, 0, 0),     # pointwise
    (3, 40, 6, 8, 33, 1, 3, 1, 1, 0, 1),      # one row of taps
    (1, 2048, 40, 60, 40, 3, 3, 1, 1, 1, 1),  # region larger than LDS: the general gather
    (2, 65, 14, 14, 20, 7, 7, 1, 1, 3, 3),    # 49 taps
]


@pytest.mark.parametrize("cfg,lean", [(c, 1) for c in range(21, 29)] + [(c, 0) for c in range(21, 25)])
@pytest.mark.parametrize("case", MATRIX_CONV_CASES)
def test_conv_matrix_core_tiles(case, cfg, lean):
    """int32, fp32, signs and pooled signs against the oracle, bit for bit; lean = 0: the staged tiles gather every
    word from memory also where the input region would fit LDS."""
    N, C, H, W, D, kH, kW, sH, sW, pH, pW = case
    print(f"conv matrix core {case} cfg={cfg} lean={lean}", flush=True)
    d = inputs.conv_inputs(inputs.ConvShape(*case), seed=sum(case))
    x = inputs.inject_specials(d["x"], 3, frac=0.001)
    st, pd = (sH, sW), (pH, pW)
    ref = oracle.conv2d_pm1(x, d["w"], st, pd)
    xp, wp = _u64dev(oracle.pack_nhwc(x)), B.bnn_pack_conv_weight(dev(d["w"]))
    sc, bi = dev(d["scale"]), dev(d["bias"])
    run = lambda **kw: B.bnn_conv2d_packed(xp, wp, C, D, kH, kW, st, pd, scale=sc, bias=bi, cfg=cfg, lean=lean, **kw)
    assert np.array_equal(host(run(out="i32")), ref)
    yref = oracle.scale_bias(ref, d["scale"], d["bias"], "nchw")
    assert np.array_equal(host(run(out="f32")), yref)
    assert np.array_equal(host(run(out="packed")).view(np.uint64), oracle.pack_nhwc(yref))
    if ref.shape[2] % 2 == 0 and ref.shape[3] % 2 == 0:
        pref = oracle.pack_nhwc(oracle.scale_bias(oracle.maxpool2x2_i32(ref), d["scale"], d["bias"], "nchw"))
        assert np.array_equal(host(run(out="packed", pool=2)).view(np.uint64), pref)


CONV_RULE_CASES = [  # C, H, W, kernel, stride
    (192, 9, 11, 1, 2), (704, 14, 14, 1, 2), (100, 8, 17, 1, 3), (128, 12, 12, 2, 2), (256, 32, 32, 2, 2),   # read once
    (256, 8, 8, 3, 1), (512, 8, 8, 3, 1),                       # small maps: four or eight waves
    (512, 14, 14, 3, 2), (704, 13, 13, 3, 2), (1024, 8, 8, 3, 2), (704, 28, 28, 3, 1),  # regions held twice, once, never
]


@pytest.mark.parametrize("tiles", [0.8, 1.9, 2.7, 4.5, 6.2])
@pytest.mark.parametrize("D", [40, 200])
@pytest.mark.parametrize("case", CONV_RULE_CASES)
def test_conv_tile_rule(case, D, tiles):
    """Every tile and gather that the rule picks by sizes against the staged 128 x 128 tile with the general gather and
    against a vector-ALU tile (integers: bit for bit)."""
    C, H, W, k, s = case
    p = k // 2 if k != 2 else 0
    OH, OW = (H + 2 * p - k) // s + 1, (W + 2 * p - k) // s + 1
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    N = max(1, round(tiles * cu * 128 / ((D + 127) // 128) / (OH * OW)))
    print(f"conv tile rule {case} D={D} N={N}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(sum(case) + D + N)
    Cw = B.packed_words(C)
    r = lambda *n: torch.randint(-2**63, 2**63 - 1, n, dtype=torch.int64, device=DEV, generator=g)
    x, w = r(N, H, W, Cw), r(D, k * k, Cw)
    if C % 64:
        x[..., -1] &= (1 << C % 64) - 1
        w[..., -1] &= (1 << C % 64) - 1
    w = w.reshape(D, k * k * Cw)
    sc, bi = torch.randn(D, device=DEV, generator=g), torch.randn(D, device=DEV, generator=g)
    run = lambda **kw: B.bnn_conv2d_packed(x, w, C, D, k, k, (s, s), (p, p), scale=sc, bias=bi, **kw)
    pools = [0, 2] if OH % 2 == 0 and OW % 2 == 0 else [0]
    for kw in [dict(out="i32"), dict(out="f32")] + [dict(out="packed", pool=q) for q in pools]:
        got = run(**kw)
        assert torch.equal(got, run(cfg=23, lean=0, **kw)), kw
        assert torch.equal(got, run(cfg=3, lean=0, **kw)), kw


@pytest.mark.parametrize("tiles", [0.9, 1.5, 2.6, 3.9, 4.6, 5.8, 7.9])
@pytest.mark.parametrize("M,K", [(33, 640), (100, 1600), (256, 2048), (300, 2111), (512, 4096), (96, 9300)])
def test_gemm_split_rule(M, K, tiles):
    """Every split that the rule picks by 32 x 32 tiles a unit and words a row, whole and half pieces, against a staged tile and
    a vector-ALU tile (integers: bit for bit)."""
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    N = max(33, int(tiles * cu / ((M + 31) // 32) * 32) - 3)
    print(f"split rule {M}x{N}x{K}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(M + N + K)
    r = lambda n: torch.randint(-2**63, 2**63 - 1, (n, B.packed_words(K)), dtype=torch.int64, device=DEV, generator=g)
    A, Bm = r(M), r(N)
    got = B.bnn_xnor_gemm(A, Bm, K)
    assert torch.equal(got, B.bnn_xnor_gemm(A, Bm, K, cfg=23))
    assert torch.equal(got, B.bnn_xnor_gemm(A, Bm, K, cfg=3))


@pytest.mark.parametrize("N,C,H,W,D,k,s,pool,out,split", [
    (381, 100, 7, 7, 96, 3, 1, 0, "packed", False),    # more than two 64 x 64 tiles a unit, since 96 rows are two tiles high
    (419, 100, 7, 9, 200, 3, 2, 0, "packed", True),    # the same, smallest maps: 32 x 32
    (435, 192, 7, 7, 96, 3, 1, 0, "i32", False),
    (569, 128, 15, 15, 128, 3, 3, 0, "packed", True),  # two a unit
    (168, 64, 7, 7, 192, 3, 1, 0, "f32", False), (168, 64, 7, 7, 192, 3, 1, 0, "i32", True),  # stores of fp32 maps
    (65, 100, 10, 10, 300, 3, 1, 0, "f32", False), (34, 128, 21, 21, 1024, 3, 3, 0, "f32", True),
    (89, 704, 8, 9, 300, 3, 2, 0, "packed", True), (13, 320, 16, 16, 96, 5, 1, 2, "packed", True)])  # long rows, odd words
def test_conv_split_rule(N, C, H, W, D, k, s, pool, out, split):
    """Which kernel takes convolutions of few tiles and short rows (256 compute units), and its values against a vector-ALU
    tile."""
    print(f"conv split rule {N}x{C}x{H}x{W} -> {D} k{k} s{s} pool={pool} {out}", flush=True)
    g = torch.Generator(device=DEV).manual_seed(N + C + D)
    x = torch.randn(N, C, H, W, device=DEV, generator=g)
    xp = B.bnn_im2col_packed(x, 1, 1).view(N, H, W, -1)
    wp = B.bnn_pack_conv_weight(torch.randn(D, C, k, k, device=DEV, generator=g))
    sc, bi = torch.randn(D, device=DEV, generator=g), torch.randn(D, device=DEV, generator=g)
    run = lambda cfg=None: B.bnn_conv2d_packed(xp, wp, C, D, k, k, (s, s), (k // 2, k // 2), pool=pool, scale=sc, bias=bi, out=out, cfg=cfg)
    got, names = kernels_of(run)
    assert torch.equal(got, run(cfg=3))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert names == ["xnor_gemm_fp4_split" if split else "xnor_gemm_fp4"]


def test_gemm_rows_beyond_the_accumulators_exact_range():
    """A wave's share of the row holds more than 2^23 values: its fp32 sums go to integers on the way."""
    K = (1 << 26) + (1 << 24) + 77
    print(f"gemm K={K}", flush=True)
    rng = np.random.default_rng(7)
    Kw = B.packed_words(K)
    A, Bm = (rng.integers(0, 1 << 64, size=(n, Kw), dtype=np.uint64) for n in (2, 3))
    A[1] = ~np.uint64(0)  # equal and opposite rows: the largest counts of both signs
    Bm[1] = ~np.uint64(0)
    Bm[2] = 0
    got = host(B.bnn_xnor_gemm(_u64dev(A), _u64dev(Bm), K))
    A[:, -1] &= np.uint64((1 << (K % 64)) - 1)
    Bm[:, -1] &= np.uint64((1 << (K % 64)) - 1)
    assert np.array_equal(got, _popcount_rows(A, Bm, K))
    assert got[1, 1] == K and got[1, 2] == -K


@pytest.mark.parametrize("N,H,W,D", [(1, 7, 9, 33), (2, 16, 16, 96), (1, 8, 8, 200), (70, 32, 32, 40), (5, 33, 31, 64),
                                     (24, 32, 32, 500), (24, 32, 32, 530)])
def test_first_layer_few_and_many_pixels(N, H, W, D):
    """The 3x3x3 layer with few pixels (chains, one channel group per workgroup) and with many (signs: half-precision products), channel
    counts off the group of 32; extreme magnitudes, signs and maps against the oracle's fma chains."""
    print(f"first layer N={N} {H}x{W} D={D}", flush=True)
    rng = np.random.default_rng(N + H + W + D)
    x = (rng.standard_normal((N, 3, H, W)) * 2.0 ** rng.integers(-40, 40, size=(N, 3, H, W))).astype(np.float32)
    w = rng.standard_normal((D, 3, 3, 3)).astype(np.float32)
    sc, bi = rng.standard_normal(D).astype(np.float32), rng.standard_normal(D).astype(np.float32)
    ref = oracle.conv2d_f32_seq(x, w, (1, 1), (1, 1), sc, bi)
    assert np.array_equal(host(B.bnn_conv2d_f32(dev(x), dev(w), (1, 1), (1, 1), dev(sc), dev(bi))), ref)
    got = as_u64(B.bnn_conv2d_f32_sign(dev(x), dev(w), dev(sc), dev(bi), (1, 1), (1, 1)))
    assert np.array_equal(got, oracle.pack_nhwc(ref))


def _first_form(N, H, W, D, stride, pad, form):
    """These sizes are for that form of the first layer's signs (on 256 compute units)."""
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert B.lib().bnn_testing_first_sign(N, H, W, D, stride, stride, pad, pad, 256) == form


@pytest.mark.parametrize("N,H,W,D,stride,pad,form", [
    (72, 32, 32, 96, 1, 1, 2),     # workgroups of four waves, two of 64 channels, the second half empty
    (13, 63, 65, 130, 1, 2, 2),    # 64 pixels cross rows and images, one word and two channels
    (64, 32, 33, 250, 1, 1, 4),    # 16 waves, the last group of 32 channels partial
    (150, 61, 59, 257, 2, 0, 3),   # eight waves, one channel in the last workgroup
    (513, 32, 32, 10, 1, 1, 3),    # several groups of pixels a wave, the last wave without any
    (4000, 5, 7, 448, 4, 1, 2)])   # 64 pixels cross many images
def test_first_layer_signs_from_split_products(N, H, W, D, stride, pad, form):
    """Enough pixels for the half-precision kernel: its bits are those of the fma chains.  Ordinary values, where a few
    outputs a wave are in doubt, then images with an area of zeros and channels that have no bias."""
    print(f"first layer signs N={N} {H}x{W} D={D} stride={stride} pad={pad}", flush=True)
    _first_form(N, H, W, D, stride, pad, form)
    rng = np.random.default_rng(N + H + W + D)
    x = rng.standard_normal((N, 3, H, W)).astype(np.float32)
    w = rng.standard_normal((D, 3, 3, 3)).astype(np.float32)
    sc, bi = rng.standard_normal(D).astype(np.float32), 0.1 * rng.standard_normal(D).astype(np.float32)
    for part in range(2):
        if part == 1:
            x[:, :, : (H + 1) // 2, : (W + 1) // 2] = 0.0
            bi[::3] = 0.0
            sc[::4] = 0.0
        ref = oracle.conv2d_f32_seq(x, w, (stride, stride), (pad, pad), sc, bi)
        got = as_u64(B.bnn_conv2d_f32_sign(dev(x), dev(w), dev(sc), dev(bi), (stride, stride), (pad, pad)))
        assert np.array_equal(got, oracle.pack_nhwc(ref))


@pytest.mark.parametrize("kind", ["specials", "nan", "ties", "large", "tiny", "filters", "scales"])
@pytest.mark.parametrize("N,D,form", [(24, 96, 0), (72, 96, 2), (64, 256, 3)])
def test_first_layer_signs_beyond_the_bound(N, D, form, kind):
    """Inputs whose signs the half-precision products cannot prove, in a few pixels or in all of them: the chains decide.  And a call
    that is left to the chains from the start."""
    print(f"first layer signs N={N} D={D} {kind}", flush=True)
    _first_form(N, 32, 32, D, 1, 1, form)
    rng = np.random.default_rng(N + D)
    x = rng.standard_normal((N, 3, 32, 32)).astype(np.float32)
    w = rng.standard_normal((D, 3, 3, 3)).astype(np.float32)
    sc, bi = (rng.random(D) + 0.5).astype(np.float32), 0.1 * rng.standard_normal(D).astype(np.float32)
    if kind == "specials":
        x = inputs.inject_specials(x, 3, frac=0.002)
    elif kind == "nan":
        x.reshape(-1)[:: 5] = np.nan
    elif kind == "ties":  # sums that are exactly 0, where the order of a sum in fp32 does not matter either
        x, w = rng.integers(-2, 3, x.shape).astype(np.float32), rng.integers(-2, 3, w.shape).astype(np.float32)
        sc, bi = np.ones(D, np.float32), np.zeros(D, np.float32)
    elif kind == "large":  # beyond fp16, and near its end
        x *= np.float32(1e6)
        x[: N // 2] *= np.float32(0.02)
    elif kind == "tiny":  # below fp16; subnormal; with and without a bias beside them
        x *= np.float32(1e-9)
        x[: N // 3] *= np.float32(1e-31)
        bi[::2] = 0.0
    elif kind == "filters":
        w[1] *= np.float32(1e30)
        w[2, 0, 0, 0] = np.inf
        w[33, 1, 1, 1] = np.nan
        w[40] *= np.float32(1e-42)
        w[41] = 0.0
        w[D - 1] *= np.float32(1e-20)
    else:
        sc[:8] = [0.0, -0.0, 1e30, -1e-30, np.inf, np.nan, 1e-44, -1.0]
        bi[:4] = [0.0, -0.0, -1e30, 1e-40]
        sc[40:48], bi[40:48] = 0.0, [0.0, -0.0, 1e-45, -1e-45, np.inf, -np.inf, np.nan, -3.0]
    with np.errstate(all="ignore"):
        ref = oracle.conv2d_f32_seq(x, w, (1, 1), (1, 1), sc, bi)
    got = as_u64(B.bnn_conv2d_f32_sign(dev(x), dev(w), dev(sc), dev(bi), (1, 1), (1, 1)))
    assert np.array_equal(got, oracle.pack_nhwc(ref))


FIRST_FORMS = [  # images of 32 x 32, channels, form
    (80, 90, 2), (64, 250, 3), (128, 200, 4),
    (600, 40, 3), (512, 40, 4)]  # two groups of pixels a wave


def _first_signs(N, D, form, x, w, sc, bi):
    """The signs of N images of 32 x 32, the ones of x over and over, in the form that the sizes are for, against the oracle's."""
    _first_form(N, 32, 32, D, 1, 1, form)
    with np.errstate(all="ignore"):
        ref = oracle.pack_nhwc(oracle.conv2d_f32_seq(x, w, (1, 1), (1, 1), sc, bi))
    xs = dev(x).repeat((N + len(x) - 1) // len(x), 1, 1, 1)[:N].contiguous()
    got = as_u64(B.bnn_conv2d_f32_sign(xs, dev(w), dev(sc), dev(bi), (1, 1), (1, 1)))
    bad = [n for n in range(N) if not np.array_equal(got[n], ref[n % len(x)])]
    assert not bad, bad


@pytest.mark.parametrize("kind", ["zeros", "zeros and biases", "sizes", "sizes and biases", "nans", "pruned", "one filter", "infinities",
                                  "ties", "specials"])
@pytest.mark.parametrize("N,D,form", FIRST_FORMS)
def test_first_layer_signs_of_whole_areas_in_doubt(N, D, form, kind):
    """What leaves more pixels in doubt than the half-precision kernel computes one by one, in every form of it: areas of zeros, sizes
    from 2^-140 to 2^120, NaN, channels without a filter, one filter that the bound does not cover."""
    print(f"first layer signs, areas: N={N} D={D} {kind}", flush=True)
    rng = np.random.default_rng(N + D)
    x = rng.standard_normal((16, 3, 32, 32)).astype(np.float32)
    w = rng.standard_normal((D, 3, 3, 3)).astype(np.float32)
    sc, bi = (rng.random(D) + 0.5).astype(np.float32), 0.1 * rng.standard_normal(D).astype(np.float32)
    sc[::5] *= np.float32(-1)
    if kind in ("zeros", "sizes", "one filter", "ties"):
        bi[:] = 0.0
    if kind.startswith("zeros"):
        x[::2] = 0.0
        x[1::4, :, 5:20, 7:] = -0.0
        x[3, :, 8, 8] = 1e-30
        bi[1::3], bi[2::9], bi[8::9] = 0.0, -0.0, -1e-38
        if kind == "zeros":
            bi[:] = np.where(np.arange(D) % 2, np.float32(0.0), np.float32(-0.0))
    elif kind.startswith("sizes"):
        x *= np.float32(2.0) ** np.array([-140, -100, -60, -49, -47, -30, -14, -3, -2, 0, 13, 16, 40, 59, 62, 120], np.float32).reshape(16, 1, 1, 1)
        x[4, :, :, 16:] *= np.float32(2.0**60)  # both in the pixels of one wave
        x[9, :, 10:20] = 0.0
        if kind != "sizes":
            bi *= np.float32(2.0) ** rng.integers(-60, 30, D).astype(np.float32)
            bi[::4] = 0.0
    elif kind == "nans":
        x[::2, 1, ::3] = np.nan
        x[1, 0, 4, 4] = np.nan
    elif kind == "pruned":
        w[::3] = 0.0
        w[4, 0] = -0.0
        sc[1::7], bi[::2] = 0.0, 0.0
        x[::5] = 0.0
        x[1] = np.inf
    elif kind == "one filter":
        w[35, 1, 1, 1] = np.inf
        w[3] *= np.float32(1e-30)
        x[::3] = 0.0
        x[1::3, :, 3:9] = np.nan
    elif kind == "infinities":
        x[::2].reshape(-1)[::997] = np.inf
        x[1::2].reshape(-1)[::53] = -np.inf
    elif kind == "ties":
        x, w = rng.integers(-2, 3, x.shape).astype(np.float32), rng.integers(-2, 3, w.shape).astype(np.float32)
        sc[:] = 1.0
    else:
        x = inputs.inject_specials(x, 3, frac=0.1)
    _first_signs(N, D, form, x, w, sc, bi)


@pytest.mark.parametrize("biased", [False, True])
def test_first_layer_signs_decided_by_subnormal_halves(biased):
    """Patches whose high halves cancel under the filter and whose low halves, subnormal in fp16, turn the sum against a 27th value:
    matrix instructions that took them as zeros would find the other sign, far beyond the bound."""
    print(f"first layer signs, subnormal halves biased={biased}", flush=True)
    N, D = 8256, 808  # one pixel an image
    rng = np.random.default_rng(3)
    w0 = np.tile(np.array([1, -1], np.float32), 13)
    a = (rng.integers(1024, 1229, (N, 13)) * 2.0**-12).astype(np.float32)  # fp16 holds them: 0.25 to 0.3
    low = (rng.random((N, 26)) * 2e-5 + 3e-5).astype(np.float32)          # below half an ulp of fp16 there (2^-13), and below 2^-14
    x = np.empty((N, 27), np.float32)
    x[:, :26] = np.repeat(a, 2, axis=1) + low * w0
    x[:, 26] = -0.5 * low.sum(axis=1)
    w = np.concatenate([w0, [1.0]]).astype(np.float32) * rng.choice([-1, 1], (D, 1)).astype(np.float32) * (rng.random((D, 1)) + 0.5).astype(np.float32)
    order = rng.permutation(27)
    x, w = x[:, order].reshape(N, 3, 3, 3), w[:, order].reshape(D, 3, 3, 3)
    sc, bi = np.ones(D, np.float32), np.zeros(D, np.float32)
    if biased:
        bi[1::2] = 1e-5 * rng.standard_normal(D // 2).astype(np.float32)
    _first_form(N, 3, 3, D, 1, 0, 2)
    ref = oracle.conv2d_f32_seq(x, w, (1, 1), (0, 0), sc, bi)
    assert np.array_equal(ref[:, :, 0, 0] >= 0, np.broadcast_to(w.reshape(D, 27)[:, np.argwhere(order == 26)[0, 0]] > 0, (N, D)))
    got = as_u64(B.bnn_conv2d_f32_sign(dev(x), dev(w), dev(sc), dev(bi), (1, 1), (0, 0)))
    assert np.array_equal(got, oracle.pack_nhwc(ref))


@pytest.mark.parametrize("e", range(-24, -1, 3))
def test_first_layer_signs_of_small_values(e):
    """Values about 2^e: halves of fp16 that are subnormal, low ones and high ones, with biases as small and with none."""
    print(f"first layer signs, values about 2^{e}", flush=True)
    rng = np.random.default_rng(100 + e)
    N, D = 80, 90
    x = (rng.standard_normal((16, 3, 32, 32)) * 2.0**e).astype(np.float32)
    w = rng.standard_normal((D, 3, 3, 3)).astype(np.float32)
    for none in (False, True):
        sc, bi = (rng.random(D) + 0.5).astype(np.float32), (rng.standard_normal(D) * 2.0 ** (e + 2)).astype(np.float32)
        bi[:: 1 if none else 3] = 0.0
        _first_signs(N, D, 2, x, w, sc, bi)


@pytest.mark.parametrize("N,D,stride,form", [(3, 196900, 2400, 1), (3, 100, 2400, 0), (1, 2200000, 2400, 1)])
def test_first_layer_signs_of_very_large_images(N, D, stride, form):
    """Images whose offsets conv_first_sign.hip does not hold: the chains, by four channel groups a workgroup where there are many
    channels, the last group partial."""
    print(f"first layer signs, very large images N={N} D={D}", flush=True)
    _first_form(N, 2400, 2400, D, stride, 1, form)
    rng = np.random.default_rng(N + D)
    x = np.zeros((N, 3, 2400, 2400), np.float32)
    x[:, :, :8, :8] = rng.standard_normal((N, 3, 8, 8))
    w = rng.standard_normal((D, 3, 3, 3)).astype(np.float32)
    sc, bi = rng.standard_normal(D).astype(np.float32), rng.standard_normal(D).astype(np.float32)
    ref = oracle.conv2d_f32_seq(np.ascontiguousarray(x[:, :, :2, :2]), w, (4, 4), (1, 1), sc, bi)  # the one pixel a stride leaves
    assert ref.shape[2:] == (1, 1)
    got = as_u64(B.bnn_conv2d_f32_sign(dev(x), dev(w), dev(sc), dev(bi), (stride, stride), (1, 1)))
    assert np.array_equal(got, oracle.pack_nhwc(ref))


@pytest.mark.parametrize("N,D", [(4, 449), (4, 256), (3, 449)])
def test_first_layer_large_maps(N, D):
    """Maps above and below 350 MB, channel counts on both sides of the rule and off the groups of 32 and 128: the
    batch repeats one image, whose map the oracle knows."""
    print(f"first layer large map N={N} D={D}", flush=True)
    H, W = 223, 227
    rng = np.random.default_rng(N + D)
    x = rng.standard_normal((1, 3, H, W)).astype(np.float32)
    w = rng.standard_normal((D, 3, 3, 3)).astype(np.float32)
    sc, bi = rng.standard_normal(D).astype(np.float32), rng.standard_normal(D).astype(np.float32)
    ref = dev(oracle.conv2d_f32_seq(x, w, (1, 1), (1, 1), sc, bi))
    out = B.bnn_conv2d_f32(dev(x).expand(N, 3, H, W).contiguous(), dev(w), (1, 1), (1, 1), dev(sc), dev(bi))
    torch.cuda.synchronize()
    assert torch.equal(out, ref.expand(N, D, H, W))


# ---------------------------------------------------------------- im2col in one launch / in two
@pytest.mark.parametrize("case", [
    # N, C, H, W, kH, kW, sH, sW, pH, pW
    (128, 64, 32, 32, 3, 3, 1, 1, 1, 1),   # two bands per image, halo rows on both sides
    (250, 3, 9, 11, 3, 3, 1, 1, 1, 1),     # one band per image, a partial granule and an empty one
    (256, 65, 4, 4, 3, 3, 1, 1, 1, 1),     # a workgroup per compute unit, odd words per pixel
    (257, 64, 4, 4, 3, 3, 1, 1, 1, 1),     # more images than compute units: two launches
    (7, 96, 20, 13, 5, 3, 2, 1, 2, 0),     # strides and paddings that differ, last band shorter
    (3, 130, 17, 9, 2, 2, 3, 2, 0, 1),     # rows that no tap reads
    (2, 40, 3, 3, 3, 3, 1, 1, 6, 6),       # bands that see padding only
    (1, 100, 40, 1, 7, 1, 1, 1, 3, 0),     # one column
    (1, 4096, 5, 5, 3, 3, 1, 1, 1, 1),     # one pixel fills the LDS budget early: two launches
    (1, 2000, 6, 2, 3, 3, 1, 1, 1, 1),
    (6, 33, 64, 5, 1, 3, 4, 1, 0, 1),      # row stride above the kernel's height
])
def test_im2col_bands(case):
    """Both sides of the rule that takes small inputs to one launch.  Exact: packed words."""
    print(f"im2col bands case={case}", flush=True)
    N, C, H, W, kH, kW, sH, sW, pH, pW = case
    rng = np.random.default_rng(sum(case))
    x = inputs.inject_specials(rng.standard_normal((N, C, H, W)).astype(np.float32), 3, frac=0.01)
    cols = as_u64(B.bnn_im2col_packed(dev(x), kH, kW, (sH, sW), (pH, pW)))
    assert np.array_equal(cols, oracle.im2col_packed(x, kH, kW, (sH, sW), (pH, pW)))


@pytest.mark.parametrize("case,bands", [
    ((1, 1, 1, 4096, 1, 101, 1, 1, 0, 50), False),   # one workgroup would emit every patch
    ((7, 4, 1, 2000, 1, 25, 1, 1, 0, 12), False),    # one per row
    ((1, 16, 1, 1024, 1, 9, 1, 1, 0, 4), False),     # little to emit, the reading too
    ((1, 1, 28, 28, 28, 28, 1, 1, 14, 14), False),   # a patch as large as the image
    ((1, 4, 3, 300, 1, 9, 1, 1, 0, 4), True),
    ((200, 1, 1, 500, 1, 51, 1, 1, 0, 25), True),    # as many pieces per workgroup, on every unit
    ((2, 3, 64, 64, 7, 7, 1, 1, 3, 3), True),
])
def test_im2col_bands_emit_no_more_than_their_share(case, bands):
    """Which of the two forms takes a call whose bands are few or long (256 compute units), and its words."""
    print(f"im2col choice case={case}", flush=True)
    N, C, H, W, kH, kW, sH, sW, pH, pW = case
    x = np.random.default_rng(sum(case)).standard_normal((N, C, H, W)).astype(np.float32)
    cols, names = kernels_of(lambda: B.bnn_im2col_packed(dev(x), kH, kW, (sH, sW), (pH, pW)))
    assert np.array_equal(as_u64(cols), oracle.im2col_packed(x, kH, kW, (sH, sW), (pH, pW)))
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        assert names == (["im2col_band"] if bands else ["encode_nchw", "im2col_gather"])
