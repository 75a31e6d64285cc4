"""GPU parity of the quantizer (Alg. 1 search, Eq. 4 scale refit, Code Cluster map of Sec. 3.3 / Eq. 1) through the C ABI:
codes, fp16 scales and the per-channel alpha / beta must equal the oracle's bit for bit (the oracle's canonical arrays
are put into device order by the library's own pack routines), on Gaussian weights, heavy-tailed weights, all-zero rows
and groups, and values that produce exact ties."""
import numpy as np
import pytest
import torch

from cases import assert_gemm_close
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FMT = {"narrow": (b.NARROW, o.F2), "wide": (b.WIDE, o.F275)}


def _weights(kind: str, N: int, K: int, seed: int) -> np.ndarray:
    rng = synth.rng(30, seed)
    if kind == "normal":
        return synth.weights_normal(N, K, rng)
    if kind == "heavy":                                   # outliers decide the group scale
        W = synth.weights_normal(N, K, rng)
        W[rng.random((N, K)) < 0.01] *= 12.0
        return W.astype(np.float32)
    if kind == "zeros":                                   # all-zero rows and groups among ordinary ones
        W = synth.weights_normal(N, K, rng)
        W[1] = 0.0
        W[3, 64:192] = 0.0
        W[N - 1, K - 64:] = 0.0
        return W
    if kind == "ties":                                    # few distinct values on a dyadic grid: many exact ties
        return (rng.integers(-8, 9, size=(N, K)) / 64.0).astype(np.float32)
    raise ValueError(kind)


def _compare(fmt_name, W):
    bfmt, ofmt = FMT[fmt_name]
    N, K = W.shape
    codes, scales, alpha, beta = o.quantize(W, ofmt)
    d = b.descriptor(K, N, [bfmt])
    want_codes = b.pack_codes(d, codes)
    want_scales = b.pack_scales(d, scales)
    got = b.quantize(torch.from_numpy(W).to(DEV), bfmt)
    torch.cuda.synchronize()
    g_codes = got.codes.cpu().numpy().reshape(-1)
    g_scales = got.scales.cpu().numpy().view(np.uint16).reshape(-1)
    if fmt_name == "narrow":
        assert np.array_equal(got.alpha.cpu().numpy().reshape(-1), alpha), "alpha differs"
        assert np.array_equal(got.beta.cpu().numpy().reshape(-1), beta), "beta differs"
    bad = np.flatnonzero(g_codes != want_codes)
    assert bad.size == 0, f"{bad.size} code bytes differ, first at {bad[:5]}"
    assert np.array_equal(g_scales, want_scales), "scales differ"
    return got, (codes, scales, alpha, beta)


@pytest.mark.parametrize("fmt_name", ["narrow", "wide"])
@pytest.mark.parametrize("kind", ["normal", "heavy", "zeros", "ties"])
def test_quantizer_matches_the_oracle(fmt_name, kind):
    K = 512 if fmt_name == "wide" else 256
    _compare(fmt_name, _weights(kind, 48, K, 1))


@pytest.mark.parametrize("fmt_name,N,K", [("narrow", 16, 1024), ("narrow", 208, 768), ("wide", 16, 1024), ("wide", 80, 1536)])
def test_shapes_and_row_stride(fmt_name, N, K):
    W = _weights("normal", N, K, 2)
    got, _ = _compare(fmt_name, W)
    # a strided source (ldw > K) gives the same result
    bfmt = FMT[fmt_name][0]
    big = torch.zeros((N, K + 64), dtype=torch.float32, device=DEV)
    big[:, :K] = torch.from_numpy(W).to(DEV)
    again = b.quantize(big[:, :K], bfmt)
    torch.cuda.synchronize()
    assert torch.equal(again.codes, got.codes) and torch.equal(again.scales, got.scales)


def test_quantize_then_multiply():
    """The quantizer's output is what ccq_gemm reads: quantize on the GPU, multiply on the GPU, compare with the oracle's
    product over the oracle's own encoding of the same matrix."""
    N, K, M = 256, 1024, 5
    W = _weights("normal", N, K, 3)
    got, (codes, scales, alpha, beta) = _compare("narrow", W)
    x = synth.activations_bf16(M, K, synth.rng(30, 9))
    y = b.gemm(got, b.bf16_tensor(x, DEV))
    torch.cuda.synchronize()
    Wd = o.decode(K, N, o.F2, codes, scales, alpha, beta)
    assert_gemm_close(b.bf16_bits(y), o.matmul(x, Wd), "quantize -> gemm")
    assert np.linalg.norm(Wd - W) / np.linalg.norm(W) < 0.45         # 2 bits per weight on Gaussian weights


@pytest.mark.parametrize("fmt_name", ["narrow", "wide"])
@pytest.mark.parametrize("kind", ["normal", "heavy", "zeros", "ties"])
def test_compressed_scales_match_the_oracle(fmt_name, kind):
    """scale_mode 1 (Sec. 3.4): quantize, then channel-wise super scale, 4-bit fields and one more search with the scale
    that is stored; codes (with the wide format's fields inside), packed narrow fields, super scales, alpha and beta."""
    bfmt, ofmt = FMT[fmt_name]
    N, K = 48, (512 if fmt_name == "wide" else 256)
    W = _weights(kind, N, K, 5)
    codes, scales, alpha, beta = o.quantize(W, ofmt)
    c2, sq, ssup = o.compress_scales(W, ofmt, codes, scales, alpha, beta)
    d = b.descriptor(K, N, [bfmt], scale_mode=1)
    got = b.quantize(torch.from_numpy(W).to(DEV), bfmt, scale_mode=1)
    torch.cuda.synchronize()
    assert np.array_equal(got.ssup.cpu().numpy().view(np.uint16).reshape(-1), ssup), "super scales differ"
    bad = np.flatnonzero(got.codes.cpu().numpy().reshape(-1) != b.pack_codes(d, c2))
    assert bad.size == 0, f"{bad.size} code bytes differ, first at {bad[:5]}"
    if fmt_name == "narrow":
        assert np.array_equal(got.scales.cpu().numpy().view(np.uint16).reshape(-1), b.pack_scales4(d, sq)), "scale fields differ"
        assert np.array_equal(got.alpha.cpu().numpy().reshape(-1), alpha) and np.array_equal(got.beta.cpu().numpy().reshape(-1), beta)
    else:
        assert got.scales is None
    # and the result multiplies: against the oracle's decode of its own compressed encoding
    x = synth.activations_bf16(3, K, synth.rng(30, 77))
    y = b.gemm(got, b.bf16_tensor(x, DEV))
    torch.cuda.synchronize()
    Wd = o.decode_cs(K, N, ofmt, c2, sq, ssup, alpha, beta)
    assert_gemm_close(b.bf16_bits(y), o.matmul(x, Wd), "quantize (compressed scales) -> gemm")


@pytest.mark.parametrize("kind", ["normal", "heavy", "zeros", "ties"])
@pytest.mark.parametrize("mode", [0, 1])
def test_hybrid_word_matches_the_oracle(kind, mode):
    """The hybrid 16-bit word (Sec. 3.2): two independent searches per word, fp16 scales or the 13-bit field of Sec. 3.4."""
    N, K = 32, 512
    W = _weights(kind, N, K, 6)
    codes, scales = o.h16_quantize(W)
    ssup = None
    if mode == 1:
        codes, ssup = o.h16_compress_scales(W, codes, scales)
    d = b.descriptor(K, N, b.H16, scale_mode=mode)
    got = b.quantize(torch.from_numpy(W).to(DEV), b.H16, scale_mode=mode)
    torch.cuda.synchronize()
    bad = np.flatnonzero(got.codes.cpu().numpy().reshape(-1) != b.pack_codes(d, codes))
    assert bad.size == 0, f"{bad.size} code bytes differ, first at {bad[:5]}"
    if mode == 0:
        assert np.array_equal(got.scales.cpu().numpy().view(np.uint16).reshape(-1), b.pack_scales(d, scales)), "scales differ"
        Wd = o.h16_decode(K, N, codes, scales)
    else:
        assert np.array_equal(got.ssup.cpu().numpy().view(np.uint16).reshape(-1), ssup), "super scales differ"
        Wd = o.h16_decode_cs(K, N, codes, ssup)
    x = synth.activations_bf16(2, K, synth.rng(30, 78))
    y = b.gemm(got, b.bf16_tensor(x, DEV))
    torch.cuda.synchronize()
    assert_gemm_close(b.bf16_bits(y), o.matmul(x, Wd), "quantize (hybrid word) -> gemm")


@pytest.mark.parametrize("mode", [0, 1])
def test_mixed_formats_match_the_oracle(mode):
    """A per-group mix of the narrow and wide formats (group_fmt shared by all rows): the Code Cluster map is fitted to the
    narrow groups' codes only, the super scale to all groups of the row."""
    N, K = 32, 2048
    G = K // 64
    gf = synth.group_format_map(G, 8, synth.rng(30, 50))
    W = _weights("heavy", N, K, 7)
    W[2, 64 * int(np.flatnonzero(gf == 1)[0]):][:64] = 0.0          # an all-zero wide group
    fmt = (o.F2, o.F275)
    codes, scales, alpha, beta = o.quantize(W, fmt, gf)
    d = b.descriptor(K, N, [b.NARROW, b.WIDE], gf, scale_mode=mode)
    got = b.quantize(torch.from_numpy(W).to(DEV), [b.NARROW, b.WIDE], scale_mode=mode, group_fmt=gf)
    torch.cuda.synchronize()
    if mode == 0:
        want_codes, want_scales = b.pack_codes(d, codes), b.pack_scales(d, scales)
        Wd = o.decode(K, N, fmt, codes, scales, alpha, beta, gf)
    else:
        c2, sq, ssup = o.compress_scales(W, fmt, codes, scales, alpha, beta, gf)
        want_codes, want_scales = b.pack_codes(d, c2), b.pack_scales4(d, sq)
        assert np.array_equal(got.ssup.cpu().numpy().view(np.uint16).reshape(-1), ssup), "super scales differ"
        Wd = o.decode_cs(K, N, fmt, c2, sq, ssup, alpha, beta, gf)
    bad = np.flatnonzero(got.codes.cpu().numpy().reshape(-1) != want_codes)
    assert bad.size == 0, f"{bad.size} code bytes differ, first at {bad[:5]}"
    assert np.array_equal(got.scales.cpu().numpy().view(np.uint16).reshape(-1), want_scales), "scales differ"
    assert np.array_equal(got.alpha.cpu().numpy().reshape(-1), alpha) and np.array_equal(got.beta.cpu().numpy().reshape(-1), beta)
    x = synth.activations_bf16(2, K, synth.rng(30, 79))
    y = b.gemm(got, b.bf16_tensor(x, DEV))
    torch.cuda.synchronize()
    assert_gemm_close(b.bf16_bits(y), o.matmul(x, Wd), "quantize (mixed formats) -> gemm")


def test_full_size_sampled_rows():
    """The 8192 x 8192 matrix of the benchmark: every row is independent of the others (scales per group, alpha / beta per
    row), so the oracle encodes a sample of rows and those are compared bit for bit, read out of the device layout
    (narrow k-tile: byte 4 kq + b of group j of the tile at (kq * 16 + row) * 16 + 4 j + b)."""
    K = N = 8192
    W = synth.weights_normal(N, K, synth.rng(30, 40))
    got = b.quantize(torch.from_numpy(W).to(DEV), b.NARROW)
    torch.cuda.synchronize()
    rows = np.array([0, 1, 15, 16, 17, 4095, 4096, 8176, 8191] + synth.rng(30, 41).integers(0, N, 7).tolist())
    codes, scales, alpha, beta = o.quantize(W[rows], o.F2)
    dev_codes = got.codes.cpu().numpy().reshape(-1)
    dev_scales = got.scales.cpu().numpy().view(np.uint16).reshape(-1)
    G = K // 64
    g, j = np.meshgrid(np.arange(G), np.arange(16), indexing="ij")
    for i, n in enumerate(rows):
        off = (n // 16) * got.info.row_tile_bytes + (g // 4) * 1024 + ((j // 4) * 16 + n % 16) * 16 + (g % 4) * 4 + j % 4
        assert np.array_equal(dev_codes[off].reshape(-1), codes[i]), f"row {n}: codes differ"
        soff = (n // 16) * (G // 4) * 64 + (np.arange(G) // 4) * 64 + (n % 16) * 4 + np.arange(G) % 4
        assert np.array_equal(dev_scales[soff], scales[i]), f"row {n}: scales differ"
    assert np.array_equal(got.alpha.cpu().numpy().reshape(-1)[rows], alpha) and np.array_equal(got.beta.cpu().numpy().reshape(-1)[rows], beta)


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("fmt", ["narrow", "wide", "h16"])
@pytest.mark.parametrize("N", [8192, 4112])
def test_large_matrix_equals_its_rows(fmt, mode, N):
    """Rows are independent: a matrix large enough for the search with two lanes per group (its workgroups fill the chip many
    times over), or with four (more than one workgroup per CU), gives the bytes that the one with sixteen lanes gives for any
    sixteen of its rows, and those are the oracle's (the tests above).  K = 2240: 35 groups, a ragged last k-tile; outliers,
    zeros and exact ties among the rows."""
    K = 2240
    g = torch.Generator(device=DEV).manual_seed(31)
    W = torch.randn(N, K, generator=g, device=DEV) * 0.02
    W[5] = torch.round(W[5] * 256) / 256
    W[16:32, :64] = 0.0
    W[4000, ::97] *= 12.0
    f = {"narrow": b.NARROW, "wide": b.WIDE, "h16": b.H16}[fmt]
    big = b.quantize(W, f, scale_mode=mode, prefill_byte=0xFF)
    for r0 in (0, 16, 3984, 4000, N - 16):
        small = b.quantize(W[r0:r0 + 16].contiguous(), f, scale_mode=mode, prefill_byte=0xFF)
        for name in ("codes", "scales", "ssup", "alpha", "beta"):
            x, y = getattr(big, name), getattr(small, name)
            assert (x is None) == (y is None)
            if x is not None:
                assert torch.equal(x.reshape(N // 16, -1)[r0 // 16], y.reshape(-1)), f"{name} of rows {r0}.. differ"


def _sparse(kind: str, N: int, K: int, seed: int = 0) -> torch.Tensor:
    g = torch.Generator(device=DEV).manual_seed(seed)
    W = torch.randn(N, K, generator=g, device=DEV) * 0.02
    if kind == "half zeros":
        W[torch.rand(N, K, generator=g, device=DEV) < 0.5] = 0.0
    elif kind == "mostly zeros":
        W[torch.rand(N, K, generator=g, device=DEV) < 0.9] = 0.0
    elif kind == "ternary":
        W = torch.sign(W) * (W.abs() > 0.012) * 0.02
    return W


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("kind", ["half zeros", "mostly zeros", "ternary"])
def test_weights_with_many_ties(kind, mode):
    """Zeros and repeated values tie on many codes: up to half of the vectors take the exact search, any number of them per
    wavefront.  Codes and scales against the oracle, every format."""
    N, K = 33, 832
    W = _sparse(kind, N, K, 5).cpu().numpy()
    for name, bf, of in (("narrow", b.NARROW, o.F2), ("wide", b.WIDE, o.F275), ("h16", b.H16, None)):
        fields = ssup = None
        if of is None:
            codes, scales = o.h16_quantize(W)
            if mode == 1:
                codes, ssup = o.h16_compress_scales(W, codes, scales)
        else:
            codes, scales, alpha, beta = o.quantize(W, of)
            if mode == 1:
                codes, fields, ssup = o.compress_scales(W, of, codes, scales, alpha, beta)
        d = b.descriptor(K, N, bf if of is None else [bf], scale_mode=mode)
        got = b.quantize(torch.from_numpy(W).to(DEV), bf, scale_mode=mode)
        assert np.array_equal(got.codes.cpu().numpy().reshape(-1), b.pack_codes(d, codes)), f"{name}: codes differ"
        if mode == 1:
            assert np.array_equal(got.ssup.cpu().numpy().view(np.uint16).reshape(-1), ssup), f"{name}: super scales differ"
        if got.scales is not None:
            want = b.pack_scales(d, scales) if mode == 0 else b.pack_scales4(d, fields)
            assert np.array_equal(got.scales.cpu().numpy().view(np.uint16).reshape(-1), want), f"{name}: scales differ"


def _best_us(W, f):
    b.quantize(W, f)
    out = []
    for _ in range(5):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        b.quantize(W, f)
        t1.record()
        torch.cuda.synchronize()
        out.append(t0.elapsed_time(t1) * 1e3)
    return min(out)


@pytest.mark.parametrize("fmt,limit", [("wide", 2.8), ("h16", 9.0)])
def test_ties_do_not_cost_a_search_each(fmt, limit):
    """The exact search takes as many vectors at once as a wavefront holds sets of states: a matrix that sends about a third
    of its vectors there (9 in 10 zeros) costs a small multiple of a dense one: 1.8 (wide) and 4.5 times (hybrid word); one vector at a time
    it was 3.9 and 26 times.  The limits lie half way, as ratios."""
    f = {"wide": b.WIDE, "h16": b.H16}[fmt]

    dense, sparse = _best_us(_sparse("dense", 8192, 4096), f), _best_us(_sparse("mostly zeros", 8192, 4096), f)
    print(f"{fmt}: dense {dense:.0f} us, mostly zeros {sparse:.0f} us")
    assert sparse < limit * dense


@pytest.mark.parametrize("fmt,limit", [("narrow", 4.0), ("wide", 1.6)])
def test_ties_in_a_small_matrix(fmt, limit):
    """Few groups are spread over many wavefronts, each with few vectors to search exactly one after the other.  256 x 4096,
    half zeros, against the same matrix dense: 3.0 and 1.35 times; with sixteen groups to a wavefront 5.2 and 1.8 times."""
    f = {"narrow": b.NARROW, "wide": b.WIDE}[fmt]
    dense, sparse = _best_us(_sparse("dense", 256, 4096), f), _best_us(_sparse("half zeros", 256, 4096), f)
    print(f"{fmt}: dense {dense:.0f} us, half zeros {sparse:.0f} us: {sparse / dense:.2f}")
    assert sparse < limit * dense


def _nearest_wide(w: np.ndarray, s: np.ndarray) -> np.ndarray:
    """Wide-format bytes [R][22] of groups w [R][64] at scales s [R]: the lowest of the codes with the smallest fp64 error."""
    c = np.arange(256)
    lv = np.stack([(c >> 4) & 15, (c >> 2) & 15, c & 15], 1).astype(np.float64) - 8.0
    v = np.concatenate([w.astype(np.float64), np.zeros((w.shape[0], 2))], 1).reshape(-1, 22, 1, 3)
    d = v - s.reshape(-1, 1, 1, 1) * lv
    return np.argmin(d[..., 0] ** 2 + d[..., 1] ** 2 + d[..., 2] ** 2, axis=2).astype(np.uint8)


@pytest.mark.parametrize("mode", [0, 1])
def test_a_weight_that_is_not_a_number_stays_in_its_code(mode):
    """Wide format: a NaN makes its own three-weight code meaningless and nothing else.  The other codes of its group are
    the nearest ones at the scale of the remaining weights (absmax / 7, as the refit sum is not a number), all other groups
    are those of the matrix without NaN."""
    N, K = 16, 704                                          # eleven groups: a ragged last k-tile
    W = synth.weights_normal(N, K, synth.rng(30, 77))
    hurt = W.copy()
    for n, k in ((0, 0), (1, 62), (2, 63), (3, 64 + 5), (3, 128 + 59), (4, 3 * 64 + 30), (5, 10 * 64 + 33), (6, 7 * 64 + 60)):
        hurt[n, k] = np.nan
    groups = hurt.reshape(-1, 64)
    nan = np.isnan(groups)
    with np.errstate(over="ignore"):
        codes, scales, _, _ = o.quantize(W, o.F275)
    codes = codes.reshape(-1, 22).copy()
    s = o.fp16_bits_to_f64(scales).reshape(-1)
    s[nan.any(1)] = np.float16(np.nanmax(np.abs(groups), axis=1).astype(np.float64) / 7.0)[nan.any(1)]
    ssup = None
    if mode == 1:
        ssup = np.float16(s.reshape(N, -1).max(1) / 15.0)
        k = np.clip(np.rint(s.reshape(N, -1) / ssup.astype(np.float64)[:, None]), 1, 15).reshape(-1)
        codes = _nearest_wide(np.where(nan, 0.0, groups), k * np.repeat(ssup.astype(np.float64), K // 64))
        codes[:, 21] = (codes[:, 21] & 0xF0) | k.astype(np.uint8)
    else:
        codes[nan.any(1)] = _nearest_wide(np.where(nan, 0.0, groups), s)[nan.any(1)]
    own = np.concatenate([nan, np.zeros((nan.shape[0], 2), bool)], 1).reshape(-1, 22, 3).any(2)   # codes that hold a NaN
    care = np.where(own, 0, 0xFF).astype(np.uint8)
    if mode == 1:
        care[:, 21] |= 0x0F
    d = b.descriptor(K, N, [b.WIDE], scale_mode=mode)
    got = b.quantize(torch.from_numpy(hurt).to(DEV), b.WIDE, scale_mode=mode, prefill_byte=0xFF)
    g_codes = got.codes.cpu().numpy().reshape(-1)
    bad = np.flatnonzero((g_codes ^ b.pack_codes(d, codes)) & b.pack_codes(d, care))
    assert bad.size == 0, f"{bad.size} code bytes differ, first at {bad[:5]}"
    if mode == 0:
        want = s.astype(np.float16).view(np.uint16).reshape(N, -1)
        assert np.array_equal(got.scales.cpu().numpy().view(np.uint16).reshape(-1), b.pack_scales(d, want))
    else:
        assert np.array_equal(got.ssup.cpu().numpy().view(np.uint16).reshape(-1), ssup.view(np.uint16))


def test_rejections_need_no_kernel():
    lib = b.load()
    assert lib.ccq_quantize_workspace_bytes(b.ctypes.byref(b.descriptor(512 + 32, 16, [b.NARROW]))) == -1            # K not a whole number of groups
    assert lib.ccq_quantize_workspace_bytes(b.ctypes.byref(b.descriptor(512 + 64, 16, [b.NARROW]))) == (16 * 9 * 16 + 16 * 9) * 2   # a ragged k-tile: real groups only
    assert lib.ccq_quantize_workspace_bytes(b.ctypes.byref(b.descriptor(512, 16, b.H16))) == 0                       # hybrid word: no workspace
    d = b.descriptor(512, 16, [b.NARROW])
    assert lib.ccq_quantize_workspace_bytes(b.ctypes.byref(d)) == (16 * 8 * 16 + 16 * 8) * 2
    d1 = b.descriptor(512, 16, [b.NARROW], scale_mode=1)
    assert lib.ccq_quantize_workspace_bytes(b.ctypes.byref(d1)) == (16 * 8 * 16 + 16 * 8) * 2 + 16 * 8 * 2 + 16 * 8
    assert lib.ccq_quantize(b.ctypes.byref(d), None, 512, None, None, None, None, None, None, 0, None) == -1

@pytest.mark.parametrize("fmt", ["narrow", "wide", "h16"])
def test_a_group_without_numbers(fmt):
    """64 NaN are not 64 zeros: every whole code of the group is all ones (no code is nearest) and its scale the smallest normal
    fp16 number, which a damaged checkpoint can be told by; in the narrow format the row's largest code is all ones too.
    The other groups are those of the matrix with a copy of its neighbour in the group's place."""
    N, K = 16, 704
    W = synth.weights_normal(N, K, synth.rng(30, 78))
    W[3, 64:128] = W[3, 128:192]
    hurt = W.copy()
    hurt[3, 64:128] = np.nan
    if fmt == "h16":
        codes, scales = o.h16_quantize(W)
    else:
        codes, scales, alpha, beta = o.quantize(W, o.F2 if fmt == "narrow" else o.F275)
    codes, scales = codes.copy().reshape(N, K // 64, -1), scales.copy().reshape(N, -1)
    codes[3, 1], scales[3, 1] = 0xFF, 0x0400
    care = np.full_like(codes, 0xFF)
    bf = {"narrow": b.NARROW, "wide": b.WIDE, "h16": b.H16}[fmt]
    got = b.quantize(torch.from_numpy(hurt).to(DEV), bf)
    g_scales = got.scales.cpu().numpy().view(np.uint16).reshape(-1)
    d = b.descriptor(K, N, bf if fmt == "h16" else [bf])
    want_scales = b.pack_scales(d, scales)
    if fmt == "narrow":
        care[3, :1] = care[3, 2:] = 0        # searched over the codes of another map
        assert float(got.beta.reshape(-1)[3]) == float(beta[3]) and float(got.alpha.reshape(-1)[3]) == np.float32((65535.0 - float(beta[3])) / 255.0)
        keep = b.pack_scales(d, np.where((np.arange(N) == 3)[:, None] & (np.arange(K // 64) != 1)[None], 0, 0xFFFF).astype(np.uint16))
        assert np.array_equal(g_scales & keep, want_scales & keep)
    else:
        care[3, 1, -1 if fmt == "wide" else -2:] = 0   # the last code is padded with zeros, which are numbers
        assert np.array_equal(g_scales, want_scales)
    bad = np.flatnonzero((got.codes.cpu().numpy().reshape(-1) ^ b.pack_codes(d, codes)) & b.pack_codes(d, care))
    assert bad.size == 0, f"{bad.size} code bytes differ, first at {bad[:5]}"


@pytest.mark.parametrize("fmt_name", ["narrow", "wide"])
@pytest.mark.parametrize("step", [0.0, 2.0 ** -22, 2.0 ** -12, 2.0 ** -6])
def test_scales_that_hardly_move(fmt_name, step):
    """Groups on their own grid (the least-squares scale is the first one, both errors are zero), next to it, and far from it; the last
    rows over the whole range of fp32 scales: which of two scales is the better is decided with and without the sums of errors."""
    N, K, Q = 32, 256, 31 if fmt_name == "narrow" else 7
    rng = synth.rng(31, 5)
    level = rng.integers(-Q, Q + 1, size=(N, K // 64, 64)).astype(np.float64)
    level[:, :, 0] = Q
    W = level * (1.0 + step * rng.standard_normal(level.shape)) * 2.0 ** -6
    W[N - 8:] *= 2.0 ** np.array([-140, -100, -30, -9, 9, 20, 60, 100])[:, None, None]
    _compare(fmt_name, W.reshape(N, K).astype(np.float32))
