"""GPU parity on shapes that do not fill whole tiles of the device layout: any K that is a multiple of the group size
(Sec. 3.1: one scale per group of 64 weights), any number of output rows, any per-group format map (Sec. 3.3
"Hybrid Bits Mix").  The pack routines pad every kind to whole k-tiles and the rows to whole row tiles; the padding
must contribute nothing, its parameters must never be read out of bounds, and nothing may be written past column N
of the output.  Every number of activation rows the library distinguishes is covered, through the dense, the
allocation-free and the grouped entry points and the quantizer."""
import numpy as np
import pytest
import torch

from cases import Case, assert_gemm_close, canon_zero, random_case, grouped_rounded_weight_sigma
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ROWS = [1, 3, 8, 16, 24, 64, 130, 300]
SENTINEL = 0x4049      # bf16 3.140625


def _run(w, x_bits, ld_extra=8, entry=b.gemm):
    """The product in an output whose rows are longer than N: returns the N result columns and checks the rest untouched."""
    M, N = x_bits.shape[0], w.N
    ld = (N + 7) // 8 * 8 + ld_extra
    y = torch.full((M + 1, ld), 3.140625, dtype=torch.bfloat16, device=DEV)
    entry(w, b.bf16_tensor(x_bits, DEV), out=y[:M, :N])
    torch.cuda.synchronize()
    bits = b.bf16_bits(y)
    assert np.all(bits[:M, N:] == SENTINEL), "columns past N were written"
    assert np.all(bits[M] == SENTINEL), "a row past M was written"
    return bits[:M, :N]


def _check(case, w, M, seed, what, entry=b.gemm):
    K = case.K
    x = synth.activations_bf16(M, K, synth.rng(14, seed + M))
    W = case.W()
    assert_gemm_close(_run(w, x, entry=entry), o.matmul(x, W), f"{what} M={M}", rounded=(x, W) if M > 16 else None)
    # decoded weights, bit exact: one-hot rows at the ends of K and inside the last (ragged) k-tile of every kind
    ks = synth.rng(14, seed + 50 + M).integers(0, K, M)
    ks[:min(M, 4)] = [K - 1, 0, K - 64, 63][:min(M, 4)]
    got = _run(w, synth.one_hot_bf16(ks, K), entry=entry)
    assert np.array_equal(canon_zero(got), canon_zero(o.to_bf16_bits(W[:, ks].T))), f"{what} M={M}: decoded weights differ"


@pytest.fixture(scope="module")
def ragged_cases():
    made = {}

    def get(kinds, K, N, n_wide=None):
        key = (tuple(kinds), K, N, n_wide)
        if key not in made:
            c = random_case(K, N, kinds, 14, stream0=K % 97 + N % 13, n_wide=n_wide)
            made[key] = (c, c.device_weight(DEV))
        return made[key]
    return get


SHAPES = [(["narrow"], 7232, 1000, None),        # 113 groups: 28 k-tiles and one group; 62 row tiles and 8 rows
          (["narrow"], 1088, 1001, None),        # an odd row count: the last quad of a row is partly real
          (["wide"], 832, 1000, None),           # 13 wide groups: one k-tile of 8 and 5
          (["narrow", "wide"], 7232, 1000, 5),   # 108 narrow groups (whole tiles) and 5 wide ones
          (["narrow", "wide"], 1600, 72, 6),     # 19 narrow and 6 wide groups: both kinds ragged
          (["narrow"], 64, 8, None),             # one group, half a row tile
          (["wide"], 64, 17, None)]


@pytest.mark.parametrize("M", ROWS)
@pytest.mark.parametrize("kinds,K,N,n_wide", SHAPES)
def test_ragged_shapes_dense(ragged_cases, kinds, K, N, n_wide, M):
    c, w = ragged_cases(kinds, K, N, n_wide)
    assert w.info.padded_N == -(-N // 16) * 16
    _check(c, w, M, 100, f"ragged {kinds} K={K} N={N}")


@pytest.mark.parametrize("K,N,M", [(1088, 1000, 2900), (320, 1001, 3100), (1088, 2056, 4000)])
def test_ragged_shapes_256_row_kernel(ragged_cases, K, N, M):
    """Thousands of rows on narrow-format weights (the 64-row kernel; ragged shapes of the 256-row one are in test_prompt_blocks.py)."""
    c, w = ragged_cases(["narrow"], K, N)
    _check(c, w, M, 200, f"ragged, many rows K={K} N={N}")


def test_ragged_explicit_launch_shapes(ragged_cases):
    """K shares over workgroups and wavefronts when the k-tile count is prime (29) or the last tile is padding."""
    c, w = ragged_cases(["narrow"], 7232, 1000)
    for M, launch in [(1, (1, 1, 4, 1)), (1, (2, 1, 8, 1)), (4, (1, 2, 2, 3)), (16, (2, 2, 1, 5)), (40, (1, 4, 1, 7))]:
        x = synth.activations_bf16(M, c.K, synth.rng(14, 300 + M))
        y = b.gemm(w, b.bf16_tensor(x, DEV), launch=b.ccq_launch(*launch))
        torch.cuda.synchronize()
        assert_gemm_close(b.bf16_bits(y), o.matmul(x, c.W()), f"ragged, launch={launch} M={M}")


def test_ragged_static_entry_point(ragged_cases):
    c, w = ragged_cases(["narrow"], 7232, 1000)
    for M in (1, 8, 24):
        _check(c, w, M, 400, "ragged, ccq_gemm_static", entry=lambda w_, x_, out: b.gemm_static(w_, x_, out))


@pytest.mark.parametrize("kinds,K,N,n_wide,M", [(["narrow"], 1088, 1000, None, 1), (["narrow"], 1088, 1000, None, 8), (["narrow"], 1088, 1000, None, 70),
                                                (["narrow"], 1088, 1000, None, 2900), (["wide"], 832, 40, None, 5), (["wide"], 832, 40, None, 33),
                                                (["narrow", "wide"], 1600, 72, 6, 1), (["narrow", "wide"], 1600, 72, 6, 16),
                                                (["narrow", "wide"], 1600, 72, 6, 100)])
def test_ragged_compressed_scales(kinds, K, N, n_wide, M):
    """Scale mode 1 (Sec. 3.4): the 4-bit fields of a ragged last k-tile, and the per-row super scales of a ragged row tile."""
    fm = {"narrow": (o.F2, b.NARROW), "wide": (o.F275, b.WIDE)}
    rng = synth.rng(14, 500 + K % 11 + N % 7)
    G = K // 64
    ofmt = fm[kinds[0]][0] if len(kinds) == 1 else (o.F2, o.F275)
    gf = synth.group_format_map(G, n_wide, rng) if len(kinds) == 2 else None
    codes = synth.random_codes(N, o.row_bytes(K, ofmt, gf), rng)
    nb = o.sq_row_bytes(K, ofmt, gf)
    sq = rng.integers(0, 256, size=(N, max(nb, 1)), dtype=np.uint8)[:, :nb]
    ssup = (o.fp16_bits_to_f64(synth.scales_log_uniform_fp16(N, 1, rng).reshape(N)) * 0.1).astype(np.float16).view(np.uint16)
    alpha, beta = synth.cluster_params(N, rng)
    W = o.decode_cs(K, N, ofmt, codes, sq, ssup, alpha, beta, gf)
    w = b.Weight.from_canonical_compressed(K, N, [fm[k][1] for k in kinds], codes, sq, ssup, alpha, beta, gf, device=DEV)
    x = synth.activations_bf16(M, K, synth.rng(14, 520 + M))
    assert_gemm_close(_run(w, x), o.matmul(x, W), f"ragged, compressed scales {kinds} M={M}", rounded=(x, W) if M > 16 else None)
    ks = synth.rng(14, 530 + M).integers(0, K, M)
    ks[:min(M, 4)] = [K - 1, 0, K - 64, 63][:min(M, 4)]
    got = _run(w, synth.one_hot_bf16(ks, K))
    assert np.array_equal(canon_zero(got), canon_zero(o.to_bf16_bits(W[:, ks].T))), f"{kinds} M={M}: decoded weights differ"


@pytest.mark.parametrize("M", [1, 4, 16, 40, 100])
def test_ragged_hybrid_word(M):
    """The 16-bit word of Sec. 3.2 with 17 groups (three k-tiles of 8, the last holds one) and 40 rows."""
    K, N = 1088, 40
    codes = synth.random_codes(N, o.h16_row_bytes(K), synth.rng(14, 600))
    scales = synth.scales_log_uniform_fp16(N, K // 64, synth.rng(14, 601))
    W = o.h16_decode(K, N, codes, scales)
    w = b.Weight.from_canonical(K, N, b.H16, codes, scales, device=DEV)
    x = synth.activations_bf16(M, K, synth.rng(14, 610 + M))
    assert_gemm_close(_run(w, x), o.matmul(x, W), f"ragged hybrid word M={M}", rounded=(x, W) if M > 16 else None)
    ks = synth.rng(14, 620 + M).integers(0, K, M)
    ks[:min(M, 4)] = [K - 1, 0, K - 64, 63][:min(M, 4)]
    got = _run(w, synth.one_hot_bf16(ks, K))
    assert np.array_equal(canon_zero(got), canon_zero(o.to_bf16_bits(W[:, ks].T))), f"hybrid word M={M}: decoded weights differ"


@pytest.mark.parametrize("kinds,K,N,counts", [(["narrow"], 1088, 1000, [5, 1, 0, 17, 38]), (["narrow"], 1088, 1000, [1, 1, 0, 1, 1]),
                                              (["narrow"], 1088, 1000, [130, 0, 70, 1, 33]), (["wide"], 832, 40, [5, 1, 0, 17, 38])])
def test_ragged_grouped(kinds, K, N, counts):
    """Experts whose matrices have ragged tiles, through the grouped entry point, with and without the host offsets."""
    E, T = len(counts), 60
    cases = [random_case(K, N, kinds, 15, stream0=10 * e) for e in range(E)]
    has_n = "narrow" in kinds
    w = b.Weight.from_canonical(K, N, [b.NARROW if has_n else b.WIDE], np.stack([c.codes for c in cases]), np.stack([c.scales for c in cases]),
                                np.stack([c.alpha for c in cases]) if has_n else None, np.stack([c.beta for c in cases]) if has_n else None,
                                device=DEV, experts=E)
    x = synth.activations_bf16(T, K, synth.rng(15, 99))
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    P = int(offs[-1])
    rows = synth.rng(15, 98).integers(0, T, size=P).astype(np.int32)
    ref = np.concatenate([o.matmul(x[rows[offs[e]:offs[e + 1]]], cases[e].W()) for e in range(E) if offs[e + 1] > offs[e]])
    sigma = grouped_rounded_weight_sigma(x, rows, offs, lambda e: cases[e].W())
    for host_offsets in (offs, None):
        y = torch.full((P + 1, N + 8), 3.140625, dtype=torch.bfloat16, device=DEV)
        b.grouped_gemm(w, b.bf16_tensor(x, DEV), torch.from_numpy(rows).to(DEV), torch.from_numpy(offs).to(DEV), host_offsets, out=y[:P, :N])
        torch.cuda.synchronize()
        bits = b.bf16_bits(y)
        assert np.all(bits[:P, N:] == SENTINEL) and np.all(bits[P] == SENTINEL)
        assert_gemm_close(bits[:P, :N], ref, f"ragged grouped {kinds} {counts}, host offsets {'given' if host_offsets is not None else 'absent'}",
                          rounded=sigma)


def _dev(t, dtype=np.uint8):
    return t.cpu().numpy().view(dtype).reshape(-1)


@pytest.mark.parametrize("kinds,N,K,n_wide,mode", [(["narrow"], 40, 1088, None, 0), (["narrow"], 40, 1088, None, 1), (["wide"], 24, 832, None, 0),
                                                   (["wide"], 24, 832, None, 1), (["narrow", "wide"], 24, 1600, 6, 0),
                                                   (["narrow", "wide"], 24, 1600, 6, 1)])
def test_ragged_quantizer_matches_the_oracle(kinds, N, K, n_wide, mode):
    """ccq_quantize on padded layouts: codes, scales (or fields and super scales), alpha and beta bit for bit against
    the oracle's encoding put into device order by the pack routines (which leave the padding zero, as the quantizer
    must: the output arrays hold 0xFF bytes beforehand), then the product."""
    fm = {"narrow": (o.F2, b.NARROW), "wide": (o.F275, b.WIDE)}
    G = K // 64
    gf = synth.group_format_map(G, n_wide, synth.rng(16, 3)) if len(kinds) == 2 else None
    ofmt = fm[kinds[0]][0] if len(kinds) == 1 else (o.F2, o.F275)
    bfmt = [fm[k][1] for k in kinds]
    W = synth.weights_normal(N, K, synth.rng(16, N + K + mode))
    W[1, K - 64:] = 0.0                                               # an all-zero last group
    codes, scales, alpha, beta = o.quantize(W, ofmt, gf)
    d = b.descriptor(K, N, bfmt, gf, scale_mode=mode)
    got = b.quantize(torch.from_numpy(W).to(DEV), bfmt if len(bfmt) == 2 else bfmt[0], scale_mode=mode, group_fmt=gf, prefill_byte=0xFF)
    torch.cuda.synchronize()
    if mode == 0:
        want_codes, want_scales = b.pack_codes(d, codes), b.pack_scales(d, scales)
        Wd = o.decode(K, N, ofmt, codes, scales, alpha, beta, gf)
    else:
        c2, sq, ssup = o.compress_scales(W, ofmt, codes, scales, alpha, beta, gf)
        want_codes = b.pack_codes(d, c2)
        want_scales = b.pack_scales4(d, sq) if "narrow" in kinds else None
        assert np.array_equal(_dev(got.ssup, np.uint16)[:N], ssup), "super scales differ"
        Wd = o.decode_cs(K, N, ofmt, c2, sq, ssup, alpha, beta, gf)
    bad = np.flatnonzero(_dev(got.codes) != want_codes)
    assert bad.size == 0, f"{bad.size} code bytes differ, first at {bad[:5]}"
    if want_scales is not None:
        assert np.array_equal(_dev(got.scales, np.uint16), want_scales), "scales differ"
    if "narrow" in kinds:
        assert np.array_equal(_dev(got.alpha, np.float32)[:N], alpha) and np.array_equal(_dev(got.beta, np.float32)[:N], beta)
    for M in (2, 40):
        x = synth.activations_bf16(M, K, synth.rng(16, 79 + M))
        assert_gemm_close(_run(got, x), o.matmul(x, Wd), f"ragged quantize -> gemm M={M}", rounded=(x, Wd) if M > 16 else None)


@pytest.mark.parametrize("mode", [0, 1])
def test_ragged_quantizer_hybrid_word(mode):
    N, K = 40, 1088
    W = synth.weights_normal(N, K, synth.rng(16, 700 + mode))
    codes, scales = o.h16_quantize(W)
    ssup = None
    if mode == 1:
        codes, ssup = o.h16_compress_scales(W, codes, scales)
    d = b.descriptor(K, N, b.H16, scale_mode=mode)
    got = b.quantize(torch.from_numpy(W).to(DEV), b.H16, scale_mode=mode, prefill_byte=0xFF)
    torch.cuda.synchronize()
    bad = np.flatnonzero(_dev(got.codes) != b.pack_codes(d, codes))
    assert bad.size == 0, f"{bad.size} code bytes differ, first at {bad[:5]}"
    if mode == 0:
        assert np.array_equal(_dev(got.scales, np.uint16), b.pack_scales(d, scales)), "scales differ"
        Wd = o.h16_decode(K, N, codes, scales)
    else:
        assert np.array_equal(_dev(got.ssup, np.uint16)[:N], ssup), "super scales differ"
        Wd = o.h16_decode_cs(K, N, codes, ssup)
    x = synth.activations_bf16(3, K, synth.rng(16, 710))
    assert_gemm_close(_run(got, x), o.matmul(x, Wd), "ragged quantize (hybrid word) -> gemm")
