"""The 64-row kernel with one share of K to a workgroup and several k-tiles in it, the last one ragged: what products large
enough to fill the chip with blocks take (more than 256 of 64 x 128).  Wide, mixed and hybrid-word weights, both scale modes,
dense (64 rows, and a thousand, of which the block kernel takes the mixes and the hybrid words) and grouped, against the oracle: products,
and decoded weights bit for bit through one-hot rows."""
import numpy as np
import pytest
import torch

from cases import assert_gemm_close, canon_zero, grouped_rounded_weight_sigma
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth
from prompt_kernels import prompt_kernel

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N = 2200                                    # 18 column blocks, the last one ragged
SHAPES = {"wide": (1088, None), "mix": (1600, 9), "h16": (1088, None)}   # K, wide groups: 3, 4 + 2 and 3 k-tiles
FMTS = {"wide": [b.WIDE], "mix": [b.NARROW, b.WIDE], "h16": b.H16}


def _stack(fmt, mode, E, N=N):
    """E experts: device weights and the oracle's decoded weights."""
    K, n_wide = SHAPES[fmt]
    G, ofmt = K // 64, o.F275 if fmt == "wide" else (o.F2, o.F275)
    gf = synth.group_format_map(G, n_wide, synth.rng(27, 0)) if fmt == "mix" else None
    codes, scales, alpha, beta, Ws = [], [], [], [], []
    for e in range(E):
        rng = synth.rng(27, 1 + e)
        codes.append(synth.random_codes(N, o.h16_row_bytes(K) if fmt == "h16" else o.row_bytes(K, ofmt, gf), rng))
        al, be = synth.cluster_params(N, rng)
        alpha.append(al)
        beta.append(be)
        if mode == 0:
            scales.append(synth.scales_log_uniform_fp16(N, G, rng))
            Ws.append(o.h16_decode(K, N, codes[e], scales[e]) if fmt == "h16" else o.decode(K, N, ofmt, codes[e], scales[e], al, be, gf))
            continue
        sup = (o.fp16_bits_to_f64(synth.scales_log_uniform_fp16(N, 1, rng).reshape(N)) * 0.1).astype(np.float16).view(np.uint16)
        fields = rng.integers(0, 256, size=(N, 0 if fmt == "h16" else o.sq_row_bytes(K, ofmt, gf)), dtype=np.uint8)
        scales.append((fields, sup))
        Ws.append(o.h16_decode_cs(K, N, codes[e], sup) if fmt == "h16" else o.decode_cs(K, N, ofmt, codes[e], fields, sup, al, be, gf))
    ab = (np.stack(alpha), np.stack(beta)) if fmt == "mix" else (None, None)
    if mode == 0:
        w = b.Weight.from_canonical(K, N, FMTS[fmt], np.stack(codes), np.stack(scales), *ab, gf, device=DEV, experts=E)
    else:
        w = b.Weight.from_canonical_compressed(K, N, FMTS[fmt], np.stack(codes), np.stack([f for f, _ in scales]), np.stack([s for _, s in scales]), *ab, gf,
                                               device=DEV, experts=E)
    return w, Ws, K


def _want_bits(W, fp32_first):
    return canon_zero(o.to_bf16_bits(W.astype(np.float32).astype(np.float64) if fp32_first else W))


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("fmt,columns,M,kernel", [("wide", N, 1000, "64-row"), ("mix", N, 1000, "block"), ("h16", N, 1000, "block"),
                                                  ("wide", 33000, 64, "64-row"), ("mix", 33000, 64, "64-row"), ("h16", 33000, 64, "64-row")])
def test_dense(fmt, columns, M, kernel, mode):
    w, (W,), K = _stack(fmt, mode, 1, columns)
    assert prompt_kernel(w.desc, M) == kernel
    x = synth.activations_bf16(M, K, synth.rng(27, 90))
    assert_gemm_close(b.bf16_bits(b.gemm(w, b.bf16_tensor(x, DEV))), o.matmul(x, W), f"{fmt} mode {mode}", rounded=(x, W))
    ks = synth.rng(27, 91).permutation(K)[:M]
    got = b.bf16_bits(b.gemm(w, b.bf16_tensor(synth.one_hot_bf16(ks, K), DEV)))
    assert np.array_equal(canon_zero(got), _want_bits(W[:, ks].T, fmt == "h16" and mode == 1))


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("fmt", ["wide", "mix", "h16"])
def test_grouped(fmt, mode):
    counts = [130, 0, 700, 65]              # 3 + 0 + 11 + 2 row blocks
    w, Ws, K = _stack(fmt, mode, len(counts))
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    P, T = int(offs[-1]), 200
    rows = synth.rng(27, 92).integers(0, T, P).astype(np.int32)
    ks = synth.rng(27, 93).integers(0, K, T)
    for x, exact in ((synth.activations_bf16(T, K, synth.rng(27, 94)), False), (synth.one_hot_bf16(ks, K), True)):
        y = b.grouped_gemm(w, b.bf16_tensor(x, DEV), torch.from_numpy(rows).to(DEV), torch.from_numpy(offs).to(DEV), offs)
        got = b.bf16_bits(y)
        parts = [(e, rows[offs[e]:offs[e + 1]]) for e in range(len(counts)) if counts[e]]
        if exact:
            want = np.concatenate([_want_bits(Ws[e][:, ks[r]].T, fmt == "h16" and mode == 1) for e, r in parts])
            assert np.array_equal(canon_zero(got), want)
        else:
            assert_gemm_close(got, np.concatenate([o.matmul(x[r], Ws[e]) for e, r in parts]), f"{fmt} mode {mode}",
                              rounded=grouped_rounded_weight_sigma(x, rows, offs, lambda e: Ws[e]))
