"""The 64/128-row kernel at the edges of its row tiles: row counts around 32, 64, 96 and 128, through the grouped entry point
with the offsets on the host, every format, against the oracle (bf16 weights, fp32 sums: the plain bound and the
rounded-weight one of assert_gemm_close)."""
import numpy as np
import pytest
import torch

from cases import assert_gemm_close, canon_zero, grouped_rounded_weight_sigma, random_case
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth
from test_gpu_compressed_scales import _case as compressed_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("kinds,K,N,n_wide", [(["narrow"], 832, 152, None), (["wide"], 1088, 152, None), (["narrow", "wide"], 1600, 40, 9)])
@pytest.mark.parametrize("counts", [[128, 32, 1, 96], [129, 33, 64, 65], [97, 127, 31, 63], [256, 95, 0, 34]])
def test_row_tile_edges(kinds, K, N, n_wide, counts):
    E, T = len(counts), 70
    cases = [random_case(K, N, kinds, 23, stream0=10 * e, n_wide=n_wide) for e in range(E)]
    for c in cases:
        c.group_fmt = cases[0].group_fmt
    has_n = "narrow" in kinds
    w = b.Weight.from_canonical(K, N, [b.NARROW if k == "narrow" else b.WIDE for k in kinds], np.stack([c.codes for c in cases]),
                                np.stack([c.scales for c in cases]), np.stack([c.alpha for c in cases]) if has_n else None,
                                np.stack([c.beta for c in cases]) if has_n else None, cases[0].group_fmt, device=DEV, experts=E)
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    P = int(offs[-1])
    rows = synth.rng(23, 98).integers(0, T, size=P).astype(np.int32)
    ks = synth.rng(23, 97).integers(0, K, T)
    for x, exact in ((synth.activations_bf16(T, K, synth.rng(23, 99)), False), (synth.one_hot_bf16(ks, K), True)):
        y = torch.full((P + 1, (N + 7) // 8 * 8), 3.0, dtype=torch.bfloat16, device=DEV)
        b.grouped_gemm(w, b.bf16_tensor(x, DEV), torch.from_numpy(rows).to(DEV), torch.from_numpy(offs).to(DEV), offs, out=y[:P, :N])
        torch.cuda.synchronize()
        assert bool((y[P] == 3.0).all())
        got = b.bf16_bits(y[:P, :N])
        if exact:   # one-hot rows pick out decoded weights
            want = np.concatenate([o.to_bf16_bits(cases[e].W()[:, ks[rows[offs[e]:offs[e + 1]]]].T) for e in range(E) if counts[e]])
            assert np.array_equal(canon_zero(got), canon_zero(want))
        else:
            ref = np.concatenate([o.matmul(x[rows[offs[e]:offs[e + 1]]], cases[e].W()) for e in range(E) if counts[e]])
            assert_gemm_close(got, ref, f"{kinds} {counts}", rounded=grouped_rounded_weight_sigma(x, rows, offs, lambda e: cases[e].W()))


@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("M", [65, 97, 128])
def test_dense_128_row_blocks(M, mode):
    """Enough columns (209 blocks of 128, the last one ragged) for the dense product to take 128-row blocks."""
    K, N = 320, 26700
    if mode == 0:
        case = random_case(K, N, ["narrow"], 24)
        W, w = case.W(), case.device_weight(DEV)
    else:
        W, w = compressed_case(["narrow"], K, N, 24)
    x = synth.activations_bf16(M, K, synth.rng(24, M))
    y = b.gemm(w, b.bf16_tensor(x, DEV))
    assert_gemm_close(b.bf16_bits(y), o.matmul(x, W), f"M={M} mode {mode}", rounded=(x, W))


@pytest.mark.parametrize("kinds,G,n_wide", [(["wide"], 25, None), (["wide"], 16, None), (["narrow", "wide"], 40, 17), (["narrow", "wide"], 12, 2),
                                            (["wide"], 88, None), (["narrow", "wide"], 100, 44)])
def test_two_shares_in_a_workgroup(kinds, G, n_wide):
    """Few blocks on wide kinds: shares of unequal length side by side (or one, where a kind has a single k-tile); the last two
    with K cut across the grid too, 11 k-tiles in ten shares, 14 + 6 in six."""
    case = random_case(64 * G, 200, kinds, 25, n_wide=n_wide)
    w = case.device_weight(DEV)
    for M in (17, 64, 70):
        x = synth.activations_bf16(M, 64 * G, synth.rng(25, M))
        assert_gemm_close(b.bf16_bits(b.gemm(w, b.bf16_tensor(x, DEV))), o.matmul(x, case.W()), f"{kinds} G={G} M={M}", rounded=(x, case.W()))
