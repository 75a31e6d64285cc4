"""The 64-row kernel (csrc/ccq_mid.hip) where its shares of K and blocks change: one to four shares in a workgroup (as many as there are
k-tiles, some of them shorter), shares in a workgroup and across the grid at once, blocks of 64 and of 128 rows with one to four row tiles
that hold rows, one and two workgroups per CU and more.  (Of the wide formats the block kernel takes some, which are named.)  Weights are exact
there, so decoded weights are held to the bit."""
import numpy as np
import pytest
import torch

from cases import assert_gemm_close, canon_zero
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth
from prompt_kernels import prompt_kernel
from test_gpu_random_shapes import _ragged_arrays, _upload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

DENSE = [
    (640, 33, 33),      # three (ragged) narrow k-tiles, two wide ones: fewer than the shares that the registers allow
    (1088, 300, 64),    # shares of unequal length
    (1088, 300, 65),
    (2112, 200, 64),    # shares across the grid too
    (2112, 200, 130),
    (576, 12000, 64),   # 94 blocks
    (576, 17000, 70),   # 266 blocks of 64 rows, 133 of 128 (three row tiles of which hold rows)
    (448, 17000, 70),
    (320, 4300, 400),   # 238 blocks of 64 rows
    (320, 9000, 500),   # more than two 64-row blocks per CU: 128-row ones, two per CU
    (128, 9000, 1300),  # more than two 128-row ones
]
BLOCK = [("wide", 1088, 300, 65), ("h16", 1088, 300, 65), ("wide", 2112, 200, 130), ("h16", 2112, 200, 130), ("h16", 576, 17000, 70)]


@pytest.mark.parametrize("K,N,M", DENSE)
@pytest.mark.parametrize("family", ["narrow", "wide", "mixed", "h16"])
@pytest.mark.parametrize("mode", [0, 1])
def test_dense(family, mode, K, N, M):
    G = K // 64
    rng = synth.rng(71, K + N + mode)
    gf = synth.group_format_map(G, max(1, G // 3), rng) if family == "mixed" else None
    a = _ragged_arrays(family, mode, K, N, gf, rng)
    w = _upload(family, mode, K, N, gf, a)
    assert prompt_kernel(w.desc, M) == ("block" if (family, K, N, M) in BLOCK else "64-row")
    x = synth.activations_bf16(M, K, synth.rng(71, M))
    ks = synth.rng(71, 9).integers(0, K, M)
    ks[:2] = [K - 1, 0]
    ld = (N + 7) // 8 * 8 + 8
    for xb in (x, synth.one_hot_bf16(ks, K)):
        y = torch.full((M + 1, ld), 3.140625, dtype=torch.bfloat16, device=DEV)
        b.gemm(w, b.bf16_tensor(xb, DEV), out=y[:M, :N])
        torch.cuda.synchronize()
        bits = b.bf16_bits(y)
        assert np.all(bits[:M, N:] == 0x4049) and np.all(bits[M] == 0x4049), "written outside the result"
        if xb is x:
            assert_gemm_close(bits[:M, :N], o.matmul(x, a["W"]), f"{family} mode {mode} K {K} N {N} M {M}", rounded=(x, a["W"]))
        else:
            assert np.array_equal(canon_zero(bits[:M, :N]), canon_zero(o.to_bf16_bits(a["W"][:, ks].T))), "decoded weights differ"


@pytest.mark.parametrize("counts", [[33, 0, 5], [200, 17, 40, 64], [70, 128, 3, 96] * 5])
@pytest.mark.parametrize("K,N", [(640, 100), (320, 2050)])
@pytest.mark.parametrize("family", ["narrow", "wide", "mixed", "h16"])
def test_grouped(family, K, N, counts):
    mode, E, T, G = (K // 64) % 2, len(counts), 60, K // 64
    rng = synth.rng(72, K + N)
    gf = synth.group_format_map(G, max(1, G // 3), rng) if family == "mixed" else None
    a = _ragged_arrays(family, mode, K, N, gf, rng)
    w = _upload(family, mode, K, N, gf, [a] * E)
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    P = int(offs[-1])
    rows = synth.rng(72, 7).integers(0, T, size=P).astype(np.int32)
    x = synth.activations_bf16(T, K, synth.rng(72, 8))
    ks = synth.rng(72, 9).integers(0, K, T)
    ld = (N + 7) // 8 * 8 + 8
    for xb in (x, synth.one_hot_bf16(ks, K)):
        y = torch.full((P + 1, ld), 3.140625, dtype=torch.bfloat16, device=DEV)
        b.grouped_gemm(w, b.bf16_tensor(xb, DEV), torch.from_numpy(rows).to(DEV), torch.from_numpy(offs).to(DEV), offs, out=y[:P, :N])
        torch.cuda.synchronize()
        bits = b.bf16_bits(y)
        assert np.all(bits[:P, N:] == 0x4049) and np.all(bits[P] == 0x4049), "written outside the result"
        if xb is x:
            assert_gemm_close(bits[:P, :N], o.matmul(x, a["W"])[rows], f"{family} K {K} N {N}", rounded=(x[rows], a["W"]))
        else:
            assert np.array_equal(canon_zero(bits[:P, :N]), canon_zero(o.to_bf16_bits(a["W"][:, ks[rows]].T))), "decoded weights differ"
