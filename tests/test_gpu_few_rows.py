"""The few-row kernel (csrc/ccq_few.hip): every launch shape (few_rows.CASES, whose shapes are checked on the host), second passes, ragged
last k-tiles, row tiles and blocks, shares without a k-tile, and dense calls on both sides of the lines that send them there.  Weights are
exact there, so products are held to the plain bound and decoded weights to the bit."""
import numpy as np
import pytest
import torch

import few_rows as fr
from cases import assert_gemm_close, canon_zero
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth
from test_gpu_random_shapes import _ragged_arrays, _upload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# (K, N, rows per expert); experts repeat two matrices, so that many of them cost the oracle two decodes
GROUPED = [
    (128, 17, [5, 0, 16, 2]),                                   # one (ragged) k-tile
    (320, 100, [16, 5, 0, 9]),                                  # a ragged second k-tile
    (1088, 17, [7, 12]),                                        # K shares of unequal length
    (2048, 40, [17, 3, 32, 16]),                                # two activation tiles, one of them for some experts
    (128, 2050, [5, 9, 1, 16, 0, 3, 6, 2] * 3),                 # a ragged last block
    (320, 2050, [18, 5, 31, 20, 0, 17, 6, 32]),                 # the same, two activation tiles
    (1088, 2050, [8, 5, 11, 16, 7, 9, 0, 6, 10, 5] * 3),        # several rounds of workgroups
    (640, 530, [33, 70, 8, 50]),                                # without the host copy: passes of 32 rows (with it: another kernel)
]


@pytest.mark.parametrize("K,N,counts", GROUPED)
@pytest.mark.parametrize("family", ["narrow", "wide", "mixed", "h16"])
@pytest.mark.parametrize("mode", [0, 1])
def test_grouped(family, mode, K, N, counts):
    E, T, G = len(counts), 40, K // 64
    rng = synth.rng(61, K + N + mode)
    gf = synth.group_format_map(G, max(1, G // 3), rng) if family == "mixed" else None
    two = [_ragged_arrays(family, mode, K, N, gf, rng) for _ in range(2)]
    w = _upload(family, mode, K, N, gf, [two[e % 2] for e in range(E)])
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    P = int(offs[-1])
    rows = synth.rng(61, 7).integers(0, T, size=P).astype(np.int32)
    of_row = np.repeat(np.arange(E), counts) % 2
    x = synth.activations_bf16(T, K, synth.rng(61, 8))
    ks = synth.rng(61, 9).integers(0, K, T)
    ks[:4] = [0, K - 1, K - 64, 63]
    hot = synth.one_hot_bf16(ks, K)
    ld = (N + 7) // 8 * 8 + 8
    rows_d, offs_d = torch.from_numpy(rows).to(DEV), torch.from_numpy(offs).to(DEV)
    few = max(counts) <= 32
    for host in (offs, None) if few else (None,):
        for xb in (x, hot):
            y = torch.full((P + 1, ld), 3.140625, dtype=torch.bfloat16, device=DEV)
            b.grouped_gemm(w, b.bf16_tensor(xb, DEV), rows_d, offs_d, host, out=y[:P, :N])
            torch.cuda.synchronize()
            bits = b.bf16_bits(y)
            assert np.all(bits[:P, N:] == 0x4049) and np.all(bits[P] == 0x4049), "written outside the result"
            for i in range(2):
                sel = np.nonzero(of_row == i)[0]
                if len(sel) == 0:
                    continue
                if xb is x:
                    assert_gemm_close(bits[sel, :N], o.matmul(x[rows[sel]], two[i]["W"]), f"{family} mode {mode} K {K} N {N} matrix {i}")
                else:
                    want = o.to_bf16_bits(two[i]["W"][:, ks[rows[sel]]].T)
                    assert np.array_equal(canon_zero(bits[sel, :N]), canon_zero(want)), "decoded weights differ"


@pytest.mark.parametrize("family,shape,K,N,E,top,step,host", fr.CASES)
def test_every_launch_shape(family, shape, K, N, E, top, step, host):
    counts = fr.counts(E, top, step)
    assert fr.grouped_shape(family, K, N, counts, host) == shape
    rng = synth.rng(63, K + N)
    mode, gf = (K // 64 + E) % 2, fr.group_map(family, K)
    a = _ragged_arrays(family, mode, K, N, gf, rng)
    w = _upload(family, mode, K, N, gf, [a] * E)
    offs = fr.offsets(counts)
    P, T = int(offs[-1]), 24
    rows = synth.rng(63, 7).integers(0, T, size=P).astype(np.int32)
    x = synth.activations_bf16(T, K, synth.rng(63, 8))
    ks = synth.rng(63, 9).integers(0, K, T)
    ks[:2] = [K - 1, 0]
    ld = (N + 7) // 8 * 8 + 8
    for xb in (x, synth.one_hot_bf16(ks, K)):
        y = torch.full((P + 1, ld), 3.140625, dtype=torch.bfloat16, device=DEV)
        b.grouped_gemm(w, b.bf16_tensor(xb, DEV), torch.from_numpy(rows).to(DEV), torch.from_numpy(offs).to(DEV), offs if host else None, out=y[:P, :N])
        torch.cuda.synchronize()
        bits = b.bf16_bits(y)
        assert np.all(bits[:P, N:] == 0x4049) and np.all(bits[P] == 0x4049), "written outside the result"
        if xb is x:
            assert_gemm_close(bits[:P, :N], o.matmul(x, a["W"])[rows], f"{family} mode {mode} shape {shape}")
        else:
            assert np.array_equal(canon_zero(bits[:P, :N]), canon_zero(o.to_bf16_bits(a["W"][:, ks[rows]].T))), "decoded weights differ"


@pytest.mark.parametrize("M", [2, 5, 16, 17, 32])
@pytest.mark.parametrize("K,N", [(576, 33), (1024, 1000), (1984, 300), (512, 9000), (4096, 24)])
@pytest.mark.parametrize("family", ["narrow", "wide", "mixed", "h16"])
def test_dense_calls_around_the_line(family, K, N, M):
    _dense(family, K, N, M)


@pytest.mark.parametrize("family,K,N,M,taken", fr.DENSE)
def test_dense_calls_at_the_lines(family, K, N, M, taken):
    assert fr.dense_shape(family, K, N, M)[1] == taken
    _dense(family, K, N, M)


def _dense(family, K, N, M):
    mode, G = (K // 64 + M) % 2, K // 64
    rng = synth.rng(62, K + N)
    gf = synth.group_format_map(G, max(1, G // 4), rng) if family == "mixed" else None
    a = _ragged_arrays(family, mode, K, N, gf, rng)
    w = _upload(family, mode, K, N, gf, a)
    x = synth.activations_bf16(M, K, synth.rng(62, M))
    ks = synth.rng(62, 9).integers(0, K, M)
    ks[:2] = [K - 1, 0]
    ld = (N + 7) // 8 * 8 + 8
    for xb in (x, synth.one_hot_bf16(ks, K)):
        y = torch.full((M + 1, ld), 3.140625, dtype=torch.bfloat16, device=DEV)
        b.gemm(w, b.bf16_tensor(xb, DEV), out=y[:M, :N])
        torch.cuda.synchronize()
        bits = b.bf16_bits(y)
        assert np.all(bits[:M, N:] == 0x4049) and np.all(bits[M] == 0x4049), "written outside the result"
        if xb is x:
            assert_gemm_close(bits[:M, :N], o.matmul(x, a["W"]), f"{family} mode {mode} K {K} N {N} M {M}", rounded=(x, a["W"]) if M > 16 else None)
        else:
            assert np.array_equal(canon_zero(bits[:M, :N]), canon_zero(o.to_bf16_bits(a["W"][:, ks].T))), "decoded weights differ"
