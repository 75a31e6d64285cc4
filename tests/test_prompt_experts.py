"""The block kernel's grouped form (csrc/ccq_block.h): experts with every count of 32-row tiles in their last block, some with none, gathered activation
rows, ragged N and K, both scale modes, against the oracle: products, and decoded weights bit for bit; eager and captured."""
import ctypes

import numpy as np
import pytest
import torch

from cases import assert_gemm_close, canon_zero
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth
from test_gpu_random_shapes import _ragged_arrays, _upload

DEV = "cuda:0"
FMTS = {"narrow": [b.NARROW], "wide": [b.WIDE], "mixed": [b.NARROW, b.WIDE], "h16": b.H16}
ONE, SOME, MANY = [31, 1, 90, 65, 0, 96, 64, 33, 128] + [97] * 11, [0, 1, 33, 65, 97, 128, 129, 64, 0] + [126] * 9, [0, 1, 32, 33, 64, 65, 96, 97, 128, 129, 300, 0]
CASES = [("narrow", 1088, 6001, MANY), ("narrow", 1088, 1909, ONE), ("wide", 576, 5365, SOME), ("wide", 576, 2805, ONE), ("mixed", 896, 3829, SOME),
         ("mixed", 896, 2421, ONE), ("h16", 576, 3189, SOME), ("h16", 576, 2037, ONE)]


def _map(family, K):
    gf = np.zeros(K // 64, dtype=np.uint8)
    gf[::3] = 1
    return gf if family == "mixed" else None


def _takes(d, counts):
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    return b.load().ccq_prompt_grouped(ctypes.byref(d), len(counts), offs.ctypes.data_as(ctypes.c_void_p))


@pytest.mark.parametrize("family,K,N,counts", CASES)
def test_cases_take_the_kernel(family, K, N, counts):
    assert _takes(b.descriptor(K, N, FMTS[family], _map(family, K)), counts) == 1


def test_other_calls_do_not():
    for K, N, counts in ((4096, 4096, [32] * 64), (448, 8192, [64] * 64), (4096, 512, [64, 64])):   # few rows, short K, too few blocks for the chip
        assert _takes(b.descriptor(K, N, b.H16), counts) == 0


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("family,K,N,counts", CASES)
def test_products_and_decoded_weights(family, K, N, counts, mode):
    gf, E, T = _map(family, K), len(counts), 210
    rng = synth.rng(93, K + N + mode)
    parts = [_ragged_arrays(family, mode, K, N, gf, rng) for _ in range(E)]
    w = _upload(family, mode, K, N, gf, parts)
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    P, ld = int(offs[-1]), (N + 7) // 8 * 8 + 8
    rows = rng.integers(0, T, size=P).astype(np.int32)
    rows[:1], rows[-1:] = T - 1, 0
    cols = np.unique(np.concatenate([np.arange(40), np.arange(N - 300, N), rng.integers(0, N, 60)]))
    hot = synth.one_hot_bf16(rng.integers(0, K, T), K)
    k_of = np.argmax(hot != 0, axis=1)
    rows_dev, offs_dev = torch.from_numpy(rows).to(DEV), torch.from_numpy(offs).to(DEV)
    for xb, exact in ((synth.activations_bf16(T, K, synth.rng(93, 1)), False), (hot, True)):
        x = b.bf16_tensor(xb, DEV)
        y = torch.full((P + 1, ld), 3.0, dtype=torch.bfloat16, device=DEV)
        b.grouped_gemm(w, x, rows_dev, offs_dev, offs, out=y[:P, :N])
        torch.cuda.synchronize()
        assert bool((y[P] == 3.0).all()) and bool((y[:, N:] == 3.0).all()), "written outside of the result"
        got = b.bf16_bits(y[:P, :N])
        for e in range(E):
            mine = slice(offs[e], offs[e + 1])
            if counts[e] == 0:
                continue
            W = parts[e]["W"]
            if exact:
                want = W.astype(np.float32).astype(np.float64) if family == "h16" and mode == 1 else W   # rounded to fp32 first there
                assert np.array_equal(canon_zero(got[mine]), canon_zero(o.to_bf16_bits(want[:, k_of[rows[mine]]].T))), f"decoded weights of expert {e} differ"
            else:
                xe = xb[rows[mine]]
                assert_gemm_close(got[mine][:, cols], o.matmul(xe, W[cols]), f"{family} K={K} N={N} mode {mode} expert {e}", rounded=(xe, W[cols]))
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
            b.grouped_gemm(w, x, rows_dev, offs_dev, offs, out=y[:P, :N], stream=side)
        for _ in range(2):
            y.fill_(1.0)
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.array_equal(b.bf16_bits(y[:P, :N]), got), "a replay differs"
