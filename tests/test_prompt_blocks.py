"""The 256-row kernel: sizes that the launch rule sends to it (which the first test asks of the host code), for each of its column
blocks, with ragged row blocks, column blocks and k-tiles, in both scale modes, eagerly and captured, against the oracle."""
import ctypes

import numpy as np
import pytest
import torch

from cases import assert_gemm_close, canon_zero, random_case
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth
from test_gpu_compressed_scales import _case as compressed_case

DEV = "cuda:0"
# K, N, M, column block: whole and ragged k-tiles (320 = one tile and one group); the last row block of every case is ragged
CASES = [(256, 1536, 2900, 192), (320, 1344, 3300, 192), (256, 1024, 6000, 128), (320, 1408, 5000, 128), (256, 2056, 7100, 256),
         (320, 1001, 14000, 256)]


def block_cols(K, N, M):
    w = b.descriptor(K, N, [b.NARROW])
    return b.load().ccq_prompt_block_cols(ctypes.byref(w), M)


@pytest.mark.parametrize("K,N,M,cols", CASES)
def test_cases_take_the_column_block_they_name(K, N, M, cols):
    assert block_cols(K, N, M) == cols


@pytest.mark.parametrize("K,N,M", [(256, 1024, 3400), (256, 2064, 4000), (320, 1001, 3100), (512, 768, 300), (256, 1536, 128)])
def test_shorter_prompts_take_the_64_row_kernel(K, N, M):
    assert block_cols(K, N, M) == 0


def _weight(K, N, mode):
    if mode == 1:
        return compressed_case(["narrow"], K, N, 51)
    c = random_case(K, N, ["narrow"], 51, stream0=N % 7)
    return c.W(), c.device_weight(DEV)


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("K,N,M,cols", CASES)
def test_products_and_decoded_weights(K, N, M, cols, mode):
    W, w = _weight(K, N, mode)
    ld = (N + 7) // 8 * 8 + 8
    ks = synth.rng(51, M).integers(0, K, M)
    ks[-4:] = [0, 63, K - 64, K - 1]
    for x, exact in ((synth.activations_bf16(M, K, synth.rng(51, 1 + M)), False), (synth.one_hot_bf16(ks, K), True)):
        y = torch.full((M + 1, ld), 3.0, dtype=torch.bfloat16, device=DEV)
        b.gemm(w, b.bf16_tensor(x, DEV), out=y[:M, :N])
        torch.cuda.synchronize()
        assert bool((y[M] == 3.0).all()) and bool((y[:, N:] == 3.0).all()), "written outside of the result"
        got = b.bf16_bits(y[:M, :N])
        if exact:
            assert np.array_equal(canon_zero(got), canon_zero(o.to_bf16_bits(W[:, ks].T))), "decoded weights differ"
        else:
            assert_gemm_close(got, o.matmul(x, W), f"K={K} N={N} M={M} mode {mode}", rounded=(x, W))


@pytest.mark.gpu
@pytest.mark.parametrize("K,N,M,cols", CASES[::2])
def test_captured_call_replays_bit_exactly(K, N, M, cols):
    _, w = _weight(K, N, 0)
    xs = [b.bf16_tensor(synth.activations_bf16(M, K, synth.rng(51, 10 + i)), DEV) for i in range(2)]
    eager = [b.bf16_bits(b.gemm(w, x)).copy() for x in xs]
    x_in, y = xs[0].clone(), torch.zeros((M, N), dtype=torch.bfloat16, device=DEV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        b.gemm(w, x_in, out=y, stream=side)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            b.gemm(w, x_in, out=y, stream=side)
    torch.cuda.synchronize()
    for rep in range(4):
        x_in.copy_(xs[rep % 2])
        y.fill_(1.0)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(b.bf16_bits(y), eager[rep % 2]), f"replay {rep} differs from the eager call"
