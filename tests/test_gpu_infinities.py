"""Infinite and very large activations in dense calls of 17 to 33 rows on the wide formats, whichever kernel takes them (a short or
wide matrix the few-row kernel up to 32 rows, otherwise the 64-row kernel; the block kernel's are in test_prompt_plans.py): an infinity gives an infinity of the weight's sign, NaN
against a zero weight, and other rows are as without it."""
import numpy as np
import pytest
import torch

from cases import assert_gemm_close
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth
from test_gpu_random_shapes import _ragged_arrays, _upload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("M", [17, 32, 33])
@pytest.mark.parametrize("K,N", [(1024, 40), (2048, 300), (1536, 9000)])   # shares of K in the workgroup; one or two row tiles per wavefront
@pytest.mark.parametrize("family", ["wide", "mixed", "h16"])
@pytest.mark.parametrize("mode", [0, 1])
def test_dense(mode, family, K, N, M):
    G = K // 64
    rng = synth.rng(91, K + mode)
    gf = None
    if family == "mixed":
        gf = np.zeros(G, np.uint8)
        gf[8:16] = 1   # whole k-tiles of both formats: padded groups would multiply the last group's activations by zero
    a = _ragged_arrays(family, mode, K, N, gf, rng)
    w = _upload(family, mode, K, N, gf, a)
    x = synth.activations_bf16(M, K, synth.rng(91, M))
    xt = b.bf16_tensor(x, DEV)
    plain = b.bf16_bits(b.gemm(w, xt))
    ks = [0, 5 * 64 + 7, 9 * 64 + 62, K - 1]        # rows of the first and of the second activation tile
    rows = [0, 3, 16, 8 if M == 17 else M - 1]
    signs = [1.0, -1.0, -1.0, 1.0]
    for m, k, s in zip(rows, ks, signs):
        xt[m, k] = s * float("inf")
    large = 7
    xt[large] = 0
    xt[large, 70] = 3e37                            # 128 times this is infinite
    got = b.gemm(w, xt).float().cpu().numpy()
    torch.cuda.synchronize()
    W = np.asarray(a["W"])
    for m, k, s in zip(rows, ks, signs):
        want = np.where(W[:, k] == 0, np.nan, np.where(s * W[:, k] > 0, np.inf, -np.inf))
        assert np.array_equal(got[m], want, equal_nan=True), (m, k)
    want = W[:, 70] * float(xt[large, 70])
    inside = np.abs(want) < 3e38                    # beyond the range of bf16: infinite
    assert np.all(np.abs(got[large] - want)[inside] <= 2.0 ** -7 * np.abs(want)[inside]) and inside.mean() > 0.5, "large activation"
    rest = [m for m in range(M) if m not in rows + [large]]
    assert_gemm_close(o.to_bf16_bits(got[rest].astype(np.float64)), o.matmul(x[rest], W), f"{family} mode {mode}", rounded=(x[rest], W))
    assert_gemm_close(plain, o.matmul(x, W), f"{family} mode {mode}, finite", rounded=(x, W))
