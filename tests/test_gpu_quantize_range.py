"""The range of a row's codes, which decides its Code Cluster map, from the few vectors that can have the smallest or the largest code (csrc/ccq_encode.hip):
alpha and beta bit for bit, with two, four and sixteen lanes per group, on rows whose extremes are one vector's, many vectors' alike, and
next to each other, ragged in rows and groups."""
import numpy as np
import pytest
import torch

from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _weights(kind, N, K):
    g = torch.Generator(device=DEV).manual_seed(N + K)
    W = torch.randn(N, K, generator=g, device=DEV) * 0.02
    if kind == "one sign":
        W = W.abs()
    elif kind == "band":      # all weights but each group's largest within a tenth of each other
        W = 0.01 + 0.0005 * W / 0.02
        W[:, ::64] = 0.05
    elif kind == "two values":
        W = torch.where(W > 0, 0.02, -0.015)
    elif kind == "zero groups":   # among groups of one sign: code 0 is theirs
        W = W.abs()
        W[:, 64:192] = 0.0
        W[1] = 0.0
    elif kind == "far":       # scales of no use to fp16: weights far beyond the levels, and far below the first
        W[::3] *= 1e12
        W[1::3] *= 1e-12
    return W


@pytest.mark.parametrize("N,K", [(17, 832), (273, 4160), (1033, 16448)])
@pytest.mark.parametrize("kind", ["normal", "one sign", "band", "two values", "zero groups", "far"])
def test_alpha_and_beta(kind, N, K):
    W = _weights(kind, N, K)
    got = b.quantize(W, b.NARROW)
    rows = np.unique(np.concatenate([np.arange(8), [N - 1], synth.rng(94, N).integers(0, N, 16)]))
    _, _, alpha, beta = o.quantize(np.ascontiguousarray(W[torch.from_numpy(rows).to(DEV)].cpu().numpy()), o.F2)
    assert np.array_equal(got.alpha.cpu().numpy().reshape(-1)[rows], alpha), "alpha differs"
    assert np.array_equal(got.beta.cpu().numpy().reshape(-1)[rows], beta), "beta differs"
