"""Prompts through ccq_gemm_static whose partial tiles do not fit its 8 MiB array: they have an array that holds any plan's, and are the calls that
ccq_gemm makes with its workspace, in bits and in time."""
import ctypes

import numpy as np
import pytest
import torch

from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth
from test_gpu_mid_rates import _ratio
from test_gpu_random_shapes import _ragged_arrays, _upload
from test_prompt_plans import FMTS, _map, _plan

DEV = "cuda:0"
PROMPT_ARRAY = 68 << 20   # kPromptPartialMost
# family, M, K, N: static over ccq_gemm's time with the rows in passes through 8 MiB: 6.2, 5.2, 4.9, 5.1, 6.9, 3.4
CALLS = [("wide", 512, 8192, 8192), ("narrow", 1024, 18432, 7168), ("h16", 777, 7232, 5001), ("h16", 2048, 11008, 4096), ("narrow", 256, 28672, 8192),
         ("narrow", 128, 7168, 18432)]


def test_no_plan_asks_for_more_than_the_array():
    rng = np.random.default_rng(95)
    most, array = 0, b.load().ccq_gemm_static_max_workspace()
    for _ in range(3000):
        family = ("narrow", "wide", "mixed", "h16")[int(rng.integers(4))]
        K, N, M = 64 * int(np.exp(rng.uniform(2.1, 6.2))), int(np.exp(rng.uniform(5, 10.3))), int(np.exp(rng.uniform(4.2, 10.0)))
        w = b.descriptor(K, N, FMTS[family], _map(family, K))
        partial = [S * M * (-(-count // 16) * 16) * 4 for _, count, _, S in _plan(w, M) if S > 1]
        most = max([most] + partial)
    assert array < most <= PROMPT_ARRAY


@pytest.mark.gpu
@pytest.mark.parametrize("family,M,K,N", CALLS)
def test_as_gemm(family, M, K, N):
    a = _ragged_arrays(family, 0, K, 256, None, synth.rng(95, K))
    small = _upload(family, 0, K, 256, None, a)
    w = b.Weight()   # the same 256 rows again and again
    w.desc = b.descriptor(K, N, FMTS[family])
    tiles = (N + 15) // 16
    for name, field in (("codes", "codes"), ("scales", "scales"), ("alpha", "code_alpha"), ("beta", "code_beta")):
        t = getattr(small, name)
        if t is not None:
            t = t.flatten()
            setattr(w, name, t.repeat(-(-tiles // 16))[:t.numel() // 16 * tiles].clone())
            setattr(w.desc, field, getattr(w, name).data_ptr())
    need, array = b.gemm_workspace_bytes(w.desc, M), b.load().ccq_gemm_static_max_workspace()
    assert _plan(w.desc, M) and array < need <= PROMPT_ARRAY
    x = b.bf16_tensor(synth.activations_bf16(M, K, synth.rng(95, M)), DEV)
    want, got = (torch.zeros((M, (N + 7) // 8 * 8), dtype=torch.bfloat16, device=DEV)[:, :N] for _ in range(2))
    ws = torch.empty(need, dtype=torch.uint8, device=DEV)
    ratio = _ratio(lambda: b.gemm_static(w, x, got), lambda: b.gemm(w, x, want, ws), calls=5, rounds=5)
    assert torch.equal(got, want) and torch.count_nonzero(got).item() > 0.9 * M * N
    assert ratio < 2.0


@pytest.mark.parametrize("family,M,K,N", [("mixed", 512, 8192, 2048), ("wide", 256, 8192, 5120), ("h16", 256, 4096, 4096)])
def test_what_was_refused_is_refused(family, M, K, N):
    """Prompts whose shares in the 64-row kernel alone are more than 8 MiB."""
    w = b.descriptor(K, N, FMTS[family], _map(family, K))
    assert _plan(w, M) and b.gemm_workspace_bytes(w, M) <= PROMPT_ARRAY
    assert b.load().ccq_gemm_static(ctypes.byref(w), None, M, K, None, N, None) == -5   # CCQ_ERR_WORKSPACE, before the pointers are looked at
