"""The native host path of the multiply calls (_ccq_call.so) behaves as the general Python path does around the launch."""
import numpy as np
import pytest
import torch

from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _weight(K, N, experts=None):
    rng = synth.rng(11, K + N)
    lead = () if experts is None else (experts,)
    codes = rng.integers(0, 256, size=lead + (N, K // 4), dtype=np.uint8)
    scales = np.full(lead + (N, K // 64), 0x2000, dtype=np.uint16)
    alpha, beta = np.full(lead + (N,), 100.0, np.float32), np.zeros(lead + (N,), np.float32)
    return b.Weight.from_canonical(K, N, [b.NARROW], codes, scales, alpha, beta, device=DEV, experts=experts)


def test_out_of_memory_is_the_allocators_exception():
    """An output that does not fit raises torch.OutOfMemoryError, as torch.empty does (the limit is the allocator's own, set
    from here: nothing is launched)."""
    K, N, M = 64, 8192, 65536                                # an output of 1 GiB
    w, we = _weight(K, N), _weight(K, N, experts=2)
    x = torch.zeros((M, K), dtype=torch.bfloat16, device=DEV)
    rows = torch.zeros(M, dtype=torch.int32, device=DEV)
    offs_host = np.array([0, M // 2, M], dtype=np.int32)
    offs = torch.from_numpy(offs_host).to(DEV)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(0.0)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            b.gemm(w, x)
        with pytest.raises(torch.OutOfMemoryError):
            b.grouped_gemm(we, x, rows, offs, offs_host)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert b.gemm(w, x[:4]).shape == (4, N)
