"""The native host path of the multiply calls (_ccq_call.so) behaves as the general Python path does around the launch."""
import ctypes

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


def test_other_threads_run_during_a_call(monkeypatch):
    """The entry points run without the interpreter lock.  CPython's own PyGILState_Check stands in for them (nothing is
    launched): it returns 0, which is CCQ_OK, only where the calling thread does not hold the lock."""
    w, we = _weight(64, 16), _weight(64, 16, experts=2)
    x = torch.zeros((4, 64), dtype=torch.bfloat16, device=DEV)
    out = torch.empty((4, 16), dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(1 << 16, dtype=torch.uint8, device=DEV)
    rows = torch.zeros(4, dtype=torch.int32, device=DEV)
    offs_host = np.array([0, 2, 4], dtype=np.int32)
    offs = torch.from_numpy(offs_host).to(DEV)
    check = ctypes.cast(ctypes.pythonapi.PyGILState_Check, ctypes.c_void_p).value
    m = b._calls()
    monkeypatch.setattr(b, "_call", None)                    # (the next call binds the library's entry points again)
    m.bind(*[check] * 5)
    try:
        got = m.gemm(w, x, out, ws), m.gemm_static(w, x, out), m.grouped_gemm(we, x, rows, offs, offs_host, out, ws)
    finally:
        b._calls()
    assert all(y is out for y in got), got
