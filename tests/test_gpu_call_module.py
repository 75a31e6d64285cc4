"""The native host path of the multiply calls (_ccq_call.so) behaves as the general Python path does around the launch."""
import ctypes

import numpy as np
import pytest
import torch
from torch.utils._python_dispatch import TorchDispatchMode

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


class _Record(TorchDispatchMode):
    def __init__(self):
        super().__init__()
        self.seen = []

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        self.seen.append(str(func))
        return func(*args, **(kwargs or {}))


def test_a_dispatch_mode_sees_what_is_allocated():
    """Memory trackers and tensor wrappers work by a TorchDispatchMode: outputs and workspaces come through it; and a tensor
    subclass is not looked into past its own attributes."""
    w, we = _weight(1024, 1003), _weight(64, 16, experts=2)
    x = b.bf16_tensor(synth.activations_bf16(40, 1024, synth.rng(11, 1)), DEV)
    rows = torch.zeros(4, dtype=torch.int32, device=DEV)
    offs_host = np.array([0, 2, 4], dtype=np.int32)
    offs = torch.from_numpy(offs_host).to(DEV)
    assert b.gemm_workspace_bytes(w.desc, 40) > 0
    want, want_e = b.gemm(w, x), b.grouped_gemm(we, x[:4, :64], rows, offs, offs_host)
    with _Record() as r:
        y = b.gemm(w, x)
    assert sum(s.startswith("aten.empty") for s in r.seen) == 2, r.seen
    with _Record() as r:
        ye = b.grouped_gemm(we, x[:4, :64], rows, offs, offs_host)
    assert sum(s.startswith("aten.empty") for s in r.seen) >= 1, r.seen
    assert torch.equal(y, want) and torch.equal(ye, want_e)
    sub = x.as_subclass(type("Sub", (torch.Tensor,), {}))
    assert b._calls().gemm(w, sub, None, None) is None
    assert torch.equal(b.gemm(w, sub), want)
