"""The launch rules of prompts: calls whose work hardly differs take about the same time.  Ratios of the best of
interleaved runs, so that neither the card nor the host shows; each limit lies half way between what the rule gives and what
it gave when it was wrong (both stated)."""
import numpy as np
import pytest
import torch

from paper_2507_07145_amd import binding as b
from prompt_kernels import prompt_kernel

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ROW_BYTES = {"narrow": 16, "wide": 22}


def _weight(fmt, K, N, mode=0, experts=None):
    rng = np.random.default_rng([K, N, mode])
    lead = () if experts is None else (experts,)
    G = K // 64
    codes = rng.integers(0, 256, lead + (N, G * ROW_BYTES[fmt]), dtype=np.uint8)
    f = [b.NARROW if fmt == "narrow" else b.WIDE]
    al, be = np.full(lead + (N,), 100.0, np.float32), np.zeros(lead + (N,), np.float32)
    if mode == 0:
        return b.Weight.from_canonical(K, N, f, codes, np.full(lead + (N, G), 0x2000, np.uint16), al, be, device=DEV, experts=experts)
    fields = rng.integers(0, 256, lead + (N, (G + 1) // 2), dtype=np.uint8)
    return b.Weight.from_canonical_compressed(K, N, f, codes, fields, np.full(lead + (N,), 0x1800, np.uint16), al, be, device=DEV, experts=experts)


def _dense(w, M):
    x = torch.randn(M, w.K, device=DEV).to(torch.bfloat16)
    out = torch.empty(M, (w.N + 7) // 8 * 8, dtype=torch.bfloat16, device=DEV)[:, :w.N]
    ws = torch.empty(max(16, b.gemm_workspace_bytes(w.desc, M)), dtype=torch.uint8, device=DEV)
    return lambda: b.gemm(w, x, out, ws)


def _grouped(w, counts):
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    P = int(offs[-1])
    x = torch.randn(512, w.K, device=DEV).to(torch.bfloat16)
    rows = torch.randint(0, 512, (P,), dtype=torch.int32, device=DEV)
    offs_dev = torch.from_numpy(offs).to(DEV)
    out = torch.empty(P, (w.N + 7) // 8 * 8, dtype=torch.bfloat16, device=DEV)[:, :w.N]
    return lambda: b.grouped_gemm(w, x, rows, offs_dev, offs, out=out)


def _ratio(f, g, calls=10, rounds=15):
    best = [np.inf, np.inf]
    for _ in range(rounds):
        for i, h in enumerate((f, g)):
            h()
            t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            t0.record()
            for _ in range(calls):
                h()
            t1.record()
            torch.cuda.synchronize()
            best[i] = min(best[i], t0.elapsed_time(t1) * 1e3 / calls)
    print(f"{best[0]:.1f} us against {best[1]:.1f} us: {best[0] / best[1]:.3f}")
    return best[0] / best[1]


def test_uneven_experts():
    """One expert with 600 rows, fifteen with 17: 300 blocks with rows, more than one per CU.  29 us against 19 us for 64
    rows each (192 blocks); taken for 168 blocks they ran two shares to a workgroup and in two rounds, 47 us."""
    w = _weight("wide", 2048, 1536, experts=16)
    assert _ratio(_grouped(w, [600] + [17] * 15), _grouped(w, [64] * 16)) < 1.9


def test_scale_modes_alike():
    """Narrow format, 128 rows: the two scale modes do the same work.  37 us each; with the compiler after four wavefronts
    per SIMD, the one with fp16 scales waited for every LDS read by itself: 43 against 37 us."""
    K = N = 8192
    assert prompt_kernel(b.descriptor(K, N, [b.NARROW]), 128) == "64-row"
    f, g = (_dense(_weight("narrow", K, N, mode), 128) for mode in (0, 1))
    assert _ratio(f, g) < 1.08


def test_uneven_shares():
    """22 k-tiles of the wide format in sixteen shares, two to a workgroup: a workgroup has two or three of them.  17.9 us
    against 14.7 us for 16 k-tiles; with the long shares side by side, four in a workgroup, 19.9 against 15.2 us."""
    assert _ratio(_dense(_weight("wide", 11008, 1000), 64), _dense(_weight("wide", 8192, 1000), 64)) < 1.28


def test_a_few_rows_more_than_a_block():
    """Narrow format, 160 rows against 128: the block kernel's blocks of as many rows, in three shares (51 and 44 us)."""
    w = _weight("narrow", 7168, 18432)
    assert prompt_kernel(w.desc, 160) == prompt_kernel(w.desc, 128) == "block"
    assert _ratio(_dense(w, 160), _dense(w, 128)) < 1.2


def test_a_few_rows_more_than_two_blocks():
    """Narrow format, K below 512, 160 rows against 128 at 144 column blocks on the 64-row kernel: 64-row blocks, two to a CU, against 128-row ones (11.2 and
    12.6 us).  At K = 7168, with 128-row blocks, 288 of them, the 160 rows took 1.4 of the 128 rows' time."""
    w = _weight("narrow", 448, 18432)
    assert prompt_kernel(w.desc, 160) == prompt_kernel(w.desc, 128) == "64-row"
    assert _ratio(_dense(w, 160), _dense(w, 128)) < 1.2
