"""The 64-row kernel (csrc/ccq_mid.hip) past the 32-bit offsets of its lean schedule and past one launch's column blocks: activation
rows far apart (a view of one position of a long sequence has a row stride of sequence times width), and more than 65535 column blocks."""
import numpy as np
import pytest
import torch

from cases import assert_gemm_close, canon_zero
from oracle import ccq_oracle as o
from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth
from test_gpu_random_shapes import _ragged_arrays, _upload

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _far(x, ld):
    """bf16 bits [rows][K] on the device with a row stride of `ld` elements; NaN everywhere else."""
    flat = torch.full(((x.shape[0] - 1) * ld + x.shape[1],), float("nan"), dtype=torch.bfloat16, device=DEV)
    view = flat.as_strided((x.shape[0], x.shape[1]), (ld, 1))
    view.copy_(b.bf16_tensor(x, DEV))
    return view


# (K, N, M, ld): the last row of a 64-row block lies past 4 GiB from ld = 2^25 on, that of a 128-row block from 2^24
DENSE = [(640, 300, 100, 1 << 23), (1088, 300, 65, 1 << 25), (320, 12000, 70, (1 << 24) + 8), (128, 9000, 520, 1 << 23), (320, 300, 140, 1 << 24)]


@pytest.mark.parametrize("K,N,M,ld", DENSE)
@pytest.mark.parametrize("family", ["narrow", "wide", "mixed", "h16"])
def test_dense(family, K, N, M, ld):
    G, mode = K // 64, M % 2
    rng = synth.rng(81, K + N)
    gf = synth.group_format_map(G, max(1, G // 3), rng) if family == "mixed" else None
    a = _ragged_arrays(family, mode, K, N, gf, rng)
    w = _upload(family, mode, K, N, gf, a)
    x = synth.activations_bf16(M, K, synth.rng(81, M))
    y = torch.full((M + 1, (N + 7) // 8 * 8), 3.140625, dtype=torch.bfloat16, device=DEV)
    b.gemm(w, _far(x, ld), out=y[:M, :N])
    torch.cuda.synchronize()
    bits = b.bf16_bits(y)
    assert np.all(bits[M] == 0x4049), "written outside the result"
    assert_gemm_close(bits[:M, :N], o.matmul(x, a["W"]), f"{family} mode {mode} K {K} N {N} M {M} ld {ld}", rounded=(x, a["W"]))


@pytest.mark.parametrize("counts", [[40, 0, 5, 33], [70, 128, 3]])
@pytest.mark.parametrize("family", ["narrow", "wide", "mixed", "h16"])
def test_grouped(family, counts):
    K, N, T, ld, mode = 320, 530, 70, 1 << 25, len(counts) % 2
    E, G = len(counts), K // 64
    rng = synth.rng(82, E)
    gf = synth.group_format_map(G, 2, rng) if family == "mixed" else None
    a = _ragged_arrays(family, mode, K, N, gf, rng)
    w = _upload(family, mode, K, N, gf, [a] * E)
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    P = int(offs[-1])
    rows = synth.rng(82, 7).integers(0, T, size=P).astype(np.int32)
    x = synth.activations_bf16(T, K, synth.rng(82, 8))
    y = torch.full((P + 1, 536), 3.140625, dtype=torch.bfloat16, device=DEV)
    for host in (offs, None):
        b.grouped_gemm(w, _far(x, ld), torch.from_numpy(rows).to(DEV), torch.from_numpy(offs).to(DEV), host, out=y[:P, :N])
        torch.cuda.synchronize()
        bits = b.bf16_bits(y)
        assert np.all(bits[P] == 0x4049), "written outside the result"
        assert_gemm_close(bits[:P, :N], o.matmul(x, a["W"])[rows], f"{family} mode {mode}", rounded=(x[rows], a["W"]))


@pytest.mark.parametrize("family,mode", [("narrow", 0), ("narrow", 1), ("wide", 0), ("h16", 1)])
def test_more_column_blocks_than_a_grid_dimension(family, mode):
    """Rows 65535 * 128 .. of W are a second launch's.  One k-tile: the same products in the same order as of those rows alone."""
    K, M, first = 64, 34, 65535 * 128
    N = first + 300
    rng = synth.rng(83, mode)
    a = _ragged_arrays(family, mode, K, 300, None, rng)
    tail = _upload(family, mode, K, 300, None, a)

    def grown(name, align):   # the same matrix below zero rows
        t = getattr(tail, name)
        per_tile = t.numel() // (tail.info.padded_N // 16)
        big = torch.zeros(1, (first // 16) * per_tile + t.numel(), dtype=t.dtype, device=DEV)
        big[0, -t.numel():] = t.flatten()
        return big

    w = b.Weight()
    w.desc = b.descriptor(K, N, {"narrow": [b.NARROW], "wide": [b.WIDE], "h16": b.H16}[family], scale_mode=mode)
    for name, field in (("codes", "codes"), ("scales", "scales"), ("alpha", "code_alpha"), ("beta", "code_beta"), ("ssup", "scale_super")):
        if getattr(tail, name) is not None:
            setattr(w, name, grown(name, 16))
            setattr(w.desc, field, getattr(w, name).data_ptr())
    x = b.bf16_tensor(synth.activations_bf16(M, K, synth.rng(83, 8)), DEV)
    y = torch.full((M, N + 4), 3.140625, dtype=torch.bfloat16, device=DEV)
    assert N % 8 == 4
    b.gemm(w, x, out=y[:, :N])
    want = b.gemm(tail, x)
    torch.cuda.synchronize()
    assert np.array_equal(b.bf16_bits(y[:, first:N]), b.bf16_bits(want))
    assert torch.count_nonzero(y[:, :first]).item() == 0 and torch.all(y[:, N:] == 3.140625).item()
