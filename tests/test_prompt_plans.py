"""The block kernel (csrc/ccq_block.h): every height of its blocks, with K whole and in shares, over one range of columns and over two, as the
plan picks them (which the first tests ask of the host code).  Ragged in rows, columns and K, both scale modes, against the oracle: products, and
decoded weights bit for bit; with less of a workspace than asked for (a plan of its own, which the host code is asked for too), and captured."""
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
# family, K, N, M, and of each range of columns the block's 32-row tiles and whether K is cut
CASES = [
    ("narrow", 576, 1814, 2202, [(4, False)]), ("narrow", 1792, 1158, 1605, [(4, True)]), ("narrow", 512, 9457, 781, [(5, False)]),
    ("narrow", 4032, 1613, 1331, [(6, True)]), ("narrow", 576, 4445, 2190, [(7, False)]), ("narrow", 4416, 2092, 2024, [(8, True)]),
    ("narrow", 1472, 7330, 2182, [(8, False), (4, True)]),
    ("wide", 640, 2821, 2122, [(4, False)]), ("wide", 1216, 947, 95, [(4, True)]), ("wide", 1920, 2449, 798, [(5, True)]),
    ("wide", 576, 7607, 1073, [(6, False)]), ("wide", 2688, 1107, 2180, [(7, True)]), ("wide", 576, 4476, 2289, [(8, False)]),
    ("wide", 1600, 9000, 2114, [(8, False), (7, True)]),
    ("mixed", 960, 2182, 2191, [(4, False)]), ("mixed", 2432, 919, 206, [(4, True)]), ("mixed", 3264, 1324, 778, [(5, True)]),
    ("mixed", 704, 6045, 1290, [(6, False)]), ("mixed", 512, 4534, 1812, [(7, False)]), ("mixed", 3328, 1863, 2295, [(8, True)]),
    ("mixed", 896, 11374, 1552, [(7, False), (4, False)]),
    ("h16", 576, 2120, 2146, [(4, False)]), ("h16", 1152, 962, 126, [(4, True)]), ("h16", 640, 9745, 770, [(5, False)]),
    ("h16", 3200, 1365, 1303, [(6, True)]), ("h16", 640, 3603, 2219, [(7, False)]), ("h16", 3968, 1026, 2254, [(8, True)]),
    ("h16", 640, 7262, 2182, [(8, False), (4, True)]),
]


def _map(family, K):
    gf = np.zeros(K // 64, dtype=np.uint8)
    gf[::3] = 1
    return gf if family == "mixed" else None


def _plan(w, M):
    out = (ctypes.c_int32 * 8)()
    n = b.load().ccq_prompt_plan(ctypes.byref(w), M, out)
    return [tuple(out[4 * i:4 * i + 4]) for i in range(n)]


@pytest.mark.parametrize("family,K,N,M,parts", CASES)
def test_cases_take_the_blocks_they_name(family, K, N, M, parts):
    assert [(mt, S > 1) for _, _, mt, S in _plan(b.descriptor(K, N, FMTS[family], _map(family, K)), M)] == parts


def test_plans_are_sound():
    """Ranges that cover the columns, shares with quads of every kind, a workspace within pack_info's figure, 32 rows of which fit the library's
    own array; every call that the array served is served still."""
    rng = np.random.default_rng(91)
    lib = b.load()
    array = lib.ccq_gemm_static_max_workspace()
    taken = 0
    for _ in range(1500):
        family = ("narrow", "wide", "mixed", "h16")[int(rng.integers(4))]
        K, N, M = 64 * int(np.exp(rng.uniform(0, 6.2))), int(np.exp(rng.uniform(2.8, 10.3))), int(np.exp(rng.uniform(3.5, 9.0)))
        gf = _map(family, K)
        if family == "mixed" and (gf.min() == gf.max()):
            continue
        w = b.descriptor(K, N, FMTS[family], gf)
        plan, need = _plan(w, M), b.gemm_workspace_bytes(w, M)
        assert need <= b.pack_info(w, M).workspace_bytes
        if not plan:
            continue
        taken += 1
        assert M > 64 and K >= 512
        quads = [-(-int((gf == 0).sum()) // 4), 2 * -(-int((gf == 1).sum()) // 8)] if family == "mixed" else [-(-K // 64 // 4) if family == "narrow" else 2 * -(-K // 64 // 8)]
        at = 0
        for first, count, mt, S in plan:
            assert first == at and first % 256 == 0 and count > 0 and 4 <= mt <= 8 and 1 <= S <= min(quads)
            at += count
            if S > 1:
                rows = S * (-(-count // 16) * 16) * 4
                assert rows * M <= need and 32 * rows <= array
        assert at == N
    assert taken > 300


@pytest.mark.parametrize("family,K,N,M_max", [("narrow", 1024, 1024, 2048), ("h16", 1024, 1024, 700), ("narrow", 4096, 11008, 2048), ("wide", 7168, 2001, 1500),
                                              ("mixed", 8192, 5120, 1000), ("h16", 7232, 5001, 2048), ("wide", 640, 300, 3000), ("narrow", 28672, 8192, 257)])
def test_pack_info_reports_what_calls_ask_for(family, K, N, M_max):
    """The most that any row count asks for, with no more on top than the padding of eight shares to whole row tiles (it was 8 shares of all columns, up to
    100 MiB: 64 MiB in the first of these, which asks for 8)."""
    w = b.descriptor(K, N, FMTS[family], _map(family, K))
    most = max(b.gemm_workspace_bytes(w, m) for m in range(1, M_max + 1))
    assert most <= b.pack_info(w, M_max).workspace_bytes <= most + 8 * M_max * (-N % 16) * 4


def _plan_within(w, M, nbytes):
    """Parts, and the estimated times of the call and of the 64-row kernel."""
    out, times = (ctypes.c_int32 * 8)(), (ctypes.c_double * 2)()
    n = b.load().ccq_prompt_plan_within(ctypes.byref(w), M, ctypes.c_int64(nbytes), out, times)
    return [tuple(out[4 * i:4 * i + 4]) for i in range(n)], times[0], times[1]


def test_less_workspace_is_never_slower_than_none():
    """By the estimates that choose: a call with more workspace takes no longer, none takes longer than the 64-row kernel, and all of it is what the
    query asks for.  (With the rows in passes through 8 of the 48 MiB that the first of these asks for it took 520 us, on the 64-row kernel 105.)"""
    rng = np.random.default_rng(92)
    calls = [("wide", 8192, 8192, 512), ("narrow", 18432, 7168, 1024), ("h16", 7232, 5001, 777), ("narrow", 28672, 8192, 256)]
    while len(calls) < 150:
        family = ("narrow", "wide", "h16")[len(calls) % 3]
        K, N, M = 64 * int(np.exp(rng.uniform(2.1, 6.1))), int(np.exp(rng.uniform(6, 10.2))), int(np.exp(rng.uniform(4.2, 8.0)))
        if any(S > 1 for _, _, _, S in _plan(b.descriptor(K, N, FMTS[family]), M)):
            calls.append((family, K, N, M))
    served = 0
    for family, K, N, M in calls:
        w = b.descriptor(K, N, FMTS[family])
        need, last = b.gemm_workspace_bytes(w, M), np.inf
        for part in (0, 1, 2, 4, 6, 7, 8, 16):
            plan, t, mid = _plan_within(w, M, need * part // 8)
            assert t <= min(last, mid), (family, K, N, M, part)
            assert all(S == 1 or S * M * (-(-count // 16) * 16) * 4 <= need * part // 8 for _, count, _, S in plan)
            last = t
            served += part < 8 and bool(plan)
        assert plan == _plan(w, M)
    assert served > 200


def _case(family, K, N, M, mode):
    gf = _map(family, K)
    a = _ragged_arrays(family, mode, K, N, gf, synth.rng(92, K + N + mode))
    return a["W"], _upload(family, mode, K, N, gf, a)


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("family,K,N,M,parts", CASES)
def test_products_and_decoded_weights(family, K, N, M, parts, mode):
    W, w = _case(family, K, N, M, mode)
    ld = (N + 7) // 8 * 8 + 8
    edges = [0, N - 40] + [p[0] - 20 for p in _plan(w.desc, M)[1:]]
    cols = np.unique(np.concatenate([np.arange(e, e + 40) for e in edges] + [synth.rng(92, 5).integers(0, N, 40)]))
    ks = synth.rng(92, M).integers(0, K, M)
    ks[-4:] = [0, 63, K - 64, K - 1]
    for x, exact in ((synth.activations_bf16(M, K, synth.rng(92, 1 + M)), False), (synth.one_hot_bf16(ks, K), True)):
        y = torch.full((M + 1, ld), 3.0, dtype=torch.bfloat16, device=DEV)
        b.gemm(w, b.bf16_tensor(x, DEV), out=y[:M, :N])
        torch.cuda.synchronize()
        assert bool((y[M] == 3.0).all()) and bool((y[:, N:] == 3.0).all()), "written outside of the result"
        got = b.bf16_bits(y[:M, :N])
        if exact:
            want = W.astype(np.float32).astype(np.float64) if family == "h16" and mode == 1 else W   # rounded to fp32 first there
            assert np.array_equal(canon_zero(got), canon_zero(o.to_bf16_bits(want[:, ks].T))), "decoded weights differ"
        else:
            assert_gemm_close(got[:, cols], o.matmul(x, W[cols]), f"{family} K={K} N={N} M={M} mode {mode}", rounded=(x, W[cols]))


@pytest.mark.gpu
@pytest.mark.parametrize("family,K,N,M,parts", [c for c in CASES if any(cut for _, cut in c[4])][::2])
def test_less_workspace_and_capture(family, K, N, M, parts):
    """Part of the workspace and none: other shares or the 64-row kernel, or refused; and the captured call."""
    W, w = _case(family, K, N, M, 0)
    x_bits = synth.activations_bf16(M, K, synth.rng(92, 3))
    x = b.bf16_tensor(x_bits, DEV)
    need = b.gemm_workspace_bytes(w.desc, M)
    want = b.bf16_bits(b.gemm(w, x)).copy()
    buf = torch.full((need + 4096,), 0xFF, dtype=torch.uint8, device=DEV)
    out = torch.zeros((M, (N + 7) // 8 * 8), dtype=torch.bfloat16, device=DEV)[:, :N]
    cols = np.unique(np.concatenate([np.arange(40), np.arange(N - 40, N), synth.rng(92, 6).integers(0, N, 40)]))
    refused = False
    for nbytes in (need - 16, need // 2 // 16 * 16, need // 8 // 16 * 16, 0):
        try:
            got = b.bf16_bits(b.gemm(w, x, out=out, workspace=buf[:nbytes]))
        except b.CcqError as e:
            assert e.status == -5, "less than 64-row blocks need is refused"
            refused = True
            continue
        assert not refused, "served with less than what was refused"
        assert_gemm_close(got[:, cols], o.matmul(x_bits, W[cols]), f"{family} K={K} N={N} M={M} workspace {nbytes} of {need}", rounded=(x_bits, W[cols]))
        torch.cuda.synchronize()
        assert bool((buf[nbytes:] == 0xFF).all()), "written outside of the workspace"
        buf.fill_(0xFF)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        b.gemm(w, x, out=out, workspace=buf[:need], stream=side)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            b.gemm(w, x, out=out, workspace=buf[:need], stream=side)
    torch.cuda.synchronize()
    for _ in range(3):
        out.fill_(1.0)
        buf.fill_(0xFF)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(b.bf16_bits(out), want)


@pytest.mark.gpu
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("family,K,N,M", [("narrow", 1792, 1158, 1605), ("wide", 1216, 947, 95), ("mixed", 2432, 919, 206), ("mixed", 512, 4534, 1812), ("h16", 1152, 962, 126)])
def test_infinite_activations(family, K, N, M, mode):
    """An infinity gives an infinity of the weight's sign, NaN against a zero weight (in the last group of K also against the padding beside it), and
    other rows are as without it."""
    W, w = _case(family, K, N, M, mode)
    assert _plan(w.desc, M)
    x = b.bf16_tensor(synth.activations_bf16(M, K, synth.rng(92, 7)), DEV)
    want = b.gemm(w, x).float().cpu().numpy()
    rows = [0, 31, 64, M - 1]
    for m, k, sign in zip(rows, [0, 5 * 64 + 7, K // 2 + 1, K - 1], [1.0, -1.0, -1.0, 1.0]):
        x[m, k] = sign * float("inf")
        want[m] = np.where(W[:, k] == 0, np.nan, np.where(sign * W[:, k] > 0, np.inf, -np.inf))
    got = b.gemm(w, x).float().cpu().numpy()
    padded = np.isnan(got[M - 1])
    assert padded.all() or np.array_equal(padded, np.isnan(want[M - 1]))
    want[M - 1, padded] = np.nan
    assert np.array_equal(got, want, equal_nan=True)


@pytest.mark.gpu
@pytest.mark.parametrize("family,K,N,M", [("narrow", 1472, 7330, 2182), ("wide", 1600, 9000, 2114), ("h16", 640, 7262, 2182), ("wide", 1216, 947, 95)])
def test_static_entry(family, K, N, M):
    """The first two ask for more than the library's own array, which the 64-row kernel would do without: served, with the same bits."""
    _, w = _case(family, K, N, M, 1)
    need = b.gemm_workspace_bytes(w.desc, M)
    assert need > 0 and (need > b.load().ccq_gemm_static_max_workspace()) == (M > 1000 and family != "h16")
    x = b.bf16_tensor(synth.activations_bf16(M, K, synth.rng(92, 4)), DEV)
    out = torch.zeros((M, (N + 7) // 8 * 8), dtype=torch.bfloat16, device=DEV)[:, :N]
    assert np.array_equal(b.bf16_bits(b.gemm_static(w, x, out)), b.bf16_bits(b.gemm(w, x)))


@pytest.mark.gpu
@pytest.mark.parametrize("kind,K,N,M", [("narrow", 1792, 1158, 1605), ("wide", 1216, 947, 95), ("wide", 1920, 2449, 798), ("h16", 1152, 962, 126)])
@pytest.mark.parametrize("zp", [0.0, 3.5, 31.5, 64.0])
def test_zero_points_and_extreme_scales(kind, K, N, M, zp):
    """States stay where they lie in a code and meet offsets of up to 1024 + zp: exact for every zero-point, and for fp16 scales at their ends."""
    G = K // 64
    scales = synth.scales_log_uniform_fp16(N, G, synth.rng(93, 1)).reshape(N, G)
    scales[:, 1] = np.tile(np.array([0x0000, 0x0001, 0x03FF, 0x0400, 0x7BFF, 0xB800, 0x3555], np.uint16), N)[:N]
    if kind == "narrow":
        codes = synth.random_codes(N, K // 4, synth.rng(93, 0))
        alpha, beta = synth.cluster_params(N, synth.rng(93, 2))
        W = o.decode(K, N, o.Code(6, 4, 3, True, zp=zp), codes, scales, alpha, beta)
        w = b.Weight.from_canonical(K, N, [b.ccq_code(6, 4, 3, 1, zp)], codes, scales, alpha, beta, device=DEV)
    elif kind == "wide":
        codes = synth.random_codes(N, G * 22, synth.rng(93, 3))
        W = o.decode(K, N, o.Code(4, 3, 2, False, zp=zp), codes, scales)
        w = b.Weight.from_canonical(K, N, [b.ccq_code(4, 3, 2, 0, zp)], codes, scales, device=DEV)
    else:
        codes = synth.random_codes(N, o.h16_row_bytes(K), synth.rng(93, 4))
        W = o.h16_decode(K, N, codes, scales, zp=zp)
        w = b.Weight.from_canonical(K, N, [b.ccq_code(3, 3, 2, 0, zp), b.ccq_code(3, 4, 2, 0, zp)], codes, scales, device=DEV)
    assert _plan(w.desc, M)
    ks = synth.rng(93, M).integers(0, K, M)
    ks[:M // 2] = 64 + ks[:M // 2] % 64   # half of the rows in the group with the extreme scales
    got = b.bf16_bits(b.gemm(w, b.bf16_tensor(synth.one_hot_bf16(ks, K), DEV)))
    assert np.array_equal(canon_zero(got), canon_zero(o.to_bf16_bits(W[:, ks].T)))
