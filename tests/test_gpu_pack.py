"""The permutation to device order on the GPU gives the bytes of the host routines, padding included: every format and
scale mode, row and k-tile remainders, group maps with one kind only, stacks that go up in several parts, read-only arrays."""
import numpy as np
import pytest

from paper_2507_07145_amd import binding as b
from paper_2507_07145_amd import synth

pytestmark = pytest.mark.gpu

GROUP_BYTES = {"narrow": 16, "wide": 22, "h16": 20}
FMTS = {"narrow": [b.NARROW], "wide": [b.WIDE], "h16": b.H16, "mix": [b.NARROW, b.WIDE]}


@pytest.mark.parametrize("K,N,E", [(64, 1, 1), (256, 16, 1), (832, 33, 3), (512, 17, 2), (4096, 272, 1)])
@pytest.mark.parametrize("fmt,n_wide", [("narrow", 0), ("wide", 0), ("h16", 0), ("mix", 0), ("mix", 1), ("mix", 5), ("mix", -1)])
@pytest.mark.parametrize("mode", [0, 1])
def test_device_permutation_is_the_hosts(K, N, E, fmt, n_wide, mode, monkeypatch):
    G, gf = K // 64, None
    if fmt == "mix":
        n_wide = G if n_wide < 0 else min(n_wide, G)
        gf = synth.group_format_map(G, n_wide, synth.rng(91, G))
        row = (G - n_wide) * 16 + n_wide * 22
    else:
        row = G * GROUP_BYTES[fmt]
    narrow = {"narrow": G, "mix": G - n_wide}.get(fmt, 0)
    rng = np.random.default_rng([K, N, E, mode])
    codes = rng.integers(0, 256, (E, N, row), dtype=np.uint8)
    codes.setflags(write=False)
    alpha = np.ones((E, N), np.float32)
    d = b.descriptor(K, N, FMTS[fmt], gf, scale_mode=mode)
    monkeypatch.setattr(b, "_PACK_CHUNK_BYTES", 2 * N * row)     # two experts at a time
    monkeypatch.setattr(b, "_PACK_HOST_BYTES", 0)                # small ones too
    if mode == 0:
        scales = rng.integers(0, 65536, (E, N, G), dtype=np.uint16)
        w = b.Weight.from_canonical(K, N, FMTS[fmt], codes, scales, alpha, alpha, gf, experts=E)
        want = [b.pack_scales(d, scales[e]) for e in range(E)]
    else:
        fields = rng.integers(0, 256, (E, N, (narrow + 1) // 2), dtype=np.uint8)
        w = b.Weight.from_canonical_compressed(K, N, FMTS[fmt], codes, fields, np.ones((E, N), np.uint16), alpha, alpha, gf, experts=E)
        want = [b.pack_scales4(d, fields[e]) for e in range(E)]
    assert np.array_equal(w.codes.cpu().numpy(), np.stack([b.pack_codes(d, codes[e]) for e in range(E)]))
    if w.scales is None:
        assert mode == 1 and narrow == 0
    else:
        assert np.array_equal(w.scales.cpu().numpy().view(np.uint16), np.stack(want))


@pytest.mark.parametrize("K,N,E,on_device", [(64, 16, 1, False), (512, 256, 1, False), (576, 256, 1, True), (64, 16, 2, True)])
def test_a_small_matrix_is_permuted_on_the_host(K, N, E, on_device, monkeypatch):
    """One matrix of up to 32 KiB of codes takes less time on the host; the bytes are the same."""
    codes = np.random.default_rng(5).integers(0, 256, (E, N, K // 4), dtype=np.uint8)
    scales, ab = np.full((E, N, K // 64), 0x2000, np.uint16), np.ones((E, N), np.float32)
    real, seen = b.load(), []

    class Lib:
        def __getattr__(self, name):
            seen.append(name)
            return getattr(real, name)

    monkeypatch.setattr(b, "load", lambda lib=Lib(): lib)
    w = b.Weight.from_canonical(K, N, [b.NARROW], codes, scales, ab, ab, experts=E)
    assert ("ccq_pack_device" in seen) == on_device
    d = b.descriptor(K, N, [b.NARROW])
    assert np.array_equal(w.codes.cpu().numpy(), np.stack([b.pack_codes(d, c) for c in codes]))
    assert np.array_equal(w.scales.cpu().numpy().view(np.uint16), np.stack([b.pack_scales(d, c) for c in scales]))
