"""Which launch form a shape takes: one launch that finishes its rows, or a second one that does.  Counted in a capture, so that a rule
that moves takes no test elsewhere along without being seen; and the outputs of the per-row forms on either side of every
line of the rule against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2311_01282_amd import fdattn, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


def kernels(H, entry, B, Hq, Hkv, Smax, chunk):
    """Kernels of one call; no buffer is touched, so all of them are the same few bytes."""
    shape = fdattn.make_shape(B, Hq, Hkv, 128, Smax, chunk, synth.default_scale(128))
    nbytes = fdattn.fd_workspace_bytes(shape)
    at = torch.zeros(4096, dtype=torch.uint8, device="cuda:0").data_ptr()
    return H.kernels_of(lambda s: getattr(fdattn, entry)(shape, at, at, at, at, synth.PHI, synth.BOUNDS, at, at, nbytes, s))


@pytest.mark.parametrize("B,heads,Smax,chunk,launches", [
    (1, 32, 1024, 128, 1), (1, 4, 64 * 128, 64, 1), (1, 4, 64 * 129, 64, 2),           # 128 chunks and one more
    (1, 32, 24 * 1024, 1024, 1), (1, 32, 25 * 1024, 1024, 2),                          # 320 MiB from 20480 keys; 768 workgroups and 800
    (2, 20, 20 * 512, 512, 1), (1, 64, 12 * 1024, 1024, 1), (1, 64, 13 * 1024, 1024, 2),
    (2, 12, 40 * 1024, 1024, 1), (1, 29, 33 * 1008, 1008, 1), (1, 30, 33 * 1008, 1008, 2),   # more than 32 chunks: 960, 957, 990
    (4, 32, 8 * 1024, 1024, 1), (4, 28, 9 * 1024, 1024, 2),                            # eight chunks, nine (1008 workgroups)
    (1, 32, 32 * 512, 512, 1), (1, 33, 32 * 512, 512, 2), (8, 33, 4 * 512, 512, 2),    # 1024 workgroups of eight wavefronts, more
    (8, 32, 8 * 256, 256, 1), (8, 32, 9 * 256, 256, 2), (40, 40, 8 * 128, 128, 1),     # of four, beyond 1024
    (8, 63, 8 * 64, 64, 1), (8, 64, 8 * 64, 64, 2), (8, 64, 8 * 112, 112, 2),          # 4096 of less than 128 keys
])
def test_per_row(H, B, heads, Smax, chunk, launches):
    assert kernels(H, "fd_decode_attn", B, heads, heads, Smax, chunk) == launches


@pytest.mark.parametrize("B,Hq,Hkv,Smax,chunk,launches", [
    (2, 64, 8, 16 * 512, 512, 1), (2, 32, 8, 17 * 256, 256, 2), (4, 64, 8, 8 * 256, 256, 1), (8, 16, 4, 9 * 64, 64, 2),
    (12, 16, 8, 8 * 64, 64, 1), (13, 16, 8, 8 * 64, 64, 2),
])
def test_grouped(H, B, Hq, Hkv, Smax, chunk, launches):
    assert kernels(H, "fd_decode_attn_gqa", B, Hq, Hkv, Smax, chunk) == launches


@pytest.mark.parametrize("B,Hq,Hkv,Smax,page,chunk,launches", [
    (8, 32, 32, 2048, 128, 256, 1), (8, 32, 32, 2304, 128, 256, 2), (7, 32, 32, 2560, 64, 512, 2), (12, 16, 8, 512, 16, 64, 1),
    (13, 16, 8, 512, 16, 64, 2), (9, 12, 4, 1280, 32, 128, 2), (2, 8, 8, 9216, 256, 256, 1), (40, 8, 4, 2048, 64, 64, 2),
])
def test_append_and_paged(H, B, Hq, Hkv, Smax, page, chunk, launches):
    shape = fdattn.make_shape(B, Hq, Hkv, 128, Smax, chunk, synth.default_scale(128))
    n = fdattn.fd_workspace_bytes(shape)
    at = torch.zeros(4096, dtype=torch.uint8, device="cuda:0").data_ptr()
    tail = (synth.PHI, synth.BOUNDS, at, at, n)
    for call in (lambda s: fdattn.fd_decode_attn_append(shape, at, at, at, at, at, at, *tail, s),
                 lambda s: fdattn.fd_decode_attn_paged(shape, at, at, at, at, page, 4096, at, *tail, s),
                 lambda s: fdattn.fd_decode_attn_paged_append(shape, at, at, at, at, at, at, page, 4096, at, *tail, s)):
        assert H.kernels_of(call) == launches


@pytest.mark.parametrize("B,heads,Smax,lens,chunk", [
    (8, 32, 512, [512, 1, 64, 300, 449, 511, 0, 130], 64),             # 2048 workgroups of eight chunks: in the launch
    (8, 64, 512, [512, 1, 64, 300, 449, 511, 0, 130], 64),             # 4096: a second one
    (8, 32, 2048, [2048, 1, 1793, 300, 256, 2000, 0, 1100], 256),      # 2048, eight chunks of 256
    (8, 32, 2304, [2304, 1, 1793, 300, 256, 2000, 0, 2049], 256),      # 2304, nine
    (40, 40, 1024, [1024 - 25 * i for i in range(40)], 128),           # 12800 of 128 keys, eight chunks
    (1, 64, 13312, [13312], 1024),                                     # 832 of 1024 keys over 320 MiB: a second launch
])
def test_outputs_on_either_side(oracle, H, B, heads, Smax, lens, chunk):
    case = synth.make_case(B=B, Hq=heads, Hkv=heads, D=128, Smax=Smax, seed=8800 + Smax + chunk, seq_lens=lens, poison_padding=True)
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = oracle.flags(case["q"], case["k"], case["seq_lens"], case["scale"], synth.PHI, *synth.BOUNDS, chunk, nthreads=8)
    assert margin.min() > 1e-2
    dc = H.DeviceCase(case, chunk=chunk)
    for rep in range(2):
        H.assert_close(dc.run("fd_decode_attn"), want, "pass %d" % rep)
        cf, rf, n, _ = dc.flags()
        assert np.array_equal(cf, ocf) and np.array_equal(rf, orf) and n == int(orf.sum())
