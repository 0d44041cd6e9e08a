"""Which (row, chunk) a workgroup of the per-row launches takes: every one exactly once, whatever the rows' and the chunks' numbers leave
over when divided among eight XCDs; launches with and without a hand-over, of fewer than eight rows, of one chunk after the
other, and the synchronized scheme's; against the fp64 oracle."""
import numpy as np
import pytest

from paper_2311_01282_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


@pytest.mark.parametrize("B,heads,Smax,chunk", [
    (1, 1, 64, 64), (1, 1, 33 * 64, 64), (1, 3, 40 * 64, 64), (2, 2, 129 * 64, 64), (7, 1, 70 * 96, 96),   # fewer than eight rows
    (1, 9, 5 * 64, 64), (3, 5, 130 * 64, 64),                                                              # rows that 8 does not divide
    (47, 4, 6 * 64, 64), (48, 22, 6 * 272, 272), (48, 22, 7 * 272, 272), (48, 22, 8 * 272, 272),           # 6, 7, 8 chunks
    (24, 22, 2 * 272, 272), (8, 16, 10 * 272, 272),                                                        # 2 and 10, two launches
    (2, 8, 31 * 1024, 1024), (2, 16, 34 * 1024, 1024),
])
def test_every_chunk_once(oracle, H, B, heads, Smax, chunk):
    rng = np.random.default_rng(Smax + B)
    lens = [Smax] + [int(x) for x in rng.integers(0, Smax + 1, B - 1)]
    case = synth.make_case(B=B, Hq=heads, Hkv=heads, D=128, Smax=Smax, seed=9800 + Smax + B, seq_lens=lens, poison_padding=True)
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    dc = H.DeviceCase(case, chunk=chunk)
    for entry in ("fd_decode_attn", "fd_decode_attn", "fd_decode_attn_sync"):
        H.assert_close(dc.run(entry), want, "%s, %d x %d rows of %d in %d" % (entry, B, heads, Smax, chunk))
