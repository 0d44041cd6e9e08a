"""Chunks whose guard fires and go on by the synchronized scheme where they stand, without being read again: logits that leave the bounds
upwards, downwards, once and again and again, in a wavefront's first block and in the last key, in launches with and without early loads, with one
block of keys in flight, with a second launch, and with an appended key; and with bounds so wide that the chunk is redone instead.
Output against the fp64 oracle, flags bit for bit."""
import numpy as np
import pytest

from paper_2311_01282_amd import synth

pytestmark = pytest.mark.gpu
TOP = 170.0


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


def _levels(pattern, n, chunk):
    """{position: logit} for a sequence of n keys."""
    last = (n - 1) // chunk * chunk                                 # first key of the last chunk
    return {
        "first": {0: 30.0},
        "last": {n - 1: 40.0},
        "stairs": {min(11 + 37 * i, n - 1): x for i, x in enumerate([30.0, 75.0, 120.0, TOP, 60.0])},
        "falling": {min(5 + 37 * i, n - 1): x for i, x in enumerate([TOP, 120.0, 75.0, 30.0, -75.0])},
        "low": {min(3 + 64 * i, n - 1): -75.0 for i in range(4)},
        "low_start": {last + i: -75.0 for i in range(min(40, n - last))},
        "all_low": {i: -70.0 - 0.2 * (i % 50) for i in range(last, n)},
        "far_below": {i: -1000.0 - 0.2 * (i % 50) for i in range(n)},
    }[pattern]


def _plant(case, pattern, chunk):
    for b, n in enumerate(case["seq_lens"]):
        if n == 0:
            continue
        h = b % case["Hq"]                                          # one row of each sequence; the others stay as they are
        q = case["q"][b, h].astype(np.float64)
        for pos, level in _levels(pattern, int(n), chunk).items():
            case["k"][b, h, pos] = (level / (case["scale"] * (q @ q)) * q).astype(np.float16)


# (batch, heads, lengths, max_seq, chunk): early loads; one launch without; one block of keys in flight and rows beyond 32 chunks;
# a second launch, chunks of the rows dealt to the XCDs in turn or one after the other
SHAPES = [
    (2, 2, [600, 129], 600, 128),
    (1, 4, [2500], 2500, 1024),
    (9, 8, [700, 1, 127, 128, 129, 640, 641, 0, 333], 700, 128),
    (2, 3, [33 * 256, 32 * 256 + 1], 33 * 256, 256),
    (40, 4, [64 * (i % 7) + i for i in range(40)], 448, 64),
    (7, 32, [2559, 0, 2560, 2048, 511, 512, 1000], 2560, 512),
    (5, 31, [2304, 1, 2200, 2049, 300], 2304, 256),
]


@pytest.mark.parametrize("B,heads,lens,Smax,chunk", SHAPES)
@pytest.mark.parametrize("pattern", ["first", "last", "stairs", "falling", "low", "low_start", "all_low", "far_below"])
@pytest.mark.parametrize("bounds", [synth.BOUNDS, (-90.0, 70.0)])
def test_out_of_bounds(oracle, H, B, heads, lens, Smax, chunk, pattern, bounds):
    case = synth.make_case(B=B, Hq=heads, Hkv=heads, D=128, Smax=Smax, seed=9500 + Smax + B, seq_lens=lens, poison_padding=True)
    _plant(case, pattern, chunk)
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = oracle.flags(case["q"], case["k"], case["seq_lens"], case["scale"], synth.PHI, *bounds, chunk, nthreads=8)
    assert margin.min() > 1e-2
    if bounds == synth.BOUNDS:
        assert orf.sum() == np.count_nonzero(case["seq_lens"])
    dc = H.DeviceCase(case, chunk=chunk)
    for entry in ("fd_decode_attn", "fd_decode_attn", "fd_decode_attn_multikernel"):
        got = dc.run(entry, bounds=bounds)
        H.assert_close_ramp(got, want, case, (0.0, 1010.0 if pattern == "far_below" else TOP), "%s, %s, chunk %d" % (entry, pattern, chunk))
        cf, rf, n, _ = dc.flags()
        assert np.array_equal(cf, ocf) and np.array_equal(rf, orf) and n == int(orf.sum())


@pytest.mark.parametrize("lens,chunk", [([256, 300, 0], 256), ([64, 65, 127], 64), ([1024, 3, 2047], 1024)])
@pytest.mark.parametrize("level", [30.0, 80.0, -75.0, -1000.0])
def test_appended_key_out_of_bounds(oracle, H, lens, chunk, level):
    from test_gpu_append import check
    case = synth.make_case(B=3, Hq=4, Hkv=4, D=128, Smax=2 * chunk, seed=9600 + chunk, seq_lens=lens, poison_padding=True)
    k_new = np.random.default_rng(9601).standard_normal((3, 4, 128)).astype(np.float16)
    for b in range(3):
        q = case["q"][b, 1].astype(np.float64)
        k_new[b, 1] = (level / (case["scale"] * (q @ q)) * q).astype(np.float16)
    check(oracle, H, case, chunk, k_new=k_new, expect_flagged=3)


def test_a_logit_that_is_not_a_number(H, oracle):
    case = synth.make_case(B=2, Hq=4, Hkv=4, D=128, Smax=900, seed=9700, seq_lens=[900, 500])
    case["k"][0, 2, 333, 7] = np.nan
    dc = H.DeviceCase(case, chunk=128)
    got = dc.run()
    cf, rf, n, rows = dc.flags()
    assert n == 1 and list(rows) == [2] and cf[0, 2].tolist() == [0, 0, 1, 0, 0, 0, 0, 0]
    assert np.isnan(got[0, 2]).all() and np.isfinite(np.delete(got.reshape(8, 128), 2, axis=0)).all()
