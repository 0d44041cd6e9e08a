"""The synchronized scheme where query heads share KV heads (the matrix-core tile of the grouped decode kernel), against the fp64
oracle: every group size's edges, ragged and empty sequences, the launch's three orders, logits that climb, fall and lie far from zero
(the tile's scale is set anew, or far below the first one), and values that are not finite numbers, which come out as from heads of their own."""
import numpy as np
import pytest

from paper_2311_01282_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


def _check(oracle, H, case, chunk, what, ramp):
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    got = H.DeviceCase(case, chunk=chunk).run("fd_decode_attn_sync")
    if ramp is None:
        H.assert_close(got, want, what)
        return
    H.assert_close_ramp(got, want, case, ramp, what)


# (batch, query heads, KV heads, lengths, max_seq, chunk): one launch of up to 256 workgroups; more, in order of length; more than 64
# sequences, in plain order; two heads sharing one on few workgroups of 64 keys (the per-row kernel) and of 96 (the tile)
@pytest.mark.parametrize("B,Hq,Hkv,lens,Smax,chunk", [
    (4, 16, 2, [1, 15, 16, 17], 80, 64),
    (3, 16, 1, [0, 700, 64], 700, 64),
    (2, 4, 2, [300, 129], 300, 128),
    (2, 15, 3, [1024, 1009], 1024, 80),
    (1, 17, 1, [200], 200, 64),
    (1, 8, 1, [4096 + 33], 4200, 4096),
    (5, 10, 5, [3000, 1, 0, 2048, 1999], 3000, 160),
    (70, 8, 4, list(range(1, 71)), 128, 64),
    (2, 12, 2, [64 * 40, 64 * 33 + 1], 64 * 40, 64),
    (1, 2, 1, [900], 900, 64),
    (1, 2, 1, [900], 900, 96),
    # as above, in launches that the tile takes: chunks beyond 1024 keys, or more than 256 workgroups of the per-row kernel, 384 of up to 128 keys (two
    # with early loads); and the edges of that rule, on both sides
    (36, 16, 2, [1, 15, 16, 17] * 9, 80, 64),
    (3, 16, 1, [0, 700, 64], 700, 528),
    (2, 4, 2, [600, 129], 600, 528),
    (20, 15, 3, [1024 - 49 * i for i in range(20)], 1024, 80),
    (3, 12, 2, [64 * 40, 64 * 33 + 1, 700], 64 * 40, 64),
    (40, 2, 1, [900 - 23 * i for i in range(40)], 900, 64),
    (40, 2, 1, [900 - 23 * i for i in range(40)], 900, 96),
    (4, 64, 4, [500, 1, 64, 333], 500, 64),
    (4, 16, 2, [2048, 1000, 3, 512], 2048, 512),
    (4, 16, 2, [2112, 1000, 3, 512], 2112, 528),
    (1, 32, 2, [2048], 2048, 128),
    (1, 32, 2, [2049], 2049, 128),
    (2, 32, 2, [1024, 900], 1024, 64),
    (2, 32, 2, [1025, 900], 1025, 64),
    (3, 16, 1, [0, 700, 64], 700, 1040),
    (2, 4, 2, [600, 129], 600, 1040),
    (1, 8, 1, [1024], 1024, 1024),
    (16, 16, 2, [512 - 16 * i for i in range(16)], 512, 512),
    (17, 16, 2, [512 - 16 * i for i in range(17)], 512, 512),
    (2, 32, 2, [576, 300], 576, 144),
    (3, 30, 2, [432, 300, 1], 432, 144),
    (1, 32, 2, [768], 768, 64),
    (1, 32, 2, [769], 769, 64),
    (1, 32, 2, [1536], 1536, 128),
    (1, 32, 2, [1537], 1537, 128),
])
@pytest.mark.parametrize("ramp", [None, (-150.0, 150.0), (150.0, -150.0), (-900.0, -880.0), (700.0, 720.0)])
def test_grouped_rows(oracle, H, B, Hq, Hkv, lens, Smax, chunk, ramp):
    case = synth.make_case(B=B, Hq=Hq, Hkv=Hkv, D=128, Smax=Smax, seed=9300 + Hq + Smax, seq_lens=lens, poison_padding=True)
    if ramp:
        H.ramp(case, *ramp)
    _check(oracle, H, case, chunk, "%d x %d/%d, %s" % (B, Hq, Hkv, ramp), ramp)


@pytest.mark.parametrize("what", ["v_inf", "v_nan", "k_nan", "k_inf", "k_minus_inf"])
@pytest.mark.parametrize("B,chunk", [(1, 128), (1, 528), (1, 1040), (10, 128)])
def test_not_finite_as_from_heads_of_their_own(H, what, B, chunk):
    G, Hkv, Smax = 4, 3, 500
    case = synth.make_case(B=B, Hq=G * Hkv, Hkv=Hkv, D=128, Smax=Smax, seed=9400, seq_lens=[Smax] * B)
    if what[0] == "v":
        case["v"][0, 1, 77, 5] = np.inf if what == "v_inf" else np.nan
    else:
        case["q"][..., 9] = np.abs(case["q"][..., 9]) + np.float16(0.25)          # no zero times infinity
        case["k"][0, 1, 77, 9] = {"k_nan": np.nan, "k_inf": np.inf, "k_minus_inf": -np.inf}[what]
    got = H.DeviceCase(case, chunk=chunk).run("fd_decode_attn_sync")
    own = dict(case, Hkv=G * Hkv, k=np.repeat(case["k"], G, axis=1), v=np.repeat(case["v"], G, axis=1))
    want = H.DeviceCase(own, chunk=chunk).run("fd_decode_attn_sync")
    fin = np.isfinite(want)
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(got[~fin], want[~fin], equal_nan=True)
    assert np.abs(got[fin] - want[fin]).max() <= H.ABS_TOL
    assert fin.all() == (what == "k_minus_inf")


@pytest.mark.parametrize("Hq,Hkv,Smax,chunk", [(16, 2, 1000, 128), (8, 4, 2000, 256), (28, 4, 4096, 2048)])
@pytest.mark.parametrize("spread", [0.05, 1.0])
def test_partial_sums_as_exact_as_from_heads_of_their_own(H, Hq, Hkv, Smax, chunk, spread):
    """f.V of the chunks against 64 bits: no further off than the per-row kernel's, whose weights are fp32 numbers.  (With weights cut to 22 bits it is,
    by 1.3 to 1.6 times.)  Both run in a fixed order, so the two errors are what they are on every run; 5 % stands for another seed."""
    B = 10                                     # enough workgroups for the tile
    case = synth.make_case(B=B, Hq=Hq, Hkv=Hkv, D=128, Smax=Smax, seed=9450, seq_lens=[Smax] * B)
    case["q"] = (spread * case["q"].astype(np.float64)).astype(np.float16)
    k, v = (np.repeat(case[n], Hq // Hkv, axis=1) for n in "kv")
    x = np.matmul(k.astype(np.float64), case["q"].astype(np.float64)[..., None])[..., 0] * case["scale"]
    errors = []
    for c in (case, dict(case, Hkv=Hq, k=k, v=v)):
        dc = H.DeviceCase(c, chunk=chunk)
        dc.run("fd_decode_attn_sync")
        num, _ = dc.partials()
        off = size = 0.0
        for i in range(num.shape[2]):
            part = slice(i * chunk, min((i + 1) * chunk, Smax))
            w = np.exp(x[..., part] - x[..., part].max(axis=-1, keepdims=True))
            exact = np.matmul(w[..., None, :], v[:, :, part].astype(np.float64))[..., 0, :]
            off += ((num[:, :, i] - exact) ** 2).sum()
            size += (exact ** 2).sum()
        errors.append(np.sqrt(off / size))
    assert errors[0] <= 1.05 * errors[1], errors
