"""Chunks whose guard fires and go on by the synchronized scheme where they stand, without being read again: logits that leave the bounds
upwards, downwards, once and again and again, in a wavefront's first block and in the last key, in launches with and without early loads, with one
block of keys in flight, with a second launch, and with an appended key; and with bounds so wide that the chunk is redone instead.
Output and the chunks' sums against fp64, flags bit for bit."""
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


def _delta(x):
    """Relative error of a per-row weight with logits up to x.  <q, k> of a key along q: four roundings in each of 16 lanes (sums of x / 16 at most),
    four levels of a tree (x / 8 .. x), the scale, the reference; the exponent's product with log2 e; up to three rescalings, with a product like that
    each: 8.2 half units in the last place of x (and of a reference that lies up to 10 further from 0).  Eight units for the exponentials."""
    return 8.25 * 2.0 ** -24 * (x + 10.0) + 2.0 ** -20


def _check_rows(dc, got, want, case, rows, chunk, cf, partials=True):
    """The rows' outputs, and their chunks' sums relative to the chunk's largest logit (flagged) or phi, each against 64 bits and within what the weights'
    errors make of it: delta times the sum of the weighted |v|.  fp32 sums add a rounding per key of a lane's column and reduction step."""
    num, den = dc.partials()
    for b, h in rows:
        n = int(case["seq_lens"][b])
        kv = h // (case["Hq"] // case["Hkv"])
        x = case["k"][b, kv, :n].astype(np.float64) @ case["q"][b, h].astype(np.float64) * case["scale"]
        v = case["v"][b, kv, :n].astype(np.float64)
        delta = _delta(np.abs(x).max()) + (chunk / 16 + 24) * 2.0 ** -24
        w = np.exp(x - x.max())
        spread = w @ np.abs(v) / w.sum()
        tol = delta * (spread + np.abs(want[b, h])) + 2.0 ** -11 * np.abs(want[b, h]) + 2.0 ** -24
        assert (np.abs(got[b, h] - want[b, h]) <= tol).all(), (b, h, np.abs(got[b, h] - want[b, h]).max())
        for c in range(-(-n // chunk) if partials else 0):
            part = slice(c * chunk, min((c + 1) * chunk, n))
            w = np.exp(x[part] - (x[part].max() if cf[b, h, c] else synth.PHI))
            assert abs(den[b, h, c] - w.sum()) <= delta * w.sum(), (b, h, c, den[b, h, c], w.sum())
            assert (np.abs(num[b, h, c] - w @ v[part]) <= delta * (w @ np.abs(v[part]))).all(), (b, h, c)


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
        cf, rf, n, _ = dc.flags()
        assert np.array_equal(cf, ocf) and np.array_equal(rf, orf) and n == int(orf.sum())
        planted = [(b, b % heads) for b in range(B) if case["seq_lens"][b]]
        # (the chain sums every chunk of a flagged row anew; its chunks are checked by their merge)
        _check_rows(dc, got, want, case, planted, chunk, cf, partials=entry == "fd_decode_attn")
        for b, h in planted:
            got[b, h] = want[b, h]
        H.assert_close(got, want, "%s, rows beside %s, chunk %d" % (entry, pattern, chunk))


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


def _by_levels(levels, heads, seed):
    """One sequence whose logits are the given numbers in every head."""
    case = synth.make_case(B=1, Hq=heads, Hkv=heads, D=128, Smax=len(levels), seed=seed)
    case["q"][...] = 0
    case["q"][..., 0] = 16.0
    case["k"][..., 0] = (np.asarray(levels) / (16.0 * case["scale"])).astype(np.float16)
    return case


def _far_apart(pattern, n):
    """Logits less phi."""
    x = np.full(n, -59.0)
    i = np.arange(n)
    if pattern == "low_chunks":                  # a chunk whose wavefronts start far below the bounds and end above the rest
        x[n // 2:3 * n // 4] = -95.0
        x[3 * n // 4:] = -57.0
    elif pattern == "low_wavefront":             # the same in some wavefronts only
        x[(i % 32 < 4) & (i < 3 * n // 4)] = -95.0
        x[(i % 32 < 4) & (i >= 3 * n // 4)] = -57.0
    elif pattern == "steps":                     # up by less than what moves a reference, again and again
        x = -100.0 + 39.0 * (i // (n // 5))
    elif pattern in ("top", "top_first"):        # sums as large as the bounds allow, then just beyond
        x[:] = 59.5
        x[n - 1 if pattern == "top" else 0] = 61.0
    elif pattern in ("bottom", "bottom_first"):
        x[:] = -63.5
        x[n - 1 if pattern == "bottom" else 0] = -65.0
    elif pattern == "top_and_bottom":            # small sums, then a chunk's largest logit, then again far below
        x[:] = -63.5
        x[n // 2] = 59.5
        x[n // 2 + 1:] = -80.0
    return x


@pytest.mark.parametrize("n,chunk", [(512, 256), (512, 64), (1024, 128), (2048, 1024), (8192, 2048), (40 * 64, 64)])
@pytest.mark.parametrize("pattern", ["low_chunks", "low_wavefront", "steps", "top", "top_first", "bottom", "bottom_first", "top_and_bottom"])
def test_references_far_apart(oracle, H, n, chunk, pattern):
    bounds, heads = (-64.0, 60.0), 3
    case = _by_levels(synth.PHI + _far_apart(pattern, n), heads, seed=9650 + n)
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = oracle.flags(case["q"], case["k"], case["seq_lens"], case["scale"], synth.PHI, *bounds, chunk, nthreads=8)
    assert margin.min() > 1e-2 and orf.all()
    dc = H.DeviceCase(case, chunk=chunk)
    for entry in ("fd_decode_attn", "fd_decode_attn_multikernel"):
        got = dc.run(entry, bounds=bounds)
        cf, rf, _, _ = dc.flags()
        assert np.array_equal(cf, ocf) and np.array_equal(rf, orf)
        _check_rows(dc, got, want, case, [(0, h) for h in range(heads)], chunk, cf, partials=entry == "fd_decode_attn")


@pytest.mark.parametrize("lens,chunk", [([256, 300, 0], 256), ([1024, 3, 2047], 1024)])
@pytest.mark.parametrize("level", [83.0, -95.0])
def test_appended_key_redone(oracle, H, lens, chunk, level):
    """Bounds too wide to go on in place: the chunk is redone, with the appended key, also one that opens its chunk."""
    from test_gpu_append import appended, run_append
    bounds = (-90.0, 70.0)
    case = synth.make_case(B=3, Hq=4, Hkv=4, D=128, Smax=2 * chunk, seed=9660 + chunk, seq_lens=lens, poison_padding=True)
    rng = np.random.default_rng(9661)
    k_new, v_new = (rng.standard_normal((3, 4, 128)).astype(np.float16) for _ in range(2))
    for b in range(3):
        q = case["q"][b, 1].astype(np.float64)
        k_new[b, 1] = (level / (case["scale"] * (q @ q)) * q).astype(np.float16)
    k2, v2, sl2 = appended(case, k_new, v_new)
    want = oracle.attn_exact(case["q"], k2, v2, sl2, case["scale"], nthreads=8)
    ocf, orf, margin = oracle.flags(case["q"], k2, sl2, case["scale"], synth.PHI, *bounds, chunk, nthreads=8)
    assert margin.min() > 1e-2 and orf.sum() == 3
    dc, got = run_append(H, case, k_new, v_new, chunk, bounds=bounds)
    assert np.array_equal(dc.k.cpu().numpy().view(np.uint16), k2.view(np.uint16))
    assert np.array_equal(dc.v.cpu().numpy().view(np.uint16), v2.view(np.uint16))
    case = dict(case, k=k2, v=v2, seq_lens=sl2)
    dc.seq_lens.copy_(dc.seq_lens.new_tensor(sl2))
    cf, rf, _, _ = dc.flags()
    assert np.array_equal(cf, ocf) and np.array_equal(rf, orf)
    H.assert_close(np.delete(got, 1, axis=1), np.delete(want, 1, axis=1), "rows beside")
    _check_rows(dc, got, want, case, [(b, 1) for b in range(3)], chunk, cf)


@pytest.mark.parametrize("page,chunk", [(64, 256), (64, 1024), (256, 2048)])
@pytest.mark.parametrize("bounds", [synth.BOUNDS, (-90.0, 70.0)])
def test_paged_redone(oracle, H, page, chunk, bounds):
    from test_gpu_paged import PagedCase
    lens = [2 * chunk, chunk + 1, chunk - 56]
    case = synth.make_case(B=3, Hq=4, Hkv=4, D=128, Smax=2 * chunk, seed=9670 + chunk, seq_lens=lens, poison_padding=True)
    _plant(case, "falling", chunk)
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = oracle.flags(case["q"], case["k"], case["seq_lens"], case["scale"], synth.PHI, *bounds, chunk, nthreads=8)
    assert margin.min() > 1e-2 and orf.sum() == 3
    pc = PagedCase(H, case, page, chunk)
    got = pc.run(bounds=bounds)
    cf, rf, _, _ = pc.dc.flags()
    assert np.array_equal(cf, ocf) and np.array_equal(rf, orf)
    _check_rows(pc.dc, got, want, case, [(b, b) for b in range(3)], chunk, cf)


def test_a_logit_that_is_not_a_number(H, oracle):
    case = synth.make_case(B=2, Hq=4, Hkv=4, D=128, Smax=900, seed=9700, seq_lens=[900, 500])
    case["k"][0, 2, 333, 7] = np.nan
    dc = H.DeviceCase(case, chunk=128)
    got = dc.run()
    cf, rf, n, rows = dc.flags()
    assert n == 1 and list(rows) == [2] and cf[0, 2].tolist() == [0, 0, 1, 0, 0, 0, 0, 0]
    assert np.isnan(got[0, 2]).all() and np.isfinite(np.delete(got.reshape(8, 128), 2, axis=0)).all()
