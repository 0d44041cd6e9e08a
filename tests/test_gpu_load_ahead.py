"""Chunks of 256 to 1024 keys whose wavefronts ask for one block of keys at a time, in rows of more than 32 chunks and in launches of more
than three workgroups per compute unit that leave the rows to a second one (elsewhere they ask for two): lengths that leave the last chunk with one key, one to all blocks (of 64 or 128 keys), odd and even counts of them; the last chunk count
without the rule and the first with it; recomputed chunks; the fused call, its chunk kernel alone and the chain of launches."""
import numpy as np
import pytest

from paper_2311_01282_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


@pytest.mark.parametrize("chunk,nc", [(256, 32), (256, 33), (256, 40), (512, 33), (208, 41), (1024, 33), (752, 35)])
@pytest.mark.parametrize("plant", [0, 2])
def test_one_block_at_a_time(oracle, H, chunk, nc, plant):
    tails = [1, 60, 65, 129, 193, 257, 385, 513, 641, 769, 897, chunk]
    lens = [(nc - 1) * chunk + t for t in tails if t <= chunk][-4:] + [5 * chunk + 70, 3]
    B, heads, Smax = len(lens), 2, nc * chunk
    case = synth.make_case(B=B, Hq=heads, Hkv=heads, D=128, Smax=Smax, seed=8600 + Smax + nc, seq_lens=lens, poison_padding=True)
    planted = synth.plant_keys(case, plant, 36.0, seed=8601 + Smax) if plant else []
    assert len(planted) == plant
    assert 8 * ((B * heads + 7) // 8) * nc > 256           # beyond the launches with early loads
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = oracle.flags(case["q"], case["k"], case["seq_lens"], case["scale"], synth.PHI, *synth.BOUNDS, chunk, nthreads=8)
    assert margin.min() > 1e-2
    dc = H.DeviceCase(case, chunk=chunk)
    for entry in ("fd_decode_attn", "fd_decode_attn", "fd_decode_attn_multikernel"):
        got = dc.run(entry)
        H.assert_close(got, want, "%s, %d chunks of %d" % (entry, nc, chunk))
        cf, rf, n, _ = dc.flags()
        assert np.array_equal(cf, ocf) and np.array_equal(rf, orf) and n == int(orf.sum())


@pytest.mark.parametrize("B,heads,chunk,nc", [(5, 31, 256, 9), (12, 8, 512, 11), (8, 14, 752, 9), (8, 15, 1024, 9)])
def test_one_block_at_a_time_in_a_large_launch(oracle, H, B, heads, chunk, nc):
    tails = [1, 65, 129, 193, 385, 513, 641, 897, chunk]
    lens = [(nc - 1) * chunk + min(tails[i % len(tails)], chunk) - (chunk * (i // 5)) for i in range(B - 1)] + [0]
    case = synth.make_case(B=B, Hq=heads, Hkv=heads, D=128, Smax=nc * chunk, seed=8700 + nc * chunk, seq_lens=lens, poison_padding=True)
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    dc = H.DeviceCase(case, chunk=chunk)
    for entry in ("fd_decode_attn", "fd_decode_attn_multikernel"):
        H.assert_close(dc.run(entry), want, "%s, %d x %d rows, %d chunks of %d" % (entry, B, heads, nc, chunk))
    dc.out.fill_(float("nan"))
    dc.run_partial()
    num, den = dc.partials()
    with np.errstate(invalid="ignore"):
        got = np.where(den.sum(-1, keepdims=True) > 0, num.astype(np.float64).sum(2) / den.astype(np.float64).sum(-1, keepdims=True), 0.0)
    H.assert_close(got, want, "the chunk kernel alone")
