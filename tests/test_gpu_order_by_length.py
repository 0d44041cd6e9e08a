"""The grouped kernel's order by sequence length (launches of more than 256 workgroups, up to 64 sequences): a
permutation of (sequence, chunk, KV head) that every workgroup works out for itself.  Head counts that do and do not divide among
the XCDs, batches at both ends of the range and one beyond it, equal lengths, empty and full sequences, lengths that
leave chunks full, nearly full or with one key, one and many chunks; rows finished inside the launch and by a second one.  A chunk that is
done twice or not at all shows in the output, in the chunk flags or in its partial sum; everything is compared with the fp64 oracle."""
import numpy as np
import pytest

from paper_2311_01282_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


def lengths(kind, B, Smax, chunk, seed):
    rng = np.random.default_rng(seed)
    if kind == "equal":
        return [Smax] * B
    if kind == "edges":                    # around multiples of the chunk, with empty and full sequences among them
        near = [0, Smax, 1, chunk, chunk + 1, max(chunk - 1, 1), min(2 * chunk, Smax), Smax - 1]
        return [near[(i * 5 + i // 8) % 8] for i in range(B)]
    return [int(x) for x in rng.integers(0, Smax + 1, B)]


@pytest.mark.parametrize("kind", ["edges", "random", "equal"])
@pytest.mark.parametrize("B,Hq,Hkv,Smax,chunk", [
    (2, 4, 2, 4160, 64),          # 4 head groups on 8 XCDs, 65 chunks each: 520 workgroups
    (1, 14, 2, 2240, 64),         # one sequence, 2 head groups, 35 chunks
    (5, 28, 4, 700, 64),          # 20 head groups
    (33, 16, 8, 192, 64),         # 264 head groups of three chunks
    (64, 10, 5, 128, 128),        # 320 head groups of a single chunk: the most sequences
    (63, 6, 3, 256, 128),         # 189 head groups, odd head count
    (65, 16, 8, 80, 80),          # a sequence too many: the general order
    (9, 16, 1, 3600, 208),        # one KV head; a chunk of 208 keys
    (7, 4, 1, 5000, 112),         # 45 chunks
    (12, 16, 8, 512, 64),         # 768 workgroups of 8 chunks: the largest launch that finishes its rows ...
    (13, 16, 8, 512, 64),         # ... and one beyond it
    (16, 4, 2, 576, 64),          # 9 chunks
])
def test_every_chunk_once(oracle, H, B, Hq, Hkv, Smax, chunk, kind):
    lens = lengths(kind, B, Smax, chunk, 9000 + B + Smax)
    case = synth.make_case(B=B, Hq=Hq, Hkv=Hkv, D=128, Smax=Smax, seed=9100 + B + chunk, seq_lens=lens, poison_padding=True)
    nc = -(-Smax // chunk)
    assert 8 * ((B * Hkv + 7) // 8) * nc > 256
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = oracle.flags(case["q"], case["k"], case["seq_lens"], case["scale"], synth.PHI, *synth.BOUNDS, chunk, nthreads=8)
    assert margin.min() > 1e-2
    dc = H.DeviceCase(case, chunk=chunk)
    for rep in range(2):                   # (arrival counters back at zero)
        got = dc.run("fd_decode_attn_gqa")
        H.assert_close(got, want, "by length, pass %d" % rep)
        cf, rf, n, _ = dc.flags()
        assert np.array_equal(cf, ocf) and np.array_equal(rf, orf) and n == int(orf.sum())
    _, den = dc.partials()
    with_keys = np.arange(nc)[None, None, :] * chunk < np.asarray(lens)[:, None, None]
    assert np.array_equal(den > 0, np.broadcast_to(with_keys, den.shape))


def dealt(B, Hkv, Smax, chunk, lens):
    """Rounds and compute units the live chunks are dealt to, or None where they are not (chunks of less than 256 keys, up to 256 full
    ones, more than three rounds of them, more live ones than fit the rounds that the full ones need, or a launch too small for them)."""
    full = sum(n // chunk for n in lens) * Hkv
    live = full + sum(n % chunk > 0 for n in lens) * Hkv
    rounds = -(-full // 256)
    if rounds not in (2, 3) or chunk < 256:
        return None
    used = (-(-live // rounds) + 7) // 8 * 8
    grid = 8 * ((B * Hkv + 7) // 8) * -(-Smax // chunk)
    return (rounds, used) if used < 256 and 256 * (rounds - 1) + used <= grid else None


@pytest.mark.parametrize("B,Hq,Hkv,Smax,chunk,lens,want", [
    (9, 16, 8, 2048, 256, [2048, 2048, 2000, 1280, 256, 0, 1796, 1800, 516], (2, 200)),      # 360 full, 32 partial
    (11, 16, 8, 2048, 256, [2048] * 4 + [520] * 6 + [1], (2, 208)),
    (11, 16, 8, 2048, 256, [2048] * 4 + [1] * 7, None),                                      # 256 full chunks: in reverse
    (11, 16, 8, 1664, 208, [1664] * 4 + [420] * 6 + [1], None),                              # chunks of less than 256 keys
    (20, 10, 5, 1024, 256, [1024] * 13 + [40] * 7, (2, 152)),                                # 260 full of 5 heads, 35 partial
    (20, 10, 5, 1152, 288, [1152] * 18 + [577, 288], None),                                  # a launch too small to be dealt
    (8, 4, 2, 10240, 256, [10240] * 3 + [2560, 2600, 0, 1, 10239], (2, 184)),
    (64, 10, 5, 2304, 256, [2304] * 12 + [0] * 34 + [280] * 18, (3, 240)),                   # three rounds
    (64, 10, 5, 2304, 256, [2304] * 17 + [0] * 34 + [280] * 13, None),                       # 830 full: a fourth round
    (64, 10, 5, 2304, 256, [2304] * 12 + [160] * 52, None),                                  # the partial chunks make a round of their own
    (6, 28, 4, 4608, 256, [4608, 4608, 3600, 4609, 4350, 0], (2, 176)),                      # 24 head groups, the last workgroup needed; a length past the cache
    (3, 16, 8, 3200, 256, [3200, 3199, 3072], None),
])
def test_more_full_chunks_than_compute_units(oracle, H, B, Hq, Hkv, Smax, chunk, lens, want):
    inside = [min(n, Smax) for n in lens]
    assert dealt(B, Hkv, Smax, chunk, inside) == want
    case = synth.make_case(B=B, Hq=Hq, Hkv=Hkv, D=128, Smax=Smax, seed=9200 + B + Smax, seq_lens=inside, poison_padding=True)
    # (a row of an empty sequence takes no key: the next seed)
    planted = next(filter(None, (synth.plant_keys(case, 1, 36.0, seed=s, allow_shared_kv=True) for s in range(9201, 9301))))
    exact = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = oracle.flags(case["q"], case["k"], case["seq_lens"], case["scale"], synth.PHI, *synth.BOUNDS, chunk, nthreads=8)
    assert margin.min() > 1e-2 and len(planted) == 1 and orf.sum() >= 1
    case["seq_lens"] = np.asarray(lens, dtype=np.int32)
    dc = H.DeviceCase(case, chunk=chunk)
    for rep in range(2):
        H.assert_close(dc.run("fd_decode_attn_gqa"), exact, "dealt %s, pass %d" % (want, rep))
        cf, rf, n, _ = dc.flags()
        assert np.array_equal(cf, ocf) and np.array_equal(rf, orf) and n == int(orf.sum())
