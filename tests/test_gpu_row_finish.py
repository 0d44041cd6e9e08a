"""The finish of a row by one wavefront of its last workgroup: chunk counts on either side of every block size (4, 8, 16,
32 chunks to a memory round trip, then several), rows with and without a recomputed chunk, the largest chunk count that is
finished inside the launch and the first that is not, and launches of more than 1024 workgroups of four wavefronts.
Every element, every flag, twice in a row (the arrival counters must be back at zero), against the fp64 oracle with the
suite's tolerance."""
import numpy as np
import pytest

from paper_2311_01282_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


def check(oracle, H, B, heads, Smax, lens, chunk, plant):
    case = synth.make_case(B=B, Hq=heads, Hkv=heads, D=128, Smax=Smax, seed=7100 + Smax + chunk, seq_lens=lens, poison_padding=True)
    planted = synth.plant_keys(case, plant, 36.0, seed=7101 + Smax) if plant else []
    assert len(planted) == plant
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = oracle.flags(case["q"], case["k"], case["seq_lens"], case["scale"], synth.PHI, *synth.BOUNDS, chunk, nthreads=8)
    assert margin.min() > 1e-2 and int(orf.sum()) >= plant
    dc = H.DeviceCase(case, chunk=chunk)
    for rep in range(2):
        got = dc.run("fd_decode_attn")
        H.assert_close(got, want, "%d chunks per row, pass %d" % (-(-Smax // chunk), rep))
        cf, rf, n, _ = dc.flags()
        assert np.array_equal(cf, ocf) and np.array_equal(rf, orf) and n == int(orf.sum())


@pytest.mark.parametrize("plant", [0, 2])
@pytest.mark.parametrize("nb", [1, 2, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 128, 129])
def test_row_of_nb_chunks(oracle, H, nb, plant):
    check(oracle, H, 2, 4, 64 * nb, [64 * nb - 3, 64 * ((nb + 1) // 2)], 64, plant)


@pytest.mark.parametrize("B,heads,Smax,lens,chunk", [
    (8, 32, 512, [512, 1, 300, 449, 2, 511, 64, 130], 64),        # 2048 workgroups of four wavefronts, finished inside the launch
    (6, 40, 1600, [1600, 1300, 1, 1457, 208, 2], 208),            # 1920, chunks of 208 keys
    (3, 32, 1024, [1024, 1, 300], 64),            # 1536 of 16 chunks per row: a second launch
    (2, 40, 4000, [4000, 2300], 208),             # 1600 of 20
    (3, 32, 5800, [5800, 300, 4097], 512),        # 1152 of eight: a second launch
    (2, 32, 8192, [8192, 1000], 512),             # 1024 of eight: inside the launch
])
def test_launches_of_more_than_1024_workgroups(oracle, H, B, heads, Smax, lens, chunk):
    check(oracle, H, B, heads, Smax, lens, chunk, 2)
