"""The merge of the synchronized scheme on either side of its two forms (32 chunks per row), at the edges of its blocks of 16 chunks,
for odd row counts, empty and short sequences in a long cache, and chunk maxima that rise and fall by more than fp32 can
rescale in one step, against the fp64 oracle."""
import numpy as np
import pytest

from paper_2311_01282_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


@pytest.mark.parametrize("nc", [1, 4, 5, 16, 17, 31, 32, 33, 47, 48, 49, 64, 65, 130])
@pytest.mark.parametrize("slope", [0.0, 120.0, -120.0])
def test_merge_of_nc_chunks(oracle, H, nc, slope):
    chunk, B, heads = 64, 3, 3
    Smax = nc * chunk
    lens = [Smax, 0, max(Smax - chunk * (nc // 3) - 5, 1)]
    case = synth.make_case(B=B, Hq=heads, Hkv=heads, D=128, Smax=Smax, seed=8900 + nc, seq_lens=lens, poison_padding=True)
    if slope:
        # logits that climb (fall) along the sequence by `slope`: one element of every key, times one of q
        t = np.linspace(0.0, 1.0, Smax) - (0.5 if slope > 0 else 0.0)
        case["q"][..., 0] = 16.0
        ramp = (t * slope / (16.0 * case["scale"])).astype(np.float16)
        for b in range(B):
            case["k"][b, :, :lens[b], 0] = ramp[:lens[b]]
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    dc = H.DeviceCase(case, chunk=chunk)
    H.assert_close(dc.run("fd_decode_attn_sync"), want, "%d chunks, slope %g" % (nc, slope))
