"""Logits up to the largest that finite fp16 operands reach (4.8e10), of either sign, where fp32 numbers lie further apart than weights can
tell: the largest logit, and every key that shares it to the bit, takes all the weight, wherever the chunks, wavefronts and blocks put it.
Against the fp64 oracle, for heads of their own and heads that share KV heads, in every decode call."""
import numpy as np
import pytest

from paper_2311_01282_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


def _case(B, Hq, Hkv, lens, Smax, size, order, seed):
    """Logits scale * <q, k_j> = size * t_j with t_j spread over (1/4, 1], neighbours at least size / 4096 apart, the largest one three times (in a
    sequence of that many keys)."""
    case = synth.make_case(B=B, Hq=Hq, Hkv=Hkv, D=128, Smax=Smax, seed=seed, seq_lens=lens, poison_padding=True)
    rng = np.random.default_rng(seed)
    root = np.sqrt(abs(size) / (128 * case["scale"]))
    sign = rng.choice([-1.0, 1.0], size=128)
    case["q"][...] = (root * sign * np.linspace(1.0, 0.5, Hq)[None, :, None]).astype(np.float16)
    for b, n in enumerate(lens):
        if n == 0:
            continue
        t = np.linspace(1.0, 0.26, n) if size > 0 else np.linspace(0.26, 1.0, n)       # falling logits
        if order == "rising":
            t = t[::-1].copy()
        elif order == "mixed":
            t = rng.permutation(t)
        top = int(np.argmax(t * np.sign(size)))
        t[rng.choice(n, size=min(n, 2), replace=False)] = t[top]
        case["k"][b, :, :n] = (np.sign(size) * root * t[:, None] * sign).astype(np.float16)
    return case


# (batch, query heads, KV heads, lengths, max_seq, chunk)
SHAPES = [
    (2, 8, 2, [700, 65], 700, 128),
    (12, 8, 2, [700, 65, 0, 699] * 3, 700, 128),
    (3, 12, 2, [1500, 0, 1024], 1500, 1024),
    (3, 12, 2, [1500, 0, 1024], 1500, 1040),
    (2, 4, 4, [700, 65], 700, 128),
    (2, 4, 4, [1500, 1000], 1500, 1024),
    (20, 16, 16, [900 - 40 * i for i in range(20)], 900, 912),
    (1, 4, 4, [1500], 1500, 2048),
]


@pytest.mark.parametrize("B,Hq,Hkv,lens,Smax,chunk", SHAPES)
@pytest.mark.parametrize("order", ["falling", "rising", "mixed"])
@pytest.mark.parametrize("size", [3e5, 2e8, -2e8, 1e9, -1e9, 4.5e10, -4.5e10])
def test_largest_logit_takes_all(oracle, H, B, Hq, Hkv, lens, Smax, chunk, order, size):
    case = _case(B, Hq, Hkv, lens, Smax, size, order, seed=9800 + Smax)
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"], nthreads=8)
    dc = H.DeviceCase(case, chunk=chunk)
    for entry in ("fd_decode_attn_sync", "fd_decode_attn", "fd_decode_attn_multikernel") + (("fd_decode_attn_gqa",) if Hq != Hkv else ()):
        H.assert_close(dc.run(entry), want, "%s, size %g, %s" % (entry, size, order))
