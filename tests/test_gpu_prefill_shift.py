"""Prompts whose tiles start 64 queries before them (launches of many tiles with a short last one): rows and flags bit for bit those of
the same prompts in a longer buffer, whose tiles start at the prompt; at the edges of the rule, in ragged batches, with tiles that are redone at either
end of the prompt, and with junk in front of and behind every head's rows."""
import numpy as np
import pytest
import torch

from paper_2311_01282_amd import fdattn, synth

pytestmark = pytest.mark.gpu
D = 128


def _prefill(q, k, v, lens):
    B, Hq, S, _ = q.shape
    shape = fdattn.make_shape(B, Hq, k.shape[1], D, S, 64, synth.default_scale(D))
    n = fdattn.fd_prefill_workspace_bytes(shape)
    ws = torch.full((n,), 0xA5, dtype=torch.uint8, device="cuda")
    out = torch.full_like(q, float("nan"))
    fdattn.fd_prefill_attn(shape, q.data_ptr(), k.data_ptr(), v.data_ptr(), lens.data_ptr(), synth.PHI, synth.BOUNDS, out.data_ptr(),
                           ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    at = fdattn.fd_prefill_get_flags(shape, ws.data_ptr(), n) - ws.data_ptr()
    tiles = (S + 63) // 64
    return out, ws[at:at + B * Hq * tiles].reshape(B, Hq, tiles)


@pytest.mark.parametrize("B,Hq,Hkv,whole", [(20, 4, 4, 6), (10, 4, 2, 7), (65, 8, 8, 0), (5, 8, 1, 6)])
@pytest.mark.parametrize("over", [1, 32, 33, 63, 64, 65])
@pytest.mark.parametrize("ragged", [False, True])
def test_as_in_a_longer_buffer(B, Hq, Hkv, whole, over, ragged):
    S = 128 * whole + over
    longer = 128 * whole + 128                                  # (no queries over: tiles start at the prompt)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9950 + S + B)
    q, k, v = (torch.randn(B, h, S, D, generator=gen, device="cuda", dtype=torch.float16) for h in (Hq, Hkv, Hkv))
    lens = torch.full((B,), S, dtype=torch.int32, device="cuda")
    if ragged:
        lens = torch.randint(0, S + 1, (B,), generator=gen, device="cuda", dtype=torch.int32)
        lens[0] = S
    for b in (0, B - 1):                                        # a logit of 36: the first tile of one prompt, the last of another
        n = int(lens[b])
        if n:
            pos = min(3, n - 1) if b else n - 1
            qv = q[b, 0, pos].float()
            k[b, 0, pos] = (36.0 * qv / qv.norm()).half()
    for b in range(B):
        for t in (q, k, v):
            t[b, :, int(lens[b]):] = float("nan")

    def pad(t):
        return torch.cat([t, torch.full((t.shape[0], t.shape[1], longer - S, D), float("nan"), dtype=t.dtype, device=t.device)], dim=2)

    got, flags = _prefill(q, k, v, lens)
    want, want_flags = _prefill(pad(q), pad(k), pad(v), lens)
    assert torch.isfinite(got).all() and flags.sum() > 0
    want = want[:, :, :S].contiguous()
    # a tile with a flag is redone as a whole, by the other scheme: of those heads the rows agree to the rounding of the output
    assert float((got.float() - want.float()).abs().max()) <= 2e-3
    same = torch.ones(B, Hq, dtype=torch.bool, device="cuda")
    same[0, :Hq // Hkv] = same[B - 1, :Hq // Hkv] = False
    assert torch.equal(got[same].view(torch.int16), want[same].view(torch.int16))
    assert np.array_equal(flags.cpu().numpy(), want_flags[:, :, :flags.shape[2]].cpu().numpy())
