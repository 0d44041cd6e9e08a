"""Launches of the prompt kernel whose heads are dealt out in groups (192 KV heads and more): every tile is computed exactly once, by
comparison, bit for bit, with the same prompts in calls of fewer heads, which take all heads together; head counts that the groups
and the XCDs do and do not divide."""
import pytest
import torch

from paper_2311_01282_amd import fdattn, synth

pytestmark = pytest.mark.gpu


def _prefill(q, k, v, lens, chunk=64):
    B, Hq, S, D = q.shape
    shape = fdattn.make_shape(B, Hq, k.shape[1], D, S, chunk, synth.default_scale(D))
    n = fdattn.fd_prefill_workspace_bytes(shape)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    out = torch.full_like(q, float("nan"))
    fdattn.fd_prefill_attn(shape, q.data_ptr(), k.data_ptr(), v.data_ptr(), lens.data_ptr(), synth.PHI, synth.BOUNDS, out.data_ptr(),
                           ws.data_ptr(), n, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("B,Hq,Hkv,S", [
    (25, 8, 8, 900),        # 200 heads of 8 tiles: groups of 32
    (67, 3, 3, 1000),       # 201 heads: XCDs and groups do not divide them
    (13, 32, 16, 700),      # two query heads to one KV head
    (24, 8, 8, 850),        # 192 heads: the first launch with groups
    (200, 1, 1, 2100),      # a group of 16 heads of 17 tiles
])
def test_every_tile_once(B, Hq, Hkv, S):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9900 + S)
    q, k, v = (torch.randn(B, h, S, 128, generator=gen, device="cuda", dtype=torch.float16) for h in (Hq, Hkv, Hkv))
    lens = torch.randint(0, S + 1, (B,), generator=gen, device="cuda", dtype=torch.int32)
    lens[0] = S
    got = _prefill(q, k, v, lens)
    step = max(1, 128 // Hkv)
    for b in range(0, B, step):
        want = _prefill(q[b:b + step].contiguous(), k[b:b + step].contiguous(), v[b:b + step].contiguous(), lens[b:b + step].contiguous())
        assert torch.equal(got[b:b + step].view(torch.int16), want.view(torch.int16)), (b, step)
