"""The merge of the synchronized scheme (Eq. 2 over a row's chunks, 16 at a time, two rows per workgroup) at the edges of its
batches, and over caches that hold little of what they could."""
import numpy as np
import pytest
import torch

import fd_harness
from paper_2311_01282_amd import fdattn, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nc", [1, 4, 5, 8, 9, 15, 16, 17, 32, 33, 49])
def test_merge_over_chunk_counts(oracle, nc):
    """An odd number of rows; beside the full sequence a short one, one that ends in the second batch and an empty one.  A
    planted key makes one chunk's maximum stand far above the others', in the last chunk where there is one."""
    S, H = 64 * nc - 5, 3
    lens = [S, max(1, S - 64), min(S, 40), 0, min(S, 64 * 17)]
    case = synth.make_case(B=len(lens), Hq=H, Hkv=H, D=128, Smax=S, seed=9100 + nc, seq_lens=lens, poison_padding=True)
    q = case["q"][0, 1].astype(np.float64)
    case["k"][0, 1, S - 1] = (36.0 * q / np.linalg.norm(q)).astype(np.float16)
    want = oracle.attn_exact(case["q"], case["k"], case["v"], case["seq_lens"], case["scale"])
    got = fd_harness.DeviceCase(case, chunk=64).run("fd_decode_attn_sync")
    fd_harness.assert_close(got, want, "synchronized merge, %d chunks" % nc)
    assert not got[3].any()


def test_merge_stops_at_the_end_of_the_row():
    """2000 keys in a cache of 131072 are 8 of 512 chunks.  The chunk kernel alone, with the same grid, takes 22.1 us on 32 heads, the
    synchronized call 25.8; a merge that walks all 512 chunks of the row would make it 44.7."""
    H, S = 32, 131072
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(77)
    rnd = lambda *shape: torch.randn(*shape, generator=gen, device=dev, dtype=torch.float16)  # noqa: E731
    q, k, v = rnd(1, H, 128), rnd(1, H, S, 128), rnd(1, H, S, 128)
    out = torch.empty_like(q)
    lens = torch.tensor([2000], dtype=torch.int32, device=dev)
    shape = fdattn.make_shape(1, H, H, 128, S, 256, synth.default_scale(128))
    nbytes = fdattn.fd_workspace_bytes(shape)
    ws = torch.empty(nbytes, dtype=torch.uint8, device=dev)
    stream = torch.cuda.current_stream(dev).cuda_stream
    fdattn.fd_workspace_init(shape, ws.data_ptr(), nbytes, stream)
    args = (shape, q.data_ptr(), k.data_ptr(), v.data_ptr(), lens.data_ptr())

    def sync():
        fdattn.fd_decode_attn_sync(*args, out.data_ptr(), ws.data_ptr(), nbytes, stream)

    def chunks_alone():
        fdattn.fd_decode_attn_partial(*args, synth.PHI, synth.BOUNDS, ws.data_ptr(), nbytes, stream)

    def us(call):
        best = float("inf")
        for _ in range(15):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                call()
            b.record()
            b.synchronize()
            best = min(best, a.elapsed_time(b) / 20 * 1e3)
        return best

    t_chunks, t_sync = us(chunks_alone), us(sync)
    print("chunks alone %.1f us, synchronized %.1f us" % (t_chunks, t_sync))
    assert t_sync < 1.5 * t_chunks, (t_sync, t_chunks)
