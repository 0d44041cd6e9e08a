"""Output rows of the prompt kernel leave through LDS and a store window of 32 rows per wavefront: every row of the buffer is
written, none past it, at the edges of that window, of the prompt and of a tile."""
import numpy as np
import pytest
import torch

from oracle import fd_prefill_oracle as pf
from paper_2311_01282_amd import fdattn, synth

pytestmark = pytest.mark.gpu
GUARD = 64 * 128          # halves past the buffer, which nothing may write


@pytest.mark.parametrize("Smax,lens", [(1, [1, 0]), (15, [15, 9]), (32, [31, 32]), (33, [33, 1]), (97, [64, 97]),
                                       (128, [128, 127]), (129, [129, 128]), (160, [129, 160]), (255, [17, 255])])
def test_rows_are_written_to_the_end_and_no_further(Smax, lens):
    import fd_harness
    B, Hq, Hkv, D = 2, 3, 1, 128
    rng = np.random.default_rng(8000 + Smax)
    q, k, v = (rng.standard_normal((B, h, Smax, D)).astype(np.float16) for h in (Hq, Hkv, Hkv))
    sl = np.asarray(lens, dtype=np.int32)
    scale = synth.default_scale(D)
    dev = torch.device("cuda:0")
    tq, tk, tv, tsl = (torch.from_numpy(a).to(dev) for a in (q, k, v, sl))
    n = B * Hq * Smax * D
    out = torch.full((n + GUARD,), float("nan"), dtype=torch.float16, device=dev)
    shape = fdattn.make_shape(B, Hq, Hkv, D, Smax, 0, scale)
    ws = torch.empty(fdattn.fd_prefill_workspace_bytes(shape), dtype=torch.uint8, device=dev)
    fdattn.fd_prefill_attn(shape, tq.data_ptr(), tk.data_ptr(), tv.data_ptr(), tsl.data_ptr(), synth.PHI, synth.BOUNDS,
                           out.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream(dev).cuda_stream)
    got = out.cpu().numpy()
    assert np.isnan(got[n:]).all()
    got = got[:n].astype(np.float64).reshape(B, Hq, Smax, D)
    for b in range(B):
        assert not got[b, :, sl[b]:].any()
    rows = np.array([r for r in pf.all_rows(B, Hq, Smax) if r[2] < sl[r[0]]], dtype=np.int32)
    want, flag, _ = pf.prefill_rows(q, k, v, sl, scale, rows, phi=synth.PHI, lo=synth.BOUNDS[0], hi=synth.BOUNDS[1], nthreads=8)
    assert not flag.any()
    fd_harness.assert_close(got[rows[:, 0], rows[:, 1], rows[:, 2]], want, "rows of %s" % ((Smax, lens),))
