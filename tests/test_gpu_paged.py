"""fd_decode_attn_paged on the GPU against the paged-cache oracle: the same attention,
with every sequence's keys and values scattered over the pages of a pool.  The pages
sit at seeded-random places; pool pages nobody uses, the unused tail of a sequence's
last page and the table entries of pages without a valid token hold poison."""
import numpy as np
import pytest
import torch

from oracle import fd_paged_oracle as po
from paper_2311_01282_amd import fdattn, synth

pytestmark = pytest.mark.gpu
LO, HI = synth.BOUNDS


@pytest.fixture(scope="module")
def H():
    import fd_harness
    return fd_harness


class PagedCase:
    def __init__(self, H, case, page, chunk, seed=77, junk_entries=True):
        self.dc = H.DeviceCase(case, chunk=chunk)        # q, lengths, workspace, and the contiguous cache for A/B
        self.page = page
        self.k_pool, self.v_pool, self.table = synth.to_pages(case, page, seed=seed)
        table = self.table.copy()
        if junk_entries:                                 # entries that must never be followed
            junk = np.array([-1, 2 ** 31 - 1, -2 ** 31, 123456], dtype=np.int64)
            idx = np.flatnonzero(table.reshape(-1) < 0)
            table.reshape(-1)[idx] = junk[np.arange(idx.size) % junk.size].astype(np.int32)
        dev = self.dc.dev
        self.kp = torch.from_numpy(self.k_pool).to(dev)
        self.vp = torch.from_numpy(self.v_pool).to(dev)
        self.tb = torch.from_numpy(table).to(dev)

    def run(self, phi=synth.PHI, bounds=synth.BOUNDS):
        dc = self.dc
        dc.out.fill_(float("nan"))
        dc.last_entry = "fd_decode_attn_paged"
        fdattn.fd_decode_attn_paged(dc.shape, dc.q.data_ptr(), self.kp.data_ptr(), self.vp.data_ptr(), self.tb.data_ptr(),
                                    self.page, self.k_pool.shape[0], dc.seq_lens.data_ptr(), phi, bounds,
                                    dc.out.data_ptr(), *dc._ws(), dc._stream())
        torch.cuda.synchronize()
        return dc.out.cpu().numpy().astype(np.float64)


def check(H, case, page, chunk, expect_flagged=0):
    pc = PagedCase(H, case, page, chunk)
    sl = case["seq_lens"]
    want = po.attn_exact(case["q"], pc.k_pool, pc.v_pool, pc.table, page, sl, case["scale"], nthreads=8)
    ocf, orf, margin = po.flags(case["q"], pc.k_pool, pc.table, page, sl, case["scale"], synth.PHI, LO, HI, chunk, nthreads=8)
    assert margin.min() > 1e-2
    got = pc.run()
    H.assert_close(got, want, "paged, page %d chunk %d" % (page, chunk))
    cf, rf, n, rows = pc.dc.flags()
    assert np.array_equal(cf, ocf) and np.array_equal(rf, orf)
    assert int(orf.sum()) == expect_flagged
    # same keys in the same order through the same sums: the contiguous entry agrees to within one fp16
    # step on EVERY element, and to the last bit on all but a few -- it may run another compiled variant
    # of the kernel (the small-launch one requests its first block before the length is known and
    # zeroes what lies beyond it), whose fp32 operations the compiler may fuse differently, and an fp32
    # sum that differs in its last bit now and then rounds to the neighbouring fp16 value
    entry = "fd_decode_attn_gqa" if 2 <= case["Hq"] // case["Hkv"] <= 16 else "fd_decode_attn"
    same = pc.dc.run(entry)
    step = np.maximum(np.abs(same), 2.0 ** -14) * 2.0 ** -10          # fp16 spacing at that magnitude
    assert (np.abs(got - same) <= step).all() and (got != same).sum() <= max(4, 1e-2 * got.size)
    return got


@pytest.mark.parametrize("B,Hq,Hkv,Smax,lens,page,chunk", [
    (2, 4, 4, 512, [512, 200], 16, 64),                # vLLM-sized pages, four per chunk
    (2, 4, 4, 512, [512, 200], 16, 256),               # sixteen pages per chunk
    (1, 8, 8, 1024, [1000], 16, 1024),                 # the limit: 64 pages per chunk, 8-wavefront workgroups
    (3, 4, 4, 1024, [1024, 1, 0], 64, 256),            # one token; empty sequence
    (2, 8, 8, 2048, [2047, 700], 256, 256),            # page = chunk
    (2, 8, 8, 2048, [2048, 1300], 1024, 256),          # several chunks share a page
    (8, 32, 32, 2048, None, 128, 256),                 # 2048 workgroups that finish their rows
    (8, 32, 32, 2304, [2304, 1, 0, 2049, 2048, 257, 1000, 2300], 128, 256),    # 2304 of nine chunks: row epilogue as a second launch
    (8, 33, 33, 1024, [1024, 1, 0, 1023, 512, 513, 255, 700], 64, 256),        # 1056 workgroups, rows that do not divide by 8
    (7, 32, 32, 2560, [2560, 1, 0, 2049, 2048, 257, 1000], 64, 512),           # 1120 of eight wavefronts: a second launch
    (2, 16, 2, 1024, [1023, 256], 16, 256),            # grouped kernel, groups of 8
    (2, 12, 4, 512, [512, 0], 64, 128),                # groups of 3; empty sequence
    (1, 64, 8, 4096, [4000], 256, 1024),               # grouped, long chunks
    (2, 16, 2, 8192, [8191, 4097], 64, 4096),          # the longest chunk over its 64 pages
    (2, 4, 4, 4096, [4096, 2049], 256, 2048),          # per-row kernel, 2048-key chunks
    (3, 16, 2, 2048, [2048, 777, 1], 64, 2048),        # grouped, one chunk per sequence (no epilogue)
    (2, 4, 4, 3072, [3000, 1700], 64, 1152),           # chunks of 1152 keys = 18 pages
    (2, 4, 4, 3072, [3000, 1700], 256, 1152),          # ... that start in the middle of a page
    (2, 16, 2, 3072, [3000, 1700], 256, 1152),         # ... through the grouped kernel
    (1, 4, 4, 2048, [2000], 16, 1008),                 # 63 pages per chunk
])
def test_paged_matches_oracle_and_contiguous(H, B, Hq, Hkv, Smax, lens, page, chunk):
    case = synth.make_case(B=B, Hq=Hq, Hkv=Hkv, D=128, Smax=Smax, seed=8100 + page + chunk, seq_lens=lens,
                           poison_padding=True)
    check(H, case, page, chunk)


@pytest.mark.parametrize("Hq,Hkv", [(8, 8), (16, 2)])
def test_paged_flag_and_recompute(H, Hq, Hkv):
    # a planted key overflows the guard of its row: flagged, recomputed through the paged loads
    case = synth.make_case(B=2, Hq=Hq, Hkv=Hkv, D=128, Smax=1024, seed=8200, seq_lens=[1024, 600], poison_padding=True)
    planted = synth.plant_keys(case, 2, 36.0, seed=8201, allow_shared_kv=Hq != Hkv)
    assert len(planted) == 2
    pc = PagedCase(H, case, 32, 256)
    want = po.attn_exact(case["q"], pc.k_pool, pc.v_pool, pc.table, 32, case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = po.flags(case["q"], pc.k_pool, pc.table, 32, case["seq_lens"], case["scale"], synth.PHI, LO, HI, 256,
                                nthreads=8)
    assert margin.min() > 1e-2 and orf.sum() >= 2
    got = pc.run()
    H.assert_close(got, want, "paged with recomputation")
    cf, rf, n, rows = pc.dc.flags()
    assert np.array_equal(cf, ocf) and np.array_equal(rf, orf)


@pytest.mark.parametrize("B,heads,nc,chunk", [(12, 16, 8, 64), (13, 16, 8, 64), (12, 16, 8, 256), (8, 32, 8, 256), (8, 32, 9, 256)])
def test_paged_recompute_in_large_launches(H, B, heads, nc, chunk):
    """Recomputed chunks of launches ordered by length (rows finished inside, by a second launch; more full chunks than compute
    units) and of large per-row launches, through the paged loads."""
    Hkv = 8 if heads == 16 else 32
    Smax = nc * chunk
    lens = [[Smax, Smax - 1, chunk, 5 * chunk + 1, Smax, 3, 2 * chunk - 1][i % 7] for i in range(B)]
    case = synth.make_case(B=B, Hq=heads, Hkv=Hkv, D=128, Smax=Smax, seed=8250 + B, seq_lens=lens, poison_padding=True)
    planted = synth.plant_keys(case, 5, 36.0, seed=8251, allow_shared_kv=True)
    pc = PagedCase(H, case, 64, chunk)
    want = po.attn_exact(case["q"], pc.k_pool, pc.v_pool, pc.table, 64, case["seq_lens"], case["scale"], nthreads=8)
    ocf, orf, margin = po.flags(case["q"], pc.k_pool, pc.table, 64, case["seq_lens"], case["scale"], synth.PHI, LO, HI, chunk, nthreads=8)
    assert margin.min() > 1e-2 and orf.sum() >= len(planted) == 5
    for rep in range(2):
        H.assert_close(pc.run(), want, "paged with recomputation, pass %d" % rep)
        cf, rf, n, rows = pc.dc.flags()
        assert np.array_equal(cf, ocf) and np.array_equal(rf, orf)


@pytest.mark.parametrize("B,Hq,Hkv,Smax,lens,page,chunk", [
    (4, 4, 4, 512, [300, 256, 511, 512], 64, 256),     # mid-page; first row of a fresh page; last free row; full (dropped)
    (3, 8, 8, 1024, [0, 1, 1023], 16, 128),            # empty sequence: the new key is the only one
    (2, 32, 32, 2048, [2047, 1000], 256, 1024),        # 8-wavefront workgroups
    (2, 16, 2, 1024, [1000, 512], 32, 256),            # grouped kernel; a fresh page that opens a chunk
    (2, 16, 2, 1024, [1000, 512], 32, 1024),           # grouped kernel, one chunk per sequence
    (8, 32, 32, 2048, None, 128, 256),                 # every sequence full: nothing appended
    (8, 32, 32, 2304, [2303, 0, 2304, 2048, 2047, 256, 1000, 1791], 128, 256),  # a second launch; new keys that open and close chunks
    (7, 32, 32, 2560, [2559, 0, 2560, 2048, 511, 512, 1000], 64, 512),          # ... of eight wavefronts
    # the grouped kernel's order by length (more than 256 workgroups, up to 64 sequences): an empty and a full sequence, new keys that
    # are a chunk of their own, the last of one, inside one
    (12, 16, 8, 512, [511, 0, 512, 64, 63, 320, 100, 449, 447, 1, 256, 500], 16, 64),   # 768 workgroups: rows finished in the launch
    (12, 64, 8, 512, [0, 1, 5, 64, 63, 32, 10, 511, 512, 128, 2, 127], 64, 128),        # 384 of groups of 8, hardly any full chunk
    (13, 16, 8, 512, [511, 0, 512, 64, 63, 320, 100, 449, 447, 1, 256, 500, 511], 16, 64),   # 832: a second launch
    (9, 12, 4, 1280, [1279, 0, 1280, 1151, 1152, 640, 127, 128, 1279], 32, 128),        # ten chunks, groups of 3: a second launch
    (11, 16, 8, 2048, [2047, 2048, 2047, 2047, 256, 520, 0, 255, 520, 520, 1], 32, 256),  # more full chunks than compute units
    (40, 8, 4, 2048, [2047 - 50 * i for i in range(40)], 64, 64),                       # 5120 workgroups: too many to be ordered
    (65, 16, 8, 128, [127 - i % 128 for i in range(65)], 16, 64),                       # a sequence too many
])
def test_paged_append(H, B, Hq, Hkv, Smax, lens, page, chunk):
    case = synth.make_case(B=B, Hq=Hq, Hkv=Hkv, D=128, Smax=Smax, seed=8300 + page + chunk, seq_lens=lens, poison_padding=True)
    rng = np.random.default_rng(8301)
    k_new = rng.standard_normal((B, Hkv, 128)).astype(np.float16)
    v_new = rng.standard_normal((B, Hkv, 128)).astype(np.float16)
    sl = np.clip(np.asarray(case["seq_lens"], dtype=np.int64), 0, Smax)
    # the cache after the step (host side): rows in place, lengths that include the new token
    after = dict(case)
    after["k"], after["v"] = case["k"].copy(), case["v"].copy()
    for b in range(B):
        if sl[b] < Smax:
            after["k"][b, :, sl[b]] = k_new[b]
            after["v"][b, :, sl[b]] = v_new[b]
    sl2 = np.minimum(sl + 1, Smax).astype(np.int32)
    after["seq_lens"] = sl2
    pc = PagedCase(H, after, page, chunk)                # pools and table of the state after the step
    want = po.attn_exact(case["q"], pc.k_pool, pc.v_pool, pc.table, page, sl2, case["scale"], nthreads=8)
    ocf, orf, margin = po.flags(case["q"], pc.k_pool, pc.table, page, sl2, case["scale"], synth.PHI, LO, HI, chunk, nthreads=8)
    assert margin.min() > 1e-2
    # the state before the step: the rows that will be written hold poison
    for b in range(B):
        if sl[b] < Smax:
            pid, r = pc.table[b, sl[b] // page], sl[b] % page
            pc.kp[pid, :, r] = float("nan")
            pc.vp[pid, :, r] = float("nan")
    dc = pc.dc
    dc.seq_lens.copy_(torch.from_numpy(sl.astype(np.int32)))
    kn, vn = torch.from_numpy(k_new).to(dc.dev), torch.from_numpy(v_new).to(dc.dev)
    dc.out.fill_(float("nan"))
    dc.last_entry = "fd_decode_attn_paged_append"
    fdattn.fd_decode_attn_paged_append(dc.shape, dc.q.data_ptr(), kn.data_ptr(), vn.data_ptr(), pc.kp.data_ptr(), pc.vp.data_ptr(),
                                       pc.tb.data_ptr(), page, pc.k_pool.shape[0], dc.seq_lens.data_ptr(), synth.PHI,
                                       synth.BOUNDS, dc.out.data_ptr(), *dc._ws(), dc._stream())
    torch.cuda.synchronize()
    H.assert_close(dc.out.cpu().numpy().astype(np.float64), want, "paged append, page %d chunk %d" % (page, chunk))
    # the pools: bit for bit the state after the step, nothing else touched (poison stays poison)
    assert np.array_equal(pc.kp.cpu().numpy().view(np.uint16), pc.k_pool.view(np.uint16))
    assert np.array_equal(pc.vp.cpu().numpy().view(np.uint16), pc.v_pool.view(np.uint16))
    dc.seq_lens.copy_(torch.from_numpy(sl2))
    cf, rf, n, rows = dc.flags()
    assert np.array_equal(cf, ocf) and np.array_equal(rf, orf)


def test_paged_long_context_and_graph_replay(H):
    # 128K tokens in 8192 pages of 16 (64 pages per chunk, 128 chunks per row), then the same call
    # recorded by a stream capture and replayed with eager calls in between
    case = synth.make_case(B=1, Hq=8, Hkv=8, D=128, Smax=131072, seq_lens=[131072 - 777], seed=8400)
    pc = PagedCase(H, case, 16, 1024)
    want = po.attn_exact(case["q"], pc.k_pool, pc.v_pool, pc.table, 16, case["seq_lens"], case["scale"], nthreads=8)
    eager = pc.run()
    H.assert_close(eager, want, "paged, 128K context")
    dc = pc.dc
    side = torch.cuda.Stream(device=dc.dev)
    graph = torch.cuda.CUDAGraph()
    out_g = torch.full_like(dc.out, float("nan"))
    side.wait_stream(torch.cuda.current_stream(dc.dev))
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            fdattn.fd_decode_attn_paged(dc.shape, dc.q.data_ptr(), pc.kp.data_ptr(), pc.vp.data_ptr(), pc.tb.data_ptr(), 16,
                                        pc.k_pool.shape[0], dc.seq_lens.data_ptr(), synth.PHI, synth.BOUNDS,
                                        out_g.data_ptr(), *dc._ws(), side.cuda_stream)
    torch.cuda.synchronize(dc.dev)
    for i in range(3):
        out_g.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize(dc.dev)
        assert np.array_equal(out_g.cpu().numpy().astype(np.float64), eager), "replay %d differs from the eager call" % i
        assert np.array_equal(pc.run(), eager)
    del graph


def test_paged_rejects_bad_arguments():
    dev = torch.device("cuda:0")
    buf = torch.zeros(1 << 22, dtype=torch.uint8, device=dev)
    p = buf.data_ptr()
    sh = fdattn.make_shape(1, 2, 2, 128, 1024, 256, 0.1)
    n = fdattn.fd_workspace_bytes(sh)
    ok = (sh, p, p, p, p, 64, 16, p, 3.0, (-60.0, 20.0), p, p, n)
    def bad(i, v):
        a = list(ok)
        a[i] = v
        return tuple(a)
    for args, code in ((bad(4, 0), fdattn.FD_ERR_NULL),                      # no table
                       (bad(5, 8), fdattn.FD_ERR_SHAPE),                     # page below 16
                       (bad(5, 48), fdattn.FD_ERR_SHAPE),                    # not a power of two
                       (bad(5, 2048), fdattn.FD_ERR_SHAPE),                  # capacity not a multiple of the page
                       (bad(6, 0), fdattn.FD_ERR_SHAPE),                     # empty pool
                       ((fdattn.make_shape(1, 2, 2, 128, 2048, 1024, 0.1),) + ok[1:5] + (8,) + ok[6:], fdattn.FD_ERR_SHAPE)):
        with pytest.raises(fdattn.FdError) as e:
            fdattn.fd_decode_attn_paged(*args)
        assert e.value.status == code
    # more than 64 pages per chunk: 128; 65; 63 and a bit when the chunk may start inside a page
    for chunk, page in ((2048, 16), (1040, 16), (4080, 64)):
        sh2 = fdattn.make_shape(1, 2, 2, 128, 4096, chunk, 0.1)
        n2 = fdattn.fd_workspace_bytes(sh2)
        with pytest.raises(fdattn.FdError) as e:
            fdattn.fd_decode_attn_paged(sh2, p, p, p, p, page, 16, p, 3.0, (-60.0, 20.0), p, p, n2)
        assert e.value.status == fdattn.FD_ERR_SHAPE
