"""The histogram kernel starts each (sequence, KV head) at a place of its own, where the runs are longer than 64 keys, or at its first
run: every key is counted once, whether the number of runs divides the workgroups or not, with as many items as workgroups hold,
fewer and more."""
import pytest

from oracle import fd_calibration_oracle as cal
from paper_2311_01282_amd import synth
from test_gpu_calibration import EDGE_EPS, check_histogram, gpu_histogram

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,Smax,lens", [
    (1, 4, 2, 40, [40]),                                  # one run per head
    (4, 8, 8, 2048, [2048, 100, 1500, 64]),               # 32 runs of 64 keys on 256 workgroups
    (3, 6, 3, 1999, [1999, 1, 1030]),                     # 32 runs, the last short; 9 heads
    (2, 24, 2, 8192, [8192, 5000]),                       # 128 runs
    (2, 34, 2, 700, [700, 321]),                          # two blocks of heads on one KV head
    (16, 16, 16, 2500, [2500 - 150 * i for i in range(16)]),   # several rounds of the workgroups
    (32, 16, 16, 1000, [1000 - 30 * i for i in range(32)]),    # 512 heads of 16 runs of 64 keys: two rounds, every head at its first run
    (32, 32, 32, 1000, [1000 - 30 * i for i in range(32)]),    # 1024 heads: 8 runs of 128 keys, each head at a place of its own
    (3, 64, 8, 20001, [20001, 2500, 64]),                      # more runs than workgroups
])
def test_every_key_is_counted_once(B, Hq, Hkv, Smax, lens):
    case = synth.make_case(B=B, Hq=Hq, Hkv=Hkv, D=128, Smax=Smax, seq_lens=lens, seed=400 + Smax, poison_padding=True)
    want, lo, hi, near = cal.logit_histogram(case["q"], case["k"], case["seq_lens"], case["scale"], -6.0, 0.125, 96,
                                             nthreads=8, edge_eps=EDGE_EPS)
    got, mm = gpu_histogram(case, -6.0, 0.125, 96)
    check_histogram(got, want, near)
    assert got.sum() == sum(lens) * Hq
    assert mm[0] == pytest.approx(lo, abs=1e-4) and mm[1] == pytest.approx(hi, abs=1e-4)


# The runs that hold keys dealt out by the lengths' prefix sums: empty sequences first, last and between, lengths at the edges of a run, a sequence
# that holds all keys, 64 sequences (the last with this order) and 65, two blocks of heads on one KV head
@pytest.mark.parametrize("B,Hq,Hkv,Smax,lens", [
    (6, 24, 24, 9000, [0, 9000, 0, 1, 4097, 0]),
    (5, 36, 2, 120000, [0, 60000, 128, 127, 129]),
    (64, 4, 4, 5000, [73 * i for i in range(64)]),
    (65, 4, 4, 5000, [73 * i for i in range(65)]),
    (3, 64, 32, 12000, [0, 0, 12000]),
    (3, 64, 32, 12000, [0, 0, 0]),
])
def test_every_key_is_counted_once_among_runs_without_keys(B, Hq, Hkv, Smax, lens):
    case = synth.make_case(B=B, Hq=Hq, Hkv=Hkv, D=128, Smax=Smax, seq_lens=lens, seed=500 + Smax, poison_padding=True)
    got, mm = gpu_histogram(case, -6.0, 0.125, 96)
    assert got.sum() == sum(lens) * Hq
    if sum(lens):
        want, lo, hi, near = cal.logit_histogram(case["q"], case["k"], case["seq_lens"], case["scale"], -6.0, 0.125, 96,
                                                 nthreads=8, edge_eps=EDGE_EPS)
        check_histogram(got, want, near)
        assert mm[0] == pytest.approx(lo, abs=1e-4) and mm[1] == pytest.approx(hi, abs=1e-4)
