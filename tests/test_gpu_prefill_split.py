"""Small prefill launches (tiles of 64 queries, the keys of 32 queries shared by two wavefronts): rows and flags against the fp64 oracle at the edges of
tiles and key steps, in ragged batches, with heads shared, and where only an even, only an odd or a late key step flags or is out of the operands' range."""
import numpy as np
import pytest

from oracle import fd_prefill_oracle as pf
from paper_2311_01282_amd import synth
from test_gpu_prefill import H, HI, LO, close, draw, run_gpu, tile_flags_from_rows  # noqa: F401 (H: the fixture)

pytestmark = pytest.mark.gpu
SCALE = float(np.float32(1.0 / np.sqrt(128.0)))


def _check(H, B, Hq, q, k, v, sl, Smax, what, flagged=None):
    rows = pf.all_rows(B, Hq, Smax)
    want, flag, margin = pf.prefill_rows(q, k, v, sl, SCALE, rows, phi=synth.PHI, lo=LO, hi=HI, nthreads=8)
    assert margin.min() > 1e-2 and (flagged is None or bool(flag.any()) == flagged)
    got, tf = run_gpu(q, k, v, sl, SCALE)
    assert np.array_equal(tf, tile_flags_from_rows(rows, flag, B, Hq, Smax))
    close(H, got.reshape(-1, 128), want, what)
    for b in range(B):
        assert not got[b, :, sl[b]:].any()


@pytest.mark.parametrize("Smax", [1, 31, 32, 33, 63, 64, 65, 95, 97, 127, 129, 193, 449])
def test_edges_of_tiles_and_steps(H, Smax):
    lens = [Smax, 0, 1, max(0, Smax - 1), Smax // 2, min(Smax, 33)]
    _check(H, 6, 4, *draw(6, 4, 2, Smax, lens, seed=7700 + Smax), Smax, "prefill of %d" % Smax, flagged=False)


# the rule: up to 256 tiles of 128 queries, up to 288 of which a head has more than four, fewer where a head has one to three, none up to 96
# queries, and what is just beyond
@pytest.mark.parametrize("B,Hq,Hkv,Smax", [(16, 16, 2, 100), (1, 257, 257, 40), (4, 12, 2, 700), (1, 49, 7, 650), (2, 24, 24, 641), (1, 128, 16, 97),
                                           (1, 128, 16, 96), (1, 129, 43, 97), (1, 64, 8, 217), (1, 65, 65, 217), (1, 64, 8, 290), (1, 65, 65, 290),
                                           (1, 85, 85, 360), (1, 64, 8, 400)])
def test_edges_of_the_rule(H, B, Hq, Hkv, Smax):
    q, k, v, sl = draw(B, Hq, Hkv, Smax, [Smax] + [max(0, Smax - 37 * b) for b in range(1, B)], seed=7800 + Smax)
    rng = np.random.default_rng(5)
    rows = np.asarray([(b, h, i) for b in range(B) for h in {0, Hq - 1, int(rng.integers(Hq))} for i in
                       {0, sl[b] - 1, *(int(x) for x in rng.integers(0, max(1, sl[b]), 60))} if i >= 0], dtype=np.int32)
    rows = rows[rows[:, 2] < sl[rows[:, 0]]]
    want, flag, _ = pf.prefill_rows(q, k, v, sl, SCALE, rows, phi=synth.PHI, lo=LO, hi=HI, nthreads=8)
    got, tf = run_gpu(q, k, v, sl, SCALE)
    assert not flag.any() and not tf.any() and np.isfinite(got).all()
    close(H, got[rows[:, 0], rows[:, 1], rows[:, 2]], want, "prefill %s" % ((B, Hq, Hkv, Smax),))
    for b in range(B):
        assert not got[b, :, sl[b]:].any()


@pytest.mark.parametrize("pos", [5, 40, 70, 100, 200, 290])          # key steps 0 .. 9, even and odd
@pytest.mark.parametrize("logit", [16.0, 38.0])                      # out of the operands' range, and of the guard's
def test_one_step_has_its_tiles_redone(H, pos, logit):
    q, k, v, sl = draw(1, 4, 2, 320, [300], seed=7900)
    q[0, 2, pos:300, 5] = np.float16(12.0)
    k[0, 1, pos] = 0
    k[0, 1, pos, 5] = np.float16(logit * np.sqrt(128.0) / 12.0)
    _check(H, 1, 4, q, k, v, sl, 320, "logit %g at key %d" % (logit, pos), flagged=logit > 20 + synth.PHI)


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_halves_of_unlike_scales(H, sign):
    """Logits of the even key steps 14 above (below) those of the odd ones: inside the guard and the range, nothing flagged."""
    q, k, v, sl = draw(2, 4, 2, 256, [256, 171], seed=7950)
    q[:, :, :, 9] = np.float16(8.0)
    for b in range(2):
        step = np.arange(sl[b]) // 32
        k[b, :, :sl[b], 9] = np.where(step % 2 == 0, sign * 7.0, -sign * 7.0)[None, :] * np.sqrt(128.0) / 8.0
    _check(H, 2, 4, q, k, v, sl, 256, "halves of unlike scales", flagged=False)
