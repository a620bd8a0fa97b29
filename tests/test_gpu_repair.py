"""GPU parity of the pulse-count repair (Sec. 2.5) where its order is hard to tell: equal deviations, deviations a few units
in the last place apart, as many pulses to move as there can be.  Every encoder against the oracle."""
import numpy as np
import pytest

import paper_2410_16926_amd as pvq
import synth_inputs as si
from oracle import pvq_oracle as oracle
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def hard_groups(n, D, K, seed):
    rng = np.random.default_rng(seed)
    g = np.empty((n, D), dtype=np.float64)
    kind = np.arange(n) % 6
    # equal magnitudes: every deviation the same
    g[kind == 0] = 1.0
    # projected values of whole numbers and a half, but for a few: as many deviations of one half as there can be
    k = kind == 1
    g[k] = rng.integers(0, 4, size=(k.sum(), D)) + 0.5
    # two magnitudes
    k = kind == 2
    g[k] = np.where(rng.random((k.sum(), D)) < 0.5, 1.0, 1.0 + 1.0 / D)
    # a few large values and many whose projection is near zero
    k = kind == 3
    g[k] = np.where(rng.random((k.sum(), D)) < 0.2, 1.0, 1e-4 * rng.random((k.sum(), D)))
    # projections just below and above a half
    k = kind == 4
    g[k] = 0.5 + 1e-3 * rng.standard_normal((k.sum(), D))
    k = kind == 5
    g[k] = rng.integers(1, 1 + max(1, 2 * K // D), size=(k.sum(), D)) + 0.48
    # neighbouring floats of the same magnitudes, up to nine units in the last place apart
    w = g.astype(np.float32)
    ulps = rng.integers(0, 10, size=w.shape) * (rng.random((n, 1)) < 0.6)
    w = (w.view(np.int32) + np.where(w > 0, ulps, 0).astype(np.int32)).view(np.float32)
    w *= rng.choice([-1.0, 1.0], size=w.shape).astype(np.float32)
    return w * np.exp2(rng.integers(-30, 30, size=(n, 1))).astype(np.float32)


@pytest.mark.parametrize("D,K,amplitude", [(8, 16, "norm"), (8, 15, "ls"), (8, 12, "norm"), (8, 3, "norm"), (8, 100, "ls"), (16, 33, "norm"), (16, 24, "ls"),
                                           (16, 5, "norm"), (32, 60, "norm"), (32, 48, "ls"), (32, 16, "norm"), (32, 1, "norm"),
                                           (64, 96, "norm"), (64, 41, "ls"), (64, 1, "norm"), (128, 187, "ls"), (128, 187, "norm"), (128, 84, "norm"), (128, 9, "ls")])
def test_order_of_deviations(D, K, amplitude):
    rows, G = 48, 36
    W0 = hard_groups(rows * G, D, K, si.BASE_SEED + 800 + D + K).reshape(rows, G * D)
    ctx = pvq.pvq_ctx_create(D, K)
    ctx.set_amplitude(amplitude)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W0), want_pulses=K <= 127)
    enc = oracle.encode(W0, D, K, 0, None, nthreads=8, amplitude="ls" if amplitude == "ls" else "l2")
    gu.assert_encode_equal(packed, enc)
    ctx.close()


@pytest.mark.parametrize("D,K,bits,G", [(8, 16, 1, 256), (8, 16, 2, 260), (8, 16, 4, 516), (8, 16, 8, 1028), (8, 16, 1, 2052), (8, 9, 2, 70), (16, 33, 8, 65), (32, 60, 1, 300)])
def test_codes_of_rows_of_any_number_of_runs(D, K, bits, G):
    # a wave writes the codes of its runs of 64 groups one, two or four at a time; the last run and the last four are ragged
    rows = 5
    W0 = np.asarray(si.gaussian_weights(rows, G * D, 0.02, seed=si.BASE_SEED + 830 + G, rotate=False, bf16=False), dtype=np.float32)
    W0[1, : 3 * D] = 0.0
    W0[2] *= np.float32(2.0) ** -60
    W0[3, D:2 * D] *= np.float32(2.0) ** -40
    ctx, oe, _ = gu.make_ctx(D, K, bits, G)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W0), want_pulses=True)
    gu.assert_encode_equal(packed, oracle.encode(W0, D, K, bits, oe, nthreads=8))
    ctx.close()


@pytest.mark.parametrize("D,K,levels,amplitude", [(64, 96, 2, "norm"), (64, 41, 5, "ls"), (64, 31, 30, "norm"), (128, 187, 3, "norm"),
                                                  (128, 84, 9, "ls"), (128, 187, 60, "norm"), (64, 300, 4, "norm")])
def test_equal_deviations_in_long_groups_of_float32_values(D, K, levels, amplitude):
    # A running maximum passes over deviations that are equal, and the places are made up for afterwards: few magnitudes, so that
    # whole runs of places are equal, at the last place, in front of it, and in more groups than have that many different ones;
    # groups of distinct values between them, which share a wave with them.
    rows, G = 24, 21
    rng = np.random.default_rng(si.BASE_SEED + 860 + K + levels)
    w = rng.choice(rng.uniform(0.2, 1.0, size=levels), size=(rows * G, D))
    w[::5] = rng.standard_normal((len(w[::5]), D))
    w[3::7] *= rng.random((len(w[3::7]), D)) < 0.1
    w = (w * rng.choice([-1.0, 1.0], size=w.shape)).astype(np.float32).reshape(rows, G * D)
    ctx = pvq.pvq_ctx_create(D, K)
    ctx.set_amplitude(amplitude)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(w), want_pulses=K <= 127)
    gu.assert_encode_equal(packed, oracle.encode(w, D, K, 0, None, nthreads=8, amplitude="ls" if amplitude == "ls" else "l2"))
    ctx.close()
