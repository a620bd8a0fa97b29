"""Amplitude codes (Sec. 3.3 Step 5) where their quotient changes between its short form and the division: row sums around
2^-60 and 2^30, sums of squares of groups around 2^-70, zeros among them."""
import numpy as np
import pytest

import synth_inputs as si
from oracle import pvq_oracle as oracle
from tests import gpu_util as gu

import paper_2410_16926_amd as pvq

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")


@pytest.mark.parametrize("D,K,amplitude", [(8, 16, "l2"), (8, 16, "ls"), (16, 33, "l2"), (32, 60, "ls")])
@pytest.mark.parametrize("bits", [1, 2, 4, 8])
def test_codes_of_rows_around_the_lines_of_the_short_quotient(D, K, amplitude, bits):
    G = 68
    rng = np.random.default_rng(si.BASE_SEED + 900 + D + bits)
    exponents = [-45, -34, -33, -32, -31, -30, -29, 0, 9, 10, 11, 12, 13, 14, 15, 16, 30]
    W = rng.standard_normal((3 * len(exponents), G * D)).astype(np.float32)
    for r, e in enumerate(exponents):
        W[3 * r: 3 * r + 3] *= np.float32(2.0) ** e
    g = W.reshape(W.shape[0], G, D)
    # in the second row of three a few groups far below the others, in the third by less or more, and zeros as well
    for r in range(1, W.shape[0], 3):
        g[r, ::7] *= np.float32(2.0) ** rng.integers(-40, -20, size=(len(g[r, ::7]), 1)).astype(np.float32)
        g[r + 1, ::5] *= np.float32(2.0) ** rng.integers(-60, -1, size=(len(g[r, ::5]), 1)).astype(np.float32)
        g[r + 1, 3::11] = 0.0
    ctx, oe, _ = gu.make_ctx(D, K, bits, G)
    ctx.set_amplitude("ls" if amplitude == "ls" else "norm")
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W), want_pulses=True)
    gu.assert_encode_equal(packed, oracle.encode(W, D, K, bits, oe, nthreads=8, amplitude=amplitude))
    ctx.close()
