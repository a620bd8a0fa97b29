"""The table decoder of groups of 8 (pvq_fast8.hip) on indices from all over their range: rows of encoded weights seldom hold
those whose bucket names more blocks than its entry has candidates, nor the ends of the tables."""
import numpy as np
import pytest

import paper_2410_16926_amd as pvq
import synth_inputs as si
from oracle import pvq_oracle as oracle
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("K,times", [(1, 1), (2, 1), (7, 1), (8, 1), (11, 1), (12, 1), (14, 1), (15, 1), (16, 1), (17, 1), (16, 200), (15, 200), (12, 200)])
def test_indices_from_all_over_their_range(K, times):
    # times = 200: tall enough for the kernel whose waves own rows
    rows, G, bits = 41, 256, oracle.index_bits(8, K)
    total = oracle.size_table(8, K)[8][K]
    rng = np.random.default_rng(si.BASE_SEED + 900 + K)
    idx = rng.integers(0, total, size=rows * G, dtype=np.uint64)
    ends = min(total, 500)
    idx[:ends] = np.arange(ends)
    idx[ends:2 * ends] = total - 1 - np.arange(ends)
    field = ((idx.reshape(rows, G, 1) >> np.arange(bits, dtype=np.uint64)) & np.uint64(1)).astype(np.uint8).reshape(rows, G * bits)
    words = np.zeros((rows, 4 * oracle.row_words(G, bits)), dtype=np.uint8)
    packed_bits = np.packbits(field, axis=1, bitorder="little")
    words[:, :packed_bits.shape[1]] = packed_bits
    y = oracle.unrank(idx, 8, K).astype(np.float64).reshape(rows, G, 8)
    amp = rng.uniform(0.5, 2.0, size=(rows, G)).astype(np.float32)
    ref = np.tile((amp[:, :, None] * y / np.sqrt((y * y).sum(axis=2, keepdims=True))).reshape(rows, G * 8), (times, 1))
    ctx = pvq.pvq_ctx_create(8, K)
    index = torch.from_numpy(words.view(np.int32).copy()).cuda().repeat(times, 1)
    scale = torch.from_numpy(amp).cuda().repeat(times, 1)
    p = pvq.Packed(rows * times, G * 8, index, scale, torch.ones(rows * times, device="cuda"))
    with gu.decoder_setting(0):
        gu.assert_decode_close(pvq.pvq_decode(ctx, p, torch.float32).cpu().numpy(), ref)
    for B in (1, 2, 5):
        xf, xb = si.activations(B, G * 8, seed=K + B)
        want, s = xf.astype(np.float64) @ ref.T, gu.product_scale(xf, ref)
        gu.assert_gemv_close(pvq.pvq_decode_gemv_on(ctx, p, gu.to_dev_bf16(xb), "table").cpu().numpy(), want, s)
    ctx.close()
