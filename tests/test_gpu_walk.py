"""The coordinate-by-coordinate decoder's kernels (pvq_walk.hip) beyond the shapes of test_gpu_parity.py."""
import numpy as np
import pytest

import paper_2410_16926_amd as pvq
import synth_inputs as si
from oracle import pvq_oracle as oracle
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_a_kernels_first_call_may_be_captured():
    # what a launch asks once per kernel must not disturb a capture (settings that no other test decodes)
    D, K, rows, cols = 32, 14, 40, 32 * 24
    W = si.gaussian_weights(rows, cols, 0.02, seed=si.BASE_SEED + 601, rotate=False)
    ctx = pvq.pvq_ctx_create(D, K)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W))
    xf, xb = si.activations(6, cols, seed=3)
    x = gu.to_dev_bf16(xb)
    out = torch.zeros((rows, cols), dtype=torch.float16, device="cuda")
    y = torch.zeros((6, rows), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        pvq.pvq_decode(ctx, packed, out=out)
        pvq.pvq_decode_gemv(ctx, packed, x, out=y)
    ref, _, _ = oracle.decode(oracle.encode(W, D, K))
    for _ in range(3):
        out.zero_(); y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert gu.ulp_f16(oracle.to_f16(ref).view(np.uint16), out.cpu().numpy().view(np.uint16)) <= 1
        gu.assert_gemv_close(y.cpu().numpy(), xf.astype(np.float64) @ ref.T, gu.product_scale(xf, ref))
    ctx.close()
