"""Products with one, two and four vectors on the table decoder where a workgroup's waves have a row or two each, or none."""
import pytest
import torch

import paper_2410_16926_amd as pvq
import synth_inputs as si

pytestmark = pytest.mark.gpu


# rows of 36, 300, 448, 512, 1024, 1028 and 2048 groups (16, 8, 8, 8, 4, 3 and 2 row lanes): one row, a row fewer and more than a row for every
# row lane of 256 workgroups, two and three each with a ragged end
@pytest.mark.parametrize("K,bits,rows,groups", [(16, 2, 1, 36), (16, 0, 95, 36), (13, 4, 33, 300), (16, 8, 1100, 448), (16, 2, 2047, 512), (16, 1, 2049, 512),
                                                (16, 0, 1023, 1024), (16, 2, 1025, 1024), (16, 4, 2051, 1024), (16, 2, 3, 1028), (16, 2, 770, 1028),
                                                (17, 0, 1500, 1028), (16, 2, 515, 2048)])
def test_products_with_few_rows_for_a_wave(K, bits, rows, groups):
    g = torch.Generator(device="cuda")
    g.manual_seed(si.BASE_SEED + 700 + rows + groups)
    ctx = pvq.pvq_ctx_create(8, K, bits, *pvq.pvq_beta_tables(8, groups, bits)) if bits else pvq.pvq_ctx_create(8, K)
    packed = pvq.pvq_encode(ctx, torch.randn((rows, 8 * groups), generator=g, device="cuda") * 0.02)
    W = pvq.pvq_decode(ctx, packed, torch.float32).double()
    for batch in (1, 2, 4):
        x = torch.randn((batch, 8 * groups), generator=g, device="cuda").to(torch.bfloat16)
        ref = x.double() @ W.T
        # float32 sums of exact products: the size of an output whose terms do not cancel times 1e-5
        bound = 1e-5 * ((x.double() ** 2) @ (W ** 2).T).sqrt()
        for y in (pvq.pvq_decode_gemv_on(ctx, packed, x, "table"), pvq.pvq_decode_gemv(ctx, packed, x)):
            assert bool(((y.double() - ref).abs() <= bound).all())
    ctx.close()
