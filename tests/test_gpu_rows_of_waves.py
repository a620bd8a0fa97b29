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


# (rows, groups, vectors, on the tables): one row a wave and one tile of the walk a unit; more rows than tiles; fewer; as many
@pytest.mark.parametrize("rows,groups,batch,table", [(512, 956, 1, False), (512, 960, 1, True), (8, 960, 1, True), (1024, 1084, 2, False), (768, 1084, 2, False),
                                                     (768, 1088, 2, True), (769, 1028, 2, False), (1024, 1280, 2, False), (1024, 1284, 2, True),
                                                     (769, 1028, 1, False), (1025, 436, 1, False), (1025, 440, 2, True), (2049, 476, 2, False), (2049, 480, 2, True),
                                                     (2049, 440, 1, True), (1100, 656, 2, True), (1400, 656, 1, False), (1400, 660, 2, True), (1030, 1000, 1, True)])
def test_lines_between_the_tables_and_the_walk_for_one_and_two_vectors(rows, groups, batch, table):
    g = torch.Generator(device="cuda")
    g.manual_seed(si.BASE_SEED + 710 + rows + groups)
    ctx = pvq.pvq_ctx_create(8, 16)
    assert pvq.pvq_decode_gemv_plan(ctx, rows, 8 * groups, batch) == [("valu_fp32" if table else "valu_fp32_generic", batch)]
    packed = pvq.pvq_encode(ctx, torch.randn((rows, 8 * groups), generator=g, device="cuda") * 0.02)
    W = pvq.pvq_decode(ctx, packed, torch.float32).double()
    x = torch.randn((batch, 8 * groups), generator=g, device="cuda").to(torch.bfloat16)
    # float32 sums of exact products: the size of an output whose terms do not cancel times 1e-5
    bound = 1e-5 * ((x.double() ** 2) @ (W ** 2).T).sqrt()
    assert bool(((pvq.pvq_decode_gemv(ctx, packed, x).double() - x.double() @ W.T).abs() <= bound).all())
    ctx.close()
