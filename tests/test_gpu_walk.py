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


@pytest.mark.parametrize("D,K", [(8, 16), (8, 127), (16, 33), (32, 60)])
def test_the_gain_is_no_further_off_than_a_rounded_root_and_quotient(D, K):
    # gain = amplitude / ||y||, seen where the pulse is a power of two and the product with it exact.  It is rounded once
    # (2^-24 of itself at most), and its correction carries half of the rounding of n2 * r (2^-24): 1.5 * 2^-24
    W = si.gaussian_weights(256, 4096, 0.02, seed=si.BASE_SEED + 610 + K, rotate=False)
    ctx = pvq.pvq_ctx_create(D, K)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W), want_pulses=True)
    got = pvq.pvq_decode(ctx, packed, torch.float32).cpu().numpy().reshape(-1, D).astype(np.float64)
    y = packed.pulses.cpu().numpy().reshape(-1, D).astype(np.float64)
    gain = packed.scale.cpu().numpy().reshape(-1, 1).astype(np.float64) / np.sqrt((y * y).sum(axis=1, keepdims=True))
    power = (y != 0) & (np.exp2(np.round(np.log2(np.maximum(np.abs(y), 1)))) == np.abs(y))
    assert power.mean() > 0.02
    err = np.abs(got / np.where(y == 0, 1, y) - gain)[power] / np.broadcast_to(gain, y.shape)[power]
    assert err.max() <= 1.5 * 2.0 ** -24, err.max() * 2.0 ** 24
    # an infinite amplitude: infinities, of the pulses' signs
    packed.scale.fill_(float("inf"))
    got = pvq.pvq_decode(ctx, packed, torch.float32).cpu().numpy().reshape(-1, D)
    assert np.array_equal(got[y != 0], np.copysign(np.inf, y[y != 0]))
    ctx.close()


@pytest.mark.parametrize("D,K,bits", [(8, 16, 2), (16, 33, 0), (32, 60, 4)])
@pytest.mark.parametrize("rows,groups,batch", [(5, 17, 1), (33, 19, 7), (21, 5, 16), (1030, 5, 5), (1030, 6, 16)])
def test_infinities_in_a_rows_last_group(D, K, bits, rows, groups, batch):
    # group counts that fill neither 16 nor 4 columns, so that the columns past the row's end hold the last group again: an
    # infinite activation there gives what float64 gives, infinities where the pulse is not 0 and no number where it is; and
    # large ones, whose dot products overflow (the group's pulses have one sign), give infinities
    cols = D * groups
    W = si.gaussian_weights(rows, cols, 0.02, seed=si.BASE_SEED + 620 + rows, rotate=False)
    W[:, -D:] = np.abs(W[:, -D:])
    ctx, oe, oc = gu.make_ctx(D, K, bits, groups)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W))
    ref, _, _ = oracle.decode(oracle.encode(W, D, K, bits, oe), oc)
    xf, _ = si.activations(batch, cols, seed=rows + batch)
    for value in (np.inf, -np.inf):
        xf[:, -3] = value
        y = pvq.pvq_decode_gemv(ctx, packed, gu.to_dev_bf16(si.f32_to_bf16_bits(xf.astype(np.float32)))).cpu().numpy()
        with np.errstate(invalid="ignore"):
            want = np.where(ref[:, -3] == 0, np.nan, value * ref[:, -3])
        assert np.array_equal(y, np.broadcast_to(want.astype(np.float32), y.shape), equal_nan=True)
    xf[:, -D:] = 3e38
    y = pvq.pvq_decode_gemv(ctx, packed, gu.to_dev_bf16(si.f32_to_bf16_bits(xf.astype(np.float32)))).cpu().numpy()
    assert np.all(y == np.inf)
    if bits == 0:
        xf[:, -D:] = 1.0
        packed.scale[:, -1] = np.inf
        y = pvq.pvq_decode_gemv(ctx, packed, gu.to_dev_bf16(si.f32_to_bf16_bits(xf.astype(np.float32)))).cpu().numpy()
        assert np.all(y == np.inf)
    ctx.close()


@pytest.mark.parametrize("D,K,bits,groups", [(8, 16, 2, 259), (16, 33, 4, 67), (32, 60, 0, 65), (32, 63, 2, 66), (16, 59, 0, 65)])
def test_products_with_many_tiles_for_a_workgroup(D, K, bits, groups):
    # more tiles of 4 and of 16 rows than workgroups at once, so that each takes several (the last one partial); group counts
    # that fill neither 16 nor 4 columns; the schedules of 32, 64 / 32, 128 / 96 / 64 / 32 and 128 / 64 / 32 bits; tables of
    # which a unit would hold three copies but for the steps LDS is given out in
    rows = 9001
    W = si.gaussian_weights(rows, D * groups, 0.02, seed=si.BASE_SEED + 640 + D, rotate=False)
    ctx, oe, oc = gu.make_ctx(D, K, bits, groups)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W))
    ref, _, _ = oracle.decode(oracle.encode(W, D, K, bits, oe, nthreads=8), oc, nthreads=8)
    for batch in (2, 7, 16):
        xf, xb = si.activations(batch, D * groups, seed=D + batch)
        want, scale = xf.astype(np.float64) @ ref.T, gu.product_scale(xf, ref)
        for _, y in gu.products(ctx, packed, gu.to_dev_bf16(xb)):
            gu.assert_gemv_close(y, want, scale)
    ctx.close()


@pytest.mark.parametrize("D,K,bits", [(32, 69, 4), (32, 105, 0), (16, 127, 2)])
@pytest.mark.parametrize("rows,groups", [(2049, 3), (5003, 20), (3100, 65)])
def test_products_with_several_teams_of_waves(D, K, bits, rows, groups):
    # tables that leave room for one workgroup to a unit, several tiles of rows for each: teams of 1, 4 and 16 waves, the
    # last turn with teams that have no tile
    W = si.gaussian_weights(rows, D * groups, 0.02, seed=si.BASE_SEED + 630 + rows, rotate=False)
    ctx, oe, oc = gu.make_ctx(D, K, bits, groups)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W))
    ref, _, _ = oracle.decode(oracle.encode(W, D, K, bits, oe, nthreads=8), oc, nthreads=8)
    for batch in (1, 5, 16):
        xf, xb = si.activations(batch, D * groups, seed=rows + batch)
        want, scale = xf.astype(np.float64) @ ref.T, gu.product_scale(xf, ref)
        x = gu.to_dev_bf16(xb)
        gu.assert_gemv_close(pvq.pvq_decode_gemv(ctx, packed, x).cpu().numpy(), want, scale)
        for tile_rows in (4, 16):
            gu.assert_gemv_close(pvq.pvq_decode_gemv_on(ctx, packed, x, "walk", tile_rows).cpu().numpy(), want, scale)
    ctx.close()


@pytest.mark.parametrize("K", [13, 33, 34, 36])
def test_rows_of_doubles(K):
    # the first and last indices, and points on and beside the axes, in the kernels that keep q as a double
    D, groups = 16, 33
    W = si.gaussian_weights(70, D * groups, 0.02, seed=si.BASE_SEED + 660 + K, rotate=False)
    for i in range(D):
        W[i, :D], W[i, D:2 * D] = 0.0, 0.0
        W[i, i], W[i, D + i] = 1.0, -1.0                    # +K and -K in one place
        W[i, D + (i + 5) % D] = 0.9 / K                     # nearly
    ctx = pvq.pvq_ctx_create(D, K)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W))
    ref, _, _ = oracle.decode(oracle.encode(W, D, K))
    gu.assert_decode_close(pvq.pvq_decode(ctx, packed, torch.float32).cpu().numpy(), ref)
    for batch in (1, 16):
        xf, xb = si.activations(batch, D * groups, seed=K + batch)
        want, scale = xf.astype(np.float64) @ ref.T, gu.product_scale(xf, ref)
        for _, y in gu.products(ctx, packed, gu.to_dev_bf16(xb)):
            gu.assert_gemv_close(y, want, scale)
    ctx.close()


@pytest.mark.parametrize("D,K,bits", [(8, 16, 2), (8, 100, 0), (16, 33, 4), (16, 60, 0), (32, 8, 1), (32, 60, 0), (32, 80, 2)])
@pytest.mark.parametrize("rows,groups", [(1, 2), (7, 7), (8, 8), (9, 9), (33, 131), (2061, 5)])
def test_products_with_tiles_of_eight_rows(D, K, bits, rows, groups):
    # two blocks of four rows share the activations of one of eight group columns: the ends of tiles, of the columns and of the
    # vectors that a block loads
    W = si.gaussian_weights(rows, D * groups, 0.02, seed=si.BASE_SEED + 670 + rows, rotate=False)
    ctx, oe, oc = gu.make_ctx(D, K, bits, groups)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W))
    ref, _, _ = oracle.decode(oracle.encode(W, D, K, bits, oe, nthreads=8), oc, nthreads=8)
    for batch in (1, 3, 4, 5, 8):
        xf, xb = si.activations(batch, D * groups, seed=rows + batch)
        want, scale = xf.astype(np.float64) @ ref.T, gu.product_scale(xf, ref)
        x = gu.to_dev_bf16(xb)
        gu.assert_gemv_close(pvq.pvq_decode_gemv_on(ctx, packed, x, "walk", 8).cpu().numpy(), want, scale)
    with pytest.raises(pvq.PvqError):
        pvq.pvq_decode_gemv_on(ctx, packed, gu.to_dev_bf16(si.activations(9, D * groups, seed=1)[1]), "walk", 8)
    ctx.close()


@pytest.mark.parametrize("rows,cols,batch,kind", [(1025, 8192, 9, "mfma_bf16"), (1025, 8192, 16, "mfma_bf16"), (1025, 8192, 8, "valu_fp32_generic"),
                                                  (1024, 8192, 9, "valu_fp32_generic"), (1024, 8704, 16, "valu_fp32_generic"),
                                                  (1025, 8000, 9, "valu_fp32_generic"), (2040, 4096, 9, "valu_fp32_generic"),
                                                  (2051, 4096, 11, "mfma_bf16")])
def test_products_at_the_line_between_the_decoders(rows, cols, batch, kind):
    # more than eight vectors from 2^20 groups on, on more than 1024 rows of whole slabs
    W = si.gaussian_weights(rows, cols, 0.02, seed=si.BASE_SEED + 680 + rows, rotate=False)
    ctx, oe, oc = gu.make_ctx(8, 16, 2, cols // 8)
    assert pvq.pvq_decode_gemv_plan(ctx, rows, cols, batch) == [(kind, batch)]
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(W))
    ref, _, _ = oracle.decode(oracle.encode(W, 8, 16, 2, oe, nthreads=8), oc, nthreads=8)
    xf, xb = si.activations(batch, cols, seed=rows + batch)
    want, scale = xf.astype(np.float64) @ ref.T, gu.product_scale(xf, ref)
    for _, y in gu.products(ctx, packed, gu.to_dev_bf16(xb)):
        gu.assert_gemv_close(y, want, scale)
    ctx.close()
