"""GPU parity of the error correction (Sec. 3.3 Step 6): the corrected weight matrix must equal the
oracle's bit for bit (every later rounding is decided from these values), and so must its code."""
import numpy as np
import pytest

import paper_2410_16926_amd as pvq
import synth_inputs as si
from oracle import pvq_oracle as oracle
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def run_correct(D, K, rows, cols, seed, amplitude="l2", scale_bits=0, ld_extra=0):
    W0 = np.asarray(si.gaussian_weights(rows, cols, 0.02, seed=seed, rotate=False, bf16=False), dtype=np.float32)
    _, U = si.calibration_hessian(cols, 2 * cols, seed + 1)
    ctx, oe, oc = gu.make_ctx(D, K, scale_bits, cols // D)
    if amplitude == "ls":
        ctx.set_amplitude("ls")
    Wd = torch.zeros((rows, cols + ld_extra), dtype=torch.float32, device="cuda")
    Wd[:, :cols] = gu.to_dev_f32(W0)
    Ud = torch.zeros((cols, cols + ld_extra), dtype=torch.float32, device="cuda")
    Ud[:, :cols] = gu.to_dev_f32(U)
    Wv, Uv = Wd[:, :cols], Ud[:, :cols]
    pvq.pvq_correct(ctx, Wv, Uv)
    torch.cuda.synchronize()
    got = Wv.cpu().numpy()
    ref, _ = oracle.correct(W0, U, D, K, amplitude=amplitude, nthreads=8)
    bad = np.argwhere(got.view(np.uint32) != ref.view(np.uint32))
    assert bad.size == 0, f"{bad.shape[0]} corrected weights differ, first at {bad[0]}: {got[tuple(bad[0])]} vs {ref[tuple(bad[0])]}"
    if ld_extra:
        assert torch.all(Wd[:, cols:] == 0)
    # and the code of the corrected matrix is the oracle's code of its corrected matrix
    packed = pvq.pvq_encode(ctx, Wv.contiguous(), want_pulses=True)
    enc = oracle.encode(ref, D, K, scale_bits, oe, nthreads=8, amplitude=amplitude)
    gu.assert_encode_equal(packed, enc)
    ctx.close()
    return W0, ref


@pytest.mark.parametrize("D,K,rows,cols,amplitude", [
    (8, 16, 200, 256, "l2"), (8, 16, 70, 512, "ls"), (8, 16, 1, 64, "l2"), (8, 16, 129, 192, "l2"),
    (16, 33, 130, 256, "l2"), (16, 33, 65, 128, "ls"), (32, 60, 64, 128, "l2"), (32, 60, 131, 320, "ls"),
    (8, 5, 300, 128, "l2")])
def test_corrected_weights_equal_the_oracles(D, K, rows, cols, amplitude):
    run_correct(D, K, rows, cols, seed=si.BASE_SEED + 500 + rows + cols, amplitude=amplitude)


def test_corrected_weights_with_amplitude_codes_and_leading_dimensions():
    # amplitude codes (Sec. 3.3 Step 5) are formed when the corrected matrix is encoded; W and U as views
    run_correct(8, 16, 96, 1024, seed=si.BASE_SEED + 541, scale_bits=2, ld_extra=12)


def test_a_wider_matrix():
    # 24 blocks of 64 columns, rows with a ragged end: the order of the updates across blocks
    run_correct(8, 16, 700, 1536, seed=si.BASE_SEED + 542)


@pytest.mark.parametrize("D,K,rows,cols", [(8, 16, 1100, 448), (16, 33, 300, 640), (32, 60, 150, 384), (8, 16, 2100, 320)])
def test_wide_updates_beside_the_next_panel(D, K, rows, cols):
    # from the third panel on a launch holds panel workgroups and update tasks of the panel before (several in
    # rows and columns, ragged ends), and the panels' t values alternate between two buffers; an odd number
    # of 64-column blocks ends in a half panel; the call is repeated on the same context
    W0, ref = run_correct(D, K, rows, cols, seed=si.BASE_SEED + 543 + rows)
    ctx = pvq.pvq_ctx_create(D, K)
    _, U = si.calibration_hessian(cols, 2 * cols, si.BASE_SEED + 543 + rows + 1)
    Ud = gu.to_dev_f32(U)
    for _ in range(2):
        Wd = gu.to_dev_f32(W0)
        pvq.pvq_correct(ctx, Wd, Ud)
        # work queued behind the call on the caller's stream sees the finished matrix
        got = (Wd + 0.0).cpu().numpy()
        assert np.array_equal(got.view(np.uint32), ref.view(np.uint32))
    ctx.close()


@pytest.mark.parametrize("D,K,rows,cols,amplitude", [(8, 16, 700, 1536, "l2"), (8, 16, 130, 448, "ls"), (16, 33, 300, 640, "l2"),
                                                     (32, 60, 150, 384, "ls"), (8, 5, 65, 320, "l2")])
def test_narrow_update_inside_the_panel_workgroups(D, K, rows, cols, amplitude):
    # The panel workgroups apply the panel before's update to their own columns, in every launch behind the first: the path of
    # all calls, here with other shapes and amplitudes than above.  The setter chooses no path (it keeps a number): what the
    # test adds is that a call between two settings gives the oracle's weights like any other.
    old = pvq.pvq_correct_set_front_tiles(1)
    try:
        run_correct(D, K, rows, cols, seed=si.BASE_SEED + 580 + rows + cols, amplitude=amplitude)
    finally:
        assert pvq.pvq_correct_set_front_tiles(old) == 1


@pytest.mark.parametrize("D,K,rows,cols", [(8, 16, 15, 384), (8, 16, 33, 448), (8, 16, 257, 512), (16, 33, 17, 384), (16, 33, 143, 448),
                                           (32, 60, 16, 448), (32, 60, 129, 320)])
def test_ragged_tiles_of_the_matrix_instructions(D, K, rows, cols):
    # rows around the 16 of an instruction and of a wave's turn of an update task, the 16 or 32 of a panel workgroup and the 64 of a
    # task's four waves; columns that end in half a panel and one task
    run_correct(D, K, rows, cols, seed=si.BASE_SEED + 630 + rows + cols, ld_extra=4)


def test_updates_of_tiny_weights_round_like_fused_multiply_adds():
    # weights around the smallest normal float: products and sums of the updates are subnormal or round there, and the
    # matrix instructions must keep every bit, as fmaf does
    D, K, rows, cols = 8, 16, 140, 512
    W0 = np.asarray(si.gaussian_weights(rows, cols, 0.02, seed=si.BASE_SEED + 641, rotate=False, bf16=False), dtype=np.float32)
    W0 *= np.exp2(-np.linspace(100, 124, rows)).astype(np.float32)[:, None]
    _, U = si.calibration_hessian(cols, 2 * cols, si.BASE_SEED + 642)
    ref, _ = oracle.correct(W0, U, D, K, nthreads=8)
    ctx = pvq.pvq_ctx_create(D, K)
    Wd = gu.to_dev_f32(W0)
    pvq.pvq_correct(ctx, Wd, gu.to_dev_f32(U))
    assert np.array_equal(Wd.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    ctx.close()


@pytest.mark.parametrize("D,K,amplitude", [(8, 16, "l2"), (8, 127, "ls"), (16, 33, "ls"), (16, 1, "l2"), (32, 60, "l2"), (32, 100, "ls")])
def test_groups_that_the_short_arithmetic_refuses(D, K, amplitude):
    # Divisions and roots of ordinary groups are short sequences that are right only between bounds; waves with other groups take
    # the general ones.  Beside ordinary rows: zeros of either sign, groups and rows of zeros, single values (whose error is
    # exactly zero in the norm's amplitude), values at and beyond the bounds' ends, and rows of U whose diagonal lies outside theirs.
    rows, cols = 150, 320
    rng = np.random.default_rng(si.BASE_SEED + 650 + D + K)
    W0 = np.asarray(si.gaussian_weights(rows, cols, 0.02, seed=si.BASE_SEED + 651, rotate=False, bf16=False), dtype=np.float32)
    W0[rng.random(W0.shape) < 0.02] = 0.0
    W0[rng.random(W0.shape) < 0.02] = -0.0
    W0[5] = 0.0
    W0[6] = -0.0
    W0[7, D:2 * D] = 0.0
    W0[8, :D] = 0.0
    W0[8, 3] = -0.75
    for r, e in zip(range(20, 52), (-126, -100, -70, -52, -50, -48, -46, -45, -44, -43, -42, 30, 40, 43, 44, 45)):
        W0[r] *= np.float32(2.0) ** e
    _, U = si.calibration_hessian(cols, 2 * cols, si.BASE_SEED + 652)
    for i, e in ((0, -22), (9, 22), (D + 1, -19), (130, 19), (200, -30), (319, 30)):
        U[i] *= np.float32(2.0) ** e
    ref, _ = oracle.correct(W0, U, D, K, amplitude=amplitude, nthreads=8)
    ctx = pvq.pvq_ctx_create(D, K)
    ctx.set_amplitude(amplitude if amplitude == "ls" else "norm")
    Wd = gu.to_dev_f32(W0)
    pvq.pvq_correct(ctx, Wd, gu.to_dev_f32(U))
    got = Wd.cpu().numpy()
    finite = np.isfinite(ref).all(axis=1)
    assert finite.sum() > rows * 0.9
    assert np.array_equal(got[finite].view(np.uint32), ref[finite].view(np.uint32))
    ctx.close()


@pytest.mark.parametrize("D,K,amplitude", [(8, 16, "l2"), (16, 33, "ls"), (32, 60, "l2")])
def test_groups_behind_groups_that_the_short_arithmetic_refuses(D, K, amplitude):
    # A wave that has met a group for the general operations has them for the next one too, until they find an ordinary one: runs
    # of such groups of every length from one on, at the start, the middle and the end of rows and panels, in some rows of a wave.
    rows, cols = 100, 448
    rng = np.random.default_rng(si.BASE_SEED + 655 + D)
    W0 = np.asarray(si.gaussian_weights(rows, cols, 0.02, seed=si.BASE_SEED + 656, rotate=False, bf16=False), dtype=np.float32)
    groups = W0.reshape(rows, cols // D, D)
    for r in range(0, rows, 3):
        run = 1 + r // 3 % 5
        for g in range(r % 7, cols // D, 2 * run):
            groups[r, g:g + run] *= np.float32(0.0 if r % 2 else 2.0 ** -60)
    W0[1] = 0.0
    W0[40:75] = 0.0
    _, U = si.calibration_hessian(cols, 2 * cols, si.BASE_SEED + 657)
    ref, _ = oracle.correct(W0, U, D, K, amplitude=amplitude, nthreads=8)
    ctx = pvq.pvq_ctx_create(D, K)
    ctx.set_amplitude(amplitude if amplitude == "ls" else "norm")
    Wd = gu.to_dev_f32(W0)
    pvq.pvq_correct(ctx, Wd, gu.to_dev_f32(U))
    assert np.array_equal(Wd.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    ctx.close()


@pytest.mark.parametrize("D,K,rows,cols", [(8, 16, 2049, 320), (8, 16, 1025, 448), (16, 33, 127, 384), (32, 60, 2177, 320)])
def test_rows_of_an_update_task(D, K, rows, cols):
    # steps of 64 rows, 16 rows a wave at a time: one row more and fewer than whole steps, and t values of a last
    # block of fewer than 16 rows
    run_correct(D, K, rows, cols, seed=si.BASE_SEED + 660 + rows)


@pytest.mark.parametrize("D,K,rows,cols", [(8, 16, 200, 384), (8, 16, 321, 448), (8, 16, 577, 448), (16, 33, 768, 384), (8, 16, 1281, 320)])
def test_rows_in_eight_chunks_or_fewer(D, K, rows, cols):
    # 4, 6, 10, 12 and 21 steps of 64 rows: in one chunk, 12 in four
    run_correct(D, K, rows, cols, seed=si.BASE_SEED + 680 + rows)


@pytest.mark.parametrize("D,K,rows,cols,ld_extra,two", [
    (8, 16, 511, 2048, 0, False), (8, 16, 512, 2048, 0, False), (8, 16, 513, 2112, 4, False), (16, 33, 1041, 2240, 8, False), (32, 60, 600, 2176, 0, False),
    (8, 16, 2048, 1984, 0, True), (8, 16, 1024, 4096, 0, True), (8, 16, 1023, 4096, 0, False), (8, 16, 1500, 2176, 4, True), (16, 33, 2041, 1408, 8, True),
    (32, 60, 1290, 2752, 0, True), (8, 16, 2049, 64, 0, None), (8, 16, 2100, 192, 0, None), (32, 60, 2180, 576, 4, True), (8, 5, 4100, 448, 0, True),
    (16, 33, 4112, 320, 0, True), (8, 16, 8200, 384, 0, True)])
def test_two_panels_a_launch(D, K, rows, cols, ld_extra, two):
    # the smallest work buffer has room for one panel a launch, twice as much for two (the rule's lines are at 2048 rows and at
    # 2^21 values behind the first 512 rows): the same bits, odd and even numbers of panels, the last one of 64 columns or 128, workgroups and shares with a ragged end,
    # and nothing written behind the buffer.  two: whether the larger buffer's second half, which a second launch of two panels has its t values in, is
    # touched (None: there is no second launch)
    g = torch.Generator(device="cuda")
    g.manual_seed(si.BASE_SEED + 670 + rows)
    W0 = torch.randn((rows, cols + ld_extra), generator=g, device="cuda") * 0.02
    U = torch.triu(torch.randn((cols, cols), generator=g, device="cuda") * (0.3 / cols ** 0.5), diagonal=1)
    U.diagonal().copy_(0.75 + 0.5 * torch.rand((cols,), generator=g, device="cuda"))
    ctx = pvq.pvq_ctx_create(D, K)
    results = []
    for size in (1024, 2048):
        whole = torch.full((rows * size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        W = W0.clone()
        pvq.pvq_correct(ctx, W[:, :cols], U, work=whole[: rows * size])
        assert bool((whole[rows * size:] == 0x5A).all())
        assert torch.equal(W[:, cols:], W0[:, cols:])
        results.append(W.view(torch.int32))
    if two is not None:
        assert bool((whole[rows * 1024: rows * 2048] == 0x5A).all()) == (not two)
    assert torch.equal(results[0], results[1])
    assert not torch.equal(results[0], W0.view(torch.int32)) or cols <= D
    ctx.close()


@pytest.mark.parametrize("rows,cols", [(2100, 320), (1570, 2048)])
@pytest.mark.parametrize("D,K,amplitude", [(8, 16, "l2"), (8, 127, "ls"), (16, 33, "ls"), (16, 58, "l2"), (32, 60, "l2"), (32, 100, "ls")])
def test_two_panels_a_launch_with_groups_that_the_short_arithmetic_refuses(D, K, amplitude, rows, cols):
    # both amplitudes in workgroups of 16 and of 32 rows; beside ordinary rows zeros of either sign, groups, runs of groups and rows of zeros, tiny
    # and huge values, in the first panel of a launch, in the second and across the two, and rows of U outside the bounds.  All such rows are compared
    # with the oracle, and ordinary ones of their workgroups
    rng = np.random.default_rng(si.BASE_SEED + 665 + D + K)
    W0 = (rng.standard_normal((rows, cols)) * 0.02).astype(np.float32)
    odd = np.arange(7, rows, 33)
    for n, r in enumerate(odd):
        g = W0[r].reshape(cols // D, D)
        kind, at = n % 8, (n // 8 * 5) % (cols // D)
        if kind == 0: W0[r] = 0.0
        elif kind == 1: W0[r] = -0.0
        elif kind == 2: g[at:] = 0.0
        elif kind == 3: g[at: at + 1 + n % 9] *= np.float32(2.0) ** -60
        elif kind == 4: W0[r] *= np.float32(2.0) ** (-126, -70, -52, -48, -45, -43)[n % 6]
        elif kind == 5: W0[r] *= np.float32(2.0) ** (30, 40, 43, 44)[n % 4]
        elif kind == 6: g[at] = 0.0; g[at, D - 1] = -0.75
        else: W0[r, rng.random(cols) < 0.3] = -0.0
    U = np.triu(rng.standard_normal((cols, cols)) * (0.3 / cols ** 0.5), 1).astype(np.float32)
    U[np.diag_indices(cols)] = (0.75 + 0.5 * rng.random(cols)).astype(np.float32)
    for i, e in ((0, -22), (9, 22), (127, -19), (130, 19), (200, -30), (255, 30)):
        U[i] *= np.float32(2.0) ** e
    some = np.unique(np.concatenate([odd, odd - 7, np.minimum(odd + 1, rows - 1), [rows - 1]]))
    ref, _ = oracle.correct(W0[some], U, D, K, amplitude=amplitude, nthreads=8)
    ctx = pvq.pvq_ctx_create(D, K)
    ctx.set_amplitude(amplitude if amplitude == "ls" else "norm")
    Wd, Ud = gu.to_dev_f32(W0), gu.to_dev_f32(U)
    work = torch.full((rows * 2048,), 0x5A, dtype=torch.uint8, device="cuda")
    pvq.pvq_correct(ctx, Wd, Ud, work=work)
    assert not bool((work[rows * 1024:] == 0x5A).all())          # two panels a launch
    got = Wd.cpu().numpy()[some]
    finite = np.isfinite(ref).all(axis=1)
    assert finite.sum() > len(some) * 0.9
    assert np.array_equal(got[finite].view(np.uint32), ref[finite].view(np.uint32))
    one = gu.to_dev_f32(W0)
    pvq.pvq_correct(ctx, one, Ud, work=work[: rows * 1024])
    fine = torch.isfinite(one).all(dim=1)
    assert torch.equal(one[fine].view(torch.int32), Wd[fine].view(torch.int32))
    ctx.close()


@pytest.mark.parametrize("D,K,rows,cols", [(8, 16, 4096, 320), (8, 16, 4097, 320), (16, 33, 2049, 448), (32, 60, 4096, 384), (8, 16, 1600, 1984)])
def test_the_library_s_own_work_buffer_with_two_panels_a_launch(D, K, rows, cols):
    # room for four buffers up to 4096 rows: the bits of a caller's work buffer of either size
    g = torch.Generator(device="cuda")
    g.manual_seed(si.BASE_SEED + 675 + rows)
    W0 = torch.randn((rows, cols), generator=g, device="cuda") * 0.02
    U = torch.triu(torch.randn((cols, cols), generator=g, device="cuda") * (0.3 / cols ** 0.5), diagonal=1)
    U.diagonal().copy_(0.75 + 0.5 * torch.rand((cols,), generator=g, device="cuda"))
    ctx = pvq.pvq_ctx_create(D, K)
    results = []
    for size in (None, 1024, 2048):
        W = W0.clone()
        if size is None:
            pvq.pvq_correct_static(ctx, W, U)
        else:
            pvq.pvq_correct(ctx, W, U, work=torch.empty((rows * size,), dtype=torch.uint8, device="cuda"))
        results.append(W.view(torch.int32))
    assert torch.equal(results[0], results[1]) and torch.equal(results[0], results[2])
    ctx.close()


@pytest.mark.parametrize("D,K,rows,cols,two", [
    (8, 16, 8192, 320, True), (8, 16, 8193, 320, True), (8, 16, 16384, 320, True), (8, 16, 16385, 320, False), (8, 16, 16400, 4096, True),
    (8, 16, 30720, 2048, False), (8, 16, 30721, 2048, True), (8, 16, 40000, 384, False), (16, 33, 8192, 320, True), (16, 33, 8193, 320, False),
    (16, 33, 8200, 4096, True), (32, 60, 12300, 320, False), (32, 60, 16390, 448, False)])
def test_more_panel_workgroups_than_have_a_place(D, K, rows, cols, two):
    # 32 rows a panel workgroup in groups of 8, else 16: 256, 512 and 960 of them and one more, few columns and many.  With the smallest work buffer
    # one panel a launch; with twice as much its second half is touched where a launch has two.  The same bits, and the oracle's for some rows
    g = torch.Generator(device="cuda")
    g.manual_seed(si.BASE_SEED + 690 + rows)
    W0 = torch.randn((rows, cols), generator=g, device="cuda") * 0.02
    U = torch.triu(torch.randn((cols, cols), generator=g, device="cuda") * (0.3 / cols ** 0.5), diagonal=1)
    U.diagonal().copy_(0.75 + 0.5 * torch.rand((cols,), generator=g, device="cuda"))
    ctx = pvq.pvq_ctx_create(D, K)
    one = W0.clone()
    pvq.pvq_correct(ctx, one, U, work=torch.empty((rows * 1024,), dtype=torch.uint8, device="cuda"))
    work = torch.full((rows * 2048,), 0x5A, dtype=torch.uint8, device="cuda")
    W = W0.clone()
    pvq.pvq_correct(ctx, W, U, work=work)
    assert torch.equal(one.view(torch.int32), W.view(torch.int32))
    assert bool((work[rows * 1024:] == 0x5A).all()) == (not two)
    some = [0, 31, rows // 2, rows - 17, rows - 1]
    ref, _ = oracle.correct(W0[some].cpu().numpy(), U.cpu().numpy(), D, K, nthreads=5)
    assert np.array_equal(W[some].cpu().numpy().view(np.uint32), ref.view(np.uint32))
    ctx.close()


@pytest.mark.parametrize("rows,cols,size", [(200, 256, 1024), (1100, 640, 1024), (2100, 640, 2048)])
def test_the_call_can_be_captured_in_a_graph_and_replayed(rows, cols, size):
    # kernels only, all on the capturing stream; every replay must reproduce the eager result for the weights
    # then in the buffer
    D, K = 8, 16
    ctx = pvq.pvq_ctx_create(D, K)
    _, U = si.calibration_hessian(cols, 2 * cols, si.BASE_SEED + 561)
    Ud = gu.to_dev_f32(U)
    W = torch.empty((rows, cols), dtype=torch.float32, device="cuda")
    work = torch.empty((rows * size,), dtype=torch.uint8, device="cuda")

    def fill(seed):
        W.copy_(gu.to_dev_f32(si.gaussian_weights(rows, cols, 0.02, seed=si.BASE_SEED + seed, rotate=False, bf16=False)))

    fill(1)
    pvq.pvq_correct(ctx, W, Ud, work=work)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    fill(1)
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            pvq.pvq_correct(ctx, W, Ud, work=work)
    torch.cuda.synchronize()
    for seed in (2, 3, 4):
        fill(seed)
        pvq.pvq_correct(ctx, W, Ud, work=work)
        torch.cuda.synchronize()
        want = W.clone()
        fill(seed)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(want, W)
    ctx.close()


def test_random_configurations():
    # seeded sweep: group size, pulse count, shape, amplitude kind, weight scale (bf16-valued weights in
    # every third case: exact ties are likelier) and damping drawn at random
    rng = np.random.default_rng(si.BASE_SEED + 570)
    for case in range(16):
        D = int(rng.choice([8, 16, 32]))
        K = int(rng.integers(1, {8: 22, 16: 40, 32: 70}[D]))
        rows = int(rng.integers(1, 400)); cols = 64 * int(rng.integers(1, 8))
        amp = str(rng.choice(["l2", "ls"]))
        sigma = float(rng.choice([1e-3, 0.02, 1.0, 50.0]))
        W0 = np.asarray(si.gaussian_weights(rows, cols, sigma, seed=3000 + case, rotate=False, bf16=False), dtype=np.float32)
        if case % 3 == 0:
            W0 = si.bf16_bits_to_f32(si.f32_to_bf16_bits(W0))
        _, U = si.calibration_hessian(cols, 2 * cols, 4000 + case, damp=float(rng.choice([0.01, 0.1])))
        ctx = pvq.pvq_ctx_create(D, K)
        if amp == "ls":
            ctx.set_amplitude("ls")
        Wd = gu.to_dev_f32(W0)
        pvq.pvq_correct(ctx, Wd, gu.to_dev_f32(U))
        ref, _ = oracle.correct(W0, U, D, K, amplitude=amp, nthreads=8)
        assert np.array_equal(Wd.cpu().numpy().view(np.uint32), ref.view(np.uint32)), (case, D, K, rows, cols, amp, sigma)
        ctx.close()


def test_corrected_code_has_the_lower_proxy_loss():
    # the point of the step (Sec. 2.1, Sec. 3.3 Step 6), end to end through the library: rotate-free synthetic
    # weights, correct, encode, decode; Tr((W - W_hat) H (W - W_hat)^T) against the plain code of the same matrix
    D, K, rows, cols = 8, 16, 48, 512
    W0 = np.asarray(si.gaussian_weights(rows, cols, 0.02, seed=93, rotate=False, bf16=False), dtype=np.float32)
    H, U = si.calibration_hessian(cols, 2 * cols, 94)
    ctx, _, _ = gu.make_ctx(D, K, 2, cols // D)

    def loss(What):
        d = W0.astype(np.float64) - What.astype(np.float64)
        return np.einsum("ri,ij,rj->", d, H, d)

    plain = pvq.pvq_decode(ctx, pvq.pvq_encode(ctx, gu.to_dev_f32(W0)), torch.float32).cpu().numpy()
    Wd = gu.to_dev_f32(W0)
    pvq.pvq_correct(ctx, Wd, gu.to_dev_f32(U))
    corrected = pvq.pvq_decode(ctx, pvq.pvq_encode(ctx, Wd), torch.float32).cpu().numpy()
    assert loss(corrected) < 0.7 * loss(plain)
    ctx.close()


@pytest.mark.parametrize("D,K", [(8, 16), (16, 33)])
def test_rounding_and_repair_ties_in_the_first_group(D, K):
    # every row starts with an adversarial group (half-integers after projection, repeated magnitudes, zeros,
    # one-hot, wide dynamic range): its point decides what the later columns receive
    rows, cols = 4096, 128
    W0 = np.asarray(si.gaussian_weights(rows, cols, 0.02, seed=97, rotate=False, bf16=False), dtype=np.float32)
    W0[:, :D] = si.adversarial_groups(rows, D, seed=98).reshape(rows, D)
    _, U = si.calibration_hessian(cols, 2 * cols, 99)
    ctx = pvq.pvq_ctx_create(D, K)
    Wd = gu.to_dev_f32(W0)
    pvq.pvq_correct(ctx, Wd, gu.to_dev_f32(U))
    ref, _ = oracle.correct(W0, U, D, K, nthreads=8)
    got = Wd.cpu().numpy()
    finite = np.isfinite(ref).all(axis=1)
    assert finite.sum() > rows * 0.9
    bad = np.argwhere(got[finite].view(np.uint32) != ref[finite].view(np.uint32))
    assert bad.size == 0, f"{bad.shape[0]} differ, first {bad[0]}"
    ctx.close()


def test_rows_that_are_not_finite_do_not_disturb_the_others():
    # rows are independent: rows of zeros, with infinities or not-a-numbers give unspecified values in those
    # rows only (and no fault); every other row still equals the oracle's
    D, K, rows, cols = 8, 16, 70, 256
    W0 = np.asarray(si.gaussian_weights(rows, cols, 0.02, seed=95, rotate=False, bf16=False), dtype=np.float32)
    W0[3] = 0.0
    W0[10, 17] = np.inf
    W0[20, 100] = np.nan
    W0[33, :8] = 3.0e38
    W0[47, 64:72] = 1.0e-44
    _, U = si.calibration_hessian(cols, 2 * cols, 96)
    ctx = pvq.pvq_ctx_create(D, K)
    Wd = gu.to_dev_f32(W0)
    pvq.pvq_correct(ctx, Wd, gu.to_dev_f32(U))
    torch.cuda.synchronize()
    got = Wd.cpu().numpy()
    ref, _ = oracle.correct(W0, U, D, K)
    clean = np.array([r for r in range(rows) if r not in (10, 20, 33)])
    assert np.array_equal(got[clean].view(np.uint32), ref[clean].view(np.uint32))
    assert np.all(got[3] == 0.0)
    ctx.close()


def test_entries_below_the_diagonal_are_not_used():
    D, K, rows, cols = 8, 16, 90, 192
    W0 = np.asarray(si.gaussian_weights(rows, cols, 0.02, seed=91, rotate=False, bf16=False), dtype=np.float32)
    _, U = si.calibration_hessian(cols, 2 * cols, 92)
    ref, _ = oracle.correct(W0, U, D, K)
    ctx = pvq.pvq_ctx_create(D, K)
    Wd = gu.to_dev_f32(W0)
    Ud = gu.to_dev_f32(U + np.tril(np.full((cols, cols), np.nan, dtype=np.float32), -1))
    pvq.pvq_correct(ctx, Wd, Ud)
    assert np.array_equal(Wd.cpu().numpy().view(np.uint32), ref.view(np.uint32))
    ctx.close()


def test_uncorrelated_inputs_leave_the_weights_alone():
    D, K, rows, cols = 8, 16, 50, 256
    W0 = np.asarray(si.gaussian_weights(rows, cols, 0.02, seed=77, rotate=False, bf16=False), dtype=np.float32)
    ctx = pvq.pvq_ctx_create(D, K)
    Wd = gu.to_dev_f32(W0)
    Ud = torch.diag(torch.linspace(0.5, 2.0, cols, device="cuda"))
    pvq.pvq_correct(ctx, Wd, Ud)
    assert np.array_equal(Wd.cpu().numpy().view(np.uint32), W0.view(np.uint32))
    ctx.close()


def test_argument_errors():
    ctx = pvq.pvq_ctx_create(8, 16)
    W = torch.zeros((4, 96), dtype=torch.float32, device="cuda")
    U = torch.eye(96, device="cuda")
    with pytest.raises(pvq.PvqError) as e:          # columns not in whole blocks of 64
        pvq.pvq_correct(ctx, W, U)
    assert e.value.status == -2
    W = torch.zeros((4, 128), dtype=torch.float32, device="cuda")
    U = torch.eye(128, device="cuda")
    with pytest.raises(pvq.PvqError) as e:          # work buffer too small
        pvq.pvq_correct(ctx, W, U, work=torch.empty((512,), dtype=torch.uint8, device="cuda"))
    assert e.value.status == -1
    pvq.pvq_correct(ctx, W[:0], U)                  # no rows: nothing to do
    ctx.close()
    wide = pvq.pvq_ctx_create(128, 187)
    with pytest.raises(pvq.PvqError) as e:
        pvq.pvq_correct(wide, W, U)
    assert e.value.status == -2
    wide.close()
