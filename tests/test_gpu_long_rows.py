"""Decoding of long groups, a lane per group with the rows of the tables brought to LDS by a wave of their own: the lines to
the decoder with a wave per group, and workgroups with few groups, at every width of the integers."""
import numpy as np
import pytest

import paper_2410_16926_amd as pvq
import synth_inputs as si
from tests import gpu_util as gu
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


# the last number of groups that a wave each decodes and the first that lanes do; rows shorter than the window and of several
# windows; half of the groups with nearly all pulses in a few coordinates, so that places lie outside the window
@pytest.mark.parametrize("D,K,groups", [(128, 3, 4096), (128, 28, 4097), (128, 84, 3072), (128, 84, 3073), (128, 187, 2048), (128, 187, 2049),
                                        (128, 188, 2561), (128, 255, 2560), (128, 255, 2561), (64, 43, 4097), (64, 44, 3072), (64, 112, 3073),
                                        (64, 113, 3585), (64, 136, 4352), (64, 136, 4353), (64, 143, 4353), (64, 144, 4353), (64, 150, 4353), (64, 150, 4800), (64, 150, 4801)])
def test_long_groups_where_lanes_take_over(D, K, groups):
    X = si.activation_matrix(groups, D, seed=D + K + groups, rotate=False, bf16=False)
    odd = si.adversarial_groups(1 << 10, D, seed=K)
    X[1::2] = odd[np.arange(groups)[1::2] % len(odd)]
    parity.run_long_groups(X, D, K)


# large batches, block after block the same, and the block by itself the oracle's (workgroups of 128 lanes): workgroups of 512 and of 448 lanes, in one launch and in launches of 512 workgroups, rows of
# the tables in LDS and in device memory (D = 64, K = 121), each with a ragged end
@pytest.mark.parametrize("D,K,times", [(64, 40, 152), (64, 40, 153), (64, 43, 170), (64, 44, 91), (64, 44, 92), (64, 112, 123), (64, 120, 92), (64, 121, 92),
                                       (128, 28, 153), (128, 84, 122), (128, 84, 123), (128, 187, 110), (128, 188, 89), (128, 188, 92), (128, 255, 110),
                                       (128, 255, 150), (128, 255, 185)])
def test_long_groups_in_workgroups_that_follow_one_another(D, K, times):
    rows, groups = 613, 7
    X = si.activation_matrix(rows, D * groups, seed=D + K, rotate=False, bf16=False)
    odd = si.adversarial_groups(1 << 10, D, seed=K)
    X.reshape(rows * groups, D)[3::29] = odd[np.arange(rows * groups)[3::29] % len(odd)]
    parity.run_long_groups(X, D, K)
    ctx = pvq.pvq_ctx_create(D, K)
    packed = pvq.pvq_encode(ctx, gu.to_dev_f32(X))
    packed.index[rows // 2] = -1                     # no codewords: zeros
    block = pvq.pvq_decode(ctx, packed, torch.float32)
    many = pvq.Packed(rows * times, packed.cols, packed.index.repeat(times, 1), packed.scale.repeat(times, 1), None)
    got = pvq.pvq_decode(ctx, many, torch.float32).view(times, rows, -1)
    assert torch.equal(got, block.expand_as(got))
    assert torch.all(block[rows // 2] == 0)
    ctx.close()
