"""Decoding of long groups, a lane per group with the rows of the tables brought to LDS by a wave of their own: the lines to
the decoder with a wave per group, and workgroups with few groups, at every width of the integers."""
import numpy as np
import pytest

import synth_inputs as si
from tests import test_gpu_parity as parity

pytestmark = pytest.mark.gpu


# the last number of groups that a wave each decodes and the first that lanes do; rows shorter than the window and of several
# windows; half of the groups with nearly all pulses in a few coordinates, so that places lie outside the window
@pytest.mark.parametrize("D,K,groups", [(128, 3, 4096), (128, 28, 4097), (128, 84, 3072), (128, 84, 3073), (128, 187, 2048), (128, 187, 2049),
                                        (128, 188, 2561), (128, 255, 2560), (128, 255, 2561), (64, 43, 4097), (64, 44, 3072), (64, 112, 3073),
                                        (64, 113, 3585), (64, 136, 4352), (64, 136, 4353), (64, 150, 4353)])
def test_long_groups_where_lanes_take_over(D, K, groups):
    X = si.activation_matrix(groups, D, seed=D + K + groups, rotate=False, bf16=False)
    odd = si.adversarial_groups(1 << 10, D, seed=K)
    X[1::2] = odd[np.arange(groups)[1::2] % len(odd)]
    parity.run_long_groups(X, D, K)
