"""Stochastic rounding at the ends of the uniform grid: blocks whose sixteen magnitudes are all equal, so that every value
is RN(amax * RN(7 / amax)), 7 or one rounding step beside it, on both signs. Values above 7 are cut to it before the draw
(with a draw of 0 they would step to 8); bit for bit against the oracle, 2^23 values, so draws of 0 occur on them."""

import numpy as np
import pytest
import torch

from oracle import ufp4_oracle as O
from paper_2606_20381_amd import ufp4 as U
from paper_2606_20381_amd import workloads as WL
from tests import parity as P

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()


@pytest.mark.parametrize("layout", ["rows", "cols"])
def test_sr_at_the_top_level(layout):
    g = torch.Generator().manual_seed(5)
    rows, cols = 4096, 2048
    mag = (1.0 + torch.randint(0, 128, (rows // 16, cols // 16), generator=g) / 128.0).repeat_interleave(16, 0)
    x = (mag.repeat_interleave(16, 1) * (1 - 2 * torch.randint(0, 2, (rows, cols), generator=g))).bfloat16()
    # one magnitude per 16 x 16 square: both layouts see blocks of equal magnitudes
    q = P.gpu_operand(x.cuda(), layout, O.UNIFORM, O.SR, False, 0, 77, 1)
    torch.cuda.synchronize()
    idx, sc = P.oracle_operand(WL.bf16_bits(x), layout, O.UNIFORM, O.SR, False, 0, 77, 1)
    assert int(np.abs(idx).min()) >= 6  # every value lies at the top
    P.assert_codes_equal(*P.gpu_rows(q), idx, sc, O.UNIFORM, layout)
