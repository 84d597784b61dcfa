"""GPU parity of ufp4_quant_stats at the edges of its launch: one block, workgroups of 256, 512 and 1024 threads with a
partial last one, and a grid that passes over the tensor more than once, where the (row, column) of a thread's block
advances by a remainder with carry. Counts exactly the oracle's; sums to a relative 1e-9 (at most 2^22.1 terms, each exact
to 2^-53 and added in another order: n * 2^-53 = 5e-10 of the sum of magnitudes)."""

import math

import numpy as np
import pytest
import torch

from oracle import ufp4_oracle as O
from paper_2606_20381_amd import ufp4 as U
from paper_2606_20381_amd import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()


# blocks: 1, 65520, 67600, 134160, 267280 (more than 256 workgroups of 1024)
@pytest.mark.parametrize("shape", [(16, 16), (1040, 1008), (1040, 1040), (2064, 1040), (4112, 1040)])
@pytest.mark.parametrize("fmt,rounding,rht,transpose", [(O.UNIFORM, O.RTNE, True, False), (O.E2M1, O.SR, False, True),
                                                        (O.UNIFORM, O.SR, False, False), (O.E2M1, O.RTNE, True, True)])
def test_stats_launch_edges(shape, fmt, rounding, rht, transpose):
    g = torch.Generator().manual_seed(shape[0] + shape[1])
    wide = torch.randn(shape[0], shape[1] + 8, generator=g).bfloat16()
    t = wide.cuda()[:, : shape[1]]
    print(f"{shape} fmt={fmt} rnd={rounding} rht={rht} t={transpose}", flush=True)
    got = U.quant_stats(t, fmt, transpose=transpose, rht=rht, sign_mask=0x35A7, rounding=rounding, seed=9, stream_id=1)
    a = O.bf16_bits_to_f32(WL.bf16_bits(wide[:, : shape[1]].contiguous()))
    want = O.quant_stats(a.T.copy() if transpose else a, fmt, rounding, rht, 0x35A7, 9, 1)
    assert got.hist == want["hist"].tolist()
    for k in ("err2", "ref2", "cross"):
        assert getattr(got, k) == pytest.approx(want[k], rel=1e-9), k


@pytest.mark.parametrize("transpose", [False, True])
@pytest.mark.parametrize("zeros", [False, True])
def test_stats_of_an_infinite_scale(transpose, zeros):
    """Blocks at the bf16 maximum whose rotated amax / 2 passes the fp32 range (E2M1 cut at 2): the scale is +inf, q of a
    zero level is NaN, and every sum with q in it is what the definition's arithmetic gives -- NaN with zero levels, +inf
    without -- while ref2 and the counts stay finite."""
    x = torch.full((16, 16), 3.3895e38).bfloat16()  # equal signs: 4 max, then fifteen zeros
    if not zeros:  # one value negated: 3.5 max, the others 0.5 max in magnitude, 0.286 of the levels' unit: 0.5
        x[:, 0] *= -1
    x = x.T.contiguous() if transpose else x
    kw = dict(max_fpx=2.0, transpose=transpose, rht=True, sign_mask=0, rounding=O.RTNE)
    got = U.quant_stats(x.cuda(), O.E2M1, **kw)
    a = O.bf16_bits_to_f32(WL.bf16_bits(x))
    with np.errstate(invalid="ignore"):  # 0 x inf
        want = O.quant_stats(a.T.copy() if transpose else a, O.E2M1, O.RTNE, True, 0, 0, 0, max_fpx=2.0)
    assert (want["hist"][0] > 0) == zeros
    assert got.hist == want["hist"].tolist() and got.ref2 == pytest.approx(want["ref2"], rel=1e-9)
    for k in ("err2", "cross"):
        g, w = getattr(got, k), want[k]
        assert math.isnan(g) if math.isnan(w) else g == w == math.inf, (k, g, w)
    assert math.isnan(want["cross"]) == zeros
