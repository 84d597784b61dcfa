"""GPU parity of the power-of-two-scale GEMM at sizes that take each of its tiles (64, 128, 256; asserted through the
library's size rule), with partial tiles on
both axes, partial K stages and a padded output, against the oracle's fp64 product on sampled rows and columns around
every tile edge.

Tolerance: levels are integers times powers of two, the matrix core adds 64 products per instruction in fp32, so at most
K / 64 = 32 roundings of 2^-24 here: below 2e-6 relative for fp32 outputs; bf16 outputs round once more (2^-9, 2^-8 asked)."""

import ctypes

import numpy as np
import pytest
import torch

from oracle import ufp4_oracle as O
from paper_2606_20381_amd import ufp4 as U
from paper_2606_20381_amd import workloads as WL
from tests import parity as P
from tests import test_size_rules as rules

pytestmark = pytest.mark.gpu

# (M, N, K) and the tile that the size rule takes
SHAPES = [
    ((33, 65, 32), 64),  # one block, one row and one column past a tile
    ((200, 136, 1056), 64),  # 33 blocks in stages of four
    ((4000, 4100, 352), 64),  # 11 blocks, more workgroups than one round
    ((2000, 2040, 2080), 128),  # 65 blocks
    ((3900, 4000, 672), 256),  # 21 blocks, partial tiles on both axes
    ((8100, 8190, 96), 256),  # a single partial stage
]


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()


def _edges(n):
    """Indices on both sides of the tile edges inside [0, n), and the last one."""
    e = {0, n - 1}
    for t in (32, 64, 128, 256):
        last = (n - 1) // t * t
        e |= {i for i in (t - 1, t, last - 1, last) if 0 <= i < n}
    return np.array(sorted(e))


@pytest.mark.parametrize("mnk,tile", SHAPES)
def test_every_mx_tile(mnk, tile):
    m, n, k = mnk
    assert rules.mx_kernel(ctypes.CDLL(U.library_path()), rules.DENSE, m, n, k)[0] == tile
    g = torch.Generator().manual_seed(m + 3 * n + 7 * k)
    x = torch.randn(m, k, generator=g).bfloat16()
    w = (torch.randn(n, k, generator=g) * 0.02).bfloat16()
    xq, wq = U.mx_quantize(x.cuda(), sign_mask=0x2345), U.mx_quantize(w.cuda(), sign_mask=0x2345)
    rows, cols = _edges(m), _edges(n)
    ia, ea = O.quantize_rows_mx(O.bf16_bits_to_f32(WL.bf16_bits(x)[rows]), O.RTNE, True, 0x2345, 0, 0, row_ids=rows)
    ib, eb = O.quantize_rows_mx(O.bf16_bits_to_f32(WL.bf16_bits(w)[cols]), O.RTNE, True, 0x2345, 0, 0, row_ids=cols)
    want = O.gemm_nt_mx(ia, ea, ib, eb)
    for dt, tol in ((torch.float32, 2e-6), (torch.bfloat16, 2.0 ** -8)):
        print(f"mx gemm {mnk} {dt}", flush=True)
        pad = (-n) % 8 + 8
        out = torch.full((m, n + pad), 7.0, dtype=dt, device="cuda")
        U.mx_gemm_fwd_y(xq, wq, out=out[:, :n])
        torch.cuda.synchronize()
        assert bool((out[:, n:] == 7.0).all())
        got = P.to_numpy(out[torch.as_tensor(rows, device="cuda")][:, torch.as_tensor(cols, device="cuda")])
        assert P.rel_fro(got, want) <= tol


@pytest.mark.parametrize("counts", [[1] * 12, [33, 0, 65, 200, 1, 31]])
def test_mx_grouped_small_tiles(counts):
    """Few tokens per group (64-row tiles, half panels): each group's rows equal the dense product of its rows, and dW
    the dense product of its token range, up to fp32 rounding."""
    g = torch.Generator().manual_seed(sum(counts))
    E, N, K, M = len(counts), 128, 160, sum(counts)
    x = torch.randn(M, K, generator=g).bfloat16().cuda()
    w = (torch.randn(E * N, K, generator=g) * 0.02).bfloat16().cuda()
    dy = (torch.randn(M, N, generator=g) * 1e-3).bfloat16().cuda()
    off, prow = U.group_offsets(counts, block=128)
    _, red = U.group_offsets(counts, block=32)
    xq = U.mx_quantize_grouped(x, off, prow, transpose=False, sign_mask=0x77)
    wq = U.mx_quantize(w, sign_mask=0x77)
    y = U.mx_gemm_fwd_y_grouped(xq, wq, off, M)
    dw = U.mx_gemm_bwd_dw_grouped(U.mx_quantize_grouped(dy, off, red, transpose=True, sign_mask=0x77),
                                  U.mx_quantize_grouped(x, off, red, transpose=True, sign_mask=0x77), off)
    torch.cuda.synchronize()
    at = 0
    for e, c in enumerate(counts):
        if c:
            xe, dye = x[at: at + c].contiguous(), dy[at: at + c]
            ref = U.mx_gemm_fwd_y(U.mx_quantize(xe, sign_mask=0x77),
                                  U.mx_quantize(w[e * N: (e + 1) * N].contiguous(), sign_mask=0x77)).double()
            assert float((y[at: at + c].double() - ref).norm() / ref.norm()) <= 4e-6
            pad = -(-c // 32) * 32
            xp, dyp = x.new_zeros(pad, K), x.new_zeros(pad, N)
            xp[:c], dyp[:c] = xe, dye
            ref = U.mx_gemm_bwd_dw(U.mx_quantize(dyp, transpose=True, sign_mask=0x77),
                                   U.mx_quantize(xp, transpose=True, sign_mask=0x77)).double()
            assert float((dw[e].double() - ref).norm() / ref.norm()) <= 4e-6
        else:
            assert bool((dw[e] == 0).all())
        at += c
