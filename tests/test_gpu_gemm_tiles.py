"""GPU parity of the block-scaled GEMM at sizes that take each of its kernels (32 x 32 and 64 x 64 direct tiles, 128 x 128
in one and two K groups, 128 x 64; asserted through the library's size rule), with partial tiles on both axes, partial K stages and a padded output, against the
oracle's fp64 product on sampled rows and columns around every tile edge.

Tolerance: the kernels add fp32 products of exact block sums in fp32, one rounding of 2^-24 per block and at most
K / 16 = 192 blocks here, so a relative Frobenius error below 192 * 2^-24 = 1.2e-5 in the worst case and about
sqrt(192) * 2^-24 = 8e-7 for independent roundings; 2e-6 is asked for fp32 outputs and 2^-8 for bf16 ones."""

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

# (M, N, K), the kernel that the size rule takes, the formats for which it does
BOTH = (O.UNIFORM, O.E2M1)
SHAPES = [
    ((33, 65, 16), "32x32", BOTH),  # a single block, one row and one column past a tile
    ((95, 64, 1552), "32x32", BOTH),  # 97 blocks over eight waves in groups of four
    ((1040, 2064, 1552), "64x64", BOTH),
    ((130, 1100, 3072), "32x32", BOTH),  # many rounds of groups
    ((1990, 2040, 2064), "128x128 in two K groups", BOTH),  # 129 blocks in stages of eight
    ((2900, 2000, 1008), "128x64", (O.UNIFORM,)),  # 63 blocks in stages of four
    ((2900, 2000, 1008), "128x128", (O.E2M1,)),
    ((250, 5328, 160), "128x64", BOTH),  # ten blocks
    ((6000, 8200, 272), "128x128", BOTH),  # 17 blocks in stages of four
    ((2700, 12768, 64), "128x128", BOTH),  # one full stage
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


@pytest.mark.parametrize("mnk,kernel,fmt", [(s, kernel, f) for s, kernel, fmts in SHAPES for f in fmts])
def test_every_gemm_kernel(mnk, kernel, fmt):
    m, n, k = mnk
    plan = ctypes.CDLL(U.library_path())
    assert rules.KERNELS[rules.gemm_kernel(plan, rules.DENSE, fmt, m, n, k)] == kernel
    g = torch.Generator().manual_seed(m + 3 * n + 7 * k + fmt)
    x = torch.randn(m, k, generator=g).bfloat16()
    w = (torch.randn(n, k, generator=g) * 0.02).bfloat16()
    xq = P.gpu_operand(x.cuda(), "rows", fmt, O.RTNE, True, 0x2345, 0, 0)
    wq = P.gpu_operand(w.cuda(), "rows", fmt, O.RTNE, True, 0x2345, 0, 0)
    rows, cols = _edges(m), _edges(n)
    ia, sa = P.oracle_operand(WL.bf16_bits(x), "rows", fmt, O.RTNE, True, 0x2345, 0, 0, rows)
    ib, sb = P.oracle_operand(WL.bf16_bits(w), "rows", fmt, O.RTNE, True, 0x2345, 0, 0, cols)
    want = O.gemm_nt(ia, sa, ib, sb, fmt)
    for dt, tol in ((torch.float32, 2e-6), (torch.bfloat16, 2.0 ** -8)):
        print(f"gemm {mnk} fmt {fmt} {dt}", flush=True)
        pad = (-n) % 8 + 8
        out = torch.full((m, n + pad), 7.0, dtype=dt, device="cuda")
        U.gemm_fwd_y(xq, wq, out=out[:, :n])
        torch.cuda.synchronize()
        assert bool((out[:, n:] == 7.0).all())
        got = P.to_numpy(out[torch.as_tensor(rows, device="cuda")][:, torch.as_tensor(cols, device="cuda")])
        assert P.rel_fro(got, want) <= tol


@pytest.mark.parametrize("counts", [[1] * 40, [33, 0, 65, 200, 1, 31], [700, 3, 400]])
def test_grouped_against_dense_per_group(counts):
    """Few tokens per group (small tiles): every group's rows equal the dense product of that group's rows up to the
    order of the fp32 sums (both within 2e-6 of the exact product), and rows past the last offset stay unwritten."""
    g = torch.Generator().manual_seed(sum(counts))
    E, N, K = len(counts), 144, 528
    x = torch.randn(sum(counts) + 3, K, generator=g).bfloat16().cuda()  # three rows past the last offset
    w = (torch.randn(E * N, K, generator=g) * 0.02).bfloat16().cuda()
    off, _ = U.group_offsets(counts)
    xq, wq = U.rht_quantize(x, sign_mask=0x77), U.rht_quantize(w, sign_mask=0x77)
    y = U.gemm_fwd_y_grouped(xq, wq, off, out=torch.full((sum(counts) + 3, N), 7.0, device="cuda"))
    torch.cuda.synchronize()
    assert bool((y[sum(counts):] == 7.0).all())
    at = 0
    for e, c in enumerate(counts):
        if c:
            xe = U.rht_quantize(x[at: at + c].contiguous(), sign_mask=0x77)
            we = U.rht_quantize(w[e * N: (e + 1) * N].contiguous(), sign_mask=0x77)
            ref = U.gemm_fwd_y(xe, we).double()
            assert float((y[at: at + c].double() - ref).norm() / ref.norm()) <= 4e-6
        at += c
