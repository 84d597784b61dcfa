"""GPU parity of the grouped GEMMs on every kernel that the size rules choose from: the five of the per-16 GEMM and the three
tiles of the power-of-two-scale one, over ragged rows (fwd_y, bwd_dx) and a ragged reduction (bwd_dw), each asserted to be
the kernel taken. Groups are empty, of one token, across panels and tiles; columns and reductions end inside a tile and a stage; rows past
the last group stay unwritten. Against the oracle's fp64 products on rows and columns around the edges of every group,
tile and panel.

Tolerance: fp32 products of exact block sums added in fp32, at most 3088 / 16 roundings of 2^-24 and 8e-7 for independent
ones: 2e-6. A group's few sampled outputs are compared together, against the norm of all of the sample."""

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

TOL = 2e-6
MASK = 0x2345
SPARE = 5  # rows of the output past the last group


@pytest.fixture(scope="module")
def plan():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    U.lib()
    return ctypes.CDLL(U.library_path())


def _counts(scale):
    return [c if c <= 1 else c * scale + (3 if scale > 1 else 0) for c in (0, 1, 77, 130, 0, 300, 64, 200, 33, 128)]


def _edges(n):
    e = {0, n - 1}
    for t in (32, 64, 128, 256):
        last = (n - 1) // t * t
        e |= {i for i in (t - 1, t, last - 1, last) if 0 <= i < n}
    return np.array(sorted(e))


def _tensors(counts, n, k, seed):
    g = torch.Generator().manual_seed(seed)
    m, groups = sum(counts), len(counts)
    x = torch.randn(m, k, generator=g).bfloat16()
    w = (torch.randn(groups * n, k, generator=g) * 0.02).bfloat16()
    dy = (torch.randn(m, n, generator=g) * 1e-3).bfloat16()
    return x, w, dy


def _starts(counts, pad=1):
    return np.concatenate([[0], np.cumsum([-(-c // pad) * pad for c in counts])]).astype(np.int64)


def _pick(t, rows, cols):
    return P.to_numpy(t[torch.as_tensor(rows, device="cuda")][:, torch.as_tensor(cols, device="cuda")])


def _check_rows(y, counts, n, product):
    """y [tokens + SPARE, n] against product(group, token rows, columns) around the edges; the spare rows untouched."""
    m, got, want = sum(counts), [], []
    assert bool((y[m:] == 7.0).all())
    start, cols = _starts(counts), _edges(n)
    for e, c in enumerate(counts):
        if c:
            rows = start[e] + _edges(c)
            got.append(_pick(y, rows, cols).ravel())
            want.append(product(e, rows, cols).ravel())
    assert P.rel_fro(np.concatenate(got), np.concatenate(want)) <= TOL


def _check_dw(dw, counts, product):
    """dw [groups, n, k] against product(group, rows, columns); groups without tokens are zero."""
    rows, cols, got, want = _edges(dw.shape[1]), _edges(dw.shape[2]), [], []
    for e, c in enumerate(counts):
        if c:
            got.append(_pick(dw[e], rows, cols).ravel())
            want.append(product(e, rows, cols).ravel())
        else:
            assert bool((dw[e] == 0).all())
    assert P.rel_fro(np.concatenate(got), np.concatenate(want)) <= TOL


def _padded_x(x, spare):
    """x with spare rows: the operand holds more rows than the offsets cover."""
    return torch.cat((x, torch.ones(spare, x.shape[1]).bfloat16()))


# kernel -> (scale of the counts, columns, reduction)
ROWS = [("128x128", 1, 784, 80), ("128x128 in two K groups", 16, 208, 1008), ("128x64", 1, 784, 208), ("32x32", 1, 80, 80),
        ("64x64", 1, 784, 336)]


@pytest.mark.parametrize("kernel,scale,n,k", ROWS)
@pytest.mark.parametrize("fmt", [O.UNIFORM, O.E2M1])
@pytest.mark.parametrize("which", ["fwd_y", "bwd_dx"])
def test_ragged_rows(plan, kernel, scale, n, k, fmt, which):
    """fwd_y: weights [groups * n, k]; bwd_dx: weights [groups * k, n] transposed, the same product with the weight's blocks
    found along the reduction."""
    counts = _counts(scale)
    m, groups = sum(counts), len(counts)
    assert rules.KERNELS[rules.gemm_kernel(plan, rules.RAGGED_M, fmt, m + SPARE, n, k, groups)] == kernel
    x, w, _ = _tensors(counts, n, k, scale + n + k)
    off, _ = U.group_offsets(counts)
    xq = P.gpu_operand(_padded_x(x, SPARE).cuda(), "rows", fmt, O.RTNE, True, MASK, 0, 0)
    y = torch.full((m + SPARE, n), 7.0, device="cuda")
    if which == "fwd_y":
        U.gemm_fwd_y_grouped(xq, P.gpu_operand(w.cuda(), "rows", fmt, O.RTNE, True, MASK, 0, 0), off, out=y)
    else:
        # W [groups * k, n] with W_e = w_e^T, quantized along its rows: W^T [n, groups * k]
        wd = w.view(groups, n, k).transpose(1, 2).reshape(groups * k, n).contiguous()
        U.gemm_bwd_dx_grouped(xq, P.gpu_operand(wd.cuda(), "cols", fmt, O.RTNE, True, MASK, 0, 0), off, out=y)
    torch.cuda.synchronize()
    xb, wb = WL.bf16_bits(x), WL.bf16_bits(w)

    def product(e, rows, cols):
        a = P.oracle_operand(xb, "rows", fmt, O.RTNE, True, MASK, 0, 0, rows)
        b = P.oracle_operand(wb, "rows", fmt, O.RTNE, True, MASK, 0, 0, e * n + cols)
        return O.gemm_nt(*a, *b, fmt)

    _check_rows(y, counts, n, product)


RED = [("128x128", O.UNIFORM, 1, 144, 784), ("128x128", O.E2M1, 1, 144, 784),
       ("128x128 in two K groups", O.UNIFORM, 16, 80, 3088), ("128x128 in two K groups", O.E2M1, 16, 80, 3088),
       ("128x64", O.UNIFORM, 1, 208, 336), ("128x64", O.E2M1, 1, 208, 336), ("32x32", O.UNIFORM, 1, 80, 80),
       ("32x32", O.E2M1, 1, 80, 80), ("64x64", O.UNIFORM, 2, 1552, 80), ("64x64", O.E2M1, 1, 144, 1552)]


@pytest.mark.parametrize("kernel,fmt,scale,n,k", RED)
def test_ragged_reduction(plan, kernel, fmt, scale, n, k):
    counts = _counts(scale)
    off, red = U.group_offsets(counts)
    assert rules.KERNELS[rules.gemm_kernel(plan, rules.RAGGED_K, fmt, n, k, red, len(counts))] == kernel
    x, _, dy = _tensors(counts, n, k, scale + n + k)
    dytq = U.quantize_grouped_t(dy.cuda(), off, red, fmt=fmt, sign_mask=MASK)
    xtq = U.quantize_grouped_t(x.cuda(), off, red, fmt=fmt, sign_mask=MASK)
    dw = torch.full((len(counts), n, k), 7.0, device="cuda")
    U.gemm_bwd_dw_grouped(dytq, xtq, off, out=dw)
    torch.cuda.synchronize()
    rows, cols = _edges(n), _edges(k)
    ia, sa, poff = P.oracle_operand_grouped(WL.bf16_bits(dy), counts, fmt, O.RTNE, True, MASK, 0, 0, rows)
    ib, sb, _ = P.oracle_operand_grouped(WL.bf16_bits(x), counts, fmt, O.RTNE, True, MASK, 0, 0, cols)

    def product(e, r, c):
        s, b = slice(poff[e], poff[e + 1]), slice(poff[e] // 16, poff[e + 1] // 16)
        return O.gemm_nt(ia[:, s], sa[:, b], ib[:, s], sb[:, b], fmt)

    _check_dw(dw, counts, product)


MX_ROWS = [(64, 1, 128, 160), (128, 1, 2048, 160), (256, 3, 2048, 224)]


@pytest.mark.parametrize("tile,scale,n,k", MX_ROWS)
def test_mx_ragged_rows(plan, tile, scale, n, k):
    counts = _counts(scale)
    m, groups = sum(counts), len(counts)
    off, prow = U.group_offsets(counts, block=128)
    assert rules.mx_kernel(plan, rules.RAGGED_M, m, n, k, groups, prow)[0] == tile
    x, w, _ = _tensors(counts, n, k, scale + n + k)
    xq = U.mx_quantize_grouped(x.cuda(), off, prow, transpose=False, sign_mask=MASK)
    xb, wb = WL.bf16_bits(x), WL.bf16_bits(w)

    def product(e, rows, cols):
        a = O.quantize_rows_mx(O.bf16_bits_to_f32(xb[rows]), O.RTNE, True, MASK, 0, 0, row_ids=rows)
        b = O.quantize_rows_mx(O.bf16_bits_to_f32(wb[e * n + cols]), O.RTNE, True, MASK, 0, 0, row_ids=e * n + cols)
        return O.gemm_nt_mx(*a, *b)

    for which in ("fwd_y", "bwd_dx"):
        y = torch.full((m + SPARE, n), 7.0, device="cuda")
        if which == "fwd_y":
            U.mx_gemm_fwd_y_grouped(xq, U.mx_quantize(w.cuda(), sign_mask=MASK), off, m, out=y[:m])
        else:
            wd = w.view(groups, n, k).transpose(1, 2).reshape(groups * k, n).contiguous()
            U.mx_gemm_bwd_dx_grouped(xq, U.mx_quantize(wd.cuda(), transpose=True, sign_mask=MASK), off, m, out=y[:m])
        torch.cuda.synchronize()
        _check_rows(y, counts, n, product)


MX_RED = [(64, 1, 144, 112), (128, 1, 1136, 368), (256, 2, 880, 1072)]


@pytest.mark.parametrize("tile,scale,n,k", MX_RED)
def test_mx_ragged_reduction(plan, tile, scale, n, k):
    counts = _counts(scale)
    off, red = U.group_offsets(counts, block=32)
    assert rules.mx_kernel(plan, rules.RAGGED_K, n, k, red, len(counts))[0] == tile
    x, _, dy = _tensors(counts, n, k, scale + n + k)
    dytq = U.mx_quantize_grouped(dy.cuda(), off, red, transpose=True, sign_mask=MASK)
    xtq = U.mx_quantize_grouped(x.cuda(), off, red, transpose=True, sign_mask=MASK)
    dw = torch.full((len(counts), n, k), 7.0, device="cuda")
    U.mx_gemm_bwd_dw_grouped(dytq, xtq, off, out=dw)
    torch.cuda.synchronize()
    ops = []
    for t, ids in ((dy, _edges(n)), (x, _edges(k))):
        a, poff = O.operand_colwise_grouped(np.ascontiguousarray(WL.bf16_bits(t)[:, ids]), counts, block=32)
        ops.append(O.quantize_rows_mx(a, O.RTNE, True, MASK, 0, 0, row_ids=ids))

    def product(e, r, c):
        s, b = slice(poff[e], poff[e + 1]), slice(poff[e] // 32, poff[e + 1] // 32)
        (ia, ea), (ib, eb) = ops
        return O.gemm_nt_mx(ia[:, s], ea[:, b], ib[:, s], eb[:, b])

    _check_dw(dw, counts, product)


def test_workgroups_per_cu_are_what_the_rules_count_on(plan):
    """A register more than a kernel's bound leaves fewer workgroups per CU than its cost row assumes."""
    costed = ctypes.c_int()
    for fmt in (O.UNIFORM, O.E2M1):
        for out in (0, 1):
            for k, name in enumerate(rules.KERNELS):
                n = plan.ufp4_plan_gemm_resident(k, fmt, out, ctypes.byref(costed))
                assert n == costed.value, (name, fmt, out, n)
        for rounding in (O.RTNE, O.SR):
            n = plan.ufp4_plan_grouped_resident(0, 0, fmt, rounding, ctypes.byref(costed))
            assert n == costed.value, (fmt, rounding, n)
    for k in range(3):
        for out in (0, 1):
            assert plan.ufp4_plan_gemm_mx_resident(k, out, ctypes.byref(costed)) == costed.value, (k, out)
    for rows in (0, 1):
        for rounding in (O.RTNE, O.SR):
            assert plan.ufp4_plan_grouped_resident(1, rows, 0, rounding, ctypes.byref(costed)) == costed.value
