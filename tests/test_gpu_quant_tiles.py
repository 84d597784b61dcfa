"""The tile kernels of the quantizers (16 x 256 tiles; 16 M x 256 / M for an RHT block of 16 M) at their edges -- one block,
tiles cut in rows and columns, panels' padding, a single column, more tiles than one row of the grid -- and the register
kernels that take large tensors: codes and scales bit for bit the oracle's, buffers prefilled so that padding must be
written."""

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


def _x(rows, cols, seed):
    g = torch.Generator().manual_seed(seed)
    t = torch.randn(rows, (cols + 7) // 8 * 8, generator=g).bfloat16()
    return t[:, :cols]  # ld a multiple of 8, a ragged column count


def _blank(rows, red, fmt):
    q = U.empty_qtensor(rows, red, fmt)
    q.codes.fill_(0xAA)
    q.scales.fill_(7.0)
    return q


def _padding_is_zero(q):
    v = q.codes[:, : q.red // 16 * 1024].reshape(q.panels, q.red // 16, 128, 8).permute(0, 2, 1, 3)
    c = v.reshape(q.panels * 128, -1)[q.rows:]
    s = q.scales[:, : q.red // 16 * 128].reshape(q.panels, q.red // 16, 128).permute(0, 2, 1)
    return bool((c == 0).all()) and bool((s.reshape(q.panels * 128, -1)[q.rows:] == 0).all())


@pytest.mark.parametrize("shape", [(16, 1), (16, 16), (48, 257), (272, 255), (128, 520), (16 * 70000, 8)])
@pytest.mark.parametrize("fmt,rounding", [(O.UNIFORM, O.RTNE), (O.UNIFORM, O.SR), (O.E2M1, O.RTNE), (O.E2M1, O.SR)])
def test_transposed_tiles(shape, fmt, rounding):
    rows, cols = shape
    x = _x(rows, cols, rows + cols)
    xd = torch.empty(rows, (cols + 7) // 8 * 8, dtype=torch.bfloat16, device="cuda")
    xd[:, :cols] = x.cuda()
    q = _blank(cols, rows, fmt)
    fn = U.rht_quantize if fmt == O.UNIFORM else U.e2m1_quantize
    fn(xd[:, :cols], transpose=True, rht=True, sign_mask=0x1234, rounding=rounding, seed=9, stream_id=1, out=q)
    torch.cuda.synchronize()
    bits = WL.bf16_bits(x.contiguous())
    if rows < 10000:
        idx, sc = P.oracle_operand(bits, "cols", fmt, rounding, True, 0x1234, 9, 1)
        P.assert_codes_equal(*P.gpu_rows(q), idx, sc, fmt, f"{shape}")
    else:  # more blocks than one row of the grid: the last 256, at their block numbers (the draws count them)
        blk0 = rows // 16 - 256
        a = np.ascontiguousarray(O.bf16_bits_to_f32(bits[16 * blk0:]).T)
        idx, sc = O.quantize_rows(a, fmt, rounding, True, 0x1234, 9, 1, block_base=blk0)
        codes, scales = P.gpu_rows(q)
        P.assert_codes_equal(codes[:, 8 * blk0:], scales[:, blk0:], idx, sc, fmt, f"{shape}")
    assert _padding_is_zero(q)


@pytest.mark.parametrize("shape", [(16, 16), (144, 272), (272, 240)])
@pytest.mark.parametrize("fmt,rounding", [(O.UNIFORM, O.RTNE), (O.UNIFORM, O.SR), (O.E2M1, O.RTNE), (O.E2M1, O.SR)])
def test_dual_tiles(shape, fmt, rounding):
    rows, cols = shape
    x = _x(rows, cols, 3 * rows + cols)
    qr, qc = _blank(rows, cols, fmt), _blank(cols, rows, fmt)
    U.quantize_dual(x.cuda(), fmt=fmt, sign_mask_rows=0x11, sign_mask_cols=0x22, rounding=rounding, seed=4, stream_rows=2,
                    stream_cols=5, out_rows=qr, out_cols=qc)
    torch.cuda.synchronize()
    bits = WL.bf16_bits(x.contiguous())
    for q, layout, mask, stream in ((qr, "rows", 0x11, 2), (qc, "cols", 0x22, 5)):
        idx, sc = P.oracle_operand(bits, layout, fmt, rounding, True, mask, 4, stream)
        P.assert_codes_equal(*P.gpu_rows(q), idx, sc, fmt, f"{shape} {layout}")
        assert _padding_is_zero(q)


@pytest.mark.parametrize("n", [32, 64, 128])
@pytest.mark.parametrize("shape", [(1, 1), (3, 130), (2, 33)])  # n-blocks, columns
@pytest.mark.parametrize("fmt,rounding", [(O.UNIFORM, O.RTNE), (O.UNIFORM, O.SR), (O.E2M1, O.SR)])
def test_wide_rht_tiles(n, shape, fmt, rounding):
    rows, cols = shape[0] * n, shape[1]
    x = _x(rows, cols, n + rows + cols)
    xd = torch.empty(rows, (cols + 7) // 8 * 8, dtype=torch.bfloat16, device="cuda")
    xd[:, :cols] = x.cuda()
    mask = 0x123456789ABCDEF00FEDCBA987654321 & ((1 << n) - 1)
    q = _blank(cols, rows, fmt)
    U.quantize_rht_block(xd[:, :cols], fmt, rht_block=n, sign_mask=mask, transpose=True, rounding=rounding, seed=6,
                         stream_id=3, out=q)
    torch.cuda.synchronize()
    a = np.ascontiguousarray(O.bf16_bits_to_f32(WL.bf16_bits(x.contiguous())).T)
    y = O.rht_rows_n(a, mask, n)
    idx, sc = O.quantize_rows(y, fmt, rounding, False, 0, 6, 3)
    P.assert_codes_equal(*P.gpu_rows(q), idx, sc, fmt, f"n={n} {shape}")
    assert _padding_is_zero(q)


@pytest.mark.parametrize("fmt,rounding", [(O.UNIFORM, O.RTNE), (O.UNIFORM, O.SR), (O.E2M1, O.RTNE)])
def test_large_tensors_keep_the_codes(fmt, rounding):
    """A tensor past the tiles' size limit (register kernels) against the same blocks taken by the tiles: the first 4096
    rows quantized by themselves give the same first blocks (the draws are numbered by block and row)."""
    rows, cols = 16384, 6656  # 109 Mi elements
    g = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(rows, cols, generator=g, device="cuda").bfloat16()
    kw = dict(rounding=rounding, seed=8)
    fn = U.rht_quantize if fmt == O.UNIFORM else U.e2m1_quantize
    big = fn(x, transpose=True, rht=True, sign_mask=3, stream_id=1, **kw)
    part = fn(x[:4096], transpose=True, rht=True, sign_mask=3, stream_id=1, **kw)
    dr, dc = U.quantize_dual(x, fmt=fmt, sign_mask_rows=3, sign_mask_cols=3, stream_rows=0, stream_cols=1, **kw)
    one = fn(x, rht=True, sign_mask=3, stream_id=0, **kw)
    torch.cuda.synchronize()
    assert torch.equal(big.codes[:, : 256 * 1024], part.codes) and torch.equal(big.scales[:, : 256 * 128], part.scales)
    assert torch.equal(dc.codes, big.codes) and torch.equal(dc.scales, big.scales)
    assert torch.equal(dr.codes, one.codes) and torch.equal(dr.scales, one.scales)


def _grouped_tensor():
    """30000 tokens of 544 columns (three column tiles) in 300 groups, empty and one-token ones among them: runs of several
    tiles per workgroup that start and end inside a block's tiles, at blocks and at groups."""
    g = torch.Generator().manual_seed(12)
    counts = torch.randint(0, 200, (300,), generator=g).tolist()
    counts[0] = counts[7] = counts[8] = 0
    counts[5], counts[-1] = 1, 0
    counts[-2] += 30000 - sum(counts) if sum(counts) < 30000 else 0
    x = torch.randn(sum(counts), 544, generator=g).bfloat16().cuda()
    return x, counts


def _pad_groups(x, counts, block):
    """The rows of x with each group zero-padded to `block`, and the row of the result that every token has."""
    at, start = [], 0
    for c in counts:
        at += range(start, start + c)
        start += -(-c // block) * block
    at = torch.tensor(at, device="cuda")
    out = torch.zeros(start, x.shape[1], dtype=x.dtype, device="cuda")
    out[at] = x
    return out, at


@pytest.mark.parametrize("fmt,rounding", [(O.UNIFORM, O.RTNE), (O.UNIFORM, O.SR), (O.E2M1, O.RTNE), (O.E2M1, O.SR)])
@pytest.mark.parametrize("extra", [0, 4800])
def test_grouped_runs_of_tiles(fmt, rounding, extra):
    """The grouped transposed operand is the plain one of the zero-padded tensor, blocks past the last group zero."""
    x, counts = _grouped_tensor()
    off, red = U.group_offsets(counts, block=16)
    xp, _ = _pad_groups(x, counts, 16)
    assert xp.shape[0] == red
    xp = torch.cat((xp, xp.new_zeros(extra, x.shape[1])))
    q = _blank(x.shape[1], red + extra, fmt)
    kw = dict(sign_mask=0x4321, rounding=rounding, seed=5, stream_id=2)
    U.quantize_grouped_t(x, off, red + extra, fmt=fmt, out=q, **kw)
    fn = U.rht_quantize if fmt == O.UNIFORM else U.e2m1_quantize
    want = fn(xp, transpose=True, rht=True, **kw)
    torch.cuda.synchronize()
    assert torch.equal(q.codes, want.codes) and torch.equal(q.scales, want.scales)


@pytest.mark.parametrize("rounding", [O.RTNE, O.SR])
def test_mx_grouped_runs_of_tiles(rounding):
    """Power-of-two scales: the grouped reduction as above, and grouped rows against the plain operand's rows (the draws
    of a row are numbered by its token)."""
    x, counts = _grouped_tensor()
    kw = dict(sign_mask=0x4321, rounding=rounding, seed=5, stream_id=2)
    off, red = U.group_offsets(counts, block=32)
    qt = U.mx_quantize_grouped(x, off, red, transpose=True, **kw)
    want = U.mx_quantize(_pad_groups(x, counts, 32)[0], transpose=True, **kw)
    torch.cuda.synchronize()
    assert torch.equal(qt.codes, want.codes) and torch.equal(qt.scales, want.scales)
    off, rows = U.group_offsets(counts, block=128)
    qr = U.mx_quantize_grouped(x, off, rows, transpose=False, **kw)
    plain = U.mx_quantize(x, **kw)
    at = _pad_groups(x, counts, 128)[1]
    torch.cuda.synchronize()
    for got, ref in ((qr.codes_rows(), plain.codes_rows()), (qr.scales_rows(), plain.scales_rows())):
        assert torch.equal(got[at], ref)
        rest = torch.ones(rows, dtype=torch.bool, device="cuda")
        rest[at] = False
        assert bool((got[rest] == 0).all())


@pytest.mark.parametrize("fmt,rounding,rht,rows,cols", [
    (O.UNIFORM, O.RTNE, True, 16400, 6570), (O.UNIFORM, O.SR, True, 16400, 2650), (O.UNIFORM, O.SR, False, 16400, 6570),
    (O.E2M1, O.RTNE, True, 16400, 4200), (O.E2M1, O.RTNE, False, 16400, 6570), (O.E2M1, O.SR, False, 20016, 6890)])
def test_large_ragged_transposed(fmt, rounding, rht, rows, cols):
    """Just past the tiles' limit of each grid, rounding and transform: a column count that ends inside a thread's eight
    columns and inside a panel. The first 2048 rows by themselves (tiles) give the same first blocks; padding is zero."""
    ld = (cols + 7) // 8 * 8
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(rows, ld, generator=g, device="cuda").bfloat16()[:, :cols]
    fn = U.rht_quantize if fmt == O.UNIFORM else U.e2m1_quantize
    kw = dict(transpose=True, rht=rht, sign_mask=0x55 if rht else 0, rounding=rounding, seed=8, stream_id=1)
    big, part = _blank(cols, rows, fmt), _blank(cols, 2048, fmt)
    fn(x, out=big, **kw)
    fn(x[:2048], out=part, **kw)
    last = fn(x[rows - 2048:], **dict(kw, rounding=O.RTNE)) if rounding == O.RTNE else None
    torch.cuda.synchronize()
    n = 2048 // 16
    assert torch.equal(big.codes[:, : n * 1024], part.codes) and torch.equal(big.scales[:, : n * 128], part.scales)
    if last is not None:
        m = rows // 16
        assert torch.equal(big.codes[:, (m - n) * 1024: m * 1024], last.codes)
        assert torch.equal(big.scales[:, (m - n) * 128: m * 128], last.scales)
    assert _padding_is_zero(big)
