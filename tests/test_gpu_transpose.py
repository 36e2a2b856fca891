"""GPU parity of the transposition (spl_transpose) and of CSC operands read
through it: B^T's pos, crd and vals bit for bit against the oracle's
transposition (one, two and three radix passes; empty matrices, empty rows
and columns, one row or column; the 2,000,000-row power-law matrix at full
size), repeated calls identical, and SpMV of a CSC matrix against the
oracle's plain CSC definition."""
import numpy as np
import pytest
import torch

import oracle
from tests import tiny
from tests.gpu_util import assert_close, host64, need_gpu
from workloads import configs

pytestmark = pytest.mark.gpu


def _spl():
    need_gpu()
    import paper_2207_13901_amd as spl
    return spl


def _dev():
    return torch.device("cuda", 0)


def _csr(spl, pos, crd, vals, shape, dtype=torch.float64):
    d = _dev()
    return spl.CSR(torch.as_tensor(np.asarray(pos, np.int32), device=d),
                   torch.as_tensor(np.asarray(crd, np.int32), device=d),
                   torch.as_tensor(np.asarray(vals, np.float64)).to(dtype).to(d), shape)


def _check(spl, B, what):
    T = spl.transpose(B)
    n, m = B.shape
    rp, rc, rv = oracle.transpose(B.pos.cpu().numpy(), B.crd.cpu().numpy(), host64(B.vals),
                                  (n, m))
    assert T.shape == (m, n)
    assert np.array_equal(T.pos.cpu().numpy(), rp), what
    assert np.array_equal(T.crd.cpu().numpy(), rc), what
    assert np.array_equal(host64(T.vals), rv), what
    assert T.vals.dtype == B.vals.dtype
    return T


@pytest.mark.parametrize("n,m,density", [(50, 7, 0.4), (300, 256, 0.05), (300, 257, 0.05),
                                         (40, 3000, 0.01), (5000, 600, 0.01), (1, 900, 0.3),
                                         (700, 1, 0.5)])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16])
def test_transpose_bit_exact(n, m, density, dtype):
    spl = _spl()
    rs = np.random.RandomState(n + m)
    pos, crd, vals = tiny.csr(rs, n, m, density, empty_rows={0} if n > 1 else (),
                              full_rows={n // 2} if m < 1000 else ())
    print(f"transpose n={n} m={m} nnz={len(crd)} {dtype}", flush=True)
    _check(spl, _csr(spl, pos, crd, vals, (n, m), dtype), (n, m, dtype))


def test_transpose_empty_and_deterministic():
    spl = _spl()
    B = _csr(spl, np.zeros(6, np.int32), np.zeros(0, np.int32), np.zeros(0), (5, 9))
    T = _check(spl, B, "empty")
    assert not T.pos.any()
    c = configs.config2(scale=0.01, N=1)
    B = spl.CSR(c["pos"].to(_dev()), c["crd"].to(_dev()), c["vals"].to(_dev()),
                (c["n"], c["n"]))
    T1 = _check(spl, B, "power law scale 0.01")
    T2 = spl.transpose(B)
    assert torch.equal(T1.pos, T2.pos) and torch.equal(T1.crd, T2.crd)
    assert torch.equal(T1.vals, T2.vals)


def test_transpose_full_size_power_law():
    # 2,000,000 columns: three radix passes over 32e6 entries
    spl = _spl()
    c = configs.config2(device="cuda", with_dense=False)
    n = c["n"]
    B = spl.CSR(c["pos"], c["crd"], c["vals"].to(torch.float32), (n, n))
    _check(spl, B, "power law full size")


@pytest.mark.parametrize("nnz,n,m,cols", [
    # one tile of 4,096 entries and its edges; 16 and 17 tiles, 64 (offsets
    # summed by the scatter) and 65 (by their own kernel); a ragged last tile
    (4095, 500, 130, "any"), (4096, 500, 130, "any"), (4097, 500, 130, "any"),
    (65536, 9000, 2000, "any"), (65537, 9000, 2000, "any"), (200_003, 9000, 70_000, "any"),
    (262_144, 9000, 2000, "any"), (262_145, 9000, 2000, "any"),
    # four passes and gaps of millions of columns; every entry in one column;
    # one row holding every entry; runs of thousands of empty rows in a tile
    (3000, 2900, 40_000_000, "any"), (70_000, 70_000, 300, "one"), (9000, 1, 70_000, "any"),
    (5000, 400_000, 257, "any"),
])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16])
def test_transpose_tile_edges(nnz, n, m, cols, dtype):
    spl = _spl()
    rs = np.random.RandomState(nnz + n)
    if cols == "one":
        row, col = np.arange(nnz), np.full(nnz, m - 1)
    elif n == 1:
        row, col = np.zeros(nnz, np.int64), np.sort(rs.choice(m, nnz, replace=False))
    else:
        key = np.unique(rs.randint(0, n * m, 2 * nnz, dtype=np.int64))
        key = np.sort(rs.choice(key, nnz, replace=False))
        row, col = key // m, key % m
    pos = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(row, minlength=n), out=pos[1:])
    print(f"transpose nnz={nnz} n={n} m={m} {cols} {dtype}", flush=True)
    _check(spl, _csr(spl, pos, col, rs.uniform(-1, 1, nnz), (n, m), dtype), (nnz, n, m, dtype))


def _spread(n, m, row, rs):
    """The n x m pattern of the entries in rows `row` (sorted; of one row,
    consecutive columns)."""
    pos = np.zeros(n + 1, np.int64)
    np.cumsum(np.bincount(row, minlength=n), out=pos[1:])
    return pos, np.arange(row.size) - pos[row], rs.uniform(-1, 1, row.size)


@pytest.mark.parametrize("span", [16_384, 16_385, 16_387, 65_536, 5_000_001])
@pytest.mark.parametrize("where", ["ends", "even", "second tile"])
def test_transpose_tiles_of_many_rows(span, where):
    """Tiles whose entries span more rows than are marked one by one (up to
    16,384), several entries to a row and long runs of empty rows among them;
    in the last case behind a tile that spans few."""
    spl = _spl()
    rs = np.random.RandomState(span)
    far = span + 7  # the last entry's row: `span` rows past the first's
    row = np.array([7] * 3 + [far] * 2) if where == "ends" else \
        np.sort(np.concatenate([np.linspace(7, far, 1500).astype(np.int64)] * 2))
    if where == "second tile":
        row = np.sort(np.concatenate([rs.randint(0, 8, 4096), row + 1]))
    print(f"transpose span={span} {where}", flush=True)
    for tail in (0, 100_000):  # empty rows at the end
        n = int(row[-1]) + 1 + tail
        _check(spl, _csr(spl, *_spread(n, 5000, row, rs), (n, 5000)), (span, where, tail))


def test_transpose_hypersparse_time():
    """Twenty million rows for 4,000 entries cost a search per entry, not a
    walk over the rows by one workgroup (which took hundreds of times as
    long as the same entries in 4,000 rows; the search takes about twice)."""
    spl = _spl()
    rs = np.random.RandomState(3)
    us = []
    for n in (4000, 20_000_000):
        row = np.sort(rs.randint(0, n, 4000))
        B = _csr(spl, *_spread(n, 300, row, rs), (n, 300))
        _check(spl, B, n)
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(10):
            spl.transpose(B)
        b.record()
        b.synchronize()
        us.append(a.elapsed_time(b) * 100)
    print(us, flush=True)
    assert us[1] < 50 * us[0], us


@pytest.mark.parametrize("kind", ["float", "int"])
def test_csc_spmv(kind):
    # A (n x m) given by columns: its CSR comes from the transposition, then
    # the CSR SpMV leaf; against the oracle's plain CSC definition
    spl = _spl()
    rs = np.random.RandomState(21)
    n, m = 3000, 1700
    cpos, crd, vals = tiny.csr(rs, m, n, 0.004, empty_rows={5}, kind=kind)
    x = rs.randint(-4, 5, m).astype(np.float64) if kind == "int" else rs.uniform(-1, 1, m)
    A = spl.CSC(*(torch.as_tensor(a, device=_dev()) for a in (cpos, crd, vals)), (n, m))
    xd = torch.as_tensor(x, device=_dev())
    ref, S = oracle.csc_spmv(cpos, crd, vals, x, n)
    for sched in (dict(kind="default"), dict(kind="row", lanes_per_row=4),
                  dict(kind="nnz", tile=512)):
        y = spl.spmv(A.to_csr(), xd, sched=spl.schedule(**sched))
        if kind == "int":
            assert np.array_equal(host64(y), ref), sched
        else:
            assert_close(host64(y), ref, S, 1e-12, f"csc spmv {sched}")
